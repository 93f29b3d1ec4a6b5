"""The bounds from which the FP64 tile engines plan a slice's series: what they
take in has to be the exponent's, and hold at every scale of its factors."""
import sys

import numpy as np
import pytest

import oracle.propagator as orc
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_07126_amd as m
    return m


@pytest.mark.parametrize("d", [33, 40, 41, 47, 48, 49, 56, 64])
@pytest.mark.parametrize("scale", [4e2, 4e6, 4e12])
def test_own_norm_where_terms_cancel(pm, d, scale):
    """Terms that cancel: the 1-norm of the exponent itself, about 0.3, asks for no
    squaring, so the plan is that of squarings forced to none, bit for bit."""
    w = synth.random_system(d, 2, n_slices=40, h=0.05, order=2, tag=1100)
    H0, Hk = scale * w.Hk[1] + w.H0, w.Hk.copy()
    w.samples[1] = -scale
    out = []
    for force in (-1, 0):
        print(f"[case] cancelling terms d={d} scale={scale} force_s={force}", file=sys.stderr, flush=True)
        with pm.Context(0, pm.PM_FP64) as ctx:
            ctx.set_hamiltonian(H0, Hk, 2)
            ctx.set_chunk(20)
            ctx.set_expm_policy(force_s=force)
            out.append(ctx.equiprop(w.samples, w.h, return_slices=True))
    assert np.array_equal(out[0][1], out[1][1]) and np.array_equal(out[0][0], out[1][0])
