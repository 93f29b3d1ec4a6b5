"""The 64-wide gradient where its chains are split: few long chains in parts that
recompute their predecessors (ragged last parts among them), and a chain per
compute unit in one part.

Tolerance: 4 * 64 sqrt(n d) 2^-53 of the gradient's scale h ||W||_F max ||H_k||_2
(rounding of the products of a slice, its two checkpoints and its series, errors
adding like a random walk); a part left out or counted twice differs by far more.
"""
import math
import sys

import numpy as np
import pytest

import oracle.propagator as orc
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n,chunk", [(33, 70, 32), (48, 67, 64), (64, 37, 40), (64, 129, 8), (64, 260, 0), (40, 520, 2)])
def test_split_chains(d, n, chunk):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_07126_amd as pm
    w = synth.random_system(d, 1, n_slices=n, h=0.02, order=2, tag=1200)
    rng = np.random.default_rng(d)
    V = rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d))
    print(f"[case] gradient d={d} N={n} chunk={chunk}", file=sys.stderr, flush=True)
    _, go = orc.control_gradient(w.H0, w.Hk, w.samples, w.h, 2, V)
    with pm.Context(0, pm.PM_FP64) as ctx:
        ctx.set_hamiltonian(w.H0, w.Hk, 2)
        ctx.set_chunk(chunk)
        c = torch.from_numpy(w.samples).cuda()
        g = torch.zeros_like(c)
        ctx.backward_dev(c, w.h, torch.from_numpy(V).cuda(), g)
        torch.cuda.synchronize()
    scale = w.h * np.linalg.norm(V) * np.linalg.norm(w.Hk[0], 2)
    err = float(np.max(np.abs(g.cpu().numpy() - go))) / scale
    tol = 4 * 64 * math.sqrt(n * d) * 2.0 ** -53
    print(f"  error {err:.2e} (bound {tol:.2e})", file=sys.stderr, flush=True)
    assert err <= tol
