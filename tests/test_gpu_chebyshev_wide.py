"""The Chebyshev series above 16 levels where its instances change (the k-slices
that a dimension reaches: 24 | 25, 28 | 29, 32, 48 | 49 .. 64), with the exponent on
the whole basis and with a commutator by product, from the shortest series to
squarings, per-slice output included.

Tolerance: 64 sqrt(n d) 2^-53 (a product of d x d unitary-scale matrices rounds to
about sqrt(d) 2^-53, a few products a slice, errors adding like a random walk; the
series' truncation, 2^-53 a slice, is below that), doubled by each squaring.
"""
import math
import sys

import numpy as np
import pytest

import oracle.propagator as orc
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [17, 24, 25, 28, 29, 32, 33, 48, 49, 64])
def test_instances(d):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_07126_amd as pm
    for order, K, h in ((2, 2, 1e-9), (2, 2, 1e-4), (2, 1, 0.02), (4, 3, 0.1), (4, 6, 0.05), (2, 2, 6.0)):
        w = synth.random_system(d, K, n_slices=23, h=h, order=order, tag=1300 + d)
        with pm.Context(0, pm.PM_FP64) as ctx:
            ctx.set_hamiltonian(w.H0, w.Hk, order)
            ctx.set_expm_method(pm.PM_EXPM_CHEBYSHEV)
            ctx.set_chunk(6)
            U, sl = ctx.equiprop(w.samples, w.h, return_slices=True)
        Uo, slo = orc.propagate(w.H0, w.Hk, w.samples, w.h, order, return_slices=True)
        nu = max(np.linalg.norm(g, 1) for g in orc.slice_exponents(w.H0, w.Hk, w.samples, w.h, order))
        s = pm.plan_chebyshev(nu)[1]
        tol = 64 * math.sqrt(w.n_slices * d) * 2.0 ** -53 * 2 ** s
        err = orc.relative_frobenius(U, Uo), float(np.max(np.abs(sl - slo)))
        print(f"[case] chebyshev d={d} K={K} order={order} h={h} s={s} errors {err[0]:.1e} {err[1]:.1e} bound {tol:.1e}",
              file=sys.stderr, flush=True)
        assert err[0] <= tol and err[1] <= 64 * math.sqrt(d) * 2.0 ** -53 * 2 ** s
