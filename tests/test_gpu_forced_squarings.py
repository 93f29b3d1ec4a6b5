"""Forced squarings in FP64 above 4 levels: the series goes on to the degree cap
when that is what the scaled exponent needs.

Exponents of 2-norm 0.5 to 1.6 times 2^s with s squarings forced and the largest
cap, 21: its remainder at 1.6 is 1.6^22 / 22! = 3e-17, below the rounding of a
slice.  Tolerances: 64 sqrt(n d) 2^-53 for a propagation of n slices (a product of
d x d unitary-scale matrices rounds to about sqrt(d) 2^-53, a few products a slice,
errors adding like a random walk), doubled by each squaring; the gradient, which
multiplies two checkpoints and a series of products, four times that relative to
its scale.
"""
import math
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


def at_norm(d, order, norm):
    """Nine slices whose largest exponent has 2-norm `norm`."""
    w = synth.random_system(d, 2, n_slices=9, h=0.1, order=order, tag=1000 + d)
    w.samples[:] = w.samples[:, :1]   # constant: the exponents scale with h
    G = orc.slice_exponents(w.H0, w.Hk, w.samples, w.h, order)
    w.h *= norm / max(np.linalg.norm(g, 2) for g in G)
    return w


@pytest.mark.parametrize("d", [5, 8, 9, 16, 24, 32, 48, 64])
@pytest.mark.parametrize("s", [0, 2])
def test_cap_is_reached(pm, d, s):
    import torch
    rng = np.random.default_rng(d)
    for order in (2, 4):
        for x in (0.5, 0.8, 1.0, 1.2, 1.4, 1.6):
            w = at_norm(d, order, x * 2 ** s)
            n = w.n_slices
            Uo, slo = orc.propagate(w.H0, w.Hk, w.samples, w.h, order, return_slices=True)
            V = rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d))
            _, go = orc.control_gradient(w.H0, w.Hk, w.samples, w.h, order, V)
            with pm.Context(0, pm.PM_FP64) as ctx:
                ctx.set_hamiltonian(w.H0, w.Hk, order)
                ctx.set_expm_policy(max_taylor_degree=21, force_s=s)
                U, sl = ctx.equiprop(w.samples, w.h, return_slices=True)
                P = ctx.trajectory(w.samples, w.h)
                c = torch.from_numpy(w.samples).cuda()
                g = torch.zeros_like(c)
                ctx.backward_dev(c, w.h, torch.from_numpy(V).cuda(), g)
                torch.cuda.synchronize()
                g = g.cpu().numpy()
            tol = 64 * math.sqrt(n * d) * 2.0 ** -53 * 2 ** s
            scale = w.h * np.linalg.norm(V) * max(np.linalg.norm(h, 2) for h in w.Hk)
            e = (orc.relative_frobenius(U, Uo), float(np.max(np.abs(sl - slo))),
                 orc.relative_frobenius(P[-1], Uo), float(np.max(np.abs(g - go))) / scale)
            print(f"[case] d={d} order={order} s={s} norm={x}*2^s errors " + " ".join(f"{v:.1e}" for v in e) +
                  f" bound {tol:.1e}", file=sys.stderr, flush=True)
            assert e[0] <= tol and e[2] <= tol
            assert e[1] <= 64 * math.sqrt(d) * 2.0 ** -53 * 2 ** s
            assert e[3] <= 4 * tol
