"""Short FP64 propagations, whose chains are one to four slices: the
product tree takes over most products and must not round worse than a chain.

With every slice propagator I + E, ||E|| = e, a product joined as X + E X adds one
rounding of X, 2^-53 of each entry at most, and the rounding of E X, below
e sqrt(d) 2^-53 in the probabilistic model.  A tree of L levels over n slices of
norm e joins nodes of norm up to e 2^l, so that relative to ||U||_F the errors of
its n / 2^l joins a level, adding like a random walk, stay below
2^-53 sqrt(n) (1 + n e sqrt(d) / 2): with n e <= 1 below 3 sqrt(n) 2^-53 (n <= 300,
d <= 64), and the exponentials' own, e sqrt(d) a few times 2^-53 a slice, are
smaller.  Full products of unitary matrices round to sqrt(d) 2^-53 each, n of them
to 2^-53 sqrt(n d), up to eight times the first term.
"""
import math
import sys

import numpy as np
import pytest

import oracle.propagator as orc
import synth

pytestmark = pytest.mark.gpu


def reference(w):
    """U(T) with the slices and every product carried less the identity."""
    E = []
    for G in orc.slice_exponents(w.H0, w.Hk, w.samples, w.h, w.order):
        X, T = np.zeros_like(G), np.eye(w.dim, dtype=complex)
        for k in range(1, 25):
            T = T @ (-1j * G) / k
            X = X + T
        E.append(X)
    while len(E) > 1:
        E = [E[i] + E[i + 1] + E[i + 1] @ E[i] for i in range(0, len(E) - 1, 2)] + E[len(E) // 2 * 2:]
    return np.eye(w.dim) + E[0]


@pytest.mark.parametrize("d", [5, 8, 12, 16, 17, 24, 27, 32, 40, 48, 57, 64])
@pytest.mark.parametrize("n", [30, 100, 300])
def test_short_propagation(d, n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_07126_amd as pm
    w = synth.random_system(d, 2, n_slices=n, h=0.3 / n, order=2, tag=1400)
    with pm.Context(0, pm.PM_FP64) as ctx:
        ctx.set_hamiltonian(w.H0, w.Hk, 2)
        U = ctx.equiprop(w.samples, w.h)
        P = ctx.trajectory(w.samples, w.h)
    ref = reference(w)
    tol = 3 * math.sqrt(n) * 2.0 ** -53
    err = orc.relative_frobenius(U, ref), orc.relative_frobenius(P[-1], ref)
    print(f"[case] d={d} N={n} errors {err[0]:.1e} {err[1]:.1e} bound {tol:.1e}", file=sys.stderr, flush=True)
    assert max(err) <= tol
