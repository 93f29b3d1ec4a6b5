"""Rounding of the stored FP64 slices of 3 and 4 levels, where a slice is c_0 I plus
sums of the size of its exponent.

For a traceless exponent of norm e << 1 (no phase to rotate) the real and the
imaginary part of an entry carry the rounding of c_0, 2^-53 at most (its last step is of
the size of one), that of the final sum, 2^-53 at most, and those of the sums before
it, a few times e 2^-53: with e below 0.05 less than 2.3 * 2^-53 a part (c_0's
imaginary part is of the size of e^3), 2.5 * 2^-53 = 2.8e-16 together.  Adding c_0
first rounds every later sum at the size of one too.
"""
import sys

import numpy as np
import pytest

import oracle.propagator as orc
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [3, 4])
@pytest.mark.parametrize("order", [2, 4])
def test_diagonal_rounds_once(d, order):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_07126_amd as pm
    w = synth.random_system(d, 2, n_slices=20000, h=0.02, order=order, tag=1600)
    eye = np.eye(d)
    H0 = w.H0 - np.trace(w.H0) / d * eye
    Hk = np.stack([h - np.trace(h) / d * eye for h in w.Hk])
    with pm.Context(0, pm.PM_FP64) as ctx:
        ctx.set_hamiltonian(H0, Hk, order)
        _, sl = ctx.equiprop(w.samples, w.h, return_slices=True)
    G = orc.slice_exponents(H0, Hk, w.samples, w.h, order)
    E = np.zeros_like(G)
    T = np.broadcast_to(eye.astype(complex), G.shape)
    for k in range(1, 16):
        T = T @ (-1j * G) / k
        E = E + T
    err = float(np.max(np.abs((sl - eye) - E)))
    print(f"[case] d={d} order={order} error {err:.2e}", file=sys.stderr, flush=True)
    assert err <= 2.5 * 2.0 ** -53
