"""The reduced-precision engine of dimensions 33..64 where its paths change: the
row tiles that a dimension reaches (33, 40 | 41, 48 | 49, 64), chains of an odd and
an even number of slices and of one, tables of weights refilled within a chain
(more than 32 slices), and pairs of slices whose degrees and squarings differ.

Tolerances: those of tests/bounds.py, with the squarings of the largest slice.
"""
import sys

import numpy as np
import pytest

import oracle.propagator as orc
import synth
from bounds import max_squarings, tol, tol_slice

pytestmark = pytest.mark.gpu

MODES = ("PM_FP32", "PM_FP32_3M", "PM_BF16_SPLIT")


@pytest.fixture(scope="module")
def pm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_07126_amd as m
    return m


def check(pm, w, prec, chunk=0):
    print(f"[case] d={w.dim} K={w.n_ctrl} N={w.n_slices} order={w.order} prec={prec} chunk={chunk}",
          file=sys.stderr, flush=True)
    Uo, slo = orc.propagate(w.H0, w.Hk, w.samples, w.h, w.order, return_slices=True)
    with pm.Context(0, prec) as ctx:
        ctx.set_hamiltonian(w.H0, w.Hk, w.order)
        if chunk:
            ctx.set_chunk(chunk)
        U, sl = ctx.equiprop(w.samples, w.h, return_slices=True)
        U2 = ctx.equiprop(w.samples, w.h)
    s = max_squarings(pm, w, prec)
    err, es = orc.relative_frobenius(U, Uo), float(np.max(np.abs(sl - slo)))
    print(f"  s={s} error {err:.2e} (bound {tol(prec, w.n_slices, w.dim, s):.2e}), slice {es:.2e}",
          file=sys.stderr, flush=True)
    assert err <= tol(prec, w.n_slices, w.dim, s)
    assert es <= tol_slice(prec, w.dim, s)
    assert np.array_equal(U, U2)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("d", [33, 40, 41, 48, 49, 63, 64])
def test_dimension_edges(pm, mode, d):
    prec = getattr(pm, mode)
    for n, order, K, chunk in ((1, 2, 1, 0), (7, 4, 2, 3), (80, 2, 2, 79)):
        check(pm, synth.random_system(d, K, n_slices=n, h=0.03, order=order, tag=800 + d), prec, chunk)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("K", [1, 4, 5])
def test_basis_groups(pm, mode, K):
    """Basis sizes around a multiple of the four matrices expanded together."""
    for order in (2, 4):
        check(pm, synth.random_system(64, K, n_slices=37, h=0.02, order=order, tag=820 + K), getattr(pm, mode), 36)


@pytest.mark.parametrize("mode", MODES)
def test_uneven_degrees(pm, mode):
    """Neighbouring slices of very different norms: every pairing of degree 1, 2,
    3, higher ones and squarings within a pair of slices."""
    amp = np.array([1e-9, 1e-7, 2e-6, 1e-4, 3e-3, 0.05, 0.4, 4.0])
    w = synth.random_system(50, 1, n_slices=2 * len(amp) ** 2, h=1.0, order=2, tag=840)
    w.H0[...] *= 1e-12
    w.samples[0] = np.stack(np.meshgrid(amp, amp, indexing="ij"), -1).reshape(-1)
    check(pm, w, getattr(pm, mode), 33)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("norm", [1e-9, 1e-6, 1e-4, 1e-2, 0.3])
def test_degrees(pm, mode, norm):
    check(pm, synth.random_system(64, 1, n_slices=9, h=norm, order=2, tag=850), getattr(pm, mode), 4)
