"""The FP64 engine of dimensions 1..4 at lengths where its chain length and the
depth of its product tree change: one slice per lane and several, ragged last
chains, one to three tree levels, with and without per-slice output.

Tolerance: the FP64 parity bound (a slice, run or tree node left out or doubled
differs by far more).
"""
import sys

import numpy as np
import pytest

import oracle.propagator as orc
import synth
from bounds import TOL64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_07126_amd as m
    return m


@pytest.mark.parametrize("d,order", [(1, 2), (2, 2), (2, 4), (2, orc.CF4), (3, 2), (3, 4), (4, 2), (4, 4), (4, orc.CF4)])
def test_lengths(pm, d, order):
    for n in (1, 2, 63, 64, 65, 255, 257, 513, 1025, 2049, 4095, 16385):
        w = synth.random_system(d, 2, n_slices=n, h=0.02, order=order, tag=900 + d)
        slices = order != orc.CF4
        with pm.Context(0, pm.PM_FP64) as ctx:
            ctx.set_hamiltonian(w.H0, w.Hk, order)
            shape = ctx.launch_shape(w.n_samples)
            print(f"[case] d={d} order={order} N={n} shape={shape}", file=sys.stderr, flush=True)
            U = ctx.equiprop(w.samples, w.h)
            out = ctx.equiprop(w.samples, w.h, return_slices=True) if slices else None
            again = ctx.equiprop(w.samples, w.h)
        e = n * (2 if order == orc.CF4 else 1)
        assert shape[1] == -(-e // shape[0]) and shape[0] % 64 == 0
        assert np.array_equal(U, again)
        ref = orc.propagate(w.H0, w.Hk, w.samples, w.h, order, return_slices=slices)
        Uo, slo = ref if slices else (ref, None)
        assert orc.relative_frobenius(U, Uo) <= TOL64
        if slices:
            assert orc.relative_frobenius(out[0], Uo) <= TOL64
            assert np.max(np.abs(out[1] - slo)) <= TOL64


def test_three_levels(pm):
    w = synth.random_system(2, 1, n_slices=300_001, h=0.01, order=2, tag=910)
    with pm.Context(0, pm.PM_FP64) as ctx:
        ctx.set_hamiltonian(w.H0, w.Hk, 2)
        assert ctx.launch_shape(w.n_samples)[2] > 64
        U = ctx.equiprop(w.samples, w.h)
    assert orc.relative_frobenius(U, orc.propagate(w.H0, w.Hk, w.samples, w.h, 2)) <= TOL64
