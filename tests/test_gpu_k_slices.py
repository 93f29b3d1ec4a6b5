"""FP64 at 25 to 29 levels, where the one-wave teams go from seven to eight
k-slices: propagation, gradient and trajectories on the whole basis and with the
commutator by product, from a single slice to chains of several.  Checks and their
tolerances are those of the other dimensions."""
import numpy as np
import pytest

import oracle.propagator as orc
import synth
from test_gpu_teams import check, cotangent, gradient_case, pm  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [25, 27, 28, 29])
@pytest.mark.parametrize("n,order,K", [(1, 2, 2), (5, 4, 2), (33, 4, 3), (41, 2, 4), (300, 2, 2), (20, orc.CF4, 2)])
def test_seven_and_eight(pm, d, n, order, K):  # noqa: F811
    w = synth.random_system(d, K, n_slices=n, h=0.05, order=order, tag=1500 + d)
    check(pm, w, slices=order != orc.CF4)
    gradient_case(pm, w, cotangent(d, n))
    P = orc.trajectory(w.H0, w.Hk, w.samples, w.h, order)
    with pm.Context(0, pm.PM_FP64) as ctx:
        ctx.set_hamiltonian(w.H0, w.Hk, order)
        out = ctx.trajectory(w.samples, w.h)
    assert np.max(np.abs(out - P)) <= 2 * 64 * np.sqrt(n) * d * 2.0 ** -53
