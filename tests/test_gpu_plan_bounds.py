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


@pytest.mark.parametrize("d,K", [(3, 2), (5, 2), (8, 3), (8, 5), (12, 2), (16, 5), (24, 2), (32, 4), (40, 2), (64, 2)])
@pytest.mark.parametrize("e", [80, -80])
def test_units(pm, d, K, e):
    """The Hamiltonian in other units: scaled by 2^-e, the slice width by 2^e (e = 80
    is joules and seconds over hbar), every exponent is the same number, so every
    plan and every result is too, bit for bit.  The controls rest over the first
    half of a chain: its bound is small, the second half's is not."""
    import torch
    rng = np.random.default_rng(d)
    V = torch.from_numpy(rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d))).cuda()
    for order in (2, 4, orc.CF4, 6):
        w = synth.random_system(d, K, n_slices=11, h=0.4, order=order, tag=1120)
        w.samples[:, : w.samples.shape[1] * 6 // 11] = 0.0
        out = []
        for x in (0, e):
            print(f"[case] units d={d} K={K} order={order} 2^{x}", file=sys.stderr, flush=True)
            with pm.Context(0, pm.PM_FP64) as ctx:
                ctx.set_hamiltonian(w.H0 * 1e-3 * 2.0 ** -x, w.Hk * 2.0 ** -x, order)
                ctx.set_chunk(12)
                h = w.h * 2.0 ** x
                res = [ctx.equiprop(w.samples, h)]
                if order in (2, 4):
                    res.append(ctx.equiprop(w.samples, h, return_slices=True)[1])
                if order != 6:
                    res.append(ctx.trajectory(w.samples, h))
                    c = torch.from_numpy(w.samples).cuda()
                    g = torch.zeros_like(c)
                    ctx.backward_dev(c, h, V, g)
                    torch.cuda.synchronize()
                    res.append(g.cpu().numpy())
            out.append(res)
        Uo = orc.propagate(w.H0 * 1e-3, w.Hk, w.samples, w.h, order)
        assert orc.relative_frobenius(out[1][0], Uo) <= 1e-10, order
        for a, b in zip(*out):
            assert np.array_equal(a, b), order


@pytest.mark.parametrize("d", [3, 5, 8, 11, 16, 17, 24, 32, 33, 64])
@pytest.mark.parametrize("kind", ["zero", "diagonal", "rank one", "one pair", "identity"])
def test_norms_of_special_matrices(pm, d, kind):
    """Norms whose bound has nothing to spare (a single eigenvalue, all alike) and a
    basis of zeros: from a short to a long series the slices keep FP64 accuracy
    (64 sqrt(n d) 2^-53, doubled by each squaring), gradients included."""
    import torch
    rng = np.random.default_rng(d)
    v = rng.standard_normal((d, 1)) + 1j * rng.standard_normal((d, 1))
    v /= np.linalg.norm(v)
    A = {"zero": np.zeros((d, d)), "diagonal": np.diag(np.linspace(-1.0, 0.9, d)), "rank one": v @ v.conj().T,
         "one pair": np.zeros((d, d), complex), "identity": np.eye(d)}[kind].astype(complex)
    if kind == "one pair":
        A[0, d - 1], A[d - 1, 0] = 1j, -1j
    w = synth.random_system(d, 1, n_slices=7, h=0.1, order=2, tag=1140)
    for H0, Hk in ((A, w.Hk), (w.H0, A[None]), (A, A[None])):
        for h in (1e-6, 0.05, 0.4, 3.0):
            print(f"[case] {kind} d={d} h={h}", file=sys.stderr, flush=True)
            V = rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d))
            with pm.Context(0, pm.PM_FP64) as ctx:
                ctx.set_hamiltonian(H0, Hk, 2)
                U = ctx.equiprop(w.samples, h)
                c = torch.from_numpy(w.samples).cuda()
                g = torch.zeros_like(c)
                ctx.backward_dev(c, h, torch.from_numpy(V).cuda(), g)
                torch.cuda.synchronize()
            Uo = orc.propagate(H0, Hk, w.samples, h, 2)
            _, go = orc.control_gradient(H0, Hk, w.samples, h, 2, V)
            tol = 64 * np.sqrt(7 * d) * 2.0 ** -53 * max(1.0, 4 * h)
            assert orc.relative_frobenius(U, Uo) <= tol
            assert np.max(np.abs(g.cpu().numpy() - go)) <= 4 * tol * h * np.linalg.norm(V) * max(1.0, np.linalg.norm(Hk[0], 2))
