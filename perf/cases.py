"""The work that users of the propagator have it do, as measurable cases.

Every case is one call (or one batch run) of the public Python entry points on
seeded synthetic inputs: GUE Hamiltonians and smooth controls (or the 3-qubit
register with one amplitude per slice), in the shapes of the repository's own
workloads (`synth`, `bench.py`).  A case is a plain dict:

  kind       "propagate" (U(T)), "slices" (U(T) and every slice propagator),
             "gradient" (dL/d samples and U(T)), "trajectory" (states at every
             slice boundary) or "batch" (many uneven instances)
  dim, ctrl  Hilbert-space dimension and number of controls
  slices     N, the number of time slices of width h
  order      2 midpoint, 4 commutator Magnus, 5 commutator-free, 6 sixth order
  precision  "fp64", "fp32", "fp32_3m" or "bf16_split"
  h, norm    slice width and 2-norm of the drift

`exact` is the same mathematics in plain torch complex128: slice exponents
from their definition, a long Taylor series with scaling and squaring, and a
balanced product tree, all carried as exp - I so that small slices keep their
relative accuracy; gradients by torch's autograd through it.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2108_07126_amd as pm

DEVICE = "cuda" if torch.cuda.is_available() else "cpu"


def _case(name, kind, dim, ctrl, slices, order, precision, h, norm=1.0, system="gue", **more):
    c = {"kind": kind, "dim": dim, "ctrl": ctrl, "slices": slices, "order": order,
         "precision": precision, "h": h, "norm": norm, "system": system}
    if name:
        c["name"] = name
    c.update(more)
    return c


def listed():
    return [
        # one shot of a driven qubit (10^4 steps): the smallest call, launch and chain latency
        _case("qubit_shot", "propagate", 2, 1, 10_000, 2, "fp64", 0.01, 3.14),
        # a long qubit record whose every step is kept (for plots, noise models): output-bound
        _case("qubit_all_steps", "slices", 2, 1, 1 << 22, 2, "fp64", 0.01, 3.14),
        # two qubits, every step kept in single precision
        _case("two_qubit_all_steps", "slices", 4, 2, 1 << 20, 2, "fp32", 0.01),
        # one gradient of the 3-qubit register (16384 parameters): the inner step of pulse optimisation
        _case("register_gradient", "gradient", 8, 4, 4096, 2, "fp64", 0.1, system="register"),
        # the register's steps kept, at a ragged length
        _case("register_all_steps", "slices", 8, 4, 100_001, 2, "fp64", 0.1, system="register"),
        # a 16-level system at the length that gives 1e-4: a short, latency-bound propagation
        _case("qudit_short", "propagate", 16, 3, 8192, 4, "fp64", 1.6e-2),
        # the 16-level system at full length (the benchmark's workload)
        _case("qudit_long", "propagate", 16, 3, 1 << 17, 4, "fp64", 1e-3),
        # states of a 16-level system over time (four initial states)
        _case("qudit_states", "trajectory", 16, 3, 32_768, 4, "fp64", 4e-3, vectors=4),
        # three qutrits (27 levels, ragged against every tile size)
        _case("three_qutrits", "propagate", 27, 4, 20_000, 4, "fp64", 5e-3, 2.0),
        # 64 levels with a strong drift: the largest matrices, double precision
        _case("d64_double", "propagate", 64, 2, 32_768, 2, "fp64", 0.01, 10.0),
        # the same system in the fastest mode, for coarse scans
        _case("d64_split", "propagate", 64, 2, 65_536, 2, "bf16_split", 0.01, 10.0),
        # a parameter study: many uneven systems in one batch
        _case("study_batch", "batch", 64, 4, 10_000, 4, "fp32_3m", 0.01, 10.0, instances=96),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["propagate", "propagate", "propagate", "propagate", "slices", "slices", "gradient",
                       "gradient", "trajectory", "batch"])
    if kind == "batch":
        return _case(None, kind, rng.choice([16, 32, 64]), rng.randint(1, 4), _log_int(rng, 1000, 10_000),
                     4, rng.choice(["fp64", "fp32_3m", "fp32", "bf16_split"]), 0.01, rng.choice([1.0, 10.0]),
                     instances=_log_int(rng, 8, 96))
    dim = rng.choice([1, 2, 2, 3, 4, 4, 5, 6, 8, 8, 9, 12, 16, 16, 20, 27, 32, 48, 64])
    ctrl = rng.randint(1, 4)
    order = rng.choice([2, 2, 2, 4, 4, 4, 5, 6])
    precision = rng.choice(["fp64", "fp64", "fp64", "fp32", "fp32_3m", "bf16_split"])
    if kind in ("gradient", "trajectory") or order == 6:
        precision = "fp64"
    if kind in ("gradient", "trajectory") and order == 6:
        order = 4
    if kind == "slices" and order == 5:
        order = 4
    d = max(dim, 8)                       # work per slice grows as d^3 above the tile's floor
    top = {"propagate": 2 ** 33 // d ** 3, "slices": 2 ** 23 // dim ** 2, "gradient": 2 ** 22 // d ** 3,
           "trajectory": 2 ** 23 // d ** 2}[kind]
    top = min(top, 1 << 21)
    n = _log_int(rng, 500 if kind != "gradient" else 200, max(top, 1000))
    h = math.exp(rng.uniform(math.log(1e-3), math.log(0.1)))
    more = {"vectors": rng.randint(1, dim)} if kind == "trajectory" else {}
    return _case(None, kind, dim, ctrl, n, order, precision, h, rng.choice([1.0, 1.0, 3.0, 10.0]), **more)


# ------------------------------------------------------------------ inputs

def _gue(rng, d, norm):
    a = (rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d))) / math.sqrt(2.0)
    a = 0.5 * (a + a.conj().T)
    return a * (norm / float(np.max(np.abs(np.linalg.eigvalsh(a)))))


def _register():
    # H0 = J (Z1Z2 + Z2Z3 + Z1Z3) + sum (w_q / 2) Z_q, controls (W/2){X1, Y1, X2, Y2}
    eye, x, y, z = (np.array(m, complex) for m in ([[1, 0], [0, 1]], [[0, 1], [1, 0]], [[0, -1j], [1j, 0]],
                                                    [[1, 0], [0, -1]]))
    kron = lambda a, b, c: np.kron(np.kron(a, b), c)
    zs = [kron(z, eye, eye), kron(eye, z, eye), kron(eye, eye, z)]
    tau = 2.0 * math.pi
    H0 = tau * 0.01 * (zs[0] @ zs[1] + zs[1] @ zs[2] + zs[0] @ zs[2])
    H0 = H0 + sum(0.5 * tau * w * zz for w, zz in zip((0.10, 0.12, 0.14), zs))
    Hk = 0.5 * tau * 0.05 * np.stack([kron(x, eye, eye), kron(y, eye, eye), kron(eye, x, eye), kron(eye, y, eye)])
    return H0, Hk


def _times(n, h, order, device):
    if order == 2:
        return (torch.arange(n, dtype=torch.float64, device=device) + 0.5) * h
    if order == 6:
        node = torch.tensor([0.5 - math.sqrt(15.0) / 10.0, 0.5, 0.5 + math.sqrt(15.0) / 10.0],
                            dtype=torch.float64, device=device)
        return ((torch.arange(n, dtype=torch.float64, device=device)[:, None] + node) * h).reshape(-1)
    return torch.arange(2 * n + 1, dtype=torch.float64, device=device) * (0.5 * h)


def _system(case, rng, device):
    """(H0, Hk) as numpy and the control samples [K][S] on the device."""
    d, K, n, h, order = case["dim"], case["ctrl"], case["slices"], case["h"], case["order"]
    if case["system"] == "register":
        H0, Hk = _register()
        c = torch.from_numpy(rng.uniform(-1.0, 1.0, size=(len(Hk), n))).to(device)
        return H0, Hk, c
    H0 = _gue(rng, d, case["norm"])
    Hk = np.stack([_gue(rng, d, 1.0) for _ in range(K)])
    f, phi = rng.uniform(0.5, 5.0, (K, 4)), rng.uniform(0.0, 2.0 * math.pi, (K, 4))
    a = rng.normal(0.0, 0.3, (K, 4))
    t = _times(n, h, order, device)
    c = torch.zeros((K, t.numel()), dtype=torch.float64, device=device)
    for k in range(K):
        for i in range(4):
            c[k] += a[k, i] * torch.sin(2.0 * math.pi * f[k, i] * t + phi[k, i])
    return H0, Hk, c.contiguous()


class _Instance:
    def __init__(self, case, rng):
        H0, Hk, c = _system(case, rng, "cpu")
        self.H0, self.Hk, self.samples, self.h, self.order = H0, Hk, c.numpy(), case["h"], case["order"]


def _instances(case, rng):
    """Uneven instances: dimensions up to case["dim"], lengths over a factor of ten, orders 2 and 4 (the
    study's layout is the case's; the systems and controls are the seed's)."""
    dims = [d for d in (2, 4, 8, 16, 32, 64) if d <= case["dim"]]
    lay = np.random.default_rng([case["instances"], case["slices"], case["dim"], case["ctrl"]])
    out = []
    for _ in range(case["instances"]):
        sub = dict(case, dim=int(lay.choice(dims)), ctrl=int(lay.integers(1, case["ctrl"] + 1)),
                   slices=int(round(case["slices"] * 10.0 ** lay.uniform(-1.0, 0.0))),
                   order=int(lay.choice([2, 4])), norm=float(case["norm"] ** lay.uniform(0.0, 1.0)))
        out.append(_Instance(sub, rng))
    return out


def _randn_c(rng, *shape):
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


def _inputs(case, seed, device):
    rng = np.random.default_rng([21080, int(seed)])
    if case["kind"] == "batch":
        return {"instances": _instances(case, rng)}
    H0, Hk, c = _system(case, rng, device)
    s = {"H0": H0, "Hk": Hk, "samples": c}
    d = case["dim"]
    if case["kind"] == "gradient":        # dL = Re Tr(W^H dU(T)) of a loss of size one
        s["W"] = torch.from_numpy(_randn_c(rng, d, d) / d).to(device)
    if case["kind"] == "trajectory":
        s["x0"] = torch.from_numpy(np.linalg.qr(_randn_c(rng, d, d))[0][:, :case["vectors"]].copy()).to(device)
    return s


def prepare(case, seed):
    s = _inputs(case, seed, DEVICE)
    s["case"] = case
    if case["kind"] == "batch":
        s["batch"] = pm.Batch(0, case["precision"])
        s["batch"].set(s["instances"])
        return s
    d, n = case["dim"], case["slices"]
    ctx = pm.Context(0, case["precision"])
    ctx.set_hamiltonian(s["H0"], s["Hk"], case["order"])
    s["ctx"] = ctx
    s["U"] = torch.zeros((d, d), dtype=torch.complex128, device=DEVICE)
    if case["kind"] == "slices":
        t = torch.complex128 if case["precision"] == "fp64" else torch.complex64
        s["out"] = torch.empty((n, d, d), dtype=t, device=DEVICE)
    if case["kind"] == "gradient":
        s["grad"] = torch.zeros_like(s["samples"])
    if case["kind"] == "trajectory":
        s["out"] = torch.empty((n + 1, d, case["vectors"]), dtype=torch.complex128, device=DEVICE)
    return s


def run(state):
    case = state["case"]
    if case["kind"] == "batch":
        state["batch"].run(torch.cuda.current_stream())
        return np.concatenate([U.ravel() for U in state["batch"].results()])
    ctx, c, h = state["ctx"], state["samples"], case["h"]
    if case["kind"] == "propagate":
        ctx.equiprop_dev(c, h, state["U"])
        return state["U"]
    if case["kind"] == "slices":
        ctx.equiprop_dev(c, h, state["U"], state["out"])
        return {"U": state["U"], "slices": state["out"]}
    if case["kind"] == "gradient":
        ctx.backward_dev(c, h, state["W"], state["grad"], state["U"])
        return {"grad": state["grad"], "U": state["U"]}
    ctx.trajectory_dev(c, h, state["out"], pm.PM_TRAJ_STATES, state["x0"])
    return state["out"]


# -------------------------------------------------------------------- work

def _samples_of(n, order):
    return n if order == 2 else (3 * n if order == 6 else 2 * n + 1)


def _work(kind, d, K, n, order, elem, vectors=0):
    exps = 2 * n if order == 5 else n
    basis = 1 + K if order != 4 else 1 + 2 * K + K * (K - 1) // 2
    # per exponential: the expansion on the basis, a fourth-degree polynomial (two products, fewer do not
    # reach these precisions) and the product into U(T); sixth order adds three commutators
    product = 8 * d ** 3
    flops = exps * (4 * basis * d * d + 3 * product) + (3 * product * n if order == 6 else 0)
    nbytes = 8 * K * _samples_of(n, order) + 16 * d * d * (1 + basis)
    if kind == "slices":
        nbytes += n * d * d * elem
    if kind == "gradient":                 # every slice's derivative in the direction of every control
        flops += exps * (4 * product + 4 * basis * d * d)
        nbytes += 8 * K * _samples_of(n, order) + 16 * d * d
    if kind == "trajectory":
        flops = exps * (4 * basis * d * d + 2 * product + 8 * d * d * vectors)
        nbytes += 16 * (n + 1) * d * vectors
    return nbytes, flops


def work(case):
    K = case["ctrl"]
    if case["kind"] == "batch":
        # the mean of the instances' draws: dimensions and control counts uniform, lengths log-uniform
        dims = [d for d in (2, 4, 8, 16, 32, 64) if d <= case["dim"]]
        n = int(case["slices"] * 0.9 / math.log(10.0))
        per = [_work("propagate", d, (1 + K) // 2, n, o, 16) for d in dims for o in (2, 4)]
        b, f = (sum(p[i] for p in per) / len(per) * case["instances"] for i in (0, 1))
        return {"bytes": int(b), "flops": int(f)}
    b, f = _work(case["kind"], case["dim"], K, case["slices"], case["order"],
                 16 if case["precision"] == "fp64" else 8, case.get("vectors", 0))
    return {"bytes": int(b), "flops": int(f)}


# ------------------------------------------------------------------- exact

def _mm(a, b):
    """Batched complex product (tiny matrices elementwise, where a batched library call is slow)."""
    d = a.shape[-1]
    if d <= 4:
        out = a[..., :, 0:1] * b[..., 0:1, :]
        for k in range(1, d):
            out = out + a[..., :, k:k + 1] * b[..., k:k + 1, :]
        return out
    return torch.bmm(a.contiguous(), b.contiguous())


def _exponents(H0, Hk, c, h, order, i0, i1):
    """The Hermitian exponents of slices i0 .. i1 - 1, in product order."""
    def H(s):
        return H0 + torch.tensordot(s.T.to(H0.dtype), Hk, dims=1)
    if order == 2:
        return h * H(c[:, i0:i1])
    if order == 6:
        a1, a2, a3 = (H(c[:, 3 * i0 + q:3 * i1:3]) for q in range(3))
        com = lambda x, y: _mm(x, y) - _mm(y, x)
        p1, p2 = -1j * h * a2, -1j * (math.sqrt(15.0) * h / 3.0) * (a3 - a1)
        p3 = -1j * (10.0 * h / 3.0) * (a3 - 2.0 * a2 + a1)
        c1 = com(p1, p2)
        c2 = com(p1, 2.0 * p3 + c1) * (-1.0 / 60.0)
        return 1j * (p1 + p3 / 12.0 + com(-20.0 * p1 - p3 + c1, p2 + c2) / 240.0)
    a1, a2, a3 = H(c[:, 2 * i0:2 * i1:2]), H(c[:, 2 * i0 + 1:2 * i1:2]), H(c[:, 2 * i0 + 2:2 * i1 + 1:2])
    if order == 4:
        return (h / 6.0) * (a1 + 4.0 * a2 + a3) + (1j * h * h / 12.0) * (_mm(a1, a3) - _mm(a3, a1))
    first, second = (h / 12.0) * (3.0 * a1 + 4.0 * a2 - a3), (h / 12.0) * (4.0 * a2 + 3.0 * a3 - a1)
    return torch.stack([first, second], dim=1).reshape(-1, *H0.shape)


def _expm1(G):
    """exp(-i G) - I by a degree-20 Taylor series on G / 2^s, ||G / 2^s|| <= 1/4, then s squarings."""
    nu = float(G.detach().abs().sum(-1).max())
    s = max(0, math.ceil(math.log2(max(nu, 1e-30) / 0.25)))
    X = (-1j * 2.0 ** -s) * G
    E = X / 20.0
    for k in range(19, 0, -1):
        E = (X + _mm(X, E)) / k
    for _ in range(s):
        E = 2.0 * E + _mm(E, E)
    return E


def _tree(E):
    """prod (I + E_j) - I over the first axis, later factors on the left."""
    while E.shape[0] > 1:
        odd = E[E.shape[0] // 2 * 2:]
        a, b = E[0:E.shape[0] // 2 * 2:2], E[1::2]
        E = torch.cat([a + b + _mm(b, a), odd])
    return E[0]


def _scan(E):
    """All prefix products minus I (Hillis-Steele)."""
    step = 1
    while step < E.shape[0]:
        a, b = E[:-step], E[step:]
        E = torch.cat([E[:step], a + b + _mm(b, a)])
        step *= 2
    return E


def _propagate(H0, Hk, c, h, order, n, keep=None):
    """U(T); with keep, every slice propagator goes there."""
    d = H0.shape[0]
    eye = torch.eye(d, dtype=torch.complex128, device=H0.device)
    chunk = max(1, (1 << 25) // (d * d))
    parts = []
    for i0 in range(0, n, chunk):
        i1 = min(n, i0 + chunk)
        E = _expm1(_exponents(H0, Hk, c, h, order, i0, i1))
        if keep is not None:
            keep[i0:i1] = eye + E
        parts.append(_tree(E))
    return eye + _tree(torch.stack(parts))


def exact(case, seed):
    s = _inputs(case, seed, DEVICE)
    h, order, n, d = case["h"], case["order"], case["slices"], case["dim"]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEVICE, torch.complex128)
    if case["kind"] == "batch":
        out = []
        for w in s["instances"]:
            c = torch.from_numpy(w.samples).to(DEVICE)
            N = c.shape[1] if w.order == 2 else (c.shape[1] - 1) // 2
            out.append(_propagate(dev(w.H0), dev(w.Hk), c, w.h, w.order, N).cpu().numpy().ravel())
        return np.concatenate(out)
    H0, Hk, c = dev(s["H0"]), dev(s["Hk"]), s["samples"]
    if case["kind"] == "propagate":
        return _propagate(H0, Hk, c, h, order, n)
    if case["kind"] == "slices":
        keep = torch.empty((n, d, d), dtype=torch.complex128, device=DEVICE)
        return {"U": _propagate(H0, Hk, c, h, order, n, keep), "slices": keep}
    if case["kind"] == "gradient":
        c = c.clone().requires_grad_(True)
        U = _propagate(H0, Hk, c, h, order, n)
        torch.sum((torch.conj(s["W"]) * U).real).backward()
        return {"grad": c.grad, "U": U.detach()}
    E = _expm1(_exponents(H0, Hk, c, h, order, 0, n))
    P = _scan(E)
    if order == 5:
        P = P[1::2]
    x0 = s["x0"]
    return torch.cat([x0[None], x0 + torch.matmul(P, x0.expand(P.shape[0], -1, -1).contiguous())])
