"""The work that programs have this library do, as cases that can be timed
and compared: single steps of 2D meshes from the smallest convergence grid to
the grid of the paper's performance runs, adaptive cycles with the refinement
indicator and the regrid, gradient rollouts, batches of scenarios, 3D steps
and finite-volume steps.

``listed()`` names the cases, ``draw()`` gives others of the same ranges,
``prepare()`` makes what a program holds before the call, ``run()`` is one
pass through the public entry points, ``work()`` counts what a pass cannot do
without and ``exact()`` computes a pass's outputs again with plain torch in
64 bits.  All states are built here, from closed forms and the seed alone.
"""
import math
import random

import numpy as np
import torch

from paper_1905_05524_amd import adg
from paper_1905_05524_amd.autodiff import theta_rollout

PERIODIC, WALL = 0, 1
# air with gravity (bubble flows) and the gas of the convergence runs
AIR = dict(gamma=1.4, Pr=0.71, R=287.0, cp=1005.0, p0=1.0e5, theta_bg=300.0, g=9.81, gravity=1, mms=0)
GAS = dict(gamma=1.4, Pr=0.7, R=0.4, cp=1.4, p0=1.0, theta_bg=1.0, g=0.0, gravity=0, mms=0)
BOX = 1000.0                       # edge of the bubble flows' domain, metres
CHUNK = 1 << 16                    # cells per chunk of the plain computation


def listed():
    return [
        # the convergence study's grid: three short launches, all latency
        dict(name="wave9_N2", kind="step", flow="wave", nx=9, nz=9, N=2),
        # the gradient workload's grid stepped forward: fewer cells than SIMDs
        dict(name="bubble27_N6", kind="step", flow="air", nx=27, nz=27, N=6),
        # a middle order on an odd grid
        dict(name="bubble65x47_N4", kind="step", flow="air", nx=65, nz=47, N=4),
        # the benchmark step
        dict(name="bubble81_N6", kind="step", flow="air", nx=81, nz=81, N=6),
        # the grid of the paper's performance runs (104 M unknowns)
        dict(name="colliding729_N6", kind="step", flow="air", nx=729, nz=729, N=6),
        # an adaptive run between two regrids: ten steps with 1:3 faces, the
        # indicator with its flags, the regrid
        dict(name="adaptive27_N6", kind="amr", nx=27, N=6, steps=10),
        # gradient of a loss with the iterates kept in device memory
        dict(name="gradient27_N6_kept", kind="gradient", nx=27, nz=27, N=6, steps=5, keep=True),
        # the same with every step's predictor recomputed, at a lower order
        dict(name="gradient41x23_N4", kind="gradient", nx=41, nz=23, N=4, steps=3, keep=False),
        # an ensemble of 64 bubbles, grids 9..81, orders 3..6, one graph replay
        dict(name="batch64", kind="batch", count=64, k_lo=9, k_hi=81),
        # the 3D bubble at the paper's order
        dict(name="bubble3d_25_N3", kind="step3", flow="air", nx=25, ny=25, nz=25, N=3),
        # a 3D periodic flow at another order, odd sizes
        dict(name="vortex3d_13_N4", kind="step3", flow="gas", nx=13, ny=11, nz=12, N=4),
        # the finite-volume run of the colliding bubbles (7^2 patches of 90^2)
        dict(name="volumes630", kind="fv", nx=630, nz=630),
    ]


def draw(rng: random.Random):
    """One more case: kinds as often as they are listed, sizes log-uniform."""
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    kind = rng.choice(["step"] * 5 + ["amr", "gradient", "gradient", "batch", "step3", "step3", "fv"])
    if kind == "step":
        flow = rng.choice(["air", "air", "air", "wave"])
        return dict(kind=kind, flow=flow, nx=size(3, 260), nz=size(3, 260), N=rng.randint(1, 7))
    if kind == "amr":
        return dict(kind=kind, nx=rng.choice([9, 12, 15, 18, 21, 24, 27, 31]), N=rng.randint(2, 6),
                    steps=rng.randint(2, 10))
    if kind == "gradient":
        return dict(kind=kind, nx=size(5, 45), nz=size(5, 45), N=rng.randint(2, 6), steps=rng.randint(1, 5),
                    keep=rng.random() < 0.5)
    if kind == "batch":
        lo = rng.randint(5, 20)
        return dict(kind=kind, count=size(3, 64), k_lo=lo, k_hi=rng.randint(lo + 5, 81))
    if kind == "step3":
        N = rng.randint(1, 5)
        top = (40, 32, 27, 17, 14)[N - 1]
        return dict(kind=kind, flow=rng.choice(["air", "gas"]), nx=size(3, top), ny=size(3, top), nz=size(3, top), N=N)
    return dict(kind=kind, nx=size(30, 1600), nz=size(30, 1600))


# ------------------------------------------------------------------- inputs
def _device():
    return torch.device("cuda") if torch.cuda.is_available() else torch.device("cpu")


def _tensor(a):
    return torch.as_tensor(np.asarray(a), dtype=torch.float64, device=_device())


def _physics(case, seed):
    """Parameters of the run, as the library takes them."""
    kind, rng = case["kind"], np.random.default_rng([seed, 1])
    if kind == "fv":
        return dict(AIR, N=0, picard_iters=0, mu=0.0, cfl=0.9)
    if case.get("flow") == "wave":
        # advected density wave with its manufactured energy source
        return dict(GAS, N=case["N"], picard_iters=0, mu=0.01, cfl=0.5, mms=1, mms_amp=float(rng.uniform(0.05, 0.15)),
                    mms_u=float(rng.uniform(0.3, 0.6)), mms_w=float(rng.uniform(0.3, 0.6)),
                    mms_kx=18 * math.pi / case["nx"], mms_kz=18 * math.pi / case["nz"], mms_p=1.0)
    if case.get("flow") == "gas":
        return dict(GAS, N=case["N"], picard_iters=0, mu=0.01, cfl=0.4)
    return dict(AIR, N=case["N"], picard_iters=0, mu=0.005 if kind == "step3" else 1e-3, cfl=0.4)


def _refined(case, seed):
    """Coarse cells of the adaptive run that start refined: a disc around the
    bubble (the same number of cells for every seed)."""
    rng = np.random.default_rng([seed, 2])
    n = case["nx"]
    xc, zc = n // 2 + rng.integers(-n // 9, n // 9 + 1), n // 2 + rng.integers(-n // 6, 1)
    return {(i, j) for j in range(n) for i in range(n) if (i - xc) ** 2 + (j - zc) ** 2 <= (0.25 * n) ** 2}


def _mesh(case, seed):
    """The mesh as the library takes it; the box's edge is the longer side."""
    kind = case["kind"]
    if kind == "step3":
        gas = case["flow"] == "gas"
        h = (2 * math.pi if gas else BOX) / max(case["nx"], case["ny"], case["nz"])
        return dict(nx=case["nx"], ny=case["ny"], nz=case["nz"], h=h, bc=[PERIODIC if gas else WALL] * 6)
    nx, nz = case["nx"], case.get("nz", case["nx"])
    wave = case.get("flow") == "wave"
    h = 1.0 / 9.0 if wave else BOX / max(nx, nz)     # the wave: one period across the domain
    m = dict(nx=nx, nz=nz, max_level=0, x0=0.0, z0=0.0, Lx=h * nx, Lz=h * nz, bc=[PERIODIC if wave else WALL] * 4)
    if kind == "amr":
        fine = _refined(case, seed)
        leaves = [(0, i, j) for j in range(nz) for i in range(nx) if (i, j) not in fine]
        leaves += [(1, 3 * i + a, 3 * j + b) for i, j in sorted(fine, key=lambda c: (c[1], c[0])) for b in range(3)
                   for a in range(3)]
        m.update(max_level=1, leaves=leaves)
    return m


def _cells(mesh):
    """Corner of every cell per direction, in cell order, and the cell sizes."""
    if "h" in mesh:
        i = np.arange(mesh["nx"] * mesh["ny"] * mesh["nz"])
        idx = (i % mesh["nx"], (i // mesh["nx"]) % mesh["ny"], i // (mesh["nx"] * mesh["ny"]))
        return [_tensor(k * mesh["h"]) for k in idx], _tensor(np.full(i.shape, mesh["h"]))
    hc = mesh["Lx"] / mesh["nx"]
    if "leaves" in mesh:
        lv = np.asarray(mesh["leaves"])
        h = hc / 3.0 ** lv[:, 0]
        return [_tensor(lv[:, 1] * h), _tensor(lv[:, 2] * h)], _tensor(h)
    i = np.arange(mesh["nx"] * mesh["nz"])
    return [_tensor((i % mesh["nx"]) * hc), _tensor((i // mesh["nx"]) * hc)], _tensor(np.full(i.shape, hc))


def _nodes(mesh, xi):
    """Coordinates of all nodes, [C, n, ..., n] per direction (last axis x)."""
    corner, h = _cells(mesh)
    d, n = len(corner), len(xi)
    out = []
    for a in range(d):
        shape = [1] * d
        shape[d - 1 - a] = n
        c = corner[a].reshape(-1, *[1] * d) + h.reshape(-1, *[1] * d) * xi.reshape(1, *shape)
        out.append(c.expand(-1, *[n] * d))
    return out


def _background(ph, z):
    """Density and pressure of the resting atmosphere of constant potential temperature."""
    ex = 1.0 - ph["g"] / (ph["cp"] * ph["theta_bg"]) * z
    p = ph["p0"] * ex ** (ph["cp"] / ph["R"])
    return p / (ph["R"] * ph["theta_bg"] * ex), p


def _bubbles(rng, pos):
    """Potential-temperature perturbation: a warm cosine bubble and a cold Gaussian one."""
    d = len(pos)
    th = torch.zeros_like(pos[0])
    for amp, size in ((rng.uniform(0.3, 0.7), rng.uniform(200.0, 300.0)), (-rng.uniform(0.1, 0.2), rng.uniform(40.0, 80.0))):
        c = rng.uniform(350.0, 650.0, d)
        r = torch.sqrt(sum((pos[a] - c[a]) ** 2 for a in range(d)))
        if amp > 0:
            th = th + torch.where(r <= size, 0.5 * amp * (1.0 + torch.cos(math.pi * r / size)), torch.zeros_like(r))
        else:
            th = th + amp * torch.exp(-(r / size) ** 2)
    return th


def _state(ph, mesh, flow, pos, seed):
    """Conserved state at the given points: [C, d+2, ...]."""
    rng = np.random.default_rng([seed, 3])
    d, gm1 = len(pos), ph["gamma"] - 1.0
    edges = [mesh["h"] * mesh[k] for k in ("nx", "ny", "nz")] if d == 3 else [mesh["Lx"], mesh["Lz"]]
    s = [2 * math.pi * p / e for p, e in zip(pos, edges)]
    if flow == "wave":
        rho = 1.0 + ph["mms_amp"] * torch.sin(ph["mms_kx"] * pos[0]) * torch.sin(ph["mms_kz"] * pos[1])
        vel = [torch.full_like(rho, ph["mms_u"]), torch.full_like(rho, ph["mms_w"])]
        E = ph["mms_p"] / gm1 + 0.5 * rho * sum(v * v for v in vel)
    elif flow == "gas":
        # vortices of the ABC kind on a smoothly varying gas
        a, b, c = rng.uniform(0.3, 1.0, 3)
        x, y, z = s
        rho = 1.0 + 0.1 * torch.sin(x + rng.uniform(0, 6)) * torch.cos(y)
        vel = [a * torch.sin(z) + c * torch.cos(y), b * torch.sin(x) + a * torch.cos(z), c * torch.sin(y) + b * torch.cos(x)]
        E = (100.0 / ph["gamma"]) / gm1 + 0.5 * rho * sum(v * v for v in vel)
    else:
        rb, pb = _background(ph, pos[-1])
        rho = rb * ph["theta_bg"] / (ph["theta_bg"] + _bubbles(rng, pos))
        # a developed circulation of a few metres per second
        amp, phase = rng.uniform(0.5, 2.0, d), rng.uniform(0, 6, d)
        vel = [amp[a] * torch.sin(s[a] / 2) ** 2 * torch.sin(s[a - 1] + phase[a]) for a in range(d)]
        E = pb / gm1 + 0.5 * rho * sum(v * v for v in vel) + rho * ph["g"] * pos[-1]
    return torch.stack([rho] + [rho * v for v in vel] + [E], dim=1).contiguous()


def _scenarios(case, seed):
    """Grid size and order of the batch's scenarios; the sizes come from the
    case, so that every seed asks for the same work."""
    rng = np.random.default_rng([case["count"], case["k_lo"], case["k_hi"]])
    return [dict(kind="step", flow="air", nx=int(rng.integers(case["k_lo"], case["k_hi"] + 1)), N=int(rng.integers(3, 7)))
            for _ in range(case["count"])]


def _centres(mesh):
    h = mesh["Lx"] / mesh["nx"]
    i = np.arange(mesh["nx"] * mesh["nz"])
    return [_tensor((i % mesh["nx"] + 0.5) * h), _tensor((i // mesh["nx"] + 0.5) * h)], h


def _perturbation(pos, seed):
    """Control of the gradient: bubbles on a smooth large-scale field."""
    rng = np.random.default_rng([seed, 4])
    th = _bubbles(rng, pos)
    for k in (1, 2):
        th = th + rng.uniform(0.02, 0.1) * torch.sin(2 * math.pi * k * pos[0] / BOX + rng.uniform(0, 6)) * \
            torch.cos(2 * math.pi * k * pos[1] / BOX + rng.uniform(0, 6))
    return th


def prepare(case, seed):
    ph, kind = _physics(case, seed) if case["kind"] != "batch" else None, case["kind"]
    if kind == "batch":
        sc = _scenarios(case, seed)
        works = [dict(phys=_physics(c, seed), mesh=_mesh(c, seed)) for c in sc]
        b = adg.Batch(works)
        for s, (c, w) in enumerate(zip(sc, works)):
            b.state(s).copy_(_state(w["phys"], w["mesh"], "air", _nodes(w["mesh"], _basis(c["N"])["xi"]), seed * 64 + s))
        b.compute_dt()
        return dict(kind=kind, batch=b, stream=torch.cuda.Stream())
    mesh = _mesh(case, seed)
    if kind == "fv":
        m = adg.FV(ph, mesh)
        m.set_state(_state(ph, mesh, "air", _centres(mesh)[0], seed))
        m.compute_dt()
        return dict(kind=kind, mesh=m)
    pos = _nodes(mesh, _basis(case["N"])["xi"])
    if kind == "gradient":
        m = adg.Mesh(ph, mesh, fixed_dt=True)
        th = _perturbation(pos, seed).contiguous().requires_grad_(True)
        m.ic_theta(th.detach())
        m.compute_dt()
        return dict(kind=kind, mesh=m, theta=th, dt=m.dt, steps=case["steps"], keep=case["keep"])
    m = (adg.Mesh3 if kind == "step3" else adg.Mesh)(ph, mesh)
    m.set_state(_state(ph, mesh, case.get("flow", "air"), pos, seed))
    m.compute_dt()
    return dict(kind=kind, mesh=m, steps=case.get("steps", 1))


def run(state):
    kind, m = state["kind"], state.get("mesh")
    if kind == "batch":
        b, s = state["batch"], state["stream"]
        # the batch's own stream (a captured step needs one) follows and is followed by the program's
        s.wait_stream(torch.cuda.current_stream())
        b.step_graph(s)
        torch.cuda.current_stream().wait_stream(s)
        return dict(Q=b.Q, clock=b.clock)
    if kind == "gradient":
        th = state["theta"]
        loss = theta_rollout(th, m, state["steps"], state["dt"], keep=state["keep"])
        (grad,) = torch.autograd.grad(loss, th)
        return dict(loss=loss.detach(), grad=grad, Q=m.Q)
    if kind == "amr":
        for _ in range(state["steps"]):
            m.step()
        tv = torch.zeros(m.C, dtype=torch.float64, device=m.device)
        flags = torch.zeros(m.C, dtype=torch.int8, device=m.device)
        stats = torch.zeros(3, dtype=torch.float64, device=m.device)
        m.tv_indicator(adg.ADG_VAR_THETA, 0.0, -0.4, tv, flags, stats)
        Q = m.Q
        m.regrid(flags)      # the next pass steps the new mesh
        return dict(Q=Q, clock=m.clock, tv=tv, flags=flags, stats=stats)
    m.step()
    return dict(Q=m.Q, clock=m.clock)


def work(case):
    """Bytes: inputs read and outputs written once.  Operations: the dense
    count of the scheme's definition (products and sums, one each)."""
    kind = case["kind"]
    if kind == "fv":
        C = case["nx"] * case["nz"]
        # per cell: 8 limited slopes, 4 + 4 flux evaluations, 2 face fluxes, the update
        return dict(bytes=64.0 * C, flops=500.0 * C)
    if kind == "batch":
        parts = [work(dict(c, nz=c["nx"])) for c in _scenarios(case, 0)]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    N, n = case["N"], case["N"] + 1
    d = 3 if kind == "step3" else 2
    v, nodes, flux = d + 2, n ** d, (99, 180)[d - 2]
    C = case["nx"] * case.get("ny", 1) * case.get("nz", case["nx"])
    if kind == "amr":
        C += 8 * 0.2 * C                      # about a fifth of the coarse cells refined
    # n sweeps (the first with one residual for all levels) and the averages
    passes = 1 + (n - 1) * n
    contraction = 2 * d * v * n * nodes
    flops = C * (passes * (2 * contraction + (flux + 18) * nodes) + n * 2 * v * n * n * nodes + n * (contraction + (flux + 36) * nodes)
                 + contraction)
    bytes_ = 16.0 * C * v * nodes
    if kind == "amr":
        return dict(bytes=case["steps"] * bytes_, flops=case["steps"] * flops)
    if kind == "gradient":
        # the reverse sweep: three contractions per level and the flux's reverse
        back = C * n * (n * (3 * contraction + 270 * nodes) + 2 * v * n * n * nodes / n + 2 * contraction + 270 * nodes)
        again = 0 if case["keep"] else flops
        return dict(bytes=16.0 * C * nodes + case["steps"] * 2 * bytes_, flops=case["steps"] * (flops + back + again))
    return dict(bytes=bytes_, flops=flops)


# ------------------------------------------------- the same in plain torch
_BASES = {}


def _basis(N):
    """Gauss-Legendre nodes and weights on [0, 1], derivative matrix, values
    at the ends, time matrix, and the tables of the 1:3 faces."""
    if (N, str(_device())) not in _BASES:
        n = N + 1
        x, w = np.polynomial.legendre.leggauss(n)
        x, w = 0.5 * (x.astype(np.longdouble) + 1), 0.5 * w.astype(np.longdouble)
        lam = np.array([1 / np.prod([x[i] - x[j] for j in range(n) if j != i]) for i in range(n)])

        def phi(m, t):
            return np.prod([(t - x[j]) / (x[m] - x[j]) for j in range(n) if j != m])

        D = np.zeros((n, n), np.longdouble)
        for i in range(n):
            for j in range(n):
                if i != j:
                    D[i, j] = lam[j] / lam[i] / (x[i] - x[j])
            D[i, i] = -D[i].sum()
        e0, e1 = (np.array([phi(m, np.longdouble(t)) for m in range(n)]) for t in (0, 1))
        K = np.outer(e1, e1) - w[None, :] * D.T
        # P = K^-1 diag(w), the inverse refined once in long double
        inv = np.linalg.inv(K.astype(np.float64)).astype(np.longdouble)
        inv = inv @ (2 * np.eye(n) - K @ inv)
        sub = np.array([[[phi(m, (k + x[q]) / 3) for m in range(n)] for q in range(n)] for k in range(3)])
        back = np.einsum("q,kqm,m->kmq", w / 3, sub, 1 / w)
        t = dict(xi=x, w=w, D=D, e0=e0, e1=e1, P=inv * w[None, :], Dw=w[None, :] * D.T / w[:, None], sub=sub, back=back)
        _BASES[(N, str(_device()))] = {k: _tensor(v.astype(np.float64)) for k, v in t.items()}
    return _BASES[(N, str(_device()))]


def _along(M, q, axis):
    """Contraction of q with the matrix M along one axis."""
    return torch.movedim(torch.matmul(torch.movedim(q, axis, -1), M.T), -1, axis)


def _pressure(ph, q, z):
    kin = sum(q[:, 1 + a] ** 2 for a in range(q.shape[1] - 2)) / (2 * q[:, 0])
    return (ph["gamma"] - 1.0) * (q[:, -1] - kin - q[:, 0] * ((ph["g"] if ph["gravity"] else 0.0) * z))


def _flux(ph, q, grad, z):
    """Fluxes along every direction and the gravity source of the vertical
    momentum, from the state and its gradients (lists over directions)."""
    d = len(grad)
    g, gm1, R = (ph["g"] if ph["gravity"] else 0.0), ph["gamma"] - 1.0, ph["R"]
    mu, kappa = ph["mu"], ph["mu"] * ph["cp"] / ph["Pr"]
    rho, E = q[:, 0], q[:, -1]
    u = [q[:, 1 + a] / rho for a in range(d)]
    p = _pressure(ph, q, z)
    rb, pb = _background(ph, z) if ph["gravity"] else (0.0, 0.0)
    du = [[(grad[b][:, 1 + a] - u[a] * grad[b][:, 0]) / rho for b in range(d)] for a in range(d)]
    T = p / (rho * R)
    dT = []
    for b in range(d):
        dp = gm1 * (grad[b][:, -1] - (0.5 * sum(v * v for v in u) + g * z) * grad[b][:, 0]
                    - rho * sum(u[a] * du[a][b] for a in range(d)) - (rho * g if b == d - 1 else 0.0))
        dT.append((dp - R * T * grad[b][:, 0]) / (rho * R))
    div = sum(du[a][a] for a in range(d))
    F = []
    for b in range(d):
        sig = [mu * ((2.0 / 3.0 * div if a == b else 0.0) - du[a][b] - du[b][a]) for a in range(d)]
        mom = [q[:, 1 + a] * u[b] + sig[a] + (p - pb if a == b else 0.0) for a in range(d)]
        en = u[b] * (E + p) + sum(u[a] * sig[a] for a in range(d)) - kappa * dT[b]
        F.append(torch.stack([q[:, 1 + b]] + mom + [en], dim=1))
    return F, -g * (rho - rb)


def _wave_source(ph, x, z, t):
    """-kappa Laplace(T) of the advected density wave at constant pressure."""
    kx, kz, A = ph["mms_kx"], ph["mms_kz"], ph["mms_amp"]
    X, Z = kx * (x - ph["mms_u"] * t), kz * (z - ph["mms_w"] * t)
    s = torch.sin(X) * torch.sin(Z)
    rho = 1.0 + A * s
    rx, rz = A * kx * torch.cos(X) * torch.sin(Z), A * kz * torch.sin(X) * torch.cos(Z)
    lap = (A * (kx * kx + kz * kz) * s / rho ** 2 + 2.0 * (rx * rx + rz * rz) / rho ** 3) * ph["mms_p"] / ph["R"]
    return -ph["mu"] * ph["cp"] / ph["Pr"] * lap


def _predict(ph, B, Q, h, pos, t, dt):
    """Volume update and face data (state and normal flux at both ends of
    every direction) of the cells given."""
    C, d, n = Q.shape[0], Q.ndim - 2, Q.shape[-1]
    hb = h.reshape(-1, *[1] * (d + 1))

    def rate(q, b, flux_only):
        grad = [_along(B["D"], q, -1 - a) / hb for a in range(d)]
        F, Sw = _flux(ph, q, grad, pos[-1])
        S = torch.zeros_like(q)
        S[:, d] = Sw
        if ph["mms"]:
            S[:, -1] = _wave_source(ph, pos[0], pos[1], t + float(B["xi"][b]) * dt)
        return (F, S) if flux_only else S - sum(_along(B["D"], F[a], -1 - a) for a in range(d)) / hb

    X = [Q] * n
    for _ in range(n):
        R = [rate(X[b], b, False) for b in range(n)]
        X = [Q + dt * sum(B["P"][a, b] * R[b] for b in range(n)) for a in range(n)]
    Qb, Sb, Fb = 0.0, 0.0, [0.0] * d
    for b in range(n):
        F, S = rate(X[b], b, True)
        w = B["w"][b]
        Qb, Sb, Fb = Qb + w * X[b], Sb + w * S, [Fb[a] + w * F[a] for a in range(d)]
    Qs = Q + dt * (sum(_along(B["Dw"], Fb[a], -1 - a) for a in range(d)) / hb + Sb)
    faces = [[tuple(torch.tensordot(v, e, dims=([v.ndim - 1 - a], [0])) for v in (Qb, Fb[a]))
              for e in (B["e0"], B["e1"])] for a in range(d)]
    return Qs, faces


def _speeds(ph, q, a, z):
    c = torch.sqrt(ph["gamma"] * _pressure(ph, q, z) / q[:, 0])
    lv = max(4.0 * ph["mu"] / 3.0, ph["gamma"] * ph["mu"] / ph["Pr"]) / q[:, 0]
    return torch.abs(q[:, 1 + a] / q[:, 0]) + c, lv


def _face_flux(ph, L, R, a, z, h, N):
    """Rusanov flux with one speed per face; L, R: (state, normal flux)."""
    top = []
    for k in (0, 1):
        v = torch.cat([_speeds(ph, s[0], a, z)[k].flatten(1) for s in (L, R)], dim=1)
        top.append(v.max(dim=1).values)
    eta = (2 * N + 1) / (h * math.sqrt(math.pi / 2))
    s = (top[0] + 2 * eta * top[1]).reshape(-1, *[1] * (L[0].ndim - 1))
    return 0.5 * (L[1] + R[1]) - 0.5 * s * (R[0] - L[0])


def _ghost(ph, q, F, a, z):
    """No-slip wall: mirrored velocity in the background state, mirrored mass
    and energy flux with the background's heat flux through horizontal walls."""
    d = q.shape[1] - 2
    rb, pb = _background(ph, z) if ph["gravity"] else (q[:, 0], _pressure(ph, q, z))
    vel = [q[:, 1 + k] / q[:, 0] for k in range(d)]
    g = ph["g"] if ph["gravity"] else 0.0
    E = pb / (ph["gamma"] - 1.0) + 0.5 * rb * sum(v * v for v in vel) + rb * g * z
    heat = ph["mu"] * ph["cp"] / ph["Pr"] * g / ph["cp"] if a == d - 1 else 0.0
    ghost = torch.stack([rb + 0.0 * q[:, 0]] + [-(rb * v) for v in vel] + [E], dim=1)
    flux = torch.cat([-F[:, :1], F[:, 1:-1], 2.0 * heat - F[:, -1:]], dim=1)
    return ghost, flux


def _links(mesh):
    """Per direction: (low cell, high cell) of conforming faces, wall faces
    (cell, side), and 1:3 faces (coarse cell, its side, fine cell, which third)."""
    if "leaves" not in mesh:
        dims = [mesh["nx"]] + ([mesh["ny"]] if "ny" in mesh else []) + [mesh["nz"]]
        idx = np.arange(int(np.prod(dims))).reshape(dims[::-1])
        out = []
        for a in range(len(dims)):
            ax = idx.ndim - 1 - a
            lo, hi = idx.take(range(dims[a] - 1), ax).ravel(), idx.take(range(1, dims[a]), ax).ravel()
            first, last = idx.take(0, ax).ravel(), idx.take(dims[a] - 1, ax).ravel()
            if mesh["bc"][2 * a] == PERIODIC:
                out.append((np.concatenate([lo, last]), np.concatenate([hi, first]), [], []))
            else:
                out.append((lo, hi, [(first, 0), (last, 1)], []))
        return out
    where = {tuple(c): k for k, c in enumerate(mesh["leaves"])}
    out = []
    for a in range(2):
        lo, hi, walls, hang = [], [], ([], []), []
        for (l, i, j), c in where.items():
            for side in (0, 1):
                q = [i, j]
                q[a] += 2 * side - 1
                if q[a] < 0 or q[a] >= (mesh["nx"], mesh["nz"])[a] * 3 ** l:
                    walls[side].append(c)
                elif (l, *q) in where:
                    if side:
                        lo.append(c)
                        hi.append(where[(l, *q)])
                elif (l - 1, q[0] // 3, q[1] // 3) in where:
                    hang.append((where[(l - 1, q[0] // 3, q[1] // 3)], 1 - side, c, q[1 - a] % 3))
        out.append((np.array(lo), np.array(hi), [(np.array(walls[s]), s) for s in (0, 1)], hang))
    return out


def _step(ph, mesh, Q, t, dt, links=None):
    """One step of the whole mesh; Q [C, d+2, n, ...]."""
    N, d = ph["N"], Q.ndim - 2
    B, n, C = _basis(N), ph["N"] + 1, Q.shape[0]
    corner, h = _cells(mesh)
    pos = _nodes(mesh, B["xi"])
    parts = [_predict(ph, B, Q[k:k + CHUNK], h[k:k + CHUNK], [p[k:k + CHUNK] for p in pos], t, dt)
             for k in range(0, C, CHUNK)]
    Qs = torch.cat([p[0] for p in parts])
    lift = 0.0
    for a, (lo, hi, walls, hang) in enumerate(links or _links(mesh)):
        data = [tuple(torch.cat([p[1][a][s][k] for p in parts]) for k in (0, 1)) for s in (0, 1)]
        zf = [corner[-1] + (h if s else 0.0) for s in (0, 1)]

        def height(cells, side, a=a, zf=zf):
            """z of the face's nodes, [faces, n, ...]"""
            if a == d - 1:
                return zf[side][cells].reshape(-1, *[1] * (d - 1))
            z = corner[-1][cells].reshape(-1, 1) + h[cells].reshape(-1, 1) * B["xi"]
            return z.reshape(-1, n, *[1] * (d - 2))

        where, G = ([], []), ([], [])       # per side: cells and their face fluxes
        if len(lo):
            lo, hi = (torch.as_tensor(v, device=Q.device) for v in (lo, hi))
            g = _face_flux(ph, [v[lo] for v in data[1]], [v[hi] for v in data[0]], a, height(lo, 1), h[lo], N)
            for side, cells in ((1, lo), (0, hi)):
                where[side].append(cells)
                G[side].append(g)
        for cells, side in walls:
            if not len(cells):
                continue
            cells = torch.as_tensor(cells, device=Q.device)
            own, z = [v[cells] for v in data[side]], height(cells, side)
            out = _ghost(ph, own[0], own[1], a, z)
            where[side].append(cells)
            G[side].append(_face_flux(ph, *((own, out) if side else (out, own)), a, z, h[cells], N))
        for side in (0, 1):                 # 1:3 faces on the coarse cells' side `side`
            rows = [r for r in hang if r[1] == side]
            if not rows:
                continue
            co, fi, k = (torch.as_tensor([r[m] for r in rows], device=Q.device) for m in (0, 2, 3))
            coarse = [torch.einsum("fqm,fvm->fvq", B["sub"][k], v[co]) for v in data[side]]
            fine = [v[fi] for v in data[1 - side]]
            g = _face_flux(ph, *((coarse, fine) if side else (fine, coarse)), a, height(fi, 1 - side), h[fi], N)
            where[1 - side].append(fi)
            G[1 - side].append(g)
            cells, inv = torch.unique(co, return_inverse=True)
            sums = torch.zeros((len(cells),) + g.shape[1:], dtype=g.dtype, device=g.device)
            where[side].append(cells)
            G[side].append(sums.index_add(0, inv, torch.einsum("fmq,fvq->fvm", B["back"][k], g)))
        for side, e in ((0, B["e0"]), (1, B["e1"])):
            full = torch.zeros_like(data[0][0]).index_copy(0, torch.cat(where[side]), torch.cat(G[side]))
            shape = [1] * d
            shape[d - 1 - a] = n
            term = (e / B["w"]).reshape(shape) * full.unsqueeze(full.ndim - a)
            lift = lift + (term if side else -term)
    return Qs - dt / h.reshape(-1, *[1] * (d + 1)) * lift


def _courant(ph, mesh, Q):
    N, d = ph["N"], Q.ndim - 2
    h, z = _cells(mesh)[1], _nodes(mesh, _basis(N)["xi"])[-1]
    both = [_speeds(ph, Q, a, z) for a in range(d)]
    lam = torch.stack([b[0].flatten(1).max(dim=1).values for b in both]).max(dim=0).values
    lv = both[0][1].flatten(1).max(dim=1).values
    o = 2 * N + 1
    return float((ph["cfl"] * h / (d * o * (lam + 2 * lv * o / h))).min())


def _theta(ph, Q, z):
    p = _pressure(ph, Q, z)
    return p / (Q[:, 0] * ph["R"]) * (ph["p0"] / p) ** (ph["R"] / ph["cp"])


def _exact_step(case, seed):
    ph, mesh = _physics(case, seed), _mesh(case, seed)
    pos = _nodes(mesh, _basis(case["N"])["xi"])
    Q, links, t = _state(ph, mesh, case.get("flow", "air"), pos, seed), _links(mesh), 0.0
    dt = _courant(ph, mesh, Q)
    for _ in range(case.get("steps", 1)):
        Q = _step(ph, mesh, Q, t, dt, links)
        t, dt = t + dt, _courant(ph, mesh, Q)
    return ph, mesh, pos, Q, _tensor([t, dt, 0.0, case.get("steps", 1)])


def _exact_indicator(ph, mesh, pos, Q):
    B, h = _basis(ph["N"]), _cells(mesh)[1]
    th = _theta(ph, Q, pos[-1])
    tv = sum(torch.abs(_along(B["D"], th, -1 - a)) for a in range(2))
    tv = torch.einsum("cji,j,i->c", tv, B["w"], B["w"]) / h
    return tv, torch.stack([torch.tensor(float(len(tv)), dtype=tv.dtype, device=tv.device), tv.mean(), tv.std(unbiased=False)])


def _exact_gradient(case, seed):
    ph, mesh = _physics(case, seed), _mesh(case, seed)
    B, links = _basis(case["N"]), _links(mesh)
    pos, h = _nodes(mesh, B["xi"]), _cells(mesh)[1]
    th = _perturbation(pos, seed).requires_grad_(True)
    rb, pb = _background(ph, pos[-1])
    rho = rb * ph["theta_bg"] / (ph["theta_bg"] + th)
    start = torch.stack([rho, 0 * rho, 0 * rho, pb / (ph["gamma"] - 1.0) + rho * ph["g"] * pos[-1]], dim=1)
    Qs = [start.detach()]
    dt = _courant(ph, mesh, Qs[0])
    for k in range(case["steps"]):
        Qs.append(_step(ph, mesh, Qs[-1], k * dt, dt, links))
    end = Qs[-1].requires_grad_(True)
    dth = _theta(ph, end, pos[-1]) - ph["theta_bg"]
    loss = torch.sqrt((h ** 2 * torch.einsum("cji,j,i->c", dth ** 2, B["w"], B["w"])).sum())
    (lam,) = torch.autograd.grad(loss, end)
    for k in range(case["steps"] - 1, -1, -1):
        q = Qs[k].detach().requires_grad_(True)
        (lam,) = torch.autograd.grad(_step(ph, mesh, q, k * dt, dt, links), q, lam)
    (grad,) = torch.autograd.grad(start, th, lam)
    return dict(loss=loss.detach(), grad=grad, Q=end.detach())


def _exact_fv(case, seed):
    """MUSCL-Hancock with the van Albada limiter; arrays [4, nz, nx]."""
    ph, mesh = _physics(case, seed), _mesh(case, seed)
    pos, h = _centres(mesh)
    nx, nz, g, gam = mesh["nx"], mesh["nz"], ph["g"], ph["gamma"]
    Q = _state(ph, mesh, "air", pos, seed).T.reshape(4, nz, nx).contiguous()
    z = pos[1].reshape(nz, nx)[:, :1]

    def press(q, zz):
        return (gam - 1.0) * (q[3] - 0.5 * (q[1] ** 2 + q[2] ** 2) / q[0] - q[0] * g * zz)

    def speed(q, zz):
        return torch.maximum(torch.abs(q[1]), torch.abs(q[2])) / q[0] + torch.sqrt(gam * press(q, zz) / q[0])

    def flux(q, zz, a):
        p, un = press(q, zz), q[1 + a] / q[0]
        pm = p - _background(ph, zz)[1]
        return torch.stack([q[1 + a], q[1] * un + (pm if a == 0 else 0.0), q[2] * un + (pm if a == 1 else 0.0),
                            un * (q[3] + p)])

    def ghost(q, zz):
        rb, pb = _background(ph, zz)
        rb, u, w = rb + 0.0 * q[0], q[1] / q[0], q[2] / q[0]
        return torch.stack([rb, -rb * u, -rb * w, pb / (gam - 1.0) + 0.5 * rb * (u * u + w * w) + rb * g * zz])

    def slope(q, lo, hi, ax):
        a, b = q - lo, hi - q
        s = a * b * (a + b) / torch.where(a * b > 0, a * a + b * b, torch.ones_like(a))
        return torch.where(a * b > 0, s, torch.zeros_like(s))

    def grown(q, ax, first, last):
        return torch.cat([first, q, last], dim=ax)

    dt = float((ph["cfl"] * h / (2 * speed(Q, z))).min())
    face, inc = [], 0.0
    zs = [z - 0.5 * h, z + 0.5 * h]
    S = torch.zeros_like(Q)
    S[2] = -g * (Q[0] - _background(ph, z)[0])
    for a, ax in ((0, 2), (1, 1)):
        f, l = Q.narrow(ax, 0, 1), Q.narrow(ax, Q.shape[ax] - 1, 1)
        zf, zl = (z, z) if a == 0 else (z[:1] - h, z[-1:] + h)
        G = grown(Q, ax, ghost(f, zf), ghost(l, zl))
        s = slope(Q, G.narrow(ax, 0, Q.shape[ax]), G.narrow(ax, 2, Q.shape[ax]), ax)
        lo, hi = Q - 0.5 * s, Q + 0.5 * s
        inc = inc + flux(lo, z if a == 0 else zs[0], a) - flux(hi, z if a == 0 else zs[1], a)
        face.append((lo, hi))
    inc = 0.5 * dt / h * inc + 0.5 * dt * S
    out = 0.0
    for a, ax in ((0, 2), (1, 1)):
        lo, hi = face[a][0] + inc, face[a][1] + inc
        cnt = Q.shape[ax]
        zf = z if a == 0 else torch.cat([zs[0], zs[1][-1:]])
        zb, ze = (z, z) if a == 0 else (zs[0][:1], zs[1][-1:])
        first, last = lo.narrow(ax, 0, 1), hi.narrow(ax, cnt - 1, 1)
        L, R = torch.cat([ghost(first, zb), hi], ax), torch.cat([lo, ghost(last, ze)], ax)
        mirror = torch.ones(4, 1, 1, dtype=Q.dtype, device=Q.device)
        mirror[0] = mirror[3] = -1.0
        FL = torch.cat([mirror * flux(first, zb, a), flux(hi, zf if a == 0 else zf[1:], a)], ax)
        FR = torch.cat([flux(lo, zf if a == 0 else zf[:-1], a), mirror * flux(last, ze, a)], ax)
        s = torch.maximum(*[torch.abs(v[1 + a] / v[0]) + torch.sqrt(gam * press(v, zf) / v[0]) for v in (L, R)])
        G = 0.5 * (FL + FR) - 0.5 * s * (R - L)
        out = out + G.narrow(ax, 1, cnt) - G.narrow(ax, 0, cnt)
    S[2] = -g * (Q[0] + inc[0] - _background(ph, z)[0])
    Q = Q - dt / h * out + dt * S
    new = float((ph["cfl"] * h / (2 * speed(Q, z))).min())
    return dict(Q=Q.reshape(4, -1).T.contiguous(), clock=_tensor([dt, new, 0.0, 1.0]))


def exact(case, seed):
    kind = case["kind"]
    if kind == "fv":
        return _exact_fv(case, seed)
    if kind == "gradient":
        return _exact_gradient(case, seed)
    if kind == "amr":
        ph, mesh, pos, Q, clock = _exact_step(case, seed)
        tv, stats = _exact_indicator(ph, mesh, pos, Q)
        # the flags are whole numbers
        return dict(Q=Q, clock=clock, tv=tv, flags=None, stats=stats)
    if kind == "batch":
        sc, Q, clocks = _scenarios(case, seed), [], []
        order = sorted(range(len(sc)), key=lambda s: sc[s]["N"])    # the state's layout: by order, then as given
        for s, c in enumerate(sc):
            ph, mesh = _physics(c, seed), _mesh(c, seed)
            q = _state(ph, mesh, "air", _nodes(mesh, _basis(c["N"])["xi"]), seed * 64 + s)
            dt = _courant(ph, mesh, q)
            q = _step(ph, mesh, q, 0.0, dt)
            Q.append(q.reshape(-1))
            clocks.append([dt, _courant(ph, mesh, q), 0.0, 1.0])
        return dict(Q=torch.cat([Q[s] for s in order]), clock=_tensor(clocks))
    _, _, _, Q, clock = _exact_step(case, seed)
    return dict(Q=Q, clock=clock)
