"""The predictors that pack several cells into a workgroup, on every path that
uses them: the parity cases, the iterate store and face data of a kept step,
the step adjoint, and the cell counts at which the default launch goes from one
kernel to another.  The kernels share the arithmetic of each value, so stores,
face data and states agree bit for bit with one cell per wavefront; against the
oracle the bars are those of the parity and adjoint tests (1e-11 of a step,
1e-12 of |J v| |w|)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_1905_05524_amd import adg
from paper_1905_05524_amd import inputs as I

import parity as P
import test_gpu_parity as T
from test_gpu_adjoint import dev

pytestmark = pytest.mark.gpu

SHAPES = [(1, 2), (2, 1), (4, 1), (0, 1), None]


def takes(N, shape):
    return shape is None or max(shape[0], 1) * (N + 1) ** 2 <= 64


def fixed_mesh(phys, mesh, shape):
    m = adg.Mesh(phys, mesh, fixed_dt=True)
    if shape is not None:
        m.set_launch(*shape)
    return m


def walls(N, nx, nz, iters=0):
    phys = dict(I.ATMO, N=N, picard_iters=iters, mu=5.0, mms=0, cfl=0.4)
    h = 1000.0 / max(nx, nz)
    mesh = dict(nx=nx, nz=nz, max_level=0, Lx=h * nx, Lz=h * nz, bc=[I.BC_WALL] * 4)
    Q = O.ic(phys, mesh, "bubbles", [I.cosine_bubble(a=400.0, xc=0.5 * h * nx, zc=0.4 * h * nz)])
    return phys, mesh, I.perturb(Q, seed=60 + N)


@pytest.mark.parametrize("kind,nx,N,shape", [(*c, s) for c in T.CASES for s in SHAPES[:3] if takes(c[2], s)])
def test_parity_cases(kind, nx, N, shape):
    w = T._case(kind, nx, N)
    Q = T._state(w, seed=500 + N)
    dt = 0.5 * O.dt(w["phys"], w["mesh"], Q)
    m = fixed_mesh(w["phys"], w["mesh"], shape)
    m.set_state(Q, t=0.2, dt=dt)
    m.step()
    P.assert_step(m.Q.cpu().numpy(), O.step(w["phys"], w["mesh"], Q, 0.2, dt), Q, what=f"{kind} N={N} {shape}")


def flow(name, N, nx, nz, iters):
    if name == "walls":
        return walls(N, nx, nz, iters)
    if name == "periodic":
        phys = dict(I.CFD, N=N, picard_iters=iters, mu=0.05, mms=0, cfl=0.5)
        mesh = dict(nx=nx, nz=nz, max_level=0, x0=0.0, z0=0.0, Lx=nx / 4.0, Lz=nz / 4.0, bc=[I.BC_PERIODIC] * 4)
        return phys, mesh, I.random_state_cfd(nx * nz, N, seed=80 + N)
    w = I.mms_small(N=N, nx=nx, mu=0.02) if name == "wave" else I.paper_mms(N, nx)
    w["phys"]["picard_iters"] = iters
    w["mesh"].update(nz=nz, Lz=w["mesh"]["Lx"] * nz / nx)
    return w["phys"], w["mesh"], O.ic(w["phys"], w["mesh"], "mms" if name == "wave" else "paper_mms", t0=0.3)


# cells not divisible by 16, 7, 4, 2 or 5, and 3
@pytest.mark.parametrize("N,nx,nz", [(1, 17, 1), (1, 5, 7), (2, 2, 4), (2, 5, 3), (3, 3, 1), (3, 3, 3), (4, 3, 1), (4, 11, 1),
                                     (5, 2, 2), (5, 5, 1), (6, 3, 1), (7, 3, 1)])
@pytest.mark.parametrize("name", ["walls", "periodic", "wave", "paper"])
def test_kept_steps_agree_bit_for_bit(N, nx, nz, name):
    """Also with steps of 20 times the CFL bound, whose iterates are mostly
    residual, so that its last bits show (in an ordinary step they rarely do):
    three sweeps of those stay finite."""
    phys, mesh, Q = flow(name, N, nx, nz, 3)
    bound = O.dt(phys, mesh, Q)

    def kept(shape, dt):
        m = fixed_mesh(phys, mesh, shape)
        m.set_state(Q, t=0.3, dt=dt)
        sb, fb = m.keep_bytes()
        # NaN where the step writes nothing, and behind the buffers
        store, fd = (torch.full((b // 8 + 64,), float("nan"), dtype=torch.float64, device="cuda") for b in (sb, fb))
        m.step_keep(store, fd)
        assert bool(torch.isnan(store[sb // 8:]).all()) and bool(torch.isnan(fd[fb // 8:]).all()), shape
        return store[:sb // 8], fd[:fb // 8], m.qstar().clone()

    for factor in (0.5, 20.0):
        ref = kept((1, 1), factor * bound)
        assert all(bool(torch.isfinite(a).all()) for a in ref), factor
        for shape in SHAPES:
            if takes(N, shape):
                assert all(torch.equal(a, b) for a, b in zip(kept(shape, factor * bound), ref)), (shape, factor)


def test_persistent_batch_agrees_bit_for_bit():
    ws = []
    for N, nx, nz in ((1, 5, 7), (2, 5, 3), (3, 3, 3), (4, 11, 1), (5, 5, 1), (6, 3, 2), (7, 3, 1)):
        phys, mesh, Q = flow("periodic", N, nx, nz, 3)
        ws.append((dict(phys=phys, mesh=mesh), Q, 20.0 * O.dt(phys, mesh, Q)))
    for mode, base in ((0, 0), (1, 0), (0, 1)):   # defaults; persistent; one cell per wavefront
        b = adg.Batch([w for w, _, _ in ws], fixed_dt=True)
        b.set_mode(mode)
        for g in range(b.n_groups if base else 0):
            b.set_launch(g, 1, 1)
        for s, (_, Q, dt) in enumerate(ws):
            b.state(s).copy_(dev(Q))
            b.clock[s, 1] = dt
        b.step()
        if (mode, base) == (0, 0):
            ref = b.Q.clone()
        assert torch.equal(b.Q, ref), (mode, base)


def adjoint_case(N, nx, nz, shape):
    """Checks <J v, w> = <v, J^T w> and returns J^T w."""
    phys, mesh, Q = walls(N, nx, nz)
    dt = 0.5 * O.dt(phys, mesh, Q)
    rng = np.random.default_rng(300 + N)
    scale = np.array([1e-4, 0.1, 0.1, 10.0])[None, :, None, None]
    v, w = rng.standard_normal(Q.shape) * scale, rng.standard_normal(Q.shape) / scale
    m = fixed_mesh(phys, mesh, shape)
    m.set_state(Q, t=0.3, dt=dt)
    lam = torch.empty_like(m.Q)
    m.step_adjoint(dev(Q), dev(w), lam)
    _, Jv = O.step_jvp(phys, mesh, Q, v, 0.3, dt)
    a, b = float(np.sum(Jv * w)), float(np.sum(v * lam.cpu().numpy()))
    assert abs(a - b) <= 1e-12 * np.linalg.norm(Jv) * np.linalg.norm(w), (a, b)
    store, fd = (torch.empty(k // 8, dtype=torch.float64, device="cuda") for k in m.keep_bytes())
    m.step_keep(store, fd)
    kept = torch.empty_like(lam)
    m.step_adjoint_kept(dev(Q), store, fd, dev(w), kept)
    assert torch.equal(kept, lam)
    return lam


@pytest.mark.parametrize("N,nx,nz", [(1, 17, 16), (2, 16, 17), (2, 3, 3), (3, 1, 259), (3, 3, 1), (4, 43, 6), (4, 3, 1),
                                     (5, 5, 1), (6, 3, 1)])
def test_step_adjoint_with_every_shape(N, nx, nz):
    ref = adjoint_case(N, nx, nz, (1, 1))
    for shape in SHAPES:
        if takes(N, shape):
            assert torch.equal(adjoint_case(N, nx, nz, shape), ref), shape


@pytest.mark.parametrize("N,nx,nz", [(1, 41, 25), (2, 37, 14), (3, 19, 27), (4, 23, 23)])
def test_step_adjoint_above_the_four_wavefront_range(N, nx, nz):
    """1,025, 518, 513 and 529 cells: the default is a packed predictor."""
    assert torch.equal(adjoint_case(N, nx, nz, None), adjoint_case(N, nx, nz, (1, 1)))


@pytest.mark.parametrize("N,C", [(1, 1024), (1, 1025), (2, 512), (2, 513), (3, 512), (3, 513), (4, 512), (4, 513), (4, 4096),
                                 (4, 4097), (5, 768), (5, 769), (5, 2048), (5, 2049), (6, 768), (6, 769), (6, 2048),
                                 (6, 2049), (7, 768), (7, 769)])
def test_both_sides_of_every_switch(N, C):
    w = I.bubble(C, N)
    w["mesh"].update(nx=C, nz=1, Lx=1000.0, Lz=1000.0 / C)
    Q = I.perturb(O.ic(w["phys"], w["mesh"], "bubbles", w["bubbles"]), seed=N)
    dt = 0.5 * O.dt(w["phys"], w["mesh"], Q)
    got = []
    for shape in (None, (1, 1)):
        m = fixed_mesh(w["phys"], w["mesh"], shape)
        m.set_state(Q, t=0.1, dt=dt)
        m.step()
        got.append(m.Q.clone())
    P.assert_step(got[0].cpu().numpy(), O.step(w["phys"], w["mesh"], Q, 0.1, dt), Q, what=f"N={N} C={C}")
    assert torch.equal(got[0], got[1])
