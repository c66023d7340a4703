"""The time-step candidates in the workspace and their minimum on both sides of
the cell count from which the minimum is taken in two stages (24,576): every
entry is the bound of its own cell (or workgroup of cells) and the clock holds
their minimum, bit for bit.  The bounds are some twenty roundings of 1.1e-16 on
a pressure without cancellation, one quarter of them under a square root: bar
1e-14, the bar of the other time-step tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_1905_05524_amd import adg
from paper_1905_05524_amd import inputs as I

pytestmark = pytest.mark.gpu

BAR = 1e-14


def bounds3(phys, h, Q):
    """CFL bound of every cell of a 3D state without gravity."""
    rho, m, E = Q[:, 0], Q[:, 1:4], Q[:, 4]
    p = (phys["gamma"] - 1.0) * (E - 0.5 * (m ** 2).sum(axis=1) / rho)
    lam = np.abs(m).max(axis=1) / rho + np.sqrt(phys["gamma"] * p / rho)
    lv = phys["mu"] * max(4.0 / 3.0, phys["gamma"] / phys["Pr"]) / rho
    o = 2.0 * phys["N"] + 1.0
    return phys["cfl"] * h / (3.0 * o * (lam.max(axis=(1, 2, 3)) + 2.0 * lv.max(axis=(1, 2, 3)) * o / h))


@pytest.mark.parametrize("N,nx,ny,nz", [(1, 32, 32, 24), (1, 24577, 1, 1), (1, 30, 29, 29), (2, 31, 28, 29)])
def test_candidates_of_a_3d_grid(N, nx, ny, nz):
    phys = dict(I.CFD, N=N, picard_iters=1, mu=0.01, mms=0, cfl=0.5)
    h = 1.0 / 32
    m = adg.Mesh3(phys, dict(nx=nx, ny=ny, nz=nz, h=h, bc=[I.BC_PERIODIC] * 6))
    m.set_state(I.random_state_cfd3(nx * ny * nz, N, seed=5), t=0.0)
    for call in ("compute_dt", "step"):
        getattr(m, call)()
        got = m.cell_dt().cpu().numpy()
        want = bounds3(phys, h, m.Q.cpu().numpy())
        assert np.max(np.abs(got - want) / want) <= BAR, call
        assert m.dt == got.min(), call


def test_bounds_of_many_finite_volume_workgroups():
    """24,580 workgroups of 256 cells."""
    nx, nz = 2560, 2458
    phys = dict(I.CFD, mu=0.0, mms=0, cfl=0.5)
    m = adg.FV(phys, dict(nx=nx, nz=nz, Lx=nx / 1024.0, Lz=nz / 1024.0, bc=[I.BC_PERIODIC] * 4))
    g = torch.Generator(device="cuda").manual_seed(9)
    u = torch.rand(m.Q.shape, generator=g, dtype=torch.float64, device="cuda")
    lo = torch.tensor([0.8, -0.3, -0.3, 2.2], dtype=torch.float64, device="cuda")
    hi = torch.tensor([1.2, 0.3, 0.3, 2.8], dtype=torch.float64, device="cuda")
    m.Q.copy_(lo + u * (hi - lo))
    off = (16 * 8 * m.C + 255) // 256 * 256
    off = (off + 8 * m.C + 255) // 256 * 256
    blocks = m.C // 256
    for calls in (("compute_dt",), ("predictor", "corrector")):
        for c in calls:
            getattr(m, c)()
        got = m.ws[off:off + 8 * blocks].view(torch.float64)
        rho, mx, mz, E = m.Q.T
        p = (phys["gamma"] - 1.0) * (E - 0.5 * (mx * mx + mz * mz) / rho)
        lam = torch.maximum(mx.abs(), mz.abs()) / rho + torch.sqrt(phys["gamma"] * p / rho)
        want = phys["cfl"] / 1024.0 / (2.0 * lam.view(blocks, 256).amax(dim=1))
        assert float(((got - want).abs() / want).max()) <= BAR, calls
        assert m.dt == float(got.min()), calls


def test_static_step_of_the_largest_mesh():
    """The largest strip of N = 1 whose sections (updates, face data,
    candidates, health flag) fit the 32 MiB of adg_step_static steps there as
    in its own workspace."""
    def sections(C):
        return sum((b * C + 255) // 256 * 256 for b in (128, 512, 8)) + 256
    C = (32 << 20) // 648
    while sections(C) > 32 << 20:
        C -= 1
    phys = dict(I.CFD, N=1, picard_iters=0, mu=0.01, mms=0, cfl=0.5)
    m = adg.Mesh(phys, dict(nx=C, nz=1, max_level=0, Lx=C / 64.0, Lz=1 / 64.0, bc=[I.BC_PERIODIC] * 4))
    m.set_state(I.random_state_cfd(C, 1, seed=3), t=0.0)
    m.compute_dt()
    Q, clock = m.Q.clone(), m.clock.clone()
    m.step_static(Q, clock)
    m.step()
    assert torch.equal(Q, m.Q) and torch.equal(clock, m.clock)


def test_minimum_across_a_regrid():
    """3,025 cells refined to 27,225 and merged again: the section for the two
    stages comes and goes with the workspace."""
    phys = dict(I.CFD, N=1, picard_iters=0, mu=0.01, mms=0, cfl=0.5)
    mesh = dict(nx=55, nz=55, max_level=1, x0=0.0, z0=0.0, Lx=1.0, Lz=1.0, bc=[I.BC_PERIODIC] * 4,
                leaves=I.uniform_leaves(55, 55))
    m = adg.Mesh(phys, mesh)
    m.set_state(I.random_state_cfd(55 * 55, 1, seed=8), t=0.0)
    for flag, cells in ((1, 27225), (-1, 3025)):
        assert m.regrid(np.full(m.C, flag, dtype=np.int8)) == cells
        m.Q[cells - 1, 3] *= 40.0
        m.compute_dt()
        want = O.dt(phys, dict(mesh, leaves=m.leaves()), m.Q.cpu().numpy())
        assert abs(m.dt - want) <= 1e-12 * want, cells


def test_two_stages_in_a_captured_step():
    phys = dict(I.CFD, N=1, picard_iters=1, mu=0.01, mms=0, cfl=0.5)
    mesh = dict(nx=30, ny=29, nz=29, h=1.0 / 32, bc=[I.BC_PERIODIC] * 6)
    Q = I.random_state_cfd3(30 * 29 * 29, 1, seed=5)
    eager, graph = adg.Mesh3(phys, mesh), adg.Mesh3(phys, mesh)
    for m in (eager, graph):
        m.set_state(Q, t=0.0)
        m.compute_dt()
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        graph.step()
    for _ in range(4):
        g.replay()
        eager.step()
        torch.cuda.synchronize()
        assert torch.equal(graph.Q, eager.Q) and torch.equal(graph.clock, eager.clock)
        assert torch.equal(graph.cell_dt(), eager.cell_dt())
