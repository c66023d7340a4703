"""The corrector and the clock at cell counts where their launches can go
wrong: around the cells of a wavefront (8, 5, 4 and 2 for N = 1 to 4, one
above), a last workgroup partly empty, and the two-stage minimum of the time
step (above 24,576 cells), against the oracle with the bars of the parity
tests (1e-11 for one step, 1e-12 for the time step)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_1905_05524_amd import adg
from paper_1905_05524_amd import inputs as I

import parity as P

pytestmark = pytest.mark.gpu


def _walls(N, nx, nz, mu=5.0):
    phys = dict(I.ATMO, N=N, picard_iters=0, mu=mu, mms=0, cfl=0.4)
    h = 1000.0 / max(nx, nz)
    mesh = dict(nx=nx, nz=nz, max_level=0, Lx=h * nx, Lz=h * nz, bc=[I.BC_WALL] * 4)
    Q = O.ic(phys, mesh, "bubbles", [I.cosine_bubble(a=300.0, xc=0.5 * h * nx, zc=0.4 * h * nz)])
    return phys, mesh, I.perturb(Q, seed=90 + N)


@pytest.mark.parametrize("N,nx,nz", [(1, 7, 1), (1, 1, 8), (1, 3, 3), (2, 4, 1), (2, 5, 1), (2, 2, 3), (3, 3, 1), (3, 5, 1),
                                     (4, 1, 1), (4, 1, 3), (5, 2, 1), (6, 3, 1), (7, 1, 2)])
def test_step_on_ragged_meshes(N, nx, nz):
    phys, mesh, Q = _walls(N, nx, nz)
    dt = 0.5 * O.dt(phys, mesh, Q)
    ref = O.step(phys, mesh, Q, 0.0, dt)
    m = adg.Mesh(phys, mesh)
    m.set_state(Q, t=0.0, dt=dt)
    m.step()
    torch.cuda.synchronize()
    P.assert_step(m.Q.cpu().numpy(), ref, Q)
    want = O.dt(phys, mesh, ref)
    assert abs(m.dt - want) <= 1e-12 * want


@pytest.mark.parametrize("nx,nz", [(192, 128), (8192, 3), (24577, 1), (173, 150), (256, 255)])
@pytest.mark.parametrize("where", [0, 1, -1])
def test_time_step_of_many_cells(nx, nz, where):
    """The smallest candidate in the first, the second or the last cell."""
    phys = dict(I.CFD, N=1, picard_iters=0, mu=0.01, mms=0, cfl=0.5)
    mesh = dict(nx=nx, nz=nz, max_level=0, Lx=nx / 64.0, Lz=nz / 64.0, bc=[I.BC_PERIODIC] * 4)
    Q = I.random_state_cfd(nx * nz, 1, seed=7)
    Q[where, 3] *= 40.0
    m = adg.Mesh(phys, mesh)
    m.set_state(Q, t=0.0)
    m.compute_dt()
    want = O.dt(phys, mesh, Q)
    assert abs(m.dt - want) <= 1e-12 * want
    m.set_state(Q, t=0.0, dt=1e-9 * want)   # the step leaves the state nearly as it is
    m.step()
    assert abs(m.dt - want) <= 1e-6 * want
