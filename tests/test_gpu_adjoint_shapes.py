"""The step adjoint at mesh sizes where its launches can go wrong: on both
sides of 256 cells (one cell and several per workgroup), counts that leave the
last workgroup partly empty, one row and one column of cells, one Picard
iteration.  <J v, w> from the oracle's forward-mode derivative against
<v, J^T w>, for a v on all cells and for one on the last cell alone; the bar
is the 1e-12 |J v| |w| of the adjoint tests, |w| over the cells where J v is
not zero."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_1905_05524_amd import adg
from paper_1905_05524_amd import inputs as I

from test_gpu_adjoint import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", [I.BC_WALL, I.BC_PERIODIC], ids=["walls", "periodic"])
@pytest.mark.parametrize("N,nx,nz,iters", [
    (1, 1, 1, 0), (1, 16, 16, 0), (1, 257, 1, 0), (1, 17, 16, 1), (2, 1, 5, 0), (2, 16, 17, 0), (2, 7, 41, 1),
    (3, 16, 16, 0), (3, 1, 259, 0), (4, 3, 2, 1), (4, 43, 6, 0), (4, 37, 7, 0), (5, 2, 1, 0), (6, 1, 2, 1), (7, 2, 2, 0)])
def test_step_adjoint_on_ragged_meshes(N, nx, nz, iters, bc):
    if bc == I.BC_WALL:
        phys = dict(I.ATMO, N=N, picard_iters=iters, mu=5.0, mms=0, cfl=0.4)
        h = 1000.0 / max(nx, nz)
        mesh = dict(nx=nx, nz=nz, max_level=0, Lx=h * nx, Lz=h * nz, bc=[bc] * 4)
        Q = O.ic(phys, mesh, "bubbles", [I.cosine_bubble(a=400.0, xc=0.5 * h * nx, zc=0.4 * h * nz)])
        Q = I.perturb(Q, seed=60 + N)
    else:
        phys = dict(I.CFD, N=N, picard_iters=iters, mu=0.05, mms=0, cfl=0.5)
        mesh = dict(nx=nx, nz=nz, max_level=0, Lx=nx / 4.0, Lz=nz / 4.0, bc=[bc] * 4)
        Q = I.random_state_cfd(nx * nz, N, seed=70 + N)
    dt = 0.5 * O.dt(phys, mesh, Q)
    rng = np.random.default_rng(200 + N)
    scale = np.array([1e-4, 0.1, 0.1, 10.0] if bc == I.BC_WALL else [1.0] * 4)[None, :, None, None]
    w = rng.standard_normal(Q.shape) / scale
    m = adg.Mesh(phys, mesh, fixed_dt=True)
    m.set_state(Q, t=0.3, dt=dt)
    lam = torch.empty_like(m.Q)
    m.step_adjoint(dev(Q), dev(w), lam)
    JTw = lam.cpu().numpy()
    v = rng.standard_normal(Q.shape) * scale
    last = np.zeros_like(v)
    last[-1] = v[-1]
    for d in (v, last):
        _, Jd = O.step_jvp(phys, mesh, Q, d, 0.3, dt)
        on = np.any(Jd != 0.0, axis=(1, 2, 3))
        bound = np.linalg.norm(Jd) * np.linalg.norm(w[on])
        a, b = float(np.sum(Jd * w)), float(np.sum(d * JTw))
        assert abs(a - b) <= 1e-12 * bound, (a, b, bound)
