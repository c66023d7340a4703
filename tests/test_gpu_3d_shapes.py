"""The 3D step at grid sizes where its launches can go wrong: cell counts that
leave the last workgroup partly empty, workgroup counts on both sides of the
multiples of eight (the XCD order of the corrector), one layer and one column
of cells (the background table of the node rows), one Picard iteration and
several.  Against the oracle, with the bars of the 3D parity tests: 1e-11 for
the predictor outputs, their step tolerance for the step."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_1905_05524_amd import adg
from paper_1905_05524_amd import inputs as I

import parity as P
import test_gpu_3d as T

pytestmark = pytest.mark.gpu

GRIDS = [(1, 7, 5, 1), (1, 17, 17, 1), (2, 1, 1, 1), (2, 10, 1, 1), (2, 11, 7, 1), (3, 29, 1, 1), (3, 3, 11, 1),
         (3, 1, 1, 9), (4, 1, 1, 1), (4, 5, 1, 3), (4, 1, 17, 1), (5, 1, 1, 1), (5, 7, 1, 1), (5, 3, 1, 3)]


@pytest.mark.parametrize("N,nx,ny,nz", GRIDS)
@pytest.mark.parametrize("iters", [0, 1])
def test_step_on_ragged_grids(N, nx, ny, nz, iters):
    phys, m, Q = T.atmo_case(N, nx, ny, nz, 40 + N)
    phys["picard_iters"] = iters
    dt = 0.5 * O.dt3(phys, m, Q)
    Qs_ref, FD_ref = O.predictor3(phys, m, Q, dt)
    ref = O.step3(phys, m, Q, 0.0, dt)
    g = adg.Mesh3(phys, m)
    g.set_state(Q, t=0.0, dt=dt)
    g.predictor()
    torch.cuda.synchronize()
    assert np.all(T.relerr(g.qstar().cpu().numpy(), Qs_ref) <= T.TOL)
    assert np.all(T.fd_err(g.face_data().cpu().numpy(), FD_ref) <= T.TOL)
    g.set_state(Q, t=0.0, dt=dt)
    g.step()
    torch.cuda.synchronize()
    P.assert_step(g.Q.cpu().numpy(), ref, Q, V=5)
