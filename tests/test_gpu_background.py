"""The background tables of the meshes: the step at cells of every height, on
both levels of an adaptive mesh and after a regrid that outgrows the tables,
against the oracle with the bars of the parity tests (1e-11 for one step)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_1905_05524_amd import adg
from paper_1905_05524_amd import inputs as I

import parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 3, 4, 6])
def test_step_after_regrids_matches_oracle(N):
    """A walled column of few coarse cells, refined everywhere (three times the
    rows and nine times the cells: new tables with a new capacity), then
    coarsened in part (the tables stay, shorter than their capacity)."""
    phys = dict(I.ATMO, N=N, picard_iters=0, mu=5.0, mms=0, cfl=0.4)
    mesh = dict(nx=2, nz=3, max_level=1, Lx=2000.0, Lz=3000.0, bc=[I.BC_WALL] * 4, leaves=I.uniform_leaves(2, 3))
    m = adg.Mesh(phys, mesh)
    m.init_state("bubbles", [I.cosine_bubble(a=800.0, xc=1000.0, zc=1200.0)])
    for k in range(2):
        leaves = [tuple(int(x) for x in r) for r in m.leaves()]
        f = [1 if k == 0 else (-1 if (l, i // 3, j // 3) == (1, 0, 0) else 0) for l, i, j in leaves]
        m.regrid(np.array(f, dtype=np.int8))
        cur = dict(mesh, leaves=[tuple(int(x) for x in r) for r in m.leaves()])
        assert m.C == len(cur["leaves"]) == (54 if k == 0 else 46)
        Q = I.perturb(m.Q.cpu().numpy(), seed=80 + N + k)
        dt = 0.5 * O.dt(phys, cur, Q)
        ref = O.step(phys, cur, Q, 0.0, dt)
        m.set_state(Q, t=0.0, dt=dt)
        m.step()
        torch.cuda.synchronize()
        P.assert_step(m.Q.cpu().numpy(), ref, Q)
