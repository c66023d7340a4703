"""The regrid plan where its shortcuts can go wrong: one, three and no levels,
all boundary combinations, families that are kept, merged in part and merged
beside finer leaves (few flags of refinement, many of coarsening).  Leaves and
transferred state against the oracle's regrid (the transfer within 1e-13, as
in the adaptive-mesh tests)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_1905_05524_amd import adg
from paper_1905_05524_amd import inputs as I

from test_gpu_amr import leaves_of, relerr

pytestmark = pytest.mark.gpu

BCS = [[I.BC_PERIODIC] * 4, [I.BC_WALL] * 4, [I.BC_WALL, I.BC_WALL, I.BC_PERIODIC, I.BC_PERIODIC]]


@pytest.mark.parametrize("seed", range(4))
@pytest.mark.parametrize("bc", BCS, ids=["periodic", "walls", "mixed"])
@pytest.mark.parametrize("nx,nz,levels", [(2, 2, 3), (5, 1, 1), (1, 1, 2), (3, 2, 0)])
def test_random_regrids_match_oracle(nx, nz, levels, bc, seed):
    rng = np.random.default_rng(seed)
    mesh = dict(nx=nx, nz=nz, max_level=levels, x0=0.0, z0=0.0, Lx=nx / 4.0, Lz=nz / 4.0, bc=bc,
                leaves=I.uniform_leaves(nx, nz))
    phys = dict(I.CFD, N=1, picard_iters=0, mu=0.02, mms=0, cfl=0.5)
    m = adg.Mesh(phys, mesh)
    m.set_state(I.random_state_cfd(nx * nz, 1, seed=seed))
    for rnd in range(6):
        cur = dict(mesh, leaves=leaves_of(m))
        Q = m.Q.cpu().numpy().copy()
        up = 0.4 if rnd < 3 else 0.03
        flags = rng.choice(np.array([-1, 0, 1], dtype=np.int8), size=m.C, p=[0.9 - up, 0.1, up])
        if rnd >= 3:   # whole families, so that some merge
            fam = {(l, i // 3, j // 3): rng.random() < 0.7 for l, i, j in cur["leaves"]}
            for c, (l, i, j) in enumerate(cur["leaves"]):
                if fam[(l, i // 3, j // 3)]:
                    flags[c] = -1
        m.regrid(flags)
        ref_leaves, ref_Q = O.regrid(phys, cur, Q, flags)
        assert leaves_of(m) == ref_leaves, rnd
        assert np.all(relerr(m.Q.cpu().numpy(), ref_Q) <= 1e-13), rnd
