"""A 3D handle without gravity has no background to tabulate: making one launches
nothing and waits for nothing beyond its uploads, so it is quicker than one with
gravity (32 and 44 us).  The best of many alternating runs, bar 90 %.  Its steps
see a background of zeros, also in memory that held something else."""
import time

import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_1905_05524_amd import adg
from paper_1905_05524_amd import inputs as I

import parity as P

pytestmark = pytest.mark.gpu


def grid3(base, N=2):
    return dict(base, N=N, picard_iters=0, mu=0.01, mms=0, cfl=0.5), \
        dict(nx=4, ny=4, nz=4, x0=0.0, y0=0.0, z0=0.0, h=0.25, bc=[I.BC_PERIODIC] * 6)


def test_no_background_without_gravity():
    best = {}
    for _ in range(200):
        for base in (I.CFD, I.ATMO):
            phys, mesh = grid3(base)
            torch.cuda.synchronize()
            t = time.perf_counter()
            m = adg.Mesh3(phys, mesh)
            t = time.perf_counter() - t
            del m
            g = base["gravity"]
            best[g] = min(t, best.get(g, t))
    assert best[0] <= 0.9 * best[1], best


@pytest.mark.parametrize("N", [1, 2, 3, 4, 5])
def test_step_after_handles_with_gravity(N):
    for _ in range(4):   # handles whose tables the allocator may give again
        adg.Mesh3(*grid3(I.ATMO, N))
    phys, mesh = grid3(I.CFD, N)
    Q = I.random_state_cfd3(64, N, seed=N)
    dt = 0.5 * O.dt3(phys, mesh, Q)
    m = adg.Mesh3(phys, mesh)
    m.set_state(Q, t=0.0, dt=dt)
    m.step()
    P.assert_step(m.Q.cpu().numpy(), O.step3(phys, mesh, Q, 0.0, dt), Q, V=5)


@pytest.mark.parametrize("nz", [1638, 1639])
def test_columns_around_the_size_of_the_upload(nz):
    """N = 2, 10 doubles per layer: up to 16,384 zeros are sent, more are cleared on
    the device."""
    for _ in range(2):
        adg.Mesh3(dict(I.ATMO, N=2, picard_iters=1, mu=0.01, mms=0, cfl=0.5),
                  dict(nx=1, ny=1, nz=nz, h=1.0, bc=[I.BC_PERIODIC] * 6))
    phys, mesh = grid3(I.CFD)
    mesh.update(nx=1, ny=1, nz=nz)
    Q = I.random_state_cfd3(nz, 2, seed=4)
    dt = 0.5 * O.dt3(phys, mesh, Q)
    m = adg.Mesh3(phys, mesh)
    m.set_state(Q, t=0.0, dt=dt)
    m.step()
    P.assert_step(m.Q.cpu().numpy(), O.step3(phys, mesh, Q, 0.0, dt), Q, V=5)
