"""Cells that a flow has driven to negative density and pressure still have a
speed of sound; their wave speed is |v| + c with |v| of the velocity, in the time
step and in the Rusanov flux, as in the oracle.  Smooth states around rho = -1,
so the bars are those of the parity tests: 1e-14 for the time step, 1e-11 of the
largest value for a step."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_1905_05524_amd import adg
from paper_1905_05524_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 6, 7])
def test_wave_speed_of_negative_density(N):
    nx, nz = 5, 3
    phys = dict(I.CFD, N=N, picard_iters=0, mu=0.0, mms=0, cfl=0.5)
    mesh = dict(nx=nx, nz=nz, max_level=0, x0=0.0, z0=0.0, Lx=nx / 4.0, Lz=nz / 4.0, bc=[I.BC_PERIODIC] * 4)
    Q = I.random_state_cfd(nx * nz, N, seed=30 + N)
    Q = -Q
    want = O.dt(phys, mesh, Q)
    assert np.isfinite(want)
    m = adg.Mesh(phys, mesh)
    m.set_state(Q, t=0.0)
    m.compute_dt()
    assert abs(m.dt - want) <= 1e-14 * want
    dt = 0.5 * want
    m.set_state(Q, t=0.0, dt=dt)
    m.step()
    ref = O.step(phys, mesh, Q, 0.0, dt)
    assert np.max(np.abs(m.Q.cpu().numpy() - ref)) <= 1e-11 * np.max(np.abs(ref))
    want = O.dt(phys, mesh, ref)
    assert abs(m.dt - want) <= 1e-12 * want
