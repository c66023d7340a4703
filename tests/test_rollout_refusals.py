"""A rollout that the library refuses leaves the mesh as it was.  On the CPU,
with a stand-in for the mesh whose initial-state map raises like that of a mesh
without gravity."""
import pytest

torch = pytest.importorskip("torch")

from paper_1905_05524_amd.autodiff import theta_rollout


class Refusing:
    fixed_dt = True
    device = torch.device("cpu")

    def __init__(self):
        self.Q = torch.arange(36.0, dtype=torch.float64).view(1, 4, 3, 3)
        self.clock = torch.tensor([0.7, 0.01, 0.0, 5.0], dtype=torch.float64)
        self.bound = self.Q

    def bind_state(self, Q):
        self.bound = Q

    def bind(self):
        self.bound = self.Q

    def keep_bytes(self):
        return 8, 8

    def ic_theta(self, theta_prime):
        raise RuntimeError("the theta' initial state needs gravity (background)")


@pytest.mark.parametrize("keep", [False, True])
def test_refused_initial_state_changes_nothing(keep):
    m = Refusing()
    Q, clock = m.Q.clone(), m.clock.clone()
    with pytest.raises(RuntimeError, match="needs gravity"):
        theta_rollout(torch.zeros(1, 3, 3, dtype=torch.float64, requires_grad=True), m, 2, 1e-3, 0.25, keep)
    assert torch.equal(m.Q, Q) and torch.equal(m.clock, clock)
    assert m.bound is m.Q
