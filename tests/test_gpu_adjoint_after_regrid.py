"""The adjoint workspace that a mesh keeps follows a regrid: of the size that
the new cells need before anything is written to it."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1905_05524_amd import adg
from paper_1905_05524_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_adjoint_workspace_grows_with_the_mesh():
    w = I.bubble(3, 2)
    w["mesh"].update(max_level=1, leaves=I.uniform_leaves(3, 3))
    m = adg.Mesh(w["phys"], w["mesh"], fixed_dt=True)
    m.init_state("bubbles", w["bubbles"])
    m.adjoint_workspace()
    assert m.regrid(np.ones(9, dtype=np.int8)) == 81
    need = ctypes.c_size_t()
    assert adg.lib().adg_adjoint_workspace_bytes(m.h, ctypes.byref(need)) == adg.ADG_OK
    assert m.adjoint_workspace().numel() >= need.value
