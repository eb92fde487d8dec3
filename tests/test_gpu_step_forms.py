"""Steps of small systems on both sides of the lines between their forms (two launches, one
launch, many steps per launch): batched, graph and separate launches give the same bits."""
import numpy as np
import pytest

from paper_2603_27279_amd import RodSim
from test_gpu_small_steps import HM, bent

pytestmark = pytest.mark.gpu

NONE = dict(dipole_on=False, contact_on=False)


@pytest.mark.parametrize("n,members,kw", [
    (1024, 1, NONE), (1025, 1, NONE), (1, 768, NONE), (1, 769, NONE), (3, 1000, NONE),
    (256, 8, dict(dipole_on=False)), (257, 7, dict(dipole_on=False)), (64, 65, dict(dipole_on=False)),
    (1024, 2, dict(contact_on=False)), (1025, 1, {}), (128, 65, {}), (129, 64, {}),
    (64, 65, HM), (65, 64, HM),
])
def test_forms_agree(n, members, kw):
    w = bent((n,), members, **kw)
    runs = []
    for mode, graph in (("batched", 0), ("batched", 3), ("separate", 0)):
        sim = RodSim(w, precision="mixed", graph_steps=graph)
        sim.dipole_layout(1)
        sim.launch_mode(mode)
        for k in (1, 4, 2):
            sim.step(k)
        sim.sync()
        runs.append(sim.state())
        sim.free()
    for k in ("x", "v", "q", "w", "F", "T"):
        np.testing.assert_array_equal(runs[0][k], runs[1][k])
        np.testing.assert_array_equal(runs[0][k], runs[2][k])
