"""Steps that the caller captures into a graph of its own and replays: the level, and
with it the field's row, comes from the device, and the candidate lists of a captured
step never count for a later call. Every replay, with eager steps between them, gives
the states of eager steps, bit for bit (the eager steps' lists are made to be rebuilt in
every call, as captured ones are: the cutoff walk adds in list order)."""
import numpy as np
import pytest
import torch

import workloads
from paper_2603_27279_amd import RodSim
from test_gpu_bond_kick import tangle
from test_gpu_small_steps import HM, bent

pytestmark = pytest.mark.gpu

SYSTEMS = {
    # many steps per launch (three members), one launch per step, Hertz-Mindlin
    "many_steps": lambda: bent((20,), 3),
    "fused_step": lambda: bent((40, 25), 2),
    "hertz_mindlin": lambda: bent((20,), 2, **HM),
    # lists that outlive a call
    "large": lambda: tangle(300, 220),
    "cutoff": lambda: tangle(30, 40, dipole_on=True, dipole_cutoff=2.5),
}


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("name", list(SYSTEMS))
def test_replays_equal_eager_steps(name, prec):
    w = SYSTEMS[name]()
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        ref = RodSim(w, precision=prec)
        sim = RodSim(w, precision=prec)
        st.synchronize()
        states = []
        for k in range(5):  # captured, captured, eager, captured, eager
            ref.step(2)
            states.append(ref.state())
            ref.energy()  # (and so new lists in the next call)
        g = torch.cuda.CUDAGraph()
        g.capture_begin()
        sim.step(2)
        g.capture_end()
        for k, captured in enumerate((True, True, False, True, False)):
            if captured:
                g.replay()
            else:
                sim.energy()
                sim.step(2)
            st.synchronize()
            for a, b in ((sim.x, "x"), (sim.v, "v"), (sim.q, "q"), (sim.om, "w"), (sim.F, "F"), (sim.T, "T")):
                assert np.array_equal(a.cpu().numpy().T, states[k][b]), (k, b)
        ref.free(); sim.free()
