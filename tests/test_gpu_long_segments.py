"""Gradients through recorded segments longer than a launch grid is high."""
import numpy as np
import pytest
import torch

import workloads
from paper_2603_27279_amd import RodSim

pytestmark = pytest.mark.gpu


def test_a_segment_of_more_levels_than_a_grid_is_high():
    """66,000 levels of three particles as one segment against segments of 1,000."""
    w = workloads.adjoint_rod(n=3)
    w["damping"] = 1.0
    grads = []
    for every in (70000, 1000):
        sim = RodSim(w, precision="fp64", tape_every=every, tape_capacity=70000)
        sim.tape_begin()
        sim.step(66000)
        sim.sync()
        g = sim.grad(gx=torch.ones_like(sim.x))
        grads.append({k: v.cpu().numpy() for k, v in g.items()})
        sim.free()
    for k, a in grads[0].items():
        b = grads[1][k]
        assert np.all(np.isfinite(b))
        # sums over 66,000 levels, whose order may differ
        assert np.max(np.abs(a - b)) <= 66000 * 2.3e-16 * max(np.max(np.abs(b)), 1e-300), k
    assert np.max(np.abs(grads[0]["field"])) > 0
