"""Gradients where the tape leaves no room for the buffers of the one-launch reverse."""
import numpy as np
import pytest
import torch

import workloads
from paper_2603_27279_amd import RodSim

pytestmark = pytest.mark.gpu

GIB = 1 << 30


def test_gradient_without_room_for_the_fused_reverse():
    """The buffers take 2.2 GiB with segments of 24,000 levels of 1,000 particles; 1 GiB
    is left. The gradient is that of the run with room, to rounding."""
    w = workloads.adjoint_rod(n=1000)
    sim = RodSim(w, precision="fp64", tape_every=24000, tape_capacity=24000)
    sim.tape_begin()
    sim.step(12)
    sim.sync()
    gx = torch.ones_like(sim.x)
    sim_out = []
    torch.cuda.empty_cache()
    held = []
    while torch.cuda.mem_get_info()[0] > 3 * GIB:
        held.append(torch.empty(min(torch.cuda.mem_get_info()[0] - 2 * GIB, 16 * GIB), dtype=torch.uint8,
                                device="cuda"))
    held.append(torch.empty(torch.cuda.mem_get_info()[0] - GIB, dtype=torch.uint8, device="cuda"))
    try:
        sim_out.append(sim.grad(gx=gx))
        torch.cuda.synchronize()
    finally:
        del held
        torch.cuda.empty_cache()
    sim_out.append(sim.grad(gx=gx))
    for k in sim_out[0]:
        a, b = (g[k].cpu().numpy() for g in sim_out)
        assert np.max(np.abs(a - b)) <= 1e-11 * max(np.max(np.abs(b)), 1e-300), k
    sim.free()
