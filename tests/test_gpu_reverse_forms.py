"""Gradients of small systems on both sides of the line between one launch and two per
reversed step: equal to rounding, and the buffers of the one-launch form are taken only
where it runs."""
import numpy as np
import pytest
import torch

from paper_2603_27279_amd import RodSim
from test_gpu_small_steps import bent

pytestmark = pytest.mark.gpu

BLOCKS = ("m_body", "field", "x0", "v0", "q0", "w0")


@pytest.mark.parametrize("n,members,kw,fused", [
    (1024, 1, {}, True), (1025, 1, {}, False), (256, 8, {}, True), (257, 7, {}, False),
    (30, 68, {}, True), (30, 69, {}, False), (256, 16, dict(contact_on=False), False),
    (200, 12, dict(dipole_on=False), False), (30, 40, dict(dipole_on=False, contact_on=False), True),
])
def test_reverse_forms_agree(n, members, kw, fused):
    w = bent((n,), members, **kw)
    grads = []
    for timed in (False, True):  # a timed run reverses with two launches per step
        sim = RodSim(w, precision="fp64", tape_every=8, tape_capacity=20)
        sim.tape_begin()
        sim.step(19)
        sim.sync()
        sim.timing(timed)
        gx = torch.ones_like(sim.x)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        sim.grad(gx=gx, want=())
        torch.cuda.synchronize()
        taken = free - torch.cuda.mem_get_info()[0]
        # (the bond Jacobians alone are 99 doubles per particle and level)
        assert (taken >= 8 * 99 * 8 * sim.n) == (fused and not timed), taken
        g = sim.grad(gx=gx)
        grads.append({k: v.cpu().numpy() for k, v in g.items()})
        sim.free()
    for k in BLOCKS:
        a, b = grads[0][k], grads[1][k]
        assert np.max(np.abs(a - b)) <= 1e-11 * max(np.max(np.abs(b)), 1e-300), k
