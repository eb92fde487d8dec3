"""Work items of the mixed path's split layout that take parts of a slot (whole tiles of
512 sources, FP64 partial sums): dipole forces and fields against FP64, launch forms bit
for bit, and gradients, for slots of one tile, of a tile and a remainder, of several,
for members that need fewer parts than others, and past 65,536 particles."""
import numpy as np
import pytest
import torch

import workloads
from paper_2603_27279_amd import RodSim, TERM_DIPOLE
from test_gpu_parity import TOL, rel_inf

pytestmark = pytest.mark.gpu


def rods(lengths, members=(0,), **kw):
    """Per member, rods of the given lengths side by side."""
    rng = np.random.default_rng(31)
    lens, org, mem = [], [], []
    for m in members:
        for r, n in enumerate(lengths[m]):
            lens.append(n)
            org.append((3.0 * (r % 24), 3.0 * (r // 24), 0.0))
            mem.append(m)
    x, off, mem = workloads.straight_rods(lens, org, (0, 0, 1), member=np.array(mem))
    n = len(x)
    bc = np.zeros(n, np.int8)
    bc[off[:-1]] = 1
    w = workloads._base(x, off, mem, np.tile([1.0, 1.0, 1.0, 0.5], (len(lens), 1)),
                        rng.normal(0, 0.1, (n, 3)), bc,
                        workloads._field_const(len(members), (0.1, 0.2, 0.3)), damping=0.1, **kw)
    return workloads._perturb(w, rng, 1e-2)


SYSTEMS = {
    "one_tile": lambda: rods([[65] * 64]),                  # 4,160: slots of 260
    "remainder": lambda: rods([[96] * 64]),                 # 6,144: 559, a tile and 47
    "three": lambda: rods([[81] * 127 + [27]]),             # 10,314: 1,474
    "four": lambda: rods([[128] * 128]),                    # 16,384: 4,096
    "members": lambda: rods([[100] * 90, [37] * 3, [60] * 40], (0, 1, 2)),
    "large": lambda: rods([[257] * 257]),                   # 66,049: one slot each
}


@pytest.mark.parametrize("name", list(SYSTEMS))
def test_parts_of_slots(name):
    w = SYSTEMS[name]()
    exact = RodSim(w, precision="fp64")
    Fe, Te, Be = exact.eval_forces(TERM_DIPOLE, with_field=True)
    states = []
    for mode in ("batched", "separate") + (("per_rod",) if name in ("remainder", "members") else ()):
        sim = RodSim(w, precision="mixed")
        sim.launch_mode(mode)
        F, T, B = sim.eval_forces(TERM_DIPOLE, with_field=True)
        for a, b in ((F, Fe), (T, Te), (B, Be)):
            assert rel_inf(a.cpu().numpy(), b.cpu().numpy()) <= TOL["mixed"], mode
        sim.step(3)
        states.append(sim.state())
        sim.free()
    exact.free()
    for st in states[1:]:
        for k in ("x", "v", "q", "w", "F", "T"):
            assert np.array_equal(states[0][k], st[k]), k


def test_gradient_through_parts():
    """Against a layout of as many work items whose slots are whole."""
    w = rods([[81] * 127 + [27]])
    g0 = np.random.default_rng(5).normal(size=(3, len(w["x0"])))
    grads = []
    for target in (1024, 4096):
        sim = RodSim(w, precision="mixed", tape_every=2, tape_capacity=5)
        sim.dipole_layout(0, target)
        sim.tape_begin()
        sim.step(5)
        g = sim.grad(gx=torch.from_numpy(g0).cuda())
        grads.append({k: v.cpu().numpy() for k, v in g.items()})
        sim.free()
    for k in grads[0]:
        assert rel_inf(grads[0][k], grads[1][k]) <= TOL["mixed"], k
