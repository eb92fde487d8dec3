"""Candidate lists that outlive a call are rebuilt after anything else has built lists or
set the positions they are measured from, also when that ran in a graph that the caller
captured earlier and replays between steps."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
import workloads
from paper_2603_27279_amd import RodSim, TERM_ALL
from paper_2603_27279_amd import _lib as L

pytestmark = pytest.mark.gpu


def closing_pairs(pairs, length):
    """Pairs of rods 2.4 apart that close at speed 1 and collide after some 140 steps."""
    org, v = [], []
    for p in range(pairs):
        for side in (0, 1):
            org.append((8.0 * (p % 32), 8.0 * (p // 32) + 2.4 * side, 0.0))
            v.append(-1.0 * side)
    x, off, mem = workloads.straight_rods([length] * len(org), org, (0, 0, 1))
    rng = np.random.default_rng(5)
    w = workloads._base(x, off, mem, np.tile([1.0, 1.0, 1.0, 0.5], (len(org), 1)),
                        rng.normal(0, 0.02, x.shape), np.zeros(len(x), np.int8),
                        workloads._field_const(1, (0.0, 0.0, 0.1)), contact_on=True, k_contact=50.0,
                        dipole_cutoff=2.0, damping=0.0, name="closing")
    w["v0"] = np.repeat(np.array(v), length)[:, None] * np.array([0.0, 1.0, 0.0])
    return w


@pytest.mark.parametrize("pairs,length,entry", [(3, 40, "forces"), (3, 40, "energy"),
                                                (330, 100, "forces"), (330, 100, "energy")])
def test_captured_evaluations_between_steps(pairs, length, entry):
    """Each step call moves the rods by 0.4 of the lists' skin, less than the distance
    that asks for new lists; over the run they move by several skins."""
    w = closing_pairs(pairs, length)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        sim = RodSim(w, precision="fp64", graph_steps=5)
        F, T = torch.zeros_like(sim.x), torch.zeros_like(sim.x)
        E = torch.zeros((1, 9), dtype=torch.float64, device="cuda")
        p = lambda t: C.c_void_p(t.data_ptr())
        st.synchronize()
        g = torch.cuda.CUDAGraph()
        g.capture_begin()
        if entry == "forces":
            L.check(sim.lib.rod_eval_forces(sim.ctx, TERM_ALL, p(F), p(T), None))
        else:
            L.check(sim.lib.rod_energy(sim.ctx, p(E), 1))
        g.capture_end()
        for _ in range(20):
            sim.step(10)
            g.replay()
        sim.sync()
        s = sim.state()
        sim.free()
        ref = RodSim(w, precision="fp64")
        ref.launch_mode("separate")  # new lists in every call
        for _ in range(20):
            ref.step(10)
        r = ref.state()
        ref.free()
    assert np.max(r["v"][:length, 1]) < -0.5  # the rods have met: the one at rest now moves
    assert np.max(np.abs(s["x"] - r["x"])) <= 1e-9
    if pairs < 10:
        o = oracle.run(w, 200)
        assert np.max(np.abs(s["x"] - o["x"])) <= 1e-9
