"""The autotuner times the launches that steps really make, on a copy of the state."""
import re

import numpy as np
import pytest

import workloads
from paper_2603_27279_amd import RodSim
from test_gpu_small_steps import HM, bent

pytestmark = pytest.mark.gpu


def chosen(report):
    m = re.search(r"^chosen: (small-member|spatial split|split) layout target_wgs=(\d+) ", report, re.M)
    return {"split": 0, "small-member": 1, "spatial split": 2}[m.group(1)], int(m.group(2))


def test_small_members_without_dipoles_keep_their_fused_steps():
    """A launch per many steps (3.5 us per step) against two launches per step (about
    10): the split layout, the only one that was considered, has no fused steps."""
    sim = RodSim(bent((20,), 3, dipole_on=False), precision="fp64")
    report = sim.autotune()
    us = dict(re.findall(r"^(small-member|split) layout .*: ([\d.]+) us", report, re.M))
    assert chosen(report)[0] == 1, report
    assert float(us["small-member"]) < 0.7 * float(us["split"]), report
    sim.free()


@pytest.mark.parametrize("lengths,members,kw", [
    ((20,), 3, {}), ((40, 25), 2, HM), ((31,), 2, dict(dipole_on=False)), ((1024,), 1, {}),
    ((700, 700, 701), 1, {}), ((1500,), 3, HM),
])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_tuning_leaves_the_run_alone(lengths, members, kw, prec):
    """State, level, histories of bond damping and of Hertz-Mindlin contact, and error
    flags: a tuned context goes on as one that was given the choice."""
    w = bent(lengths, members, **kw)
    w["bond_damping"] = np.tile([0.2, 0.1, 0.3, 0.15], (len(lengths) * members, 1))
    w["damping"] = 0.0
    a, b = (RodSim(w, precision=prec, graph_steps=4) for _ in range(2))
    a.step(5)
    b.step(5)
    small, target = chosen(a.autotune())
    b.dipole_layout(small, max(target, 1))
    assert a.get_step() == 5
    for sim in (a, b):
        sim.step(9)
        sim.sync()
    sa, sb = a.state(), b.state()
    for k in ("x", "v", "q", "w", "F", "T"):
        np.testing.assert_array_equal(sa[k], sb[k])
    a.free()
    b.free()
