"""The fused steps of small systems (one launch per step, or many steps per launch for
the smallest members) against the separate kernels, bit for bit, and the oracle, at
the sizes where their tiles and lane groups end."""
import numpy as np
import pytest

import oracle
import workloads
from paper_2603_27279_amd import RodSim

pytestmark = pytest.mark.gpu


def bent(lengths, members, seed=11, **kw):
    """Coils whose turns touch, several rods per member: contacts, dipoles, a
    gradient field, a clamped and a driven particle."""
    rng = np.random.default_rng(seed)
    pts, off, mem = [], [0], []
    for m in range(members):
        for r, n in enumerate(lengths):
            ph = np.arange(n) * 0.66
            pts.append(np.stack([1.5 * np.cos(ph) + 3.4 * r, 1.5 * np.sin(ph), 0.125 * ph], 1))
            off.append(off[-1] + n)
            mem.append(m)
    x = np.concatenate(pts)
    n = len(x)
    bc = np.zeros(n, np.int8)
    bc[0] = 1
    if n > 3:
        bc[n - 1] = 2
    f = workloads._field_const(members, (0.1, 0.3, -0.2), g=np.diag([0.02, -0.03, 0.01]), length=3)
    f[1] *= 1.5
    w = workloads._base(x, off, mem, np.tile([1.0, 1.0, 2.0, 0.4], (len(mem), 1)),
                        rng.normal(0, 0.04, (n, 3)), bc, f, contact_on=True, drive_period=400,
                        drive_axis=np.array([0.0, 0.0, 1.0]), name="bent")
    w["v0"] = rng.normal(0, 0.02, (n, 3)) * (bc == 0)[:, None]
    w.update(kw)
    return workloads._perturb(w, rng, 1e-2)


HM = dict(contact_model="hertz_mindlin", contact_hm=np.array([2.0, 0.3, 0.5, 0.05, 0.02]))


# one particle; the group widths of the many-step kernel (16, 32) and just past them;
# its rods per member; the four- and sixteen-particle workgroups (up to and past 2048
# particles) and members that end inside one; more than 32 rounds of 64 candidates
@pytest.mark.parametrize("lengths,members,kw", [
    ((1,), 1, {}), ((2,), 1, {}), ((16,), 3, {}), ((9, 8), 2, {}), ((32,), 2, {}), ((30, 3), 3, {}),
    ((31,), 1, dict(dipole_on=False)), ((25,), 2, dict(exclude_depth=40)),
    ((20,), 2, dict(contact_on=False)), ((33,), 2, dict(dipole_on=False)),
    ((40, 25), 2, dict(exclude_depth=3)), ((13, 50), 5, HM), ((20,), 2, HM),
    ((1024, 1024), 1, {}), ((301, 382), 3, {}), ((682, 1), 3, HM), ((2048,), 2, {}),
])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_fused_small_steps(lengths, members, kw, prec):
    w = bent(lengths, members, **kw)
    if sum(lengths) % 2:
        w["bond_damping"] = np.tile([0.2, 0.1, 0.3, 0.15], (len(lengths) * members, 1))
        w["damping"] = 0.0
    runs = []
    for mode, graph in (("batched", 0), ("batched", 4), ("separate", 0)):
        sim = RodSim(w, precision=prec, graph_steps=graph)
        sim.launch_mode(mode)
        for n in (1, 4, 2, 9):
            sim.step(n)
        sim.sync()
        runs.append(sim.state())
        sim.free()
    for k in ("x", "v", "q", "w", "F", "T"):
        np.testing.assert_array_equal(runs[0][k], runs[1][k])
        np.testing.assert_array_equal(runs[0][k], runs[2][k])
    o = oracle.run(w, 16)
    motion = np.max(np.abs(o["x"] - w["x0"])) or 1.0
    assert np.max(np.abs(runs[0]["x"] - o["x"])) / motion <= (1e-9 if prec == "fp64" else 1e-4)
    assert runs[0]["step"] == 16


@pytest.mark.parametrize("n", [24, 70])
def test_layout_change_and_inspection_between_steps(n):
    """Force evaluations, energies, pair queries and a layout change between fused
    steps leave the state alone and see it whole."""
    w = bent((n,), 2)
    a, b = RodSim(w, precision="fp64"), RodSim(w, precision="fp64")
    a.step(7)
    b.step(3)
    b.eval_forces()
    b.energy()
    pairs = b.contact_pairs()
    assert np.array_equal(pairs, oracle.contact_pairs(w, b.state()["x"]))
    b.dipole_layout(1, 64)
    b.step(4)
    sa, sb = a.state(), b.state()
    for k in ("x", "v", "q", "w", "F", "T"):
        np.testing.assert_array_equal(sa[k], sb[k])
    F, T = b.eval_forces()
    assert np.max(np.abs(F.cpu().numpy().T - sb["F"])) > 0  # full-step velocities now
    a.free()
    b.free()
