"""A candidate list or a cell table past its capacity is reported at every check, not
only at the first after the lists were built: later calls on the same lists too."""
import numpy as np
import pytest

import workloads
from paper_2603_27279_amd import RodSim
from paper_2603_27279_amd._lib import ROD_E_OVERFLOW, RodError

pytestmark = pytest.mark.gpu


def fixed(xs, **kw):
    """Single fixed particles at xs."""
    n = len(xs)
    x, off, mem = workloads.straight_rods([1] * n, xs, (1, 0, 0))
    return workloads._base(x, off, mem, np.tile([1.0, 1.0, 1.0, 0.5], (n, 1)),
                           np.random.default_rng(1).normal(0, 0.01, (n, 3)), np.ones(n, np.int8),
                           workloads._field_const(1, (0, 0, 0)), contact_on=True, k_contact=1e-3, **kw)


def crowd():
    """400 particles that all lie within each other's dipole cutoff: lists of 399."""
    return fixed(np.random.default_rng(4).uniform(0, 5, (400, 3)), dipole_cutoff=7.0)


def clusters():
    """66,000 particles in 4,400 clusters of 15, each in one cell: seven of each do not
    fit, 30,800 in all, while no particle has more than 14 candidates."""
    g = np.arange(17) * 5.0 + 0.6
    c = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)[:4400]
    xs = np.repeat(c, 15, axis=0) + np.random.default_rng(2).uniform(-0.2, 0.2, (66000, 3))
    return fixed(xs, dipole_on=False)


@pytest.mark.parametrize("system", [crowd, clusters])
def test_reported_at_every_check(system):
    sim = RodSim(system(), precision="fp64", graph_steps=2)
    for n in (2, 1, 2, 3):
        sim.step(n)
        with pytest.raises(RodError) as e:
            sim.sync()
        assert e.value.code == ROD_E_OVERFLOW
    sim.free()
