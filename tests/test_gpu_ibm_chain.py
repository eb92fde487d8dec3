"""The chain of fused steps in coupled cycles (batched launches: kicks between force
launches that also spread the step before) against separate launches: one substep (no
kick) and several, both precisions, Hertz-Mindlin contact, and a system past 65,536
particles (contact by candidate lists, one particle per thread in the kick). The two
orders of launches do the same arithmetic on the rods; the fluid's force sums differ in
the order of their FP64 additions."""
import numpy as np
import pytest

import workloads
from test_gpu_ibm import fluid, rods, run_gpu

pytestmark = pytest.mark.gpu

HM = dict(contact_on=True, contact_model="hertz_mindlin", contact_hm=np.array([20.0, 0.3, 0.5, 0.0, 0.0]))


def both(w, f0, cycles, nsub, prec):
    st, f = run_gpu(w, f0, cycles, nsub, 0.8, mode="batched", prec=prec)
    st2, f2 = run_gpu(w, f0, cycles, nsub, 0.8, mode="separate", prec=prec)
    assert st["step"] == st2["step"] == cycles * nsub
    # a cycle's fluid velocity differs by the rounding of the force sums before it
    # (about 1e-16 of forces of 1e-3 to 1 over a few cells): far below 1e-12
    for k in ("x", "v", "w", "F"):
        scale = max(1.0, np.max(np.abs(st2[k])))
        assert np.max(np.abs(st[k] - st2[k])) <= 1e-12 * scale, k
    assert np.max(np.abs(f - f2)) <= 1e-13


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("nsub,contact", [(1, {}), (2, {}), (5, HM)])
def test_chain_equals_separate_launches(prec, nsub, contact):
    w = rods([7, 7, 90], [(3.0, 4.0, 5.0), (3.0, 4.95, 5.0), (2.0, 8.0, 9.0)], nsub, 21, **contact)
    both(w, fluid((20, 13, 15), 22), 3, nsub, prec)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_large_system(prec):
    """65,600 particles of 2,050 rods in two layers whose rods touch."""
    lens, org = [32] * 2050, []
    for r in range(2050):
        org.append((1.0 + 33.0 * (r % 2), 2.0 + 1.5 * ((r // 2) % 41), 2.0 + 0.97 * (r // 82)))
    w = rods(lens, org, 3, 23, contact_on=True, dipole_on=False)
    both(w, fluid((68, 66, 32), 24), 2, 3, prec)
