"""Which small systems are given the second set of state planes of one-launch steps: by
particles, members and force terms, at the edges of the rule (no GPU needed)."""
import ctypes as C

import numpy as np
import pytest

import workloads
from paper_2603_27279_amd import _lib as L
from test_capi import _desc

HM = dict(contact_on=True, contact_model=1, contact_hm=(C.c_double * 5)(2.0, 0.3, 0.5, 0.05, 0.02))
TERMS = {
    "none": dict(dipole_on=False, contact_on=False), "contact": dict(dipole_on=False, contact_on=True),
    "hm": dict(HM, dipole_on=False), "dipole": dict(dipole_on=True, contact_on=False),
    "dipole+contact": dict(dipole_on=True, contact_on=True), "dipole+hm": dict(HM, dipole_on=True),
}


def workspace(members, n, terms, precision):
    lens = [n] * members
    org = [(0.0, 0.0, 0.0)] * members
    x, off, mem = workloads.straight_rods(lens, org, (0, 0, 1), member=np.arange(members))
    w = workloads._base(x, off, mem, np.tile([1.0, 1.0, 1.0, 0.5], (members, 1)), 0 * x,
                        np.zeros(len(x), np.int8), workloads._field_const(members, (0, 0, 0.1)))
    w["contact_on"] = w["dipole_on"] = False
    d, keep = _desc(w, precision=precision, **TERMS[terms])
    b = C.c_size_t()
    assert L.load().rod_query_workspace(C.byref(d), C.byref(b)) == L.ROD_OK
    return b.value


PER_MEMBER = 8 * 8 + 4 + 4 * 3 + 4 + 8 * 9 + 8 * 9  # tables and sums of a rod that is a member


# (members, particles, terms): with the planes or without, FP64 and mixed
@pytest.mark.parametrize("members,n,terms,fp64,mixed", [
    (16, 256, "none", True, True), (12, 257, "none", False, False), (64, 128, "none", False, False),
    (500, 5, "none", False, False), (100, 200, "none", False, False),
    (16, 256, "contact", True, True), (16, 512, "contact", False, False),
    (128, 64, "contact", True, True), (129, 64, "contact", False, False),
    (256, 16, "hm", True, True), (16, 512, "hm", False, False), (256, 64, "hm", False, False),
    (32, 200, "dipole", True, True), (4, 1024, "dipole", True, True), (3, 1025, "dipole", False, False),
    (128, 96, "dipole", False, True), (100, 200, "dipole", False, False),
    (4, 1024, "dipole+contact", False, True), (8, 512, "dipole+contact", True, True), (16, 512, "dipole+contact", False, False),
    (400, 64, "dipole+contact", True, True), (400, 20, "dipole+contact", False, False),
    (16, 512, "dipole+hm", False, False), (400, 64, "dipole+hm", True, True),
    (511, 64, "dipole+hm", True, True), (512, 64, "dipole+hm", False, False),
])
def test_planes_of_one_launch_steps(members, n, terms, fp64, mixed):
    """Against one member of as many particles, more than the layout takes."""
    N = members * n
    assert N > 2048
    for prec, planes, want in ((L.ROD_FP64, 16, fp64), (L.ROD_MIXED, 18, mixed)):
        extra = workspace(members, n, terms, prec) - workspace(1, N, terms, prec)
        assert extra - PER_MEMBER * (members - 1) == (8 * planes * N if want else 0)


@pytest.mark.parametrize("members,n,terms,want", [
    (8, 256, "contact", True), (7, 257, "contact", False), (2, 1024, "dipole", True),
    (1, 1500, "dipole", False), (1, 1024, "dipole", True), (8, 256, "dipole+contact", True),
    (1, 2048, "dipole+contact", False), (1, 1024, "dipole+contact", True), (5, 33, "contact", True),
])
def test_planes_up_to_2048_particles(members, n, terms, want):
    """Against single particles, which take many steps per launch and no planes."""
    N = members * n
    for prec, planes in ((L.ROD_FP64, 16), (L.ROD_MIXED, 18)):
        extra = workspace(members, n, terms, prec) - workspace(N, 1, terms, prec)
        assert extra + PER_MEMBER * (N - members) == (8 * planes * N if want else 0)


def test_planes_without_pair_terms():
    """1,024 particles without dipoles or contact take one-launch steps and 1,025 do not."""
    for prec, planes in ((L.ROD_FP64, 16), (L.ROD_MIXED, 18)):
        drop = workspace(1, 1024, "none", prec) - workspace(1, 1025, "none", prec)
        assert abs(drop - 8 * planes * 1024) <= 1500
