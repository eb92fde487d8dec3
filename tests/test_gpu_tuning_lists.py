"""The autotuner times every distinct work list: equal numbers of work items can be other
slots in other parts."""
import re

import pytest

import workloads
from paper_2603_27279_amd import RodSim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,prec,targets", [
    # 128 blocks of 64 targets in 4, 8, 16, 32 and 64 slots
    (8192, "fp64", [512, 1024, 2048, 4096, 8192]),
    # the first three all 2048 items: 4 slots of 4 parts, 8 of 2, 16 whole ones
    (8192, "mixed", [512, 1024, 2048, 4096, 8192]),
    (16384, "mixed", [512, 1024, 2048, 4096, 8192, 16384, 32768]),
])
def test_every_distinct_work_list_is_timed(n, prec, targets):
    w = workloads.twisted_rod(n=n)
    sim = RodSim(w, precision=prec)
    report = sim.autotune()
    for name in ("split", "spatial split"):
        got = [int(t) for t in re.findall(rf"^{name} layout target_wgs=(\d+) ", report, re.M)]
        assert got == targets, (name, report)
    sim.free()
