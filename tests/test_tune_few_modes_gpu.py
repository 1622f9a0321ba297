"""iwfpm_tune's time is that of the route which the plan's applies take: on a
few-mode plan the convolution's, a third or less of the transforms' on this grid
in float64 (70 against 330 us), so half of theirs separates the two."""

import pytest

import paper_2404_04507_amd as lib
from paper_2404_04507_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_tune_times_the_route_of_the_applies(tmp_path, monkeypatch):
    prob = W.c2_2d(lam=0.5)
    print(f"case: tune N={prob.N}", flush=True)
    monkeypatch.setenv("IWFPM_TUNE_CACHE", str(tmp_path / "tune"))
    with lib.Plan.from_problem(prob) as few:
        first, schedule = few.tune(nvec=16), few.schedule()
    line = (tmp_path / "tune").read_text().split()
    monkeypatch.delenv("IWFPM_TUNE_CACHE")
    with lib.Plan.from_problem(prob, schedule="threepass") as transforms:
        theirs = transforms.tune(nvec=16)
    assert 0.0 < first < 0.5 * theirs, (first, theirs)
    # the file keeps the schedule's own time, and the schedule is kept for solves
    assert float(line[-2]) > 0.5 * theirs and not schedule["fused"]
