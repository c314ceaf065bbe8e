"""A G2P in the launch of the next sub-step's P2G (consecutive sub-steps without
a binning between them) against separate launches: the same sub-steps taken
one call each never join.  FP32 states agree bit for bit (the same arithmetic
per particle; FP64 window sums rounded to FP32); FP64 states to the order of
FP64 sums, 1e-16 a term over at most 7 sub-steps: 1e-13."""
import sys

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _run(ddm, w, prec, sort_every, calls, record):
    cfg, inst = ddm.from_workload(w, max_steps=8, checkpoint_every=4, precision=prec, sort_every=sort_every)
    sim = ddm.Simulator(cfg, [inst])
    sim.init_state(W.bed_positions(w))
    for n in calls:
        sim.rollout(n) if record else sim.step(n)
    err = sim.check()
    assert err.flags == 0
    return sim.packed_state(0)


# one binning at the start, binnings inside the run, more particles than a
# workgroup of either width takes at once
@pytest.mark.parametrize("sort_every", [0, 3])
@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("case", ["tiny2d", "tiny3d", "dig"])
def test_joined_launches_equal_separate_ones(case, prec, sort_every):
    import paper_2510_17335_amd as ddm
    w = {"tiny2d": lambda: W.tiny(2), "tiny3d": lambda: W.tiny(3, shovel=True), "dig": lambda: W.dig_3d(steps=8)}[case]()
    w.precision = prec
    print("case", case, prec, sort_every, flush=True)
    sys.stdout.flush()
    one = _run(ddm, w, prec, sort_every, [1] * 7, False)
    for record in (False, True):
        many = _run(ddm, w, prec, sort_every, [7], record)
        if prec == "f32" and not record:
            assert np.array_equal(one, many)
        else:
            # (a recorded run bins at its checkpoints as well, which reorders sums)
            tol = 1e-13 if prec == "f64" else 1e-5
            assert np.linalg.norm(one - many) <= tol * np.linalg.norm(one)
