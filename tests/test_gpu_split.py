"""Which tile runs: the split tiles of small FP32 quadrotor batches belong to the
default partition alone, hjpd_get_launch_timing names the tile that ran, and a
plan that was asked for runs as it says.  The rule's line (12 waves of the batch
per CU) on both sides, groups that refill, and graph replay; a point's results
are the same bits throughout."""
import numpy as np
import pytest

import workloads as W
from test_gpu_plan import _equal, _inputs, _run, _solver

pytestmark = pytest.mark.gpu

PLAN = [(8, 8, 1), (16, 16, 1), (32, 16, 2), (64, 32, 2)]  # the default partition of N_max = 64


def _batch(n, cap, tol=1e-30, hi=64):
    w = W.quadrotor12(n)
    w.N = np.random.default_rng(4).integers(17, hi + 1, n).astype(np.int32)
    w.t = 0.05 * w.N
    w.N_max, w.max_iter, w.tol = hi, cap, tol
    return w


def _tiles(s):
    return {(a["N_lo"], a["N_hi"]): (a["L"], a["K"]) for a in s.launch_timings()}


def _limit(lanes):
    import torch
    return 64 * 12 * torch.cuda.get_device_properties(0).multi_processor_count // lanes


@pytest.mark.parametrize("hi,over", [(32, 0), (32, 1), (64, 0), (64, 1)])
def test_default_partition_on_both_sides_of_the_line(hi, over):
    """The line lies where the widest split tile of the partition makes 12 waves per CU."""
    import torch
    n = _limit(hi) + over
    w = _batch(n, 6, hi=hi)
    s = _solver(w, torch.float32, timing=True)
    plan = [p for p in PLAN if p[0] <= hi]
    assert s.plan()[0] == plan
    inp = _inputs(w, torch.float32)
    a = _run(s, inp, traj=True)
    t = _tiles(s)
    assert t[(17, 32)] == ((16, 2) if over else (32, 1))
    assert hi == 32 or t[(33, 64)] == ((32, 2) if over else (64, 1))
    s.set_plan(plan)
    b = _run(s, inp, traj=True)
    t = _tiles(s)
    assert t[(17, 32)] == (16, 2) and (hi == 32 or t[(33, 64)] == (32, 2))
    _equal(a, b)
    s.close()


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_plans_asked_for_run_as_they_say(dtype):
    import torch
    td = torch.float32 if dtype == "f32" else torch.float64
    w = _batch(70, 5)
    inp = _inputs(w, td)
    s = _solver(w, td, timing=True)
    _run(s, inp)
    split = _tiles(s)[(17, 32)] == (32, 1)
    assert split == (dtype == "f32")  # no split tile is built in FP64
    s.set_plan(PLAN)
    with pytest.raises(Exception):
        s.set_plan([(64, 8, 1)])      # refused: the plan before it stays, as it was
    _run(s, inp)
    assert _tiles(s)[(17, 32)] == (16, 2) and _tiles(s)[(33, 64)] == (32, 2)
    s.close()
    s = _solver(w, td, timing=True)
    with pytest.raises(Exception):
        s.set_plan([(64, 8, 1)])
    _run(s, inp)
    assert (_tiles(s)[(17, 32)] == (32, 1)) == split
    s.autotune(*inp, probe_iters=3)
    _run(s, inp)
    lo = 1
    for hi, L, K in s.plan()[0]:
        assert _tiles(s)[(lo, min(hi, 64))] == (L, K)
        lo = hi + 1
    s.close()


def test_launch_timing_outlives_the_plan_it_was_taken_with():
    import torch
    w = _batch(40, 3)
    s = _solver(w, torch.float32, timing=True)
    s.set_plan(PLAN)
    _run(s, _inputs(w, torch.float32))
    before = _tiles(s)
    s.set_plan([(64, 32, 2)])
    assert _tiles(s) == before
    s.close()


def test_split_groups_refill_and_replay():
    """3,072 points make more groups than the split grid holds; the replayed
    graph is of the split kernels."""
    import torch
    w = _batch(_limit(64), 40, tol=1.0)
    inp = _inputs(w, torch.float32)
    s = _solver(w, torch.float32)
    s.set_plan(PLAN)
    want = _run(s, inp)
    s.close()
    assert len(np.unique(want["iters"])) > 2
    s = _solver(w, torch.float32, graph=True)
    out = s.alloc(w.n)
    for _ in range(3):
        out.phi.zero_()
        s.solve(*inp, out=out)
        torch.cuda.synchronize()
        _equal({"phi": out.phi.cpu().numpy(), "iters": out.iters.cpu().numpy(),
                "status": out.status.cpu().numpy()}, want)
    s.close()
