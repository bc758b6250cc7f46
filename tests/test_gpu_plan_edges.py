"""Plans at the edges of their scans and lists: the box tables and every list equal the oracle's, bit for bit, also when
plans are built and destroyed in turn (released buffers are used again by the next plan)."""
import threading

import numpy as np
import pytest
import torch

import oracle
from paper_2202_01085_amd import f3m, inputs
from parity_util import TOL_F3M, assert_close, say
from test_gpu_parity import check_plan_bit_exact

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


# a scan is one block up to 2048 elements (256 counts per sort tile of 8192 keys: 65 536 keys); the largest box comes
# from one block up to 16 384 boxes; lists of more than three dimensions have rows of 1 to thousands of candidates,
# 64 at a time
@pytest.mark.parametrize("n,D,p,zeta,more", [
    (65_536, 3, 4, 16, {}), (65_537, 3, 4, 16, {}), (2_048, 1, 3, 1, {}), (2_049, 2, 3, 1, {}),
    (40_000, 2, 3, 2, {}),                                   # more than 16 384 leaf boxes
    (3_000, 4, 3, 8, {}), (5_000, 5, 2, 4, {}), (6_000, 6, 2, 16, {}), (4_001, 7, 2, 8, {}),
    (4_001, 4, 3, 16, dict(small_field=40)),
    (3_001, 3, 4, 16, dict(small_field=60)),
    (3_001, 4, 3, 16, dict(force_all_near=True, max_depth=2)),
])
def test_plan_tables(n, D, p, zeta, more):
    say("plan edges n=%d D=%d zeta=%d %r" % (n, D, zeta, more))
    X = inputs.points_normal(n, D, 91 + D)
    T = oracle.Tree(X.numpy(), theta=2.0, zeta=zeta, **more)
    plan = f3m.Plan(X.to(DEV), 1.0, p, 2.0, leaf_max=zeta, **more)
    check_plan_bit_exact(plan, T)
    plan.close()


def test_plans_in_turn_and_from_two_threads():
    """Buffers of a plan that is gone serve the next one, on other streams and threads too: the same bits every time."""
    sizes = [30_000, 3_000, 70_001]
    Xs = [inputs.points_uniform(n, 3, 95).to(DEV) for n in sizes]
    bs = [inputs.rhs_normal(n, 96).to(DEV) for n in sizes]

    def one(k):
        plan = f3m.Plan(Xs[k], 0.4, 4, 2.0)
        y = plan.kmvm(bs[k])
        plan.close()
        return y

    want = [one(k) for k in range(3)]
    torch.cuda.synchronize()
    T = oracle.Tree(Xs[1].cpu().numpy(), theta=2.0, zeta=128)
    assert_close(want[1].cpu().numpy(), T.apply(bs[1].cpu().numpy(), float(np.float32(0.4)), 4), TOL_F3M, "vs CPU F3M")
    bad = []

    def work():
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for i in range(6):
                y = one(i % 3)
                s.synchronize()
                if not torch.equal(y, want[i % 3]):
                    bad.append(i)

    threads = [threading.Thread(target=work) for _ in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


# overlap and the solver: the far field's last pass adds the near field, which another stream may have computed
@pytest.mark.parametrize("n,zeta,gamma", [(20_000, 128, 0.5), (30_001, 12, 1.7), (400, 128, 0.5)])
def test_solver_with_and_without_overlap(n, zeta, gamma):
    X = inputs.points_uniform(n, 3, 97).to(DEV)
    b = inputs.rhs_normal(n, 98).to(DEV)
    got = []
    for overlap in (False, True):
        plan = f3m.Plan(X, gamma, 4, 2.0, leaf_max=zeta, overlap=overlap)
        x, it, hist = plan.cg_solve(b, 0.1 * n, tol=0.0, max_iter=4)
        t = plan.stage_times()
        assert all(np.isfinite(v) and v >= 0.0 for v in t.values())
        got.append(x)
        res = float((plan.kmvm(x) + 0.1 * n * x - b).norm() / b.norm())
        assert abs(res - float(hist[-1])) <= 1e-5
        plan.close()
    assert torch.equal(got[0], got[1])


def test_downward_time_leaves_out_the_wait_for_the_near_field():
    """Large leaf boxes of depth 2: the near field takes some 5 ms and holds the chip, the far field gets through beside it
    shortly before its end, and with overlap the solver's last pass waits for the rest (0.13 of 0.15 ms), which is not its
    own time (0.02 ms)."""
    X = inputs.points_uniform(500_000, 3, 99).to(DEV)
    b = inputs.rhs_normal(500_000, 100).to(DEV)
    times = []
    for overlap in (False, True):
        plan = f3m.Plan(X, 0.5, 4, 2.0, leaf_max=10_000, overlap=overlap)
        for _ in range(2):
            plan.cg_solve(b, 5e4, tol=0.0, max_iter=3)
        t = plan.stage_times()
        say("overlap %d: p2p %.3f l2p %.3f ms, depth 2 %r" % (overlap, t["p2p"], t["l2p"], plan.level_times(2)))
        assert plan.info().depth == 2 and abs(plan.level_times(2)[2] - t["l2p"]) <= 1e-6
        times.append(t)
        plan.close()
    assert times[1]["p2p"] > 2.0 and times[1]["l2p"] <= 2.0 * times[0]["l2p"] + 0.03
