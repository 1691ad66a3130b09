"""Inputs that misjudge the sample.  With the sampled places fixed, the answer
comes from the input itself (both directions, one and two levels, calls of one
launch of buckets and of two); without, the same input is not misjudged, since
the process samples other places."""
import sys

import numpy as np
import pytest

import synth
import test_sampled
from checks import check_exact, to_np
from test_sampled import sampled_positions

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

drt = pytest.importorskip("paper_2109_08219_amd")


def say(*a):
    print("[case]", *a, file=sys.stderr, flush=True)


@pytest.fixture
def fixed():
    drt.fix_sample(0)
    try:
        yield
    finally:
        drt.fix_sample(None)


def rescued(call):
    """Whether a call with the run capacity capped had to collect from the input."""
    drt.check()
    drt.set_run_cap(50)
    try:
        call()
        drt.check()
        return False
    except drt.DrTopkError as e:
        assert e.flags & 18
        return True
    finally:
        drt.set_run_cap(0)


def misjudged(n, M, dt, high):
    bit = np.array(1 << (63 if dt == "u64" else 31), np.uint64 if dt == "u64" else np.uint32)
    x, _ = synth.keys(f"uniform_{dt}", n, 31)
    x = x & ~bit if high else x | bit
    x[sampled_positions(n, M)] ^= bit
    return x


# one bucket; some hundred buckets; more of them than one launch takes with its rare ways
@pytest.mark.parametrize("high", [True, False])
@pytest.mark.parametrize("dt,n,k,M", [("u32", 1 << 20, 1024, 65536), ("u64", 1 << 20, 1024, 65536),
                                      ("u32", 1 << 20, 200000, 8192), ("u64", 1 << 20, 200000, 8192),
                                      ("u32", (1 << 24) + 5, 1 << 21, 8192), ("u64", (1 << 22) + 3, 1 << 18, 8192)])
def test_rescue(dt, n, k, M, high, fixed):
    x = misjudged(n, M, dt, high)
    t = torch.from_numpy(x).cuda()
    say("rescue", dt, "n", n, "k", k, "high", high)
    assert rescued(lambda: drt.topk_select(t, k))
    v, i = drt.topk_select(t, k, check=True)
    check_exact(x, k, dt, to_np(v), to_np(i), f"{dt} n={n} k={k} high={high}")
    kth = drt.kth_select(t, k, check=True)
    assert to_np(kth).tobytes() == to_np(v)[-1:].tobytes()
    drt.fix_sample(None)
    say("other places", dt, "n", n, "k", k, "high", high)
    if n == 1 << 20:  # (with buckets of thousands of keys, one may be collected in runs, which the cap shows as well)
        assert not rescued(lambda: drt.topk_select(t, k))
    v, i = drt.topk_select(t, k, check=True)
    check_exact(x, k, dt, to_np(v), to_np(i), f"other places {dt} n={n} k={k} high={high}")


def test_rescue_of_two_levels(fixed):
    test_sampled.test_two_levels_misjudged()


def test_graph_replays_keep_their_places(fixed):
    # captured with fixed places, replayed on an input that they misjudge and on one that they do not
    n, k = 1 << 20, 1024
    t = torch.empty(n, dtype=torch.int32, device="cuda").random_(0, 1 << 30)
    vals, idx = torch.empty(k, dtype=torch.int32, device="cuda"), torch.empty(k, dtype=torch.int32, device="cuda")
    drt.topk_select_noalloc(t, k, vals, idx, dtype="u32")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        drt.topk_select_noalloc(t, k, vals, idx, dtype="u32")
    drt.fix_sample(None)
    for rep in range(4):
        x = misjudged(n, 65536, "u32", rep % 3 == 0) if rep % 2 == 0 else synth.keys("uniform_u32", n, rep)[0]
        t.copy_(torch.from_numpy(x.view(np.int32)))
        say("replay", rep)
        g.replay()
        torch.cuda.synchronize()
        check_exact(x, k, "u32", to_np(vals).view(np.uint32), to_np(idx), f"replay {rep}")


@pytest.mark.parametrize("dt,n,k,high", [("u32", 2_400_000, 2048, 7715), ("u64", 1_120_000, 1024, 3650)])
def test_more_candidates_than_a_workgroup_sorts(dt, n, k, high, fixed):
    # one bucket by the plan; its buffer holds some more than a workgroup sorts at
    # once, and the cut lets `high` through: the lowest of them are 129 sampled keys
    rng = np.random.default_rng(3)
    x, _ = synth.keys(f"uniform_{dt}", n, 31)
    bit = np.array(1 << (63 if dt == "u64" else 31), x.dtype)
    x &= ~bit
    p = sampled_positions(n, 65536)
    x[rng.choice(p, 129, replace=False)] = bit
    rest = rng.choice(np.setdiff1d(np.arange(n), p), high - 129, replace=False)
    x[rest] |= bit | np.array(1, x.dtype)
    t = torch.from_numpy(x).cuda()
    say("one bucket in runs", dt, n, k)
    assert rescued(lambda: drt.topk_select(t, k))  # (the cap shows runs as well)
    v, i = drt.topk_select(t, k, check=True)
    check_exact(x, k, dt, to_np(v), to_np(i), f"one bucket in runs {dt}")
