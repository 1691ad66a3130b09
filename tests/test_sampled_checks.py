"""Internal checks of plain calls reach drtopk_check.

The run-capacity testing hook makes, from the host, what a misjudged sample's
rescue or a run of an oversized bucket collects smaller than it needs: the
kernels drop the writes past the cap, raise flag 16 (capacity) and 2 (fewer
elements than the histogram promised), and exit normally.  The flags must arrive
through plain calls of every entry point, per stream, and be cleared by the
check."""
import sys

import numpy as np
import pytest

import synth
from checks import check_exact, to_np
from test_sampled import sampled_positions

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

drt = pytest.importorskip("paper_2109_08219_amd")


def say(*a):
    print("[case]", *a, file=sys.stderr, flush=True)


@pytest.fixture
def capped():
    drt.check()  # nothing left over from earlier tests on this stream
    drt.set_run_cap(50)
    drt.fix_sample(0)
    try:
        yield
    finally:
        drt.set_run_cap(0)
        drt.fix_sample(None)


def misjudged(n, M, dt="u32"):
    """The sampled keys lie below all others: the cut keeps far too many."""
    x, _ = synth.keys(f"uniform_{dt}", n, 31)
    top = np.array(1 << (63 if dt == "u64" else 31), x.dtype)
    x |= top
    x[sampled_positions(n, M)] ^= top
    return x


def flagged(stream=None):
    with pytest.raises(drt.DrTopkError) as e:
        drt.check(stream)
    assert e.value.flags & 18 == 18, e.value.flags
    drt.check(stream)  # cleared


# one workgroup; one bucket; buckets of rows
@pytest.mark.parametrize("dt", ["u32", "u64"])
@pytest.mark.parametrize("n,k,M", [(20000, 100, 256), (1 << 20, 1024, 65536), (1 << 20, 200000, 8192)])
def test_rescue_is_checked(n, k, M, dt, capped):
    x = misjudged(n, M, dt)
    t = torch.from_numpy(x).cuda()
    say("capped rescue", dt, n, k)
    drt.topk_select(t, k)  # plain call: returns OK, enqueue only
    flagged()
    drt.set_run_cap(0)
    v, i = drt.topk_select(t, k, check=True)
    check_exact(x, k, dt, to_np(v), to_np(i), f"{dt} n={n} k={k} after the cap is lifted")


def test_runs_of_an_oversized_bucket_are_checked(capped):
    n, k = (1 << 24) + 5, 1 << 21  # 16-bit values: dozens of buckets above a workgroup's capacity
    x = torch.randn(n, device="cuda").bfloat16().float()
    say("capped runs")
    drt.topk_select(x, k)
    flagged()
    drt.set_run_cap(0)
    v, i = drt.topk_select(x, k, check=True)
    order = x.sort(descending=True, stable=True).indices[:k]
    assert torch.equal(i.long(), order) and torch.equal(v, x[order])


def test_flags_are_per_stream_and_of_every_entry(capped):
    n, k = 1 << 20, 1024
    t = torch.from_numpy(misjudged(n, 65536)).cuda()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        say("capped call on a side stream")
        drt.topk_select(t, k, stream=s)
    drt.check()
    flagged(s)
    say("capped payload call")
    drt.topk_select_payload(t, torch.arange(n, device="cuda"), k)
    flagged()
    say("capped call without allocation")
    vals, idx = torch.empty(k, dtype=torch.int32, device="cuda"), torch.empty(k, dtype=torch.int32, device="cuda")
    drt.topk_select_noalloc(t, k, vals, idx, dtype="u32")
    flagged()


def test_server_fails_flagged_request(capped):
    n, k = (1 << 22) + 1, 1024
    t = torch.from_numpy(misjudged(n, 65536)).cuda()
    b = drt.Batch([(t, k)])
    with drt.Server(streams=1, max_batch=1) as srv:
        say("server: capped request")
        ticket = srv.submit(b, 0)
        with pytest.raises(drt.DrTopkError) as e:
            srv.wait(ticket)
        assert e.value.status == 3
        with pytest.raises(drt.DrTopkError):
            srv.drain()
