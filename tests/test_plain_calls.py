"""Calls as users make them: no counters and no explicit method parameters
(a call that asks for either runs the delegate method or the radix select).
The problems of the random sweep and the sizes of the single-problem and 64-bit
tests against the oracle element by element; shares of millions of keys, where
buckets are parts of the space between samples and some hold more than a
workgroup sorts at once, against a stable sort; and full sizes, positions
beyond 2^31 among them, against the delegate method."""
import sys

import numpy as np
import pytest

import synth
import test_random_sweep
from checks import check_exact, to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

drt = pytest.importorskip("paper_2109_08219_amd")


def say(*a):
    print("[case]", *a, file=sys.stderr, flush=True)


def compare(t, x, dt, k, largest, tag):
    say(tag)
    v, i = drt.topk_select(t, k, largest=largest, check=True)
    kth = drt.kth_select(t, k, largest=largest, check=True)
    check_exact(x, k, dt, to_np(v), to_np(i), tag, largest=largest)
    assert to_np(kth).tobytes() == to_np(v)[-1:].tobytes(), tag


@pytest.mark.parametrize("part", range(4))
def test_random_sweep_plain(part):
    for kind, n, k, largest, _, s in test_random_sweep.draw_cases(150, 777 + part):
        x, dt = synth.keys(kind, n, s)
        compare(torch.from_numpy(x).cuda(), x, dt, k, largest, f"{kind} n={n} k={k} largest={largest}")


@pytest.mark.parametrize("kind", ["uniform_u32", "normal_f32", "sorted_f32", "revsorted_f32", "heavydup_u32",
                                  "uniform_i32", "smallrange_i32"])
def test_sizes_and_k(kind):
    for n in (1, 3, 64, 1000, 8192, 8193, 65537, 300007, (1 << 20) + 13):
        x, dt = synth.keys(kind, n, 1000 + n)
        t = torch.from_numpy(x).cuda()
        for j, k in enumerate(sorted({k for k in (1, 2, 33, 1024, 8192, 8193, 20000, n) if 1 <= k <= n})):
            compare(t, x, dt, k, (n + j) % 2 == 0, f"{kind} n={n} k={k}")


@pytest.mark.parametrize("kind", ["uniform_u64", "uniform_i64", "normal_f64", "sorted_f64", "heavydup_u64",
                                  "smallrange_i64", "highword_u64"])
def test_sizes_and_k_wide(kind):
    for n in (1, 7, 1000, 8193, 65539, 300007, (1 << 22) + 17):
        x, dt = synth.keys(kind, n, 5000 + n)
        t = torch.from_numpy(x).cuda()
        for j, k in enumerate(sorted({k for k in (1, 17, 1000, 5000, n) if 1 <= k <= n})):
            compare(t, x, dt, k, (n + j) % 2 == 0, f"{kind} n={n} k={k}")


# ---------------------------------------------------------------------------
# Rank of every key, larger first, as a whole number (floats by totalOrder).
def rank_of(x, dt, largest):
    if dt[0] == "f":
        b = x.view(torch.int32 if dt == "f32" else torch.int64).long()
        r = b ^ ((b >> 63) & (0x7FFFFFFF if dt == "f32" else 0x7FFFFFFFFFFFFFFF))
    elif dt == "u32":
        r = x.long() & 0xFFFFFFFF
    elif dt == "u64":
        r = x ^ (-1 << 63)
    else:
        r = x.long()
    return r if largest else ~r


def share_keys(kind, n, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    normal = torch.randn(n, device="cuda", generator=g)
    if kind == "normal_f32":
        return normal, "f32"
    if kind == "bf16_f32":  # 16-bit values held in 32 bits: thousands of keys share each
        return normal.bfloat16().float(), "f32"
    if kind == "sorted_f32":
        return normal.sort().values, "f32"
    if kind == "clusters_i32":  # five values far apart
        return torch.randint(-2, 3, (n,), dtype=torch.int32, device="cuda", generator=g) * 10 ** 9, "i32"
    if kind == "ties_u32":
        return torch.randint(0, 16, (n,), dtype=torch.int32, device="cuda", generator=g), "u32"
    if kind == "uniform_u32":
        return torch.randint(-2 ** 31, 2 ** 31, (n,), dtype=torch.int32, device="cuda", generator=g), "u32"
    if kind == "normal_f64":
        return torch.randn(n, dtype=torch.float64, device="cuda", generator=g), "f64"
    if kind == "bf16_f64":
        return normal.bfloat16().double(), "f64"
    if kind == "ties_i64":
        return torch.randint(0, 16, (n,), dtype=torch.int64, device="cuda", generator=g), "i64"
    return torch.randint(-2 ** 62, 2 ** 62, (n,), dtype=torch.int64, device="cuda", generator=g), "u64"


@pytest.mark.parametrize("kind", ["normal_f32", "bf16_f32", "sorted_f32", "clusters_i32", "ties_u32", "uniform_u32",
                                  "normal_f64", "bf16_f64", "ties_i64", "uniform_u64"])
def test_shares_of_millions(kind):
    wide = kind.endswith("64")
    # an eighth, a sixteenth and the middle of millions: buckets that are parts of
    # the space between samples, up to 1300 of them (then a second launch takes the
    # ones too large for a workgroup); and a list of few, each bucket's workgroup
    # reading all of it
    sizes = [(1_500_001, 100_000), ((1 << 22) + 3, 1 << 18)] if wide else [
        (3_000_001, 375_000), ((1 << 24) + 5, 1 << 21), ((1 << 25) + 7, 10_000)]
    for n, k in sizes:
        x, dt = share_keys(kind, n, n % 1000)
        pay = torch.arange(n, dtype=torch.int64, device="cuda") * 3 + 1
        for largest in (True, False):
            order = rank_of(x, dt, largest).sort(descending=True, stable=True).indices
            say("share", kind, "n", n, "k", k, "largest", largest)
            v, i, p = drt.topk_select_payload(x, pay, k, dtype=dt, largest=largest)
            w, j = drt.topk_select(x, k, dtype=dt, largest=largest, check=True)
            bits = torch.int64 if wide else torch.int32
            assert torch.equal(i.long(), order[:k]) and torch.equal(j.long(), order[:k])
            assert torch.equal(v.view(bits), x[order[:k]].view(bits)) and torch.equal(w.view(bits), v.view(bits))
            assert torch.equal(p, pay[order[:k]])
            for r in (k, n // 2, n - k):
                say("k-th", kind, "n", n, "k", r, "largest", largest)
                kth = drt.kth_select(x, r, dtype=dt, largest=largest, check=True)
                assert torch.equal(kth.view(bits), x[order[r - 1:r]].view(bits)), (kind, n, r)


# ---------------------------------------------------------------------------
def against_delegates(x, dt, k, largest=True):
    say("against the delegate method:", dt, "n", x.numel(), "k", k, "largest", largest)
    v, i = drt.topk_select(x, k, dtype=dt, largest=largest, check=True)
    wv, wi, _ = drt.topk_select(x, k, dtype=dt, largest=largest, stats=True, check=True)
    bits = torch.int64 if x.element_size() == 8 else torch.int32
    assert torch.equal(i, wi) and torch.equal(v.view(bits), wv.view(bits)), (dt, x.numel(), k, largest)
    kth = drt.kth_select(x, k, dtype=dt, largest=largest, check=True)
    assert torch.equal(kth.view(bits), v[-1:].view(bits))


def test_full_size_32_bit():
    n = 1 << 30
    x = torch.empty(n, dtype=torch.int32, device="cuda").random_(-2 ** 31, 2 ** 31)
    for k in (2, 1024, 131072):
        against_delegates(x, "u32", k)
    against_delegates(x, "i32", 1024, False)
    x = torch.randn(n, device="cuda")
    for k in (1024, 131072):
        against_delegates(x, "f32", k)
    x = x[:1 << 29].sort().values
    against_delegates(x, "f32", 16384)
    against_delegates(x, "f32", 16384, False)
    x = torch.randint(0, 16, (1 << 29,), dtype=torch.int32, device="cuda")
    against_delegates(x, "u32", 16384)


def test_full_size_64_bit():
    n = (1 << 28) + 3
    x = torch.randn(n, dtype=torch.float64, device="cuda")
    for k in (1, 1024, 131072):
        against_delegates(x, "f64", k)
    x = torch.empty(1 << 29, dtype=torch.int64, device="cuda").random_(-2 ** 62, 2 ** 62)
    against_delegates(x, "i64", 16384)
    against_delegates(x, "u64", 16384, False)


def test_positions_beyond_2_31():
    n = (1 << 31) + 12345
    x = torch.empty(n, dtype=torch.int32, device="cuda")
    for i in range(0, n, 1 << 28):
        x[i:i + (1 << 28)].random_(-2 ** 31, 2 ** 31)
    x[-5:] = torch.tensor([-1, -2, -1, 7, -3], dtype=torch.int32, device="cuda")  # among the highest as uint32
    for k in (2, 1000, 100_003):
        against_delegates(x, "u32", k)
    against_delegates(x, "i32", 5000, False)
