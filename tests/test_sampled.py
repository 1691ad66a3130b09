"""The sampled path (plain topk_select / kth_select calls) element by element against the oracle: its smallest inputs, tile and stage
remainders, unaligned heads, open and two-sided windows, one bucket, many
buckets and two levels, keys clustered on few values, ties and all-equal keys,
every bit pattern of a float, and inputs whose sampled positions misjudge the
rest in either direction (the answer then comes from the input itself)."""
import sys

import numpy as np
import pytest

import synth
from checks import check_exact, to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

drt = pytest.importorskip("paper_2109_08219_amd")


def say(*a):
    print("[case]", *a, file=sys.stderr, flush=True)


def keys_of(kind, n, seed):
    rng = np.random.default_rng(seed)
    if kind == "bits_f32":  # every class of float: NaNs, infinities, zeros, subnormals
        return rng.integers(0, 1 << 32, n, dtype=np.uint32).view(np.float32), "f32"
    if kind == "bits_f64":
        return rng.integers(0, 1 << 64, n, dtype=np.uint64).view(np.float64), "f64"
    if kind == "sparse_f32":  # 1% of the keys nonzero
        return (rng.integers(1, 1000, n) * (rng.random(n) < 0.01)).astype(np.float32), "f32"
    if kind == "clusters_i32":  # five far-apart values
        return (rng.integers(-2, 3, n) * 10 ** 9).astype(np.int32), "i32"
    if kind == "edge_u32":  # the type's lowest and highest values, tied
        return np.where(rng.random(n) < 0.5, np.uint32(0), np.uint32(0xFFFFFFFF)).astype(np.uint32), "u32"
    if kind == "equal_u64":
        return np.full(n, 5, np.uint64), "u64"
    return synth.keys(kind, n, seed)


KINDS = ["uniform_u32", "bits_f32", "normal_f32", "sorted_f32", "heavydup_u32", "sparse_f32", "clusters_i32", "edge_u32",
         "normal_f64", "bits_f64", "heavydup_u64", "equal_u64"]


def compare(x, dt, k, largest, tag, off=0):
    t = torch.from_numpy(x).cuda()
    if off:
        buf = torch.empty(t.numel() + off, dtype=t.dtype, device="cuda")
        buf[off:] = t
        t = buf[off:]
    say(tag)
    v, i = drt.topk_select(t, k, largest=largest, check=True)
    kth = drt.kth_select(t, k, largest=largest, check=True)
    check_exact(x, k, dt, to_np(v), to_np(i), tag, largest=largest)
    assert to_np(kth).tobytes() == to_np(v)[-1:].tobytes(), tag


@pytest.mark.parametrize("kind", KINDS)
def test_against_oracle(kind):
    # (n, k): the smallest inputs of both samples, remainders of a tile and a
    # stage, k a fixed share, the middle, k = n, and k that leave one bucket
    cases = [(16384, 2049), (16385, 16385), (65537, 300), (131072, 3000), (131071, 130000), (524288 + 1, 262145),
             (1048576 - 8191, 131000), (1 << 21, 20)]
    for j, (n, k) in enumerate(cases):
        x, dt = keys_of(kind, n, 9000 + j)
        off = 0 if x.dtype.itemsize == 8 else j % 4
        compare(x, dt, k, j % 3 != 1, f"{kind} n={n} k={k} off={off}", off)


@pytest.mark.parametrize("kind", KINDS)
def test_one_workgroup(kind):
    # the sizes one workgroup takes: every element sorted (its LDS exactly full
    # and beyond), the cut by 256 samples, heads and remainders of 16-byte loads,
    # few and most of the elements wanted
    cases = [(1, 1), (3, 2), (257, 256), (1024, 3), (1025, 1025), (4096, 4095), (4097, 5), (8192, 8192), (8193, 100),
             (40001, 2), (65536, 1500), (65535, 2500)]
    for j, (n, k) in enumerate(cases):
        x, dt = keys_of(kind, n, 9100 + j)
        off = 0 if x.dtype.itemsize == 8 else j % 4
        compare(x, dt, k, j % 3 != 1, f"{kind} n={n} k={k} off={off}", off)


# sample i of M lies in stratum [i n / M, (i + 1) n / M) at this hash of i
def sampled_positions(n, M):
    h = np.arange(M, dtype=np.uint64)
    x = h.copy()
    m32 = np.uint64(0xFFFFFFFF)
    x = ((x ^ (x >> np.uint64(16))) * np.uint64(0x7FEB352D)) & m32
    x = ((x ^ (x >> np.uint64(15))) * np.uint64(0x846CA68B)) & m32
    x ^= x >> np.uint64(16)
    lo, hi = h * np.uint64(n) // np.uint64(M), (h + np.uint64(1)) * np.uint64(n) // np.uint64(M)
    return (lo + ((x * (hi - lo)) >> np.uint64(32))).astype(np.int64)


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("high", [True, False])
def test_misjudged_samples(wide, high):
    # the sampled positions hold only keys above (high) or below all others:
    # too few elements reach the cut, or more than the buffer holds do
    n, dt = 1 << 20, "u64" if wide else "u32"
    for k, M in ((1024, 65536), (200000, 8192)):
        x, _ = synth.keys(f"uniform_{dt}", n, 31)
        x = x >> 1 if high else x | (1 << (63 if wide else 31))
        p = sampled_positions(n, M)
        x[p] ^= np.array(1 << (63 if wide else 31), x.dtype)
        compare(x, dt, k, True, f"misjudged {dt} k={k} high={high}")


@pytest.mark.parametrize("high", [True, False])
def test_misjudged_samples_of_one_workgroup(high):
    n, k = 50000, 300
    x, _ = synth.keys("uniform_u32", n, 33)
    x = x >> 1 if high else x | (1 << 31)
    x[sampled_positions(n, 256)] ^= np.uint32(1 << 31)
    compare(x, "u32", k, True, f"misjudged one workgroup high={high}")


@pytest.mark.parametrize("dtype", ["f32", "i64"])
def test_two_levels(dtype):
    # more than 4096 (8-byte keys: 2048) elements a sample: the candidates are
    # sampled again; compared with the delegate method and its checks
    t = {"f32": torch.float32, "i64": torch.int64}[dtype]
    n = (1 << 28) + 12345 if dtype == "f32" else (1 << 27) + 12345
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    x = torch.randn(n, device="cuda", generator=g)
    x = x if t == torch.float32 else (x * 1e5).to(t)  # int64: many ties
    for k, largest in ((30, True), (5000, False), (100003, True)):
        say("two levels", dtype, "k", k, "largest", largest)
        v, i = drt.topk_select(x, k, largest=largest, check=True)
        wv, wi, _ = drt.topk_select(x, k, largest=largest, stats=True, check=True)
        kth = drt.kth_select(x, k, largest=largest, check=True)
        assert torch.equal(v, wv) and torch.equal(i, wi) and kth[0] == wv[-1], (dtype, k)


def test_two_levels_misjudged():
    n = (1 << 28) + (1 << 20)
    x = torch.zeros(n, dtype=torch.float32, device="cuda")
    x[torch.from_numpy(sampled_positions(n, 65536)).cuda()] = 2.0  # 65536 tied samples at the top
    x[123456789] = 1.0
    for k in (100000, 65537):  # reaches past them: the cut keeps far fewer than k
        say("two levels misjudged k", k)
        v, i = drt.topk_select(x, k, check=True)
        wv, wi, _ = drt.topk_select(x, k, stats=True, check=True)
        assert torch.equal(v, wv) and torch.equal(i, wi)


def test_graph_replay():
    n, k = 1 << 20, 1024
    x = torch.randn(n, device="cuda")
    vals, idx = torch.empty(k, device="cuda"), torch.empty(k, dtype=torch.int32, device="cuda")
    drt.topk_select_noalloc(x, k, vals, idx)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        drt.topk_select_noalloc(x, k, vals, idx)
    for rep in range(4):
        say("graph replay", rep)
        x.normal_()
        vals.zero_()
        g.replay()
        torch.cuda.synchronize()
        order = x.sort(descending=True, stable=True).indices[:k]
        assert torch.equal(idx.long(), order) and torch.equal(vals, x[order])
