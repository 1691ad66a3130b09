"""Problems of a batch that one workgroup takes in one pass, element by element against the oracle: the sizes where the
first cut comes from no sample, a small or a large one, chunk remainders and unaligned bases, ties and all-equal keys,
ordered inputs, inputs whose sampled places misjudge the rest in either direction, and large problems that stay whole
because the batch has many."""
import sys

import numpy as np
import pytest

import synth
from checks import check_exact, to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

drt = pytest.importorskip("paper_2109_08219_amd")


def run(hosts, largest, repeat=1):
    """hosts: (x, dtype, k, offset).  `repeat` > 1: each problem that often, to the same outputs' values."""
    tensors = []
    for x, dt, k, off in hosts:
        t = torch.from_numpy(np.concatenate([np.zeros(off, x.dtype), x])).cuda()[off:]
        tensors += [(t, k, dt, largest)] * repeat
    b = drt.Batch(tensors)
    b.run(check=True)
    for i, (x, dt, k, off) in enumerate(hosts):
        for j in (i * repeat, i * repeat + repeat - 1):
            tag = f"n={x.shape[0]} k={k} {dt} off={off} largest={largest}"
            print("[case]", tag, file=sys.stderr, flush=True)
            check_exact(x, k, dt, to_np(b.values(j)), to_np(b.indices(j)), tag, largest=largest)


# sorted whole or selected first; below and at the LDS's capacity, chunk remainders, the samples' limits
SIZES = [(1, 1), (2, 2), (511, 511), (1024, 1024), (1025, 128), (1025, 129), (4096, 512), (4096, 513),
         (4097, 1), (4097, 2048), (7680, 2048), (7681, 2048), (7681, 1), (8192 + 5, 700), (65537, 2047), (131071, 2048),
         (131072, 2048), (200003, 33)]


@pytest.mark.parametrize("largest", [True, False])
@pytest.mark.parametrize("kind", ["uniform_u32", "normal_f32", "sorted_f32", "heavydup_u32", "bits_f32", "equal_u32", "edge_i32"])
def test_against_oracle(kind, largest):
    hosts = []
    for j, (n, k) in enumerate(SIZES):
        rng = np.random.default_rng(n + k)
        if kind == "bits_f32":
            x, dt = rng.integers(0, 1 << 32, n, dtype=np.uint32).view(np.float32), "f32"
        elif kind == "equal_u32":
            x, dt = np.full(n, [0, 7, 0xFFFFFFFF][j % 3], np.uint32), "u32"
        elif kind == "edge_i32":
            x, dt = np.where(rng.random(n) < 0.5, -2 ** 31, 2 ** 31 - 1).astype(np.int32), "i32"
        else:
            x, dt = synth.keys(kind, n, n + k)
        hosts.append((x, dt, k, j % 4))
    run(hosts[:13], largest)          # descriptors as arguments
    run(hosts, largest, repeat=8)     # staged descriptors


def sampled_places(n):
    """Places that the first cut's sample reads."""
    h = np.arange(128 * (1 if n < 1 << 17 else 3), dtype=np.uint64)
    g = h.copy()
    m = np.uint64(0xFFFFFFFF)
    h = (h ^ (h >> np.uint64(16))) * np.uint64(0x7FEB352D) & m
    h = (h ^ (h >> np.uint64(15))) * np.uint64(0x846CA68B) & m
    h ^= h >> np.uint64(16)
    G = np.uint64(len(g))
    lo, hi = g * np.uint64(n) // G, (g + np.uint64(1)) * np.uint64(n) // G
    p = (lo + (h * (hi - lo) >> np.uint64(32))) & ~np.uint64(15)
    p = (p[:, None] + np.arange(16, dtype=np.uint64)).reshape(-1).astype(np.int64)
    return np.unique(p[p < n])


@pytest.mark.parametrize("n,k", [(40001, 2000), (150000, 2048)])
@pytest.mark.parametrize("way", ["high", "low"])
def test_misjudged(n, k, way):
    rng = np.random.default_rng(n)
    p = sampled_places(n)
    x = rng.integers(1 << 20, 1 << 21, n, dtype=np.uint32)
    if way == "high":   # fewer than k reach the cut: every high key is one of the sample
        x[rng.permutation(p)[:k // 3]] = rng.integers(1 << 30, 1 << 31, k // 3, dtype=np.uint32)
    else:               # the sample is below everything: the cut keeps nearly all
        x[p] = rng.integers(0, 1 << 10, p.size, dtype=np.uint32)
    run([(x, "u32", k, 0)] * 2, True, repeat=20)


def test_large_whole():
    # 520 equal problems: each at most a slot's share, so none is split
    x, dt = synth.keys("normal_f32", 300001, 5)
    y, dy = synth.keys("sorted_f32", 300001, 6)
    run([(x, dt, 2048, 0), (y, dy, 777, 0)], True, repeat=520)
