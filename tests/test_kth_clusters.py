"""k-th values whose bucket holds its keys in clusters inside clusters, on either
side of zero or of a shared prefix: the sort of a bucket divides the bin of the
wanted rank again until few keys are left in it.  Against a sort."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

drt = pytest.importorskip("paper_2109_08219_amd")


def say(*a):
    print("[case]", *a, file=sys.stderr, flush=True)


def nested(dtype, n, rng):
    sign = np.where(rng.random(n) < 0.5, -1.0, 1.0)
    if np.issubdtype(dtype, np.floating):
        reach = 512 if dtype == np.float64 else 64
        level = rng.choice([e for e in (1, 8, 64, 512) if e <= reach], n)
        return (sign * (0.5 + rng.random(n)) * 2.0 ** -level.astype(np.float64)).astype(dtype)
    bits = np.iinfo(dtype).bits
    top = bits - 2
    level = rng.integers(0, 1 + top // 10, n)
    r = (rng.integers(0, 2 ** 62, n, dtype=np.uint64) >> (62 - np.maximum(top - 10 * level, 1)).astype(np.uint64))
    if np.issubdtype(dtype, np.unsignedinteger):
        mid = 1 << (bits - 1)
        return np.where(sign < 0, np.uint64(mid) - np.minimum(r, np.uint64(mid)), np.uint64(mid) + r).astype(dtype)
    return (sign.astype(np.int64) * r.astype(np.int64)).astype(dtype)


@pytest.mark.parametrize("name", ["float32", "uint32", "int32", "float64", "uint64", "int64"])
def test_kth_of_clusters(name):
    dtype = np.dtype(name)
    rng = np.random.default_rng(len(name) + dtype.itemsize)
    for n in (300, 3000, 7000, 20000, 70001, 1 << 20):
        x = nested(dtype, n, rng)
        for kind in ("nested", "sorted"):
            if kind == "sorted":
                x = np.sort(x)
            want = np.sort(x)
            t = torch.from_numpy(x).cuda()
            for k in sorted({1, 2, n // 7, n // 3, n // 2 - 1, n // 2, n // 2 + 1, 5 * n // 6, n}):
                say(name, n, kind, k)
                got = drt.kth_select(t, k, check=True).cpu().numpy()
                assert got.tobytes() == want[n - k:n - k + 1].tobytes(), (name, n, kind, k)
                got = drt.kth_select(t, k, largest=False, check=True).cpu().numpy()
                assert got.tobytes() == want[k - 1:k].tobytes(), (name, n, kind, k)
