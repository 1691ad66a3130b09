"""Whole problems of a batch by either way of a workgroup, next to each other in
one launch (descriptors as arguments and staged), and those that overflow the
delegate method (ordered and tied keys), which are streamed: element by element
against the oracle, unaligned bases and k-selection alone among them."""
import sys

import numpy as np
import pytest

import oracle
import synth
from checks import check_exact, to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

drt = pytest.importorskip("paper_2109_08219_amd")

# (n, k): few of many, most of a few, either side of the rule's lines
SIZES = [(64, 64), (1000, 512), (1024, 200), (3000, 190), (4096, 90), (4096, 600), (4097, 1), (5000, 40), (6144, 30),
         (6145, 3000 // 2), (7680, 8), (7681, 40), (8192, 500), (9001, 64), (12000, 600), (17999, 2), (31000, 4),
         (50001, 2), (65536, 1), (65536, 700)]


@pytest.mark.parametrize("table", [True, False])  # tuned plans (radix selects among them) and Rule 4's
@pytest.mark.parametrize("count", [20, 60, 300])
def test_mixed_ways(count, table):
    kinds = ["uniform_u32", "normal_f32", "sorted_f32", "heavydup_u32", "smallrange_i32"]
    hosts = []
    for j in range(count):
        n, k = SIZES[j % len(SIZES)]
        x, dt = synth.keys(kinds[(j + j // len(SIZES)) % len(kinds)], n, 60 + j % 40)
        hosts.append((x, dt, k, j % 4, j % 3 != 0))
    tensors = [(torch.from_numpy(np.concatenate([np.zeros(off, x.dtype), x])).cuda()[off:], k, dt, largest)
               for x, dt, k, off, largest in hosts]
    saved = drt.tune_get()
    try:
        if not table:
            drt.tune_set([])
        print("[case] mixed ways", count, "table", table, file=sys.stderr, flush=True)
        b = drt.Batch(tensors)
        b.run(check=True)
        kth = drt.Batch(tensors, kth_only=True)
        kth.run(check=True)
    finally:
        drt.tune_set(saved)
    for i, (x, dt, k, off, largest) in enumerate(hosts):
        tag = f"#{i} n={x.shape[0]} k={k} {dt} off={off} largest={largest}"
        check_exact(x, k, dt, to_np(b.values(i)), to_np(b.indices(i)), tag, largest=largest)
        want = np.asarray(oracle.kth_value(x, k, dt, largest)).tobytes()
        assert to_np(kth.kth_value(i)).tobytes() == want == to_np(b.kth_value(i)).tobytes(), tag


@pytest.mark.parametrize("way", ["low", "few"])
def test_only_one_way(way):
    # every problem by the delegate method (k small, few lists), ordered so that it overflows
    n, k = (65536, 2) if way == "few" else (40001, 8)
    x, dt = synth.keys("sorted_f32" if way == "few" else "heavydup_u32", n, 5)
    t = torch.from_numpy(x).cuda()
    for count in (2, 40):
        b = drt.Batch([(t, k)] * count)
        b.run(check=True)
        for i in (0, count - 1):
            check_exact(x, k, dt, to_np(b.values(i)), to_np(b.indices(i)), f"{way} {count} #{i}")
