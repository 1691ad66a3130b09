"""A batch with more tiles of split problems than run at once: items claimed by
a grid that stays (the whole problems then run the delegate method, the radix
select or a sort inside a workgroup).  Against the oracle element by element,
with one and two delegates per subrange, unaligned bases, ties and ordered keys,
next to many short problems."""
import sys

import numpy as np
import pytest

import synth
from checks import check_exact, to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

drt = pytest.importorskip("paper_2109_08219_amd")


def tiles(n, k):
    """Workgroups of a split problem by its plan: 2^18 keys each, fewer where a tile's
    delegates (at most 4096) cover fewer; problems up to 2^16 keys are not split."""
    r, alpha, beta = drt.batched_plan(n, k)
    if r != 2 or n <= 1 << 16 or alpha < 4:
        return 1
    log = min(alpha + 12 - (beta > 1), max(alpha, 18))
    return -(-n // (1 << log))


@pytest.mark.parametrize("beta", [1, 2])
def test_more_tiles_than_run_at_once(beta):
    rng = np.random.default_rng(100 + beta)
    base = {}
    for kind in ("uniform_u32", "normal_f32", "heavydup_u32", "sorted_f32"):
        x, dt = synth.keys(kind, 1 << 21, 50 + beta)
        base[kind] = (x, dt, torch.from_numpy(x).cuda())
    lists = []
    for i in range(300):  # long ones: slices of four arrays at any offset
        kind = ("uniform_u32", "normal_f32", "uniform_u32", "normal_f32", "heavydup_u32", "sorted_f32")[i % 6]
        n = int(2.0 ** rng.uniform(19, 20.9))
        lists.append((kind, int(rng.integers(0, (1 << 21) - n)), n, 1 + int(rng.integers(0, 2048))))
    for i in range(400):  # short ones, whole: sorted, by delegates, by radix select
        n = int(2.0 ** rng.uniform(4, 16))
        lists.append((("uniform_u32", "normal_f32", "heavydup_u32")[i % 3], int(rng.integers(0, (1 << 21) - n)), n,
                      1 + int(rng.integers(0, min(n, 2048)))))
    saved = drt.tune_get()
    try:
        if beta == 2:
            drt.tune_set([])
            entries = set()
            for _, _, n, k in lists:
                r, a, _ = drt.batched_plan(n, k)
                if r == 2:
                    entries.add((drt.FORM_BATCHED, int(np.log2(n)), int(np.log2(k)), max(a, 4), 2))
            drt.tune_set(sorted(entries))
            assert sum(drt.batched_plan(n, k)[2] == 2 for _, _, n, k in lists) > len(lists) // 2
        total, share = sum(n for _, _, n, _ in lists), 2 * torch.cuda.get_device_properties(0).multi_processor_count
        split = sum(tiles(n, k) for _, _, n, k in lists if n * share > total and tiles(n, k) > 1)
        assert split > 2 * share, split  # more than two rounds over the device
        print("[case] tiles", split, "beta", beta, file=sys.stderr, flush=True)
        b = drt.Batch([(base[kind][2][off:off + n], k) for kind, off, n, k in lists])
        b.run(check=True)
    finally:
        drt.tune_set(saved)
    for i, (kind, off, n, k) in enumerate(lists):
        x, dt, _ = base[kind]
        check_exact(x[off:off + n], k, dt, to_np(b.values(i)), to_np(b.indices(i)), f"#{i} {kind} n={n} k={k} off={off}")
