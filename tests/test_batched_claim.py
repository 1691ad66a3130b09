"""Split problems with somewhat more tiles than run at once, next to whole ones:
their tiles are claimed by as many workgroups as run at once, in the launch that
gives each whole problem a workgroup of its own.  Against the oracle element by
element."""
import sys

import numpy as np
import pytest

import synth
from checks import check_exact, to_np
from test_batched_split import tiles

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

drt = pytest.importorskip("paper_2109_08219_amd")


@pytest.mark.parametrize("long", [100, 190])  # below and above one round of the device
def test_tiles_beside_whole_problems(long):
    rng = np.random.default_rng(long)
    base = {}
    for kind in ("uniform_u32", "normal_f32", "heavydup_u32", "sorted_f32"):
        x, dt = synth.keys(kind, 1 << 20, 70)
        base[kind] = (x, dt, torch.from_numpy(x).cuda())
    lists = []
    for i in range(long):  # four tiles each
        kind = ("uniform_u32", "normal_f32", "uniform_u32", "normal_f32", "heavydup_u32", "sorted_f32")[i % 6]
        n = int(rng.integers(900_000, 1 << 20))
        lists.append((kind, int(rng.integers(0, (1 << 20) - n)), n, 1 + int(rng.integers(0, 2048))))
    for i in range(150):  # whole, by either way
        n = int(2.0 ** rng.uniform(4, 16))
        lists.append((("uniform_u32", "normal_f32", "heavydup_u32")[i % 3], int(rng.integers(0, (1 << 20) - n)), n,
                      1 + int(rng.integers(0, min(n, 2048)))))
    slots = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    total = sum(n for _, _, n, _ in lists)
    split = sum(tiles(n, k) for _, _, n, k in lists if n * slots > total and tiles(n, k) > 1)
    print("[case] tiles", split, "of", slots, file=sys.stderr, flush=True)
    assert (split <= slots) if long == 100 else (slots < split <= 2 * slots), split
    b = drt.Batch([(base[kind][2][off:off + n], k) for kind, off, n, k in lists])
    for _ in range(3):
        b.vals.fill_(0x55555555)
        b.run(check=True)
    for i, (kind, off, n, k) in enumerate(lists):
        x, dt, _ = base[kind]
        check_exact(x[off:off + n], k, dt, to_np(b.values(i)), to_np(b.indices(i)), f"#{i} {kind} n={n} k={k} off={off}")
