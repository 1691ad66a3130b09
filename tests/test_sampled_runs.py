"""Buckets larger than a workgroup, sorted in runs of leading bins: where a run
ends, and an input of more than 2^31 keys whose bucket spans most of the key
space (its 64-bit composites then fill their type, so the width of all bins
together does not fit it)."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_2109_08219_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

CUT = r"""
#include "sample_win.h"
#include <cstdio>
typedef unsigned __int128 u128;
// The last composite of the first `bins` bins, by 128-bit arithmetic (C: at most 96 bits used).
template <typename C> int check(C mx, C mn) {
  int bl = 0;
  for (C d = mx - mn; d; d >>= 1) ++bl;
  const int sh = bl > 11 ? bl - 11 : 0;
  int bad = 0;
  for (uint32_t bins = 1; bins <= 2048; ++bins) {
    const u128 width = (u128)bins << sh, span = (u128)(mx - mn) + 1;
    const C want = width >= span ? mn : (C)((u128)mx - width + 1);
    if (drtopk::leading_bins_cut<C>(mx, mn, bins, sh) != want) ++bad;
  }
  return bad;
}
int main() {
  int bad = 0;
  const uint64_t edge[] = {0, 1, 2047, 2048, 2049, (1ull << 32) - 1, 1ull << 53, (1ull << 63) - 1, 1ull << 63,
                           (1ull << 63) + 1, ~0ull - (1ull << 53), ~0ull - 1, ~0ull};
  for (uint64_t a : edge)
    for (uint64_t b : edge)
      if (a >= b) {
        bad += check<uint64_t>(a, b);
        bad += check<u128>((u128)a << 32 | 5, (u128)b << 32);
      }
  printf("%d\n", bad);
  return bad != 0;
}
"""


@pytest.mark.skipif(not shutil.which(HIPCC) and not os.path.exists(HIPCC), reason="hipcc not found")
def test_where_a_run_ends(tmp_path):
    src = tmp_path / "cut.hip"
    src.write_text(CUT)
    exe = tmp_path / "cut"
    subprocess.run([HIPCC, *build.HIPCC_FLAGS, "--cuda-host-only", "-I", build.CSRC, "-I",
                    os.path.join(build.ROOT, "include"), "-o", str(exe), str(src)], check=True, capture_output=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout == "0\n", out.stdout + out.stderr


@pytest.mark.gpu
def test_bucket_across_the_key_space():
    # a million keys at the top of uint32, all others below 2^20: the bucket that
    # holds the last of the first and the first of the second has more keys than
    # a workgroup sorts at once, but in its first run, in one trial of 500
    torch = pytest.importorskip("torch")
    import paper_2109_08219_amd as drt
    n, ca, cb = (1 << 32) - 4096, 1_050_000, 1_050_000
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    x = torch.empty(n, dtype=torch.int32, device="cuda")
    for i in range(0, n, 1 << 28):
        x[i:i + (1 << 28)].random_(0, 1 << 20, generator=g)
    pos = torch.arange(ca, device="cuda") * (n // ca) + 7
    x[pos] = 0
    rest = torch.cat([c[c >= (1 << 20) - 512] for c in x.split(1 << 28)])
    rest = rest.sort(descending=True).values[:cb]
    assert rest.numel() == cb
    vals = torch.empty(ca + cb, dtype=torch.int32, device="cuda")
    idx = torch.empty(ca + cb, dtype=torch.int32, device="cuda")
    for trial in range(2000):
        if trial % 100 == 0:
            print("[case] bucket across the key space, trial", trial, file=sys.stderr, flush=True)
        top = -1 - torch.randint(0, 1 << 20, (ca,), dtype=torch.int32, device="cuda", generator=g)  # as uint32: the highest
        x[pos] = top
        vals.fill_(0x55555555)
        drt.topk_select(x, ca + cb, vals, idx, dtype="u32")
        assert torch.equal(vals[:ca], top.sort(descending=True).values) and torch.equal(vals[ca:], rest), f"trial {trial}"
    at = idx.long() & 0xFFFFFFFF
    assert bool((x[at] == vals).all()) and bool(((at[1:] > at[:-1]) | (vals[1:] != vals[:-1])).all())
