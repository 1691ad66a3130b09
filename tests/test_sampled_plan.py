"""The sampled path's plan: the chance that the candidates do not fit their
buffers is below exp(-24) over the sizes and shares that it takes (fewer
samples than planned among as many elements as the buffer holds: at most a
Poisson tail), at both levels."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2109_08219_amd import build

scipy_stats = pytest.importorskip("scipy.stats")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PLAN = r"""
#include "sample_host.h"
#include <cstdio>
using namespace drtopk;
int main() {
  const int dts[] = {DRTOPK_U32, DRTOPK_U64};
  for (int dt : dts)
    for (int kth = 0; kth < 2; ++kth)
      for (double n = 1 << 14; n < 4.29e9; n *= 1.37)
        for (double k = 2; k <= n; k *= 1.31) {
          SPlan p;
          sample_plan(reinterpret_cast<void*>(64), (uint64_t)n, (uint32_t)k, dt, kth != 0, &p);
          if (!p.on || p.one) continue;
          const double m = p.top ? 16.0 * p.m : p.m, gap = (double)p.n / m;
          const uint32_t span = p.win.r - p.win.a;
          printf("%llu %u %u %.9g %u\n", (unsigned long long)p.n, p.k, span, gap, p.levels == 2 ? p.cap1 : p.cap);
          if (p.levels == 2)  // the second level, for any number of candidates of the first
            for (int i = 0; i <= 8; ++i) {
              const double count = p.k + (p.cap1 - (double)p.k) * i / 8;
              SWin w = {};
              sample_window(count, p.k, 4096, kth != 0, &w);
              printf("%.0f %u %u %.9g %u\n", count, p.k, w.r - w.a, count / 4096, p.cap);
            }
        }
}
"""


@pytest.mark.skipif(not shutil.which(HIPCC) and not os.path.exists(HIPCC), reason="hipcc not found")
def test_candidates_fit(tmp_path):
    if not os.path.exists(build.LIB):
        pytest.skip("library not built")
    src, exe = tmp_path / "plan.hip", tmp_path / "plan"
    src.write_text(PLAN)
    subprocess.run([HIPCC, *build.HIPCC_FLAGS, "--cuda-host-only", "-I", build.CSRC, "-I",
                    os.path.join(build.ROOT, "include"), "-c", "-o", str(tmp_path / "plan.o"), str(src)],
                   check=True, capture_output=True)
    subprocess.run([HIPCC, "-o", str(exe), str(tmp_path / "plan.o"), build.LIB, f"-Wl,-rpath,{build.HERE}"],
                   check=True, capture_output=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    rows = np.array([[float(v) for v in line.split()] for line in out.splitlines()])
    assert len(rows) > 2000
    n, k, span, gap, cap = rows.T
    whole = cap >= n  # every element fits
    tail = scipy_stats.poisson.logcdf(span - 1, (cap + 1) / gap)
    bad = np.flatnonzero(~whole & (tail > -23.99))
    assert bad.size == 0, (bad.size, rows[bad[0]].tolist(), float(tail[bad].max()))
