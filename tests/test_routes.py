"""The rules in routes.h against the measurements that they stand on: sizes at
which one way is the slower one by more than the runs of either differ do not
take it."""
import os
import shutil
import subprocess

import pytest

from paper_2109_08219_amd import build

CXX = shutil.which("g++") or shutil.which("c++")
pytestmark = pytest.mark.skipif(CXX is None, reason="no C++ compiler")


def ask(tmp_path, expr, cells):
    src, exe = tmp_path / "ask.cpp", tmp_path / "ask"
    src.write_text('#include "routes.h"\n#include <cstdio>\nint main() {\n  using namespace drtopk;\n' +
                   "".join(f'  printf("%d\\n", (int){expr(c)});\n' for c in cells) + "}\n")
    subprocess.run([CXX, "-std=c++17", "-I", build.CSRC, "-o", str(exe), str(src)], check=True, capture_output=True)
    return [int(v) for v in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()]


# (n, k, items): one pass or a sort of all took 1.05 to 3.3 times as long, as float32 normal, uint32 uniform
# or 16-bit values in 32 bits
SLOWER = [(64, 64, 8), (200, 200, 30), (500, 500, 8), (1000, 512, 30), (1000, 384, 8), (1500, 384, 8),
          (2000, 512, 30), (2000, 512, 500), (3000, 192, 8), (3000, 1024, 500), (4096, 128, 8), (4096, 512, 60),
          (4096, 512, 2000), (4097, 2048, 30), (4500, 2048, 8), (5000, 2048, 60), (7680, 8, 8), (7680, 32, 30),
          (7681, 8, 8), (8192, 8, 30), (8192, 24, 1), (10000, 64, 8), (12000, 1, 2000), (12000, 24, 30),
          (16000, 48, 60), (16000, 96, 8), (20000, 4, 8), (31000, 1, 2000), (31000, 4, 30), (50000, 2, 8),
          (65536, 8, 30), (100000, 8, 100), (200000, 1, 60)]
# a tenth or more faster at each of them
FASTER = [(64, 8, 30), (500, 62, 8), (1000, 16, 8), (1000, 128, 2000), (1024, 768, 30), (2000, 96, 8),
          (4096, 32, 30), (4096, 64, 2000), (4097, 24, 8), (5000, 24, 30), (6000, 32, 2000), (5000, 512, 250),
          (7680, 1500, 30), (7681, 512, 500), (8192, 2048, 8), (16000, 2048, 30), (16000, 1024, 2000),
          (20000, 48, 30), (31000, 512, 8), (31000, 16, 2000), (50000, 1024, 60), (65536, 512, 500),
          (65536, 2048, 8), (100000, 64, 500)]


# (n, k) of single calls of 4-byte keys: by the batched form's kernel; cut by a sample where all keys fit the LDS
SINGLE = [(1000, 100, 0, 0), (1000, 126, 1, 0), (3000, 375, 0, 0), (4096, 256, 0, 0), (4096, 512, 0, 1),
          (4096, 2048, 1, 0), (4097, 16, 0, 0), (6000, 256, 0, 1), (8192, 64, 0, 0), (8192, 512, 0, 1),
          (8192, 1024, 0, 1), (8192, 1025, 1, 0), (8192, 2049, 0, 0), (8193, 16, 1, 0), (8193, 64, 0, 0),
          (50000, 4, 1, 0), (50000, 64, 0, 0), (65537, 4, 0, 0)]


def test_single_rules(tmp_path):
    got = ask(tmp_path, lambda c: f"one_delegates({c[0]}, {c[1]})", SINGLE)
    assert got == [c[2] for c in SINGLE]
    small = [c for c in SINGLE if c[0] <= 8192 and not c[2]]
    assert ask(tmp_path, lambda c: f"one_cuts({c[0]}, {c[1]})", small) == [c[3] for c in small]


def test_batch_rule(tmp_path):
    got = ask(tmp_path, lambda c: f"batch_streams({c[0]}, {c[1]}, {c[2]})", SLOWER + FASTER)
    assert got == [0] * len(SLOWER) + [1] * len(FASTER), [c for c, g in zip(SLOWER + FASTER, got) if g != (c in FASTER)]
