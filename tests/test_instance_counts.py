"""The 32-bit instance count and the capacity planned from it, at the edges of 32 bits: the
functions of csrc/gs_common.h that the kernels and the host share, compiled for the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = """
#include <cstdio>
#include "gs_common.h"
int main() {
  unsigned long long t;
  while (std::scanf("%llu", &t) == 1)
    std::printf("%u %lld\\n", gs::instance_word(t), (long long)gs::planned_capacity((int64_t)t));
}
"""
TOO_MANY = 2**32 - 1


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_totals_past_32_bits_fit_no_capacity(tmp_path):
    src, exe = tmp_path / "counts.hip", tmp_path / "counts"
    src.write_text(SRC)
    subprocess.run(["hipcc", "--cuda-host-only", "-std=c++17", "-I", os.path.join(ROOT, "paper_2404_06926_amd", "csrc"),
                    "-o", str(exe), str(src)], check=True, capture_output=True)
    totals = [0, 1, 65535, 65536, 2**31, 2**32 - 3, 2**32 - 2, 2**32 - 1, 2**32, 2**32 + 24_704, 5 * 2**32, 2**62]
    out = subprocess.run([str(exe)], input="\n".join(map(str, totals)), capture_output=True, text=True, check=True).stdout
    assert len(out.splitlines()) == len(totals)
    for total, line in zip(totals, out.splitlines()):
        word, cap = map(int, line.split())
        if total < TOO_MANY:
            assert word == total and cap >= total and cap >= 65536
            assert cap <= max(total + total // 4, 65536)
        else:
            assert word == TOO_MANY
        assert cap < TOO_MANY  # a count that stands for too many is above every capacity
