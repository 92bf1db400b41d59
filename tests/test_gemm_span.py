"""The rule that gives the GEMMs their buffer loads, built for the host: the
128- and 256-tile kernels, whose last step addresses at most 64 k past the
range, take every operand that leaves their offsets room; no operand that
either kind of kernel takes lets an offset reach 2^32, where it would wrap
back into the operand."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_09200_amd", "csrc")
PROG = r"""
#include <cstdio>
#include <initializer_list>
#include "gemm_span.h"
using namespace lat;
int main() {
  const int64_t lim = (int64_t)1 << 31;
  // strides from 3.4M elements, and operands within 320 k rows of 2 GiB, of
  // the 64-k step; the few-tile kernel's loads three steps ahead refuse them
  std::printf("%d%d %d%d %d%d\n", operand_in_buffer(4200000, 4200000, 8, true, BUF_AHEAD),
              operand_in_buffer(4200000, 4200000, 8, true, BUF_AHEAD_DMA),
              operand_in_buffer(16384, 16384, 65400, true, BUF_AHEAD),
              operand_in_buffer(16384, 16384, 65400, true, BUF_AHEAD_DMA),
              operand_in_buffer(16384, 65536, 16200, false, BUF_AHEAD),
              operand_in_buffer(16384, 65536, 16200, false, BUF_AHEAD_DMA));
  long bad = 0, most = 0;
  for (int64_t ld = 8; ld < (int64_t)1 << 25; ld = ld * 5 / 4 / 8 * 8 + 8)
    for (int K = 1; K < 100000; K = K * 3 / 2 + 1)
      for (int mn = 0; mn < 2; ++mn)
        for (int ahead : {BUF_AHEAD, BUF_AHEAD_DMA}) {
          const int64_t R = mn ? ld : (lim / 2 / ld) - 1;
          if (R < 1 || (!mn && K > ld) || !operand_in_buffer(ld, (int)R, K, mn, ahead)) continue;
          const int64_t k = (int64_t)(K - 1 + ahead);
          const int64_t last = (mn ? k * ld + R + 255 : (R - 1) * ld + k) * 2 + 16;
          if (last >= 2 * lim) ++bad;
          ++most;
        }
  std::printf("bad %ld of %ld\n", bad, most);
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_reach_of_buffer_loads(tmp_path):
    src = tmp_path / "prog.cpp"
    src.write_text(PROG)
    exe = str(tmp_path / "prog")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout.split()
    assert out[:3] == ["10", "10", "10"], out
    assert out[3:5] == ["bad", "0"] and int(out[6]) > 100, out


def test_each_kernel_uses_its_own_reach():
    with open(os.path.join(CSRC, "gemm.hip")) as f:
        text = f.read()
    uses = [line.strip() for line in text.splitlines() if "gemm_use_buf(g, " in line]
    small = [u for u in uses if "BUF_AHEAD_DMA" in u]
    tiles = [u for u in uses if "BUF_AHEAD)" in u]
    assert len(small) == 1 and len(tiles) == 2 and len(uses) == 3, uses
