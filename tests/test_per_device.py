"""Settings that belong to a device (a kernel's LDS limit) are made once on
each device, whatever the thread, and a failure is returned by every call on
that device and by none on another: the launchers' holder, built for the host."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_09200_amd", "csrc")
PROG = r"""
#include <atomic>
#include <cstdio>
#include <thread>
#include <vector>
#include "per_device.h"
static lat::PerDevice<int> limit;
int main() {
  std::atomic<int> made[3] = {};
  std::atomic<int> wrong{0};
  auto use = [&](int device) {
    const int r = limit.get(device, [&] { ++made[device]; return device == 1 ? 7 : 0; });
    if (r != (device == 1 ? 7 : 0)) ++wrong;
  };
  std::vector<std::thread> t;
  for (int i = 0; i < 8; ++i) t.emplace_back([&, i] { for (int q = 0; q < 300; ++q) use((q + i) % 3); });
  for (auto& x : t) x.join();
  std::printf("%d %d %d wrong %d beyond %d\n", made[0].load(), made[1].load(), made[2].load(), wrong.load(),
              limit.get(1000, [] { return 3; }));
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_once_per_device_and_failures_stay(tmp_path):
    src = tmp_path / "prog.cpp"
    src.write_text(PROG)
    exe = str(tmp_path / "prog")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(src), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout
    assert out.split() == "1 1 1 wrong 0 beyond 3".split(), out


def test_launchers_set_limits_per_device():
    for name in sorted(os.listdir(CSRC)):
        with open(os.path.join(CSRC, name)) as f:
            text = f.read()
        if name != "per_device.h":
            assert "once_flag" not in text, f"{name}: a setting made once per process"
