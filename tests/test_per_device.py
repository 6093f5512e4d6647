"""csrc/per_device.h on the CPU: a value is made once for each device, also
under several threads."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_12292_amd", "csrc")

MAIN = r"""
#include <atomic>
#include <cstdio>
#include <thread>
#include <vector>
#include "per_device.h"
int main() {
  bgl::PerDevice<int> v;
  std::atomic<int> made[3] = {{0}, {0}, {0}};
  std::atomic<int> wrong{0};
  std::vector<std::thread> threads;
  for (int t = 0; t < 8; ++t)
    threads.emplace_back([&, t] {
      for (int i = 0; i < 300; ++i) {
        const int dev = (t + i) % 3;
        if (v.get(dev, [&] { ++made[dev]; return 10 + dev; }) != 10 + dev) ++wrong;
      }
    });
  for (auto& t : threads) t.join();
  std::printf("%d %d %d %d\n", int(made[0]), int(made[1]), int(made[2]), int(wrong));
  return 0;
}
"""


def test_made_once_per_device(tmp_path):
    src = tmp_path / "main.cpp"
    src.write_text(MAIN)
    exe = tmp_path / "main"
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    if r.returncode != 0 and "g++" in r.stderr and "not found" in r.stderr:
        pytest.skip("no host compiler")
    assert r.returncode == 0, r.stderr
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60).stdout.split()
    assert out == ["1", "1", "1", "0"]


def test_resident_kernels_are_set_up_per_device():
    """The attribute that lets a launch have more than 64 KB of LDS is set
    through PerDevice, not once per process."""
    with open(os.path.join(CSRC, "eval.hip")) as f:
        text = f.read()
    assert text.count("hipFuncSetAttribute") == 1
    before = text[:text.index("hipFuncSetAttribute")]
    assert "limit_raised.get(dev" in before[-200:] and "call_once" not in text
