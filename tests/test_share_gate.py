"""The order in which whole-solve launches share a device (csrc/mlb_gate.hpp, host code): a launch that needs the
whole of it enters although smaller ones keep coming, shares never add up to more than one, and one that fits
passes one that does not."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <atomic>
#include <chrono>
#include <cstdio>
#include <thread>
#include <vector>
#include "mlb_gate.hpp"

using namespace std::chrono_literals;

int main() {
  mlb::ShareGate g;
  std::atomic<int> held{0}, most{0};   // in hundredths
  auto hold = [&](double share, std::chrono::microseconds t) {
    g.enter(share);
    const int now = held += (int)(100 * share + 0.5);
    int m = most;
    while (now > m && !most.compare_exchange_weak(m, now)) {
    }
    std::this_thread::sleep_for(t);
    held -= (int)(100 * share + 0.5);
    g.leave(share);
  };
  // smaller ones in overlapping turns: there is never a moment without one, until the large one waits
  std::atomic<bool> stop{false};
  std::atomic<long> turns{0};
  std::vector<std::thread> ts;
  for (int k = 0; k < 6; ++k)
    ts.emplace_back([&, k] {
      std::this_thread::sleep_for(std::chrono::microseconds(300 * k));
      while (!stop) {
        hold(0.25, 2000us);
        ++turns;
      }
    });
  std::this_thread::sleep_for(50ms);
  std::atomic<bool> in{false};
  long before = turns, after = 0;
  std::thread large([&] {
    for (int k = 0; k < 5; ++k) hold(1.0, 1000us);
    in = true;
  });
  for (int k = 0; k < 2000 && !in; ++k) std::this_thread::sleep_for(1ms);
  const bool entered = in;
  after = turns;
  stop = true;
  for (auto& t : ts) t.join();
  large.join();
  // one that fits passes one that does not
  g.enter(0.6);
  std::atomic<bool> big{false}, small{false};
  std::thread a([&] { g.enter(0.9); big = true; g.leave(0.9); });
  std::this_thread::sleep_for(20ms);
  std::thread b([&] { g.enter(0.3); small = true; g.leave(0.3); });
  for (int k = 0; k < 2000 && !small; ++k) std::this_thread::sleep_for(1ms);
  const bool passed = small && !big;
  g.leave(0.6);
  a.join();
  b.join();
  std::printf("entered %d turns %ld most %d passed %d\n", (int)entered, after - before, (int)most, (int)passed);
  return entered && most <= 100 && passed ? 0 : 1;
}
"""


def test_share_gate(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if not cxx:
        pytest.skip("no C++ compiler")
    (tmp_path / "gate.cpp").write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-pthread", "-I", os.path.join(ROOT, "paper_1106_3678_amd", "csrc"),
                    "-o", str(tmp_path / "gate"), str(tmp_path / "gate.cpp")], check=True)
    r = subprocess.run([str(tmp_path / "gate")], capture_output=True, text=True, timeout=60)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
