"""The limit of dynamic LDS is an attribute per device: the guard of the launchers raises it on every device that a process
uses, with several threads calling at once, and again where it failed."""
import glob
import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_02570_amd", "csrc")

PROGRAM = r"""
#include "wsvd_lds_limit.h"
#include <thread>
#include <vector>
enum Status { kOk = 0, kFailed = 1 };
int main() {
  static LdsLimit limit, other;
  int calls[70] = {};
  bool fail = true;
  auto on = [&](LdsLimit& l, int device) { return l(device, [&] { calls[device]++; return fail ? kFailed : kOk; }); };
  if (on(limit, 0) != kFailed || calls[0] != 1) return 1;
  fail = false;
  if (on(limit, 0) != kOk || calls[0] != 2) return 2;                    // a failure is not remembered
  if (on(limit, 0) != kOk || calls[0] != 2) return 3;                    // a success is
  if (on(limit, 1) != kOk || calls[1] != 1) return 4;                    // another device has its own
  if (on(other, 0) != kOk || calls[0] != 3) return 5;                    // and so has another kernel
  for (int i = 0; i < 3; i++)
    if (on(limit, 64) != kOk) return 6;
  if (calls[64] != 3) return 7;
  std::atomic<int> raised[16] = {}, before[16] = {};
  std::vector<std::thread> threads;
  for (int t = 0; t < 8; t++)
    threads.emplace_back([&, t] {
      for (int i = 0; i < 2000; i++) {
        const int device = 8 + (i + t) % 8;
        limit(device, [&] { raised[device]++; return kOk; });
        if (!raised[device]) before[device]++;                           // a launch that got ahead of the attribute
      }
    });
  for (auto& t : threads) t.join();
  for (int d = 8; d < 16; d++)
    if (raised[d] < 1 || raised[d] > 8 || before[d]) return 8;
  return 0;
}
"""


def test_limit_is_raised_once_per_device(tmp_path):
    src, exe = tmp_path / "limit.cpp", tmp_path / "limit"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], timeout=60).returncode == 0


def test_every_launcher_goes_through_the_guard():
    for path in glob.glob(os.path.join(CSRC, "*.hip")):
        assert not re.search(r"hipFuncSetAttribute|static bool \w+ *=", open(path).read()), path
