"""csrc/device_once.hpp on the CPU: once per device, from several threads."""

import os
import subprocess

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2508_02343_amd", "csrc",
                      "device_once.hpp")
MAIN = """
#include <cstdlib>
#include <thread>
#include <vector>
#include "%s"
static mm::DeviceOnce once;
int main() {
  std::atomic<int> ran[66] = {};
  if (once.run(3, [&] { ran[3]++; return 7; }) != 7) return 1;  // a failure is reported and not remembered
  std::vector<std::thread> t;
  for (int k = 0; k < 8; ++k)
    t.emplace_back([&] {
      for (int i = 0; i < 2000; ++i) {
        const int d = i %% 5;
        if (once.run(d, [&] { ran[d]++; return 0; }) != 0 || ran[d] <= (d == 3)) std::_Exit(2);
      }
    });
  for (auto& x : t) x.join();
  for (int d = 0; d < 5; ++d)
    if (ran[d] > 9) return 3;  // at most once for each thread
  for (int i = 0; i < 2; ++i) once.run(65, [&] { ran[65]++; return 0; });
  return ran[65] == 2 && ran[5] == 0 ? 0 : 4;  // devices beyond the mask: every time
}
"""


def test_once_per_device(tmp_path):
    src, exe = tmp_path / "once.cpp", tmp_path / "once"
    src.write_text(MAIN % HEADER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=thread", "-pthread", "-o", str(exe), str(src)],
                   check=True)
    assert subprocess.run([str(exe)], timeout=60).returncode == 0
