"""Host-side helpers of the library that need no GPU, compiled on their own."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1711_09846_amd", "csrc")


def _run(tmp_path, source):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()


def test_once_per_device(tmp_path):
    """An attribute that belongs to a device is set on every one of them, a failure is not remembered."""
    out = _run(tmp_path, r"""
#include <cstdio>
#include <thread>
#include <vector>
#include "per_device.h"
int main() {
  std::atomic<uint64_t> done{0};
  int calls[66] = {};
  auto at = [&](int device, int result) { return pbt::once_per_device(done, device, [&] { ++calls[device]; return result; }); };
  const int failed = at(0, 7), then = at(0, 0);
  printf("%d %d\n", failed, then);
  for (int round = 0; round < 3; ++round)
    for (int d : {0, 1, 63, 64, 65}) at(d, 0);
  printf("%d %d %d %d %d\n", calls[0], calls[1], calls[63], calls[64], calls[65]);
  std::atomic<uint64_t> shared{0};
  std::atomic<int> set{0};
  std::vector<std::thread> threads;
  for (int k = 0; k < 8; ++k) threads.emplace_back([&, k] { for (int n = 0; n < 1000; ++n) pbt::once_per_device(shared, k % 4, [&] { ++set; return 0; }); });
  for (auto& t : threads) t.join();
  printf("%d\n", shared.load() == 15 && set >= 4 && set <= 8 ? 1 : 0);
}
""")
    assert out == ["7", "0", "2", "1", "1", "3", "3", "1"]


def test_no_launch_remembers_an_attribute_for_the_whole_process():
    for name in os.listdir(CSRC):
        if name.endswith((".h", ".hip")):
            assert "static hipError_t attr" not in open(os.path.join(CSRC, name)).read(), name
