"""LDS beyond 64 KB is asked for on every device that a kernel runs on, whichever thread comes first (csrc/once_per_device.h), on the CPU."""
import glob
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2201_05596_amd", "csrc")
PROGRAM = r"""
#include <atomic>
#include <cstdio>
#include <thread>
#include <vector>
#include "once_per_device.h"
int main() {
    moe::OncePerDevice once;
    std::atomic<int> asked[70] = {}, early{0};
    std::vector<std::thread> threads;
    for (int t = 0; t < 4; ++t)
        threads.emplace_back([&, t] {
            for (int i = 0; i < 20000; ++i) {
                const int device = (i + t * 7) % 8;
                if (!once(device, [&] { return ++asked[device] > 1; })) continue;        // the first time it fails
                if (asked[device] < 2) ++early;                                          // through without a success on this device
            }
        });
    for (auto& t : threads) t.join();
    for (int device : {63, 64, 64, 69, 69}) once(device, [&] { ++asked[device]; return true; });
    once(63, [&] { ++asked[63]; return true; });
    for (int d = 0; d < 8; ++d) early += asked[d] < 2 || asked[d] > 5;
    std::printf("%d %d %d %d\n", early.load(), asked[63].load(), asked[64].load(), asked[69].load());
}
"""


def test_asked_on_every_device(tmp_path):
    src, exe = tmp_path / "once.cc", tmp_path / "once"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split() == ["0", "1", "2", "2"]


def test_every_launch_asks_through_it():
    sources = {f: open(f).read() for f in glob.glob(CSRC + "/*.h*")}
    assert [os.path.basename(f) for f, text in sources.items() if "hipFuncSetAttribute(" in text] == ["moe_internal.h"]
