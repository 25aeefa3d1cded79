"""The tags that the decode gate's hand-over flags carry (csrc/call_tag.h), on the CPU: scratch memory that holds indices,
counts or an earlier call's flags must never look like the present call's."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2201_05596_amd", "csrc")
PROGRAM = r"""
#include <cstdio>
#include <thread>
#include <vector>
#include "call_tag.h"
int main() {
    std::vector<std::vector<uint64_t>> tags(4);
    std::vector<std::thread> threads;
    for (auto& t : tags) threads.emplace_back([&t] { for (int i = 0; i < 5000; ++i) t.push_back(moe::next_call_tag()); });
    for (auto& t : threads) t.join();
    for (auto& t : tags) for (uint64_t v : t) std::printf("%llu\n", (unsigned long long)v);
}
"""


def test_tags_are_wide_and_never_repeat(tmp_path):
    src, exe = tmp_path / "tags.cc", tmp_path / "tags"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    runs = [[int(v) for v in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()] for _ in range(2)]
    for tags in runs:
        assert len(set(tags)) == len(tags) == 20000          # four threads: none twice
        assert min(tags) >= 1 << 32                          # no small whole number (chance of one such tag: 5e-6)
    assert not set(runs[0]) & set(runs[1])                   # nothing in common with another process
