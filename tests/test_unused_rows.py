"""The entries of slot_token past an expert's rows, as a work-group of 1024 threads visits them (for_unused_rows in csrc/route_device.h), on the CPU: each
once and none beside them -- one expert and as many as there are threads, counts of none, some and all of the capacity, capacities up to
2^31 - 1, where a thread's next row is past what 32 signed bits hold."""
import os
import subprocess

from paper_2201_05596_amd.build import CSRC, FLAGS, HIPCC

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "route_device.h"
int main() {
    const int most = 0x7fffffff;
    struct Case { int E, C, left; };                            // left: rows without a token, at most
    std::vector<Case> cases;
    for (int E : {1, 2, 3, 8, 63, 64, 65, 127, 128, 255, 256, 257, 511, 512, 513, 1000, 1023, 1024})
        for (int C : {1, 2, 3, 8, 9, 31, 64, 65, 256, 300, most / E, most / E - 1}) cases.push_back({E, C, 700});
    for (const Case& c : cases) {
        std::vector<int32_t> rows(c.E);
        long long want = 0, seen = 0;
        const int base = c.C > c.left ? c.C - c.left : 0;       // the table itself would hold 2^31 entries
        for (int e = 0; e < c.E; ++e) {
            rows[e] = e % 3 == 0 ? base : e % 3 == 1 ? c.C : base + (e * 37) % (c.C - base + 1);
            want += c.C - rows[e];
        }
        std::vector<char> hit((size_t)c.E * (c.C - base));
        for (int tid = 0; tid < 1024; ++tid)
            moe::for_unused_rows(rows.data(), c.E, c.C, tid, 1024, [&](int e, long long i) {
                const bool inside = e >= 0 && e < c.E && i >= rows[e] && i < c.C;
                if (!inside || hit[(size_t)e * (c.C - base) + (i - base)]++) {
                    std::printf("E=%d C=%d thread %d: entry %lld of expert %d %s\n", c.E, c.C, tid, i, e, inside ? "twice" : "outside");
                    std::exit(1);
                }
                ++seen;
            });
        if (seen != want) {
            std::printf("E=%d C=%d: %lld of %lld entries\n", c.E, c.C, seen, want);
            return 1;
        }
    }
}
"""


def test_every_unused_entry_once(tmp_path):
    src, exe = tmp_path / "unused.hip", tmp_path / "unused"
    src.write_text(PROGRAM)
    # wrapping sums, as the GPU's: a sum past 31 bits shows as an entry outside
    subprocess.run([HIPCC, *FLAGS, "--offload-host-only", "-fwrapv", str(src), "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, run.stdout
