"""How the streaming kernel's work-groups share the tiles of a grouped product (tile_of_block and blocks_dealt in csrc/ffn_common.h), on the CPU: every
row tile, column tile and part of K of every group exactly once -- one group to more than twice the XCDs, one to seventeen row tiles, K whole
and split, and with fewer parts than the grid was sized for."""
import os
import subprocess

from paper_2201_05596_amd.build import FLAGS, HIPCC

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "ffn_common.h"
int main() {
    for (int G : {1, 2, 3, 7, 8, 9, 17})
        for (int n_tiles : {1, 2, 3, 8, 9})
            for (int m_tiles = 1; m_tiles <= 17; ++m_tiles)
                for (int ksplit = 1; ksplit <= 8; ++ksplit)
                    for (int parts = 1; parts <= ksplit; ++parts) {
                        moe::WsGemmArgs a{};
                        a.G = G; a.ksplit = ksplit;
                        const int inner = m_tiles * parts;
                        const long long grid = moe::tile_grid_blocks(a, n_tiles, m_tiles * ksplit);
                        const int blocks = moe::blocks_dealt((int)grid, m_tiles * ksplit, inner);
                        std::vector<int> dealt((size_t)G * n_tiles * inner);
                        bool inside = blocks <= grid;
                        for (int b = 0; b < blocks; ++b) {
                            const moe::TileId t = moe::tile_of_block(a, n_tiles, inner, b);
                            if (!t.live) continue;
                            inside = inside && t.g >= 0 && t.g < G && t.nt >= 0 && t.nt < n_tiles && t.inner >= 0 && t.inner < inner;
                            if (inside) ++dealt[((size_t)t.g * n_tiles + t.nt) * inner + t.inner];
                        }
                        for (int n : dealt) inside = inside && n == 1;
                        if (!inside) {
                            std::printf("%d groups, %d column tiles, %d row tiles, %d of %d parts\n", G, n_tiles, m_tiles, parts, ksplit);
                            return 1;
                        }
                    }
}
"""


def test_every_tile_once(tmp_path):
    src, exe = tmp_path / "dealing.hip", tmp_path / "dealing"
    src.write_text(PROGRAM)
    subprocess.run([HIPCC, *FLAGS, "--offload-host-only", str(src), "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, run.stdout
