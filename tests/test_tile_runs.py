"""The order in which the blocks of a launch with an unaligned input take their tiles
(csrc/ktanh_order.h), compiled for the CPU: every tile once, and each XCD's blocks in runs of neighbours."""
import subprocess

from paper_1909_07729_amd import build

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include <vector>
#include "ktanh_order.h"
using namespace ktanh_device;
int main()
{
    for (unsigned long long tiles : {1ull, 511ull, 512ull, (1ull << 15) - 1, 1ull << 15, (1ull << 15) + 511, 51201ull,
                                     (1ull << 18) - 1, 1ull << 18, (1ull << 18) + 5, 307200ull, (1ull << 19) - 8, 1ull << 19,
                                     (1ull << 19) + 12345, 3ull << 18, (1ull << 20) + (1ull << 18) + 3})
        for (bool windows : {false, true}) {
            const TileOrder order = windows ? tile_order_for(tiles) : TileOrder{0u, 18u};
            const unsigned runs = run_tiles_for(tiles);
            if (runs > tiles || runs % kSpan != 0 || (runs != 0) != (tiles >= (1ull << 15)) || order.whole > runs)
                return 1;
            std::vector<unsigned char> seen(tiles, 0);
            for (unsigned b = 0; b < tiles; ++b) {
                const unsigned t = tile_of_block_in_runs(b, runs, order.whole, order.lg_seg);
                if (t >= tiles || seen[t]) return 2;
                seen[t] = 1;
                // the block that the same XCD runs next takes the next tile, but at the end of a run
                if (b + 8 < runs && (b & (kSpan - 1)) / 8 != kRun - 1 &&
                    tile_of_block_in_runs(b + 8, runs, order.whole, order.lg_seg) != t + 1) return 3;
            }
            if (tile_of_block_in_runs(0, runs, order.whole, order.lg_seg) != 0) return 4;
        }
    std::puts("ok");
    return 0;
}
"""


def test_runs_take_every_tile_once(tmp_path):
    src, exe = tmp_path / "runs.cpp", tmp_path / "runs"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-fsanitize=undefined", "-fno-sanitize-recover",
                    "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0 and done.stdout.strip() == "ok", (done.returncode, done.stderr[-2000:])
