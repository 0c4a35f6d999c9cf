"""The order in which the assignment hands out its tiles, as facts the compiler checks: every tile exactly once, no block more than the
share its list of undecided vectors has room for, and every stretch of rows on the XCD of the row-pass block that takes them."""
import os
import subprocess

from paper_1509_05194_amd import build

CHECKS = r'''
#include "assign_half.hpp"
using namespace hclae;
constexpr int kMost = 1 << 12;
constexpr bool ok(int ntiles, int grid, int ls)
{
    bool seen[kMost] = {};
    int64_t entries = 0;
    for (int b = 0; b < grid; ++b) {
        int mine = 0;
        for (int w = 0; w < kAssignWaves; ++w) {
            const int count = half_tiles_of(b, w, ntiles, grid, ls);
            for (int j = 0; j < count; ++j) {
                const int t = half_tile(b, w + kAssignWaves * j, grid, ls);
                if (t < 0 || t >= ntiles || seen[t]) return false;
                if (ls >= 0 && ((t >> ls) & 7) != (b & 7)) return false;
                seen[t] = true;
            }
            if (half_tile(b, w + kAssignWaves * count, grid, ls) < ntiles) return false;
            mine += count;
        }
        if (mine > half_share(ntiles, grid, ls)) return false;
        entries += (int64_t)half_share(ntiles, grid, ls) * kTileVec;
    }
    for (int t = 0; t < ntiles; ++t)
        if (!seen[t]) return false;
    return entries <= half_list_entries((int64_t)(ntiles - 1) * kTileVec + 1, (int64_t)grid * kAssignWaves);
}
static_assert(ok(1, 1, -1) && ok(3, 1, -1) && ok(7, 2, -1) && ok(1023, 256, -1) && ok(2049, 256, -1), "in order");
static_assert(ok(64, 16, 0) && ok(65, 16, 1) && ok(1000, 16, 1) && ok(131, 32, 2), "small devices");
static_assert(ok(1024, 256, 0) && ok(1025, 256, 2) && ok(2047, 256, 1) && ok(1024, 256, 7) && ok(4095, 256, 6) && ok(3001, 256, 3), "256 CUs");
static_assert(half_order(256, 256, 128) == 2 && half_order(256, 256, 64) == 1 && half_order(256, 256, 32) == 0, "rows of a pass block");
static_assert(half_order(256, 256, 16) == -1 && half_order(100, 256, 64) == -1 && half_order(12, 12, 64) == -1, "in order otherwise");
static_assert(half_order(256, 256, 2048) == 6 && half_order(64, 64, 2048) == -1, "a stretch is at most half a round");
'''


def test_every_tile_once(tmp_path):
    src = tmp_path / "order.hip"
    src.write_text(CHECKS)
    p = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-std=c++17", "--offload-arch=gfx950", "--cuda-host-only",
                        "-fsyntax-only", "-fconstexpr-steps=100000000", "-I", build.CSRC, str(src)], capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stderr
