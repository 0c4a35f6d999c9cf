"""The launch arithmetic of the fused encoder up to the largest N a context accepts, as facts the compiler checks."""
import os
import subprocess

from paper_1509_05194_amd import build

CHECKS = r'''
#include "encode.hpp"
using namespace hclae;
constexpr bool ok(int64_t N)
{
    const int64_t tiles = encode_tiles(N), blocks = encode_blocks(N);
    return tiles * kTileVec >= N && (tiles - 1) * kTileVec < N          // every vector has its tile, no tile is empty
        && tiles <= 0x7fffffff && blocks >= 1 && blocks <= tiles        // the kernel counts tiles in int, every block has one
        && blocks * 64 * 8 < ((int64_t)1 << 32);                        // threads of a launch, eight waves to a block
}
static_assert(ok(1) && ok(31) && ok(32) && ok(33) && ok(1000000), "small");
static_assert(ok(33554431) && ok(33554432) && ok(33554433), "where blocks begin to stride");
static_assert(ok(268435455) && ok(536870912) && ok(536870913) && ok(1073741825), "2^32 threads with a block per tile");
static_assert(ok(2147483616) && ok(2147483617) && ok(2147483647), "the largest N");
static_assert(encode_tiles(2147483647) == 67108864, "2^26 tiles");
'''


def test_every_tile_has_a_block_and_every_launch_fits(tmp_path):
    src = tmp_path / "grid.hip"
    src.write_text(CHECKS)
    p = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-std=c++17", "--offload-arch=gfx950", "--cuda-host-only",
                        "-fsyntax-only", "-I", build.CSRC, str(src)], capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stderr
