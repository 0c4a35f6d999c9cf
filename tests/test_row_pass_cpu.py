"""The row passes that leave fp16 operands run two blocks of 512 threads per CU where a row is one chunk of columns, at 128 coordinates and in
the kernel for long rows: at most 128 registers, as the compiler reports them, and but for the last none in scratch memory."""
import os
import re
import subprocess

from paper_1509_05194_amd import build

SOURCE = r'''
#include "stream.hpp"
using namespace hclae;
#define ROW(MODE, DT) template __global__ void hclae::k_row_pass<MODE, true, DT, true, true>(float *, const float *, const uint8_t *, const float *, \
    const float *, int64_t, int, int, int, int, RowGeom, uint8_t *, double *, long long *, unsigned *, RowPass16);
#define WIDE(MODE) template __global__ void hclae::k_row_pass_wide<MODE, true, true, true>(float *, const float *, const uint8_t *, const float *, \
    const float *, int64_t, int, int, int, int, uint8_t *, double *, long long *, unsigned *, RowPass16);
ROW(0, 128) ROW(1, 128) ROW(0, kOneChunk) ROW(1, kOneChunk) WIDE(0) WIDE(1)
'''


def test_two_blocks_per_cu(tmp_path):
    src = tmp_path / "rows.hip"
    src.write_text(SOURCE)
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    p = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags + ["--cuda-device-only", "-c", "-Rpass-analysis=kernel-resource-usage",
                        "-I", build.CSRC, "-o", str(tmp_path / "rows.o"), str(src)], capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stderr
    kernels = [k for k in re.split(r"Function Name: ", p.stderr)[1:] if "k_row_pass" in k.split()[0]]
    assert len(kernels) == 6
    for k in kernels:
        figures = {name: int(n) for name, n in re.findall(r"remark:\s+([A-Za-z ]+?)(?: \[[^\]]*\])?: (\d+)", k)}
        assert figures["VGPRs"] <= 128 and (figures["VGPRs Spill"] == 0 or "k_row_pass_wide" in k), k[:200]
