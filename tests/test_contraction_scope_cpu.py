"""The eigen-solver forbids fused multiply-adds to itself, and only to itself: device code that comes after its header in the
same translation unit (dictionary variances, multi-path scoring) is compiled as it would be without it."""
import os
import subprocess

import pytest

from paper_1509_05194_amd import build


@pytest.mark.parametrize("include", [False, True], ids=["alone", "after_the_eigen_solver"])
def test_device_code_after_the_eigen_solver_is_contracted(include, tmp_path):
    src = tmp_path / "after.hip"
    head = '#include "%s"\n' % os.path.join(build.CSRC, "eigen.hpp") if include else ""
    src.write_text(head + "#include <hip/hip_runtime.h>\n"
                   "__global__ void after(const double *a, double *c) { c[0] = a[0] * a[1] + c[1]; }\n")
    asm = tmp_path / "after.s"
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-O3", "-std=c++17", "--offload-arch=gfx950", "-S",
                    "--cuda-device-only", "-o", str(asm), str(src)], check=True, capture_output=True, timeout=300)
    text = asm.read_text()
    assert "v_fma" in text and "v_mul_f64" not in text
