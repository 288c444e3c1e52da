"""LDS positions that the preconditioned CG's sweep of general cells reads
(host build of the column code, under AddressSanitizer)."""
import os
import subprocess

import pytest

from test_sanitize_host import CSRC, NATIVE, ROOT, SAN, _run, _sanitizers_available


def test_arms_leaving_the_plane_stay_in_it(tmp_path):
    if not _sanitizers_available(tmp_path):
        pytest.skip("gcc without ASan/UBSan runtime")
    if not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("HIP headers not installed")
    exe = tmp_path / "pcg_columns"
    subprocess.run(["g++", "-std=c++17", *SAN, "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", str(exe),
                    os.path.join(NATIVE, "pcg_columns_main.cpp"), os.path.join(CSRC, "plan_geometry.cpp"),
                    os.path.join(CSRC, "nk_stencil.cpp")], check=True)
    _run(exe)
