"""Parts of the preconditioned CG in a host build, under AddressSanitizer: the
LDS positions that its sweep of general cells reads, and the precision of its
solution update."""
import os
import subprocess

import pytest

from test_sanitize_host import CSRC, NATIVE, ROOT, SAN, _run, _sanitizers_available


def _build_and_run(tmp_path, main, *sources):
    if not _sanitizers_available(tmp_path):
        pytest.skip("gcc without ASan/UBSan runtime")
    if not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("HIP headers not installed")
    exe = tmp_path / "main"
    subprocess.run(["g++", "-std=c++17", *SAN, "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", str(exe), os.path.join(NATIVE, main),
                    *(os.path.join(CSRC, s) for s in sources)], check=True)
    _run(exe)


def test_arms_leaving_the_plane_stay_in_it(tmp_path):
    _build_and_run(tmp_path, "pcg_columns_main.cpp", "plan_geometry.cpp", "nk_stencil.cpp")


def test_solution_update_in_the_solutions_precision(tmp_path):
    _build_and_run(tmp_path, "pcg_update_main.cpp")
