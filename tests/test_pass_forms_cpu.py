"""Every level pass has a kernel in the form picked for it, or the problem is
refused (CPU only): the launch code linked with a marching form that takes
nothing (tests/host/pass_forms_driver.cpp) must not accept a problem whose
passes it would leave out."""

import os
import subprocess

import pytest

from paper_2602_01888_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_pass_without_a_kernel_is_refused(tmp_path):
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    clang = os.path.join(rocm, "llvm", "bin", "clang++")
    if not (os.path.exists(build.HIPCC) and os.path.exists(clang)):
        pytest.skip("no ROCm toolchain")
    objs = [build.object_of(s) for s in build.SOURCES if s != "march.hip"]
    exe = str(tmp_path / "pass_forms_driver")
    subprocess.run([clang, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(rocm, "include"), "-I", os.path.join(ROOT, "include"),
                    "-I", build.CSRC, "-o", exe,
                    os.path.join(ROOT, "tests", "host", "pass_forms_driver.cpp")] + objs +
                   ["-L", os.path.join(rocm, "lib"), "-lamdhip64",
                    "-Wl,-rpath," + os.path.join(rocm, "lib")], check=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    assert "all checks ran" in r.stdout
