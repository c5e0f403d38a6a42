"""The library products never get an algorithm that needs more workspace than they
have: hipBLASLt's heuristics return such algorithms whatever the preference says (a
product of 1558 rows, 2560 -> 19456, then wrote 8 MiB past a layer's workspace and
faulted).  csrc/model/blas.hip is built with stubs of the hipBLASLt calls
(tests/sanitize/blas_driver.cpp) and run on the CPU under the sanitizers."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def test_algorithms_fit_the_workspace(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists(os.path.join(ROCM, "include", "hipblaslt", "hipblaslt.h")):
        pytest.skip("g++ or the hipBLASLt headers not available")
    model = os.path.join(ROOT, "paper_2606_13361_amd", "csrc", "model")
    exe = str(tmp_path / "blas_driver")
    subprocess.run([gxx, "-x", "c++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-I" + model, "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROCM, "include"), os.path.join(model, "blas.hip"),
                    os.path.join(ROOT, "tests", "sanitize", "blas_driver.cpp"), "-o", exe], check=True)
    p = subprocess.run([exe], env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"), capture_output=True, text=True, timeout=120)
    assert p.returncode == 0 and "all checks passed" in p.stdout, p.stdout + p.stderr
