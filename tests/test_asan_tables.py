"""The tables that the posterior kernels test and read, under
AddressSanitizer and UndefinedBehaviorSanitizer (CPU only): the boxes along the
nodes' axes hold their nodes, the headers their chunks, the probe operands and
chunk records are the nodes' values, and the skip depths keep their bounds
(tests/c/skip_tables_asan.cpp with the library's host plan source)."""
import os
import shutil
import subprocess

import pytest

from tests.test_asan import ROCM, ROOT, _run


def test_skip_tables_under_sanitizers(tmp_path):
    hipcc = shutil.which("hipcc") or os.path.join(ROCM, "bin", "hipcc")
    clangxx = os.path.join(ROCM, "llvm", "bin", "clang++")
    if not (os.path.exists(hipcc) and os.path.exists(clangxx)):
        pytest.skip("ROCm compilers not found")
    obj, exe = str(tmp_path / "st.o"), str(tmp_path / "skip_tables_asan")
    # host pass only; each sanitizer flag goes to the host compiler
    subprocess.run([hipcc, "-x", "hip", "--offload-arch=gfx950", "--cuda-host-only", "-std=c++17", "-O1", "-g",
                    "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
                    "-Xarch_host", "-fno-sanitize-recover=all", "-Xarch_host", "-fno-omit-frame-pointer",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1706_07263_amd", "csrc"),
                    "-c", os.path.join(ROOT, "tests", "c", "skip_tables_asan.cpp"), "-o", obj],
                   check=True, capture_output=True)
    subprocess.run([clangxx, "-fsanitize=address,undefined", obj, "-o", exe, "-L", os.path.join(ROCM, "lib"),
                    "-lamdhip64", "-Wl,-rpath," + os.path.join(ROCM, "lib")], check=True)
    assert "skip tables asan ok" in _run(exe)
