"""Calls that need device memory only to be faster still work when the device has none left.

The library's host sources are linked against tests/full_device_driver.cpp, a HIP runtime whose
device memory is host memory and whose hipMalloc can fail: spins are read and written without the
staging buffer, training takes records in smaller chunks and losses in shorter runs of epochs."""
import os
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2503_10302_amd", "csrc")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
CLANG = "/opt/rocm/llvm/bin/clang++"

pytestmark = pytest.mark.skipif(not (os.path.exists(HIPCC) and os.path.exists(CLANG)), reason="needs hipcc and clang")


def test_calls_on_a_full_device(tmp_path):
    srcs = [os.path.join(CSRC, "sg_api.cpp"), os.path.join(CSRC, "sg_mlp_api.cpp"),
            os.path.join(ROOT, "tests", "full_device_driver.cpp")]
    objs = [str(tmp_path / (os.path.basename(s) + ".o")) for s in srcs]

    def compile_one(a):
        subprocess.run([HIPCC, "--offload-arch=gfx950", "-std=c++17", "-O1", "-ffp-contract=off", "-fPIC",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c", a[0], "-o", a[1]],
                       check=True, capture_output=True, text=True)

    with ThreadPoolExecutor(max_workers=3) as ex:
        list(ex.map(compile_one, zip(srcs, objs)))
    exe = str(tmp_path / "full_device")
    subprocess.run([CLANG, *objs, "-o", exe, "-Wl,--unresolved-symbols=ignore-all", "-lpthread", "-lm"],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
