"""Dispatch of the GEMM for more than 64 rows, on the CPU: gemm.hip's host code against a recording stand-in for the
HIP runtime (gemm_routes.hip)."""
import ctypes
import os
import re
import subprocess

import pytest

import paper_2608_11226_amd as R

PKG = os.path.dirname(os.path.abspath(R.__file__))
HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="no ROCm compiler here")


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    d = tmp_path_factory.mktemp("routes")
    (d / "code").write_bytes(bytes(64))  # in the place of the device code, which is not compiled
    obj, lib = d / "routes.o", d / "routes.so"
    subprocess.run([HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-fPIC", f"-I{PKG}/csrc",
                    f"-I{os.path.dirname(PKG)}/include", "-Xclang", "-fcuda-include-gpubinary", "-Xclang", str(d / "code"),
                    "-c", os.path.join(HERE, "gemm_routes.hip"), "-o", str(obj)], check=True, capture_output=True)
    subprocess.run(["g++", "-shared", str(obj), "-o", str(lib)], check=True, capture_output=True)
    so = ctypes.CDLL(str(lib))
    so.last_kernel.restype = ctypes.c_char_p
    return so


def test_a_plan_that_cannot_hold_the_matrix_is_refused(routes):
    # tiles of eight 16-row blocks over 64 blocks: eight workgroups and more can, seven and fewer can not
    for nt in (8, 9, 64):
        assert routes.launch_plan(nt, 128, 1024, 256) == 0 and b"k_gemm_pp" in routes.last_kernel()
    for nt in (7, 1, 0, 65):  # too few, none planned, more than blocks
        assert routes.launch_plan(nt, 128, 1024, 256) != 0 and routes.last_kernel() == b""
