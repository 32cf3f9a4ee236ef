"""Dispatch of the GEMM for more than 64 rows, on the CPU: gemm.hip's host code against a recording stand-in for the
HIP runtime (gemm_routes.hip)."""
import ctypes
import os
import re
import subprocess

import pytest

import paper_2608_11226_amd as R
from gpu_helpers import TILE_ROWS

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


SWIGLU, ADD = "swiglu", "add"
TILE = {"5,2,2,4": "10x8", "4,4,4,2": "16x8", "4,4,2,4": "8x16", "5,4,2,4": "10x16", "4,8,4,2": "16x16", "5,8,4,2": "20x16"}


def _routes(routes, q4, rows, shape):
    """(tile, what its epilogue does, whether the last 16-row block is ragged) of every launch of the row tests"""
    _, d, nh, nkv, hd, ff, V, _ = shape
    seen = set()
    for M in rows:
        for quant, N, K, splits, swiglu, residual in ((q4, nh * hd + 2 * nkv * hd, d, 16, 0, 0), (q4, d, nh * hd, 16, 0, 1),
                                                      (q4, 2 * ff, d, 1, 1, 0), (q4, d, ff, 16, 0, 1), (0, V, d, 1, 0, 0)):
            s = routes.project(quant, M, N, K, splits, swiglu, residual)
            assert s >= 0
            t = re.search(r"k_gemm_ppILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi\d+ELb(\d)ELb(\d)", routes.last_kernel().decode())
            assert int(t[5]) == swiglu and int(t[6]) == quant
            if quant == q4:
                seen.add((TILE[",".join(t.group(1, 2, 3, 4))], SWIGLU if swiglu else ADD if s == 0 else "", M % 16 > 0))
    return seen


@pytest.mark.parametrize("q4", [0, 1])
def test_the_row_tests_reach_every_tile(routes, q4):
    seen = set()
    for t in TILE_ROWS.values():
        seen |= _routes(routes, q4, t[q4], t[2])
    tiles = [t for t in TILE.values() if not q4 or t not in ("16x16", "20x16")]
    for tile in tiles:  # plain and SwiGLU epilogue of every tile, at ragged row counts
        assert (tile, "", True) in seen or (tile, ADD, True) in seen, tile
        assert (tile, SWIGLU, True) in seen, tile
    # the product added to the residual stream, at 128- and 256-row activation tiles
    assert {t for t, what, ragged in seen if what == ADD and ragged} >= {"10x8", "16x8", "8x16", "10x16" if q4 else "20x16"}


@pytest.mark.parametrize("M,N,K,tile", [(256, 768, 256, "10x8"), (129, 1024, 256, "10x8"),
                                        (256, 37888, 3584, "10x16"), (256, 27648, 5120, "8x16")])
def test_short_k_takes_small_tiles(routes, M, N, K, tile):
    assert routes.project(0, M, N, K, 1, 1, 0) == 1
    t = re.search(r"k_gemm_ppILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E", routes.last_kernel().decode())
    assert TILE[",".join(t.groups())] == tile


def test_a_plan_that_cannot_hold_the_matrix_is_refused(routes):
    # tiles of eight 16-row blocks over 64 blocks: eight workgroups and more can, seven and fewer can not
    for nt in (8, 9, 64):
        assert routes.launch_plan(nt, 128, 1024, 256) == 0 and b"k_gemm_pp" in routes.last_kernel()
    for nt in (7, 1, 0, 65):  # too few, none planned, more than blocks
        assert routes.launch_plan(nt, 128, 1024, 256) != 0 and routes.last_kernel() == b""
