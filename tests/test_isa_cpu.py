"""Direct loads into LDS in the compiled kernels: the wait state after M0 and M0 as a clobber.

``global_load_lds`` takes its LDS address from M0, and on gfx950 a scalar write of M0 needs one wait state (any
instruction, or ``s_nop 0``) before it; a scalar register that a vector instruction wrote needs five.  The compiler
inserts these for its own builtin but does not look inside inline assembly, which is how the kernels issue these loads,
so the built code is checked instruction by instruction."""
import os
import re
import subprocess

import pytest

import paper_2608_11226_amd as R

PKG = os.path.dirname(os.path.abspath(R.__file__))
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

pytestmark = pytest.mark.skipif(not (os.path.exists(OBJDUMP) and os.path.exists(HIPCC)), reason="no ROCm compiler here")


def _instructions(text):
    lines = (l.split("//")[0].split(";")[0].strip() for l in text.splitlines())
    return [l for l in lines if re.match(r"[a-z]+_\w+( |$)", l)]


def _loads_without_wait_state(ins):
    """(direct loads into LDS, writes of M0 or of their base registers that stand too close before them)"""
    at = [i for i, s in enumerate(ins) if s.startswith(("global_load_lds", "buffer_load")) and "lds" in s]
    bad = [ins[i - 1] for i in at if re.match(r"\w+ m0,", ins[i - 1])]
    for i in at:
        base = re.search(r"s\[(\d+):(\d+)\]", ins[i])
        regs = ["m0"] + ([f"s{r}" for r in range(int(base[1]), int(base[2]) + 1)] if base else [])
        states = 0
        for s in reversed(ins[max(0, i - 5):i]):
            if states >= 5:
                break
            if re.match(rf"v_\w+ ({'|'.join(regs)}),", s):
                bad.append(s)
            nop = re.match(r"s_nop (\d+)", s)
            states += int(nop[1]) + 1 if nop else 1
    return len(at), bad


def test_every_direct_load_into_lds_has_its_wait_state(tmp_path):
    lib = tmp_path / "librollout.so"
    os.symlink(os.path.join(PKG, "librollout.so"), lib)
    subprocess.run([OBJDUMP, "--offloading", lib.name], cwd=tmp_path, check=True, capture_output=True)
    loads, bad = 0, []
    for code in sorted(tmp_path.glob("*gfx950")):
        out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--mcpu=gfx950", code.name], cwd=tmp_path, check=True,
                             capture_output=True, text=True)
        n, b = _loads_without_wait_state(_instructions(out.stdout))
        loads += n
        bad += b
    assert loads > 0, "no direct load into LDS found: the check looks at the wrong code"
    assert not bad, f"{len(bad)} writes stand too close before {loads} loads, e.g. {bad[0]}"


# Two direct loads to one LDS address by the compiler's builtin, with a helper's load elsewhere between them: the
# compiler has to write M0 again for the second.
KERNEL = """
#include "internal.h"
using namespace rollout;
__global__ void k(const char* a, float* out) {
  __shared__ float ls[1024];
  typedef __attribute__((address_space(3))) void lds_t;
  typedef __attribute__((address_space(1))) const void glb_t;
  __builtin_amdgcn_global_load_lds((glb_t*)a, (lds_t*)ls, 16, 0, 0);
  HELPER
  __builtin_amdgcn_global_load_lds((glb_t*)(a + 8192), (lds_t*)ls, 16, 0, 0);
  __syncthreads();
  out[threadIdx.x] = ls[threadIdx.x] + ls[512 + threadIdx.x];
}
"""


@pytest.mark.parametrize("helper", ["dma_lds16(a + 16 * threadIdx.x, ls + 512);",
                                    "dma_lds16_at(a, 16 * threadIdx.x, ls + 512);"])
def test_the_compiler_knows_that_the_helpers_write_m0(helper, tmp_path):
    src = tmp_path / "k.hip"
    src.write_text(KERNEL.replace("HELPER", helper))
    inc = [f"-I{os.path.join(PKG, 'csrc')}", f"-I{os.path.join(os.path.dirname(PKG), 'include')}"]
    out = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", *inc, "-Xclang", "-target-feature",
                          "-Xclang", "-packed-fp32-ops", "--cuda-device-only", "-S", src.name, "-o", "-"],
                         cwd=tmp_path, check=True, capture_output=True, text=True)
    ins = _instructions(out.stdout)
    at = [i for i, s in enumerate(ins) if s.startswith("global_load_lds")]
    assert len(at) == 3
    assert any(re.match(r"\w+ m0,", s) for s in ins[at[1] + 1:at[2]]), "M0 is not written again after the helper"
    assert not _loads_without_wait_state(ins)[1]
