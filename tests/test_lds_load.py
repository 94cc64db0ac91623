"""The direct loads to LDS write m0 in inline assembly, and the compiler knows: a kernel that
holds a value of its own there (another direct load's LDS address, the same before and after)
gets it back.  Compiled to assembly only."""
import importlib.util
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1909_01554_amd", "csrc")

KERNEL = """
#include "lds_load.h"
__global__ void probe(const unsigned* a, unsigned* out) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[2048];
  typedef __attribute__((address_space(3))) unsigned char* lds_ptr;
  typedef __attribute__((address_space(3))) unsigned* lds_words;
  typedef const __attribute__((address_space(1))) unsigned* words;
  const lds_words own = (lds_words)(lds_ptr)smem;
  __builtin_amdgcn_global_load_lds((words)a + threadIdx.x, own, 4, 0, 0);
  bmm::load_lds16(%s (unsigned)(unsigned long)(lds_ptr)(smem + 1024));
  __builtin_amdgcn_global_load_lds((words)a + 64 + threadIdx.x, own, 4, 256, 0);
  __syncthreads();
  out[threadIdx.x] = *(unsigned*)(smem + 4 * threadIdx.x);
}
"""


@pytest.mark.parametrize("form", ["a, threadIdx.x * 16u,", "a + 4 * threadIdx.x,"])
def test_m0_is_set_again_after_a_direct_load(tmp_path, form):
    spec = importlib.util.spec_from_file_location(
        "_bmm_build_flags", os.path.join(ROOT, "paper_1909_01554_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc not available")
    src, asm = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text("#include <hip/hip_runtime.h>\n" + KERNEL % form)
    r = subprocess.run([build.HIPCC] + [f for f in build.FLAGS if f != "-fPIC"] +
                       ["-I", CSRC, "-S", "--cuda-device-only", str(src), "-o", str(asm)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    assert "reserved registers" not in r.stderr
    code = asm.read_text().split("s_endpgm")[0]
    loads = [m for m in re.finditer(r"global_load_lds_\w+", code)]
    assert [m.group() for m in loads] == ["global_load_lds_dword", "global_load_lds_dwordx4",
                                          "global_load_lds_dword"]
    assert re.search(r"s_mov_b32 m0, ", code[loads[1].end():loads[2].start()])
