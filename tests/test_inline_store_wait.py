"""The results' buffer stores are inline assembly, where the compiler does not see that a vector instruction has just written a scalar register
that the store reads (five wait states on this chip).  A kernel that moves the resource and the offset from vector to scalar registers right
ahead of the store, compiled to assembly: the wait has to be there by itself."""
import re
import subprocess

import pytest

from paper_2303_11257_amd import build

SOURCE = """
#include "us_device.h"
using namespace us;
extern "C" __global__ void k(const v4i* in, const int* off, const V* data) {
  const v4i w = in[threadIdx.x];
  const V d = data[threadIdx.x];
  const int o = off[threadIdx.x];
  const v4i r = {__builtin_amdgcn_readfirstlane(w.x), __builtin_amdgcn_readfirstlane(w.y), __builtin_amdgcn_readfirstlane(w.z), __builtin_amdgcn_readfirstlane(w.w)};
  wt_buffer_store(r, (uint32_t)o, __builtin_amdgcn_readfirstlane(o), d);
}
"""


@pytest.mark.parametrize("vector,store", [("v4i", "buffer_store_dwordx4"), ("v2i", "buffer_store_dwordx2")])
def test_store_waits_for_scalar_registers(tmp_path, vector, store):
    src, asm = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text(SOURCE.replace("V*", vector + "*").replace("V d", vector + " d"))
    subprocess.run([build.HIPCC, *build.FLAGS, "-I", build.CSRC, "--offload-device-only", "-S", str(src), "-o", str(asm)], check=True)
    lines = [t for t in (re.sub(r"[;/].*", "", line).strip() for line in asm.read_text().splitlines()) if re.match(r"[sv]_|buffer_|global_", t)]
    at = next(i for i, t in enumerate(lines) if t.startswith(store))
    wait = 0
    for t in reversed(lines[:at]):
        if t.startswith("v_readfirstlane"):
            break
        wait += int(t.split()[1]) + 1 if t.startswith("s_nop") else 1
    else:
        pytest.fail("no vector instruction writes a scalar register here")
    assert wait >= 5, lines[max(0, at - 8):at + 1]
    # ... and the data registers stay as they are for two more wait states
    assert lines[at + 1] == "s_nop 1"
