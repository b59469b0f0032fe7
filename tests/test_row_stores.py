"""How rows are stored (csrc/internal.h): what the compiler makes of store_chunk."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2302_09915_amd", "csrc")

PROBE = """
#include "internal.h"
using namespace tamoe;
template <int ST> __global__ void probe(vec16* p, uint32_t z) {
    vec16 v = {threadIdx.x, z, z, z};
    p += threadIdx.x;
    for (int i = 0; i < 4; ++i) {
        store_chunk<ST>(p, v);
        __builtin_amdgcn_sched_barrier(0);
        v.w ^= v.x;   // into the register that was stored, nothing else between
        v.x += v.y;
        asm volatile("" ::: "memory");
    }
}
template __global__ void probe<kStoreBack>(vec16*, uint32_t);
template __global__ void probe<kStoreStream>(vec16*, uint32_t);
template __global__ void probe<kStoreThrough>(vec16*, uint32_t);
template __global__ void probe<kStoreOut>(vec16*, uint32_t);
"""


def _gaps(lines):
    """Wait states between each 16-byte store and the first instruction that writes its data registers."""
    out = []
    for i, line in enumerate(lines):
        m = re.match(r"global_store_dwordx4 \S+ v\[(\d+):(\d+)\],", line)
        if m is None:
            continue
        data, states = range(int(m[1]), int(m[2]) + 1), 0
        for after in lines[i + 1:]:
            nop = re.match(r"s_nop (\d+)", after)
            w = re.match(r"v_\w+ v(?:(\d+)|\[(\d+):(\d+)\]),", after)
            if w and any(r in data for r in range(int(w[1] or w[2]), int(w[1] or w[3]) + 1)):
                out.append(states)
                break
            states += int(nop[1]) + 1 if nop else 1
    return out


def test_data_of_a_store_is_not_overwritten_early(tmp_path):
    """A store of 16 bytes still reads its data in the two wait states behind it.  The compiler keeps them free behind
    its own stores; behind those it does not see, as many have to be part of them."""
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not found")
    src, asm = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PROBE)
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, "--cuda-device-only", "-S", str(src), "-o", str(asm)],
                   check=True, capture_output=True, timeout=300)
    gaps = {}
    for name, body in re.findall(r"^_Z5probeILi(\d+)E\w+:(.*?)s_endpgm", asm.read_text(), flags=re.S | re.M):
        lines = [s.split(";")[0].strip() for s in body.splitlines()]
        gaps[int(name)] = _gaps([s for s in lines if re.match(r"(v|s|global)_", s)])
    assert sorted(gaps) == [0, 2, 16, 19] and all(len(g) >= 3 for g in gaps.values()), gaps
    need = min(gaps[0])   # the compiler's own
    assert need >= 2 and all(min(g) >= need for g in gaps.values()), gaps
