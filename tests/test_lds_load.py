"""What the compiler makes of load_to_lds (csrc/mfma_util.h), whose inline assembly it cannot look into: read from the
assembly of code compiled here, no GPU needed."""
import glob
import os
import re
import subprocess

import pytest

from paper_2312_17482_amd import build

PROBE = r"""
#include "mfma_util.h"
using namespace mb;
// Descriptor words that come out of vector lanes right in front of the load, and loads the compiler knows of, which
// need the same m0, in front of it and behind it.
__global__ void probe(const uint32_t* p, uint32_t* out, uint32_t soff) {
  __shared__ __attribute__((aligned(1024))) uint32_t smem[4096];
  const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint32_t*)smem);
  const uint32_t x = p[threadIdx.x];
  u32x4 r;
  for (int i = 0; i < 4; ++i) r[i] = __builtin_amdgcn_readlane(x, i);
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, 4096, 0x00020000);
  const auto known = [&](int off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)smem, 4, off, 0, 0, 0);
  };
  known(threadIdx.x * 4);
  load_to_lds(lds0 + 1024, threadIdx.x * 16, r, soff);
  known(threadIdx.x * 4 + 256);
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  out[threadIdx.x] = smem[threadIdx.x];
}
"""
WAIT_STATES = 5   # from a vector instruction that writes a scalar register to a memory instruction that reads it


def assembly(source, out):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    subprocess.run([build.HIPCC] + build.FLAGS + ["-S", "--cuda-device-only", str(source), "-o", str(out)], check=True,
                   capture_output=True, timeout=110)
    lines = (l.split(";")[0].strip() for l in open(out))
    return [l for l in lines if re.match(r"(s|v|buffer|global|flat|ds|scratch)_\w+|[\w.$]+:$", l)]


def scalars(operand):
    """The scalar registers that an operand names, as numbers."""
    m = re.match(r"s(\d+)$", operand) or re.match(r"s\[(\d+):(\d+)\]$", operand)
    return set(range(int(m.group(1)), int(m.groups()[-1]) + 1)) if m else set()


def operands(line):
    return [x.strip() for x in re.split(r",\s*(?![^\[]*\])", line.split(None, 1)[1])] if " " in line or "\t" in line else []


def too_early(code):
    """Loads into LDS with a scalar operand that a vector instruction wrote fewer than five wait states before, along any
    way through the code: (load, writer, wait states)."""
    sources = {}                                     # label -> branches to it
    for i, l in enumerate(code):
        if re.match(r"s_c?branch", l):
            sources.setdefault(l.split()[-1], []).append(i)
    found = []

    def back(load, wanted, i, states):               # instructions in front of i, `states` wait states before the load
        while i > 0 and states < WAIT_STATES and wanted:
            i -= 1
            l = code[i]
            if l.endswith(":"):
                for branch in sources.get(l[:-1], []):
                    back(load, wanted, branch, states + 1)
                continue
            op = l.split()[0]
            if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
                return                               # nothing falls through to here
            ops = operands(l)
            written = scalars(ops[0]) if ops else set()
            if op.startswith("v_"):
                if "_co_" in op or "div_scale" in op:
                    written |= scalars(ops[1])
                if written & wanted:
                    found.append((code[load], l, states))
                    return
            elif op.startswith("s_") and not re.match(r"s_(nop|waitcnt|cmp|bitcmp|barrier|c?branch|setprio|sleep)", op):
                wanted = wanted - written            # written again by the scalar unit, which waits by itself
            states += int(l.split()[1]) + 1 if op == "s_nop" else 1

    loads = [i for i, l in enumerate(code) if re.match(r"buffer_load_dword\w* .*\blds$", l)]
    for i in loads:
        ops = operands(code[i])
        back(i, set().union(*(scalars(x.split()[0]) for x in ops)), i, 0)
    return len(loads), found


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    d = tmp_path_factory.mktemp("lds_load")
    (d / "probe.hip").write_text(PROBE)
    return assembly(d / "probe.hip", d / "probe.s")


def test_the_compiler_knows_what_m0_holds(probe):
    """The load behind load_to_lds needs the m0 of the one in front of it: it is set again in between."""
    at = next(i for i, l in enumerate(probe) if l.startswith("buffer_load_dwordx4"))
    known = [i for i, l in enumerate(probe) if re.match(r"buffer_load_dword .* lds", l)]
    assert len(known) == 2 and known[0] < at < known[1]
    assert any(re.match(r"s_mov_b32 m0,", l) for l in probe[at + 1:known[1]])


def test_a_descriptor_just_read_out_of_vector_lanes_is_found(probe):
    loads, found = too_early(probe)
    assert loads == 3 and any("v_readlane" in w for _, w, _ in found)


def test_the_search_follows_branches_and_rewritten_registers():
    def n(text):
        return len(too_early([l.strip() for l in text.strip().splitlines()])[1])
    load = "buffer_load_dwordx4 v0, s[4:7], s9 offen lds"
    assert n("v_readfirstlane_b32 s9, v1\ns_nop 3\n" + load) == 1
    assert n("v_readfirstlane_b32 s9, v1\ns_nop 4\n" + load) == 0
    assert n("v_readlane_b32 s6, v1, 3\ns_mov_b32 s6, s20\n" + load) == 0
    assert n("v_readlane_b32 s8, v1, 3\n" + load) == 0
    assert n("v_cmp_gt_u32_e64 s[4:5], v1, v2\n" + load) == 1
    assert n("v_readlane_b32 s7, v1, 3\ns_branch .L1\n.L0:\ns_nop 7\n.L1:\n" + load) == 1


def test_no_load_of_the_library_comes_too_early(tmp_path):
    sources = [f for f in glob.glob(os.path.join(build.CSRC, "*.hip")) if "load_to_lds" in open(f).read()]
    assert sources
    for f in sources:
        loads, found = too_early(assembly(f, tmp_path / "code.s"))
        print(os.path.basename(f), loads, "loads into LDS", flush=True)
        assert loads > 100 and not found, found[:10]
