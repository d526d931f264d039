"""What the attention kernels' inline assembly has to see to itself, read from the listing that the compiler makes of
them for gfx950: the hazard recogniser does not look into an asm block."""

import os
import re
import subprocess

import pytest

from paper_2511_23113_amd import build as b

PLAIN_STORE = """
#include <hip/hip_runtime.h>
typedef float f32x4 __attribute__((ext_vector_type(4)));
__global__ void plain_store(f32x4* to, const f32x4* from) {
  f32x4 v = from[threadIdx.x];
  to[threadIdx.x] = v;
  __builtin_amdgcn_sched_barrier(0);
  v *= 2.f;
  asm volatile("" ::"v"(v));
}
"""


def listing(src, out, extra=()):
    cmd = [b._hipcc(), "-x", "hip", "-S", "--cuda-device-only", src, "-o", out, "-I", b.CSRC, "-I", os.path.join(b.ROOT, "include")]
    subprocess.run(cmd + b.HIP_FLAGS + list(extra), check=True, capture_output=True, timeout=300)
    with open(out) as f:
        return [line.strip() for line in f]


@pytest.fixture(scope="module")
def kernel_listing(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "attn_fwd.s"
    return listing(os.path.join(b.CSRC, "attn_fwd.hip"), str(out), b.EXTRA_FLAGS["attn_fwd.hip"])


def asm_blocks(lines):
    block = None
    for line in lines:
        if line == ";;#ASMSTART":
            block = []
        elif line == ";;#ASMEND":
            yield block
            block = None
        elif block is not None:
            block.append(line)


def nop_states(lines):
    return sum(int(m[1], 0) + 1 for m in (re.match(r"s_nop (\w+)", line) for line in lines) if m)


WIDE_STORE = re.compile(r"global_store_dwordx[34]\s")


def test_wide_stores_keep_their_data_as_long_as_the_compiler_does(kernel_listing, tmp_path):
    # the compiler's own count: between a 16-byte store and a write to the registers it stores
    (tmp_path / "plain.hip").write_text(PLAIN_STORE)
    plain = listing(str(tmp_path / "plain.hip"), str(tmp_path / "plain.s"))
    store = next(i for i, line in enumerate(plain) if WIDE_STORE.match(line))
    data = re.search(r"v\[(\d+):", plain[store])[1]
    write = next(i for i, line in enumerate(plain) if i > store and re.match(rf"v_\w+ v{data},", line))
    needed = nop_states(plain[store:write])
    assert needed > 0
    stores = [(blk, i) for blk in asm_blocks(kernel_listing) for i, line in enumerate(blk) if WIDE_STORE.match(line)]
    assert stores
    assert min(nop_states(blk[i:]) for blk, i in stores) >= needed


def test_m0_is_the_copies_own(kernel_listing):
    # a group of copies keeps its LDS destination in M0 across whole steps; its asm blocks set M0, nothing else does
    set_here = sum("m0" in re.split(r"[ ,\[\]]+", line.split(";")[0]) for blk in asm_blocks(kernel_listing) for line in blk)
    all_set = sum("m0" in re.split(r"[ ,\[\]]+", line.split(";")[0]) for line in kernel_listing)
    assert set_here == all_set > 0


def test_a_slices_barrier_waits_for_reads_and_copies(kernel_listing):
    # by a builtin, in front of the builtin barrier: nothing but the markers of empty asm blocks stands between the two
    code = [line for line in kernel_listing if line and not line.startswith(";")]
    waits = [line for line, after in zip(code, code[1:]) if after == "s_barrier" and re.match(r"s_waitcnt vmcnt\(\d+\) lgkmcnt\(0\)$", line)]
    # an item's first two slices and a round of the ring: two kernels at d = 128 with the longer wait throughout, two with
    # the shorter one (4) in the ring; at d = 64 one kernel, its first slice and a round
    for n, at_least in ((16, 2 * 6 + 2 * 2), (4, 2 * 4), (8, 1 + 4)):
        assert waits.count(f"s_waitcnt vmcnt({n}) lgkmcnt(0)") >= at_least
