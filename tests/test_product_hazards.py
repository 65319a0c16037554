"""Wait states ahead of the matrix products, on the CPU, in the assembly that the build's own
flags give for the HIP sources.

A vector instruction's result may be read by a matrix product (v_mfma) two wait states after
it was issued at the earliest: an instruction in between counts one, s_nop N counts N + 1. The
compiler keeps that distance for every vector instruction that it knows as one, but not for
inline asm, whose results therefore must not be a product's operand."""
import os
import re
import subprocess

import pytest

from paper_2604_07980_amd import build

WAIT_STATES = 2
REG = re.compile(r"\b([av])(?:(\d+)\b|\[(\d+):(\d+)\])")


def _regs(operand):
    """The vector registers that an operand names, as (file, number)."""
    out = set()
    for kind, one, lo, hi in REG.findall(operand):
        out.update((kind, k) for k in (range(int(lo), int(hi) + 1) if lo else (int(one),)))
    return out


def hazards(asm):
    """(products, those that read a vector result too early) of an assembly text."""
    now, written, products, found = 0, {}, 0, []
    for line in asm.splitlines():
        line = line.split(";")[0].strip()
        if not line or line.startswith(".") or line.endswith(":"):
            continue
        name, _, rest = line.partition(" ")
        ops = [o.strip() for o in rest.split(", ")]
        if name.startswith("v_mfma"):
            products += 1
            late = [r for o in ops[1:] for r in _regs(o) if now - written.get(r, -9) <= WAIT_STATES]
            if late:
                found.append((line, late))
            for r in _regs(ops[0]):
                written.pop(r, None)                # products among themselves are another rule
        elif name.startswith("v_"):
            for r in _regs(ops[0]):
                written[r] = now
        now += int(ops[0], 0) + 1 if name == "s_nop" else 1
    return products, found


def test_the_audit_itself():
    mfma = "v_mfma_scale_f32_32x32x64_f8f6f4 a[0:15], v[4:7], v[8:11], a[0:15], v1, v1"
    near = "v_bitop3_b32 v7, v1, v2, v3 bitop3:0xea\n%s" + mfma
    assert hazards(near % "") == (1, [(mfma, [("v", 7)])])
    assert len(hazards(near % "s_nop 0\n")[1]) == 1
    assert hazards(near % "s_nop 1\n") == (1, [])
    assert hazards(near % "s_add_i32 s0, s0, 1\nv_mov_b32_e32 v20, 0\n") == (1, [])


KERNELS = """#include "match_kernels.hpp"
using namespace ocsr;
template <class M>
constexpr auto kernel = &match_level_kernel<M, 4, false>;
const void* kernels[] = {
    (const void*)kernel<dev::PairMatcher<3>>, (const void*)kernel<dev::PairMatcher<8>>,
    (const void*)kernel<dev::QuadMatcher<2>>, (const void*)kernel<dev::MatrixMatcher<2, 4, true>>,
    (const void*)kernel<dev::MatrixMatcher<4, 8, true>>};
"""


@pytest.mark.parametrize("source", ["dense.hip", "matchers.hip"])
def test_products_wait_for_their_operands(tmp_path, source):
    path, out = os.path.join(build.CSRC, source), tmp_path / "out.s"
    if not os.path.exists(path):                    # the block matchers, a few of them
        path = tmp_path / source
        path.write_text(KERNELS)
    subprocess.run([build.HIPCC, *build.FLAGS, "--offload-device-only", "-S", str(path), "-o", str(out)],
                   check=True, capture_output=True)
    products, found = hazards(out.read_text())
    assert products > 50
    assert not found, f"{len(found)} of {products} products read a result too early, first: {found[0]}"
