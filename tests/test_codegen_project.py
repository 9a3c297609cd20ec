"""The projection kernels whose accumulators are named registers (no GPU needed): nothing but its own statements may touch that
file, so the generated code must hold no other move into it and no spill.  The build looks at its own code in the same way; that
it would see each kind of foreign use is checked on code that has been changed."""
import re

import pytest

from paper_2502_02406_amd import build as B
from test_codegen import _asm, _kernels

_KERNELS = sorted(B.NAMED_ACCUMULATORS.items())


@pytest.mark.parametrize("src,kernel", _KERNELS)
def test_named_accumulators_are_nobody_elses(src, kernel):
    B.check_named_accumulators(_asm(src), kernel)
    for body in _kernels(_asm(src), kernel):
        assert "v_accvgpr_write" not in body and "v_accvgpr_mov" not in body and "scratch_" not in body
        # every read is one of the 256 of a tile's packing, which stands in the code twice
        assert len(re.findall(r"v_accvgpr_read", body)) == 512


_MFMA = r"v_mfma_f32_32x32x16_bf16 a\[32:47\], (v\[\d+:\d+\]), (v\[\d+:\d+\]), a\[32:47\]"


@pytest.mark.parametrize("pattern,instead", [
    (r"\tv_accvgpr_read_b32 (v\d+), a\[7\]\n", r"\tv_accvgpr_read_b32 \1, a[8]\n"),             # a register is not read
    (r"\ts_barrier\n", "\ts_barrier\n\tv_accvgpr_write_b32 a200, v0\n"),                         # something else is kept there,
    (r"\ts_barrier\n", "\ts_barrier\n\tds_read_b128 a[4:7], v0\n"),                              # loaded there,
    (r"\ts_barrier\n", "\ts_barrier\n\tv_accvgpr_read_b32 v3, a[3]\n"),                          # or read from there
    (r"\ts_barrier\n", "\ts_barrier\n\tscratch_store_dword off, v0, off\n"),                     # a spill
    (_MFMA, r"v_mfma_f32_32x32x16_bf16 a[32:47], a[0:3], \2, a[32:47]"),                         # an operand from that file
    (_MFMA, r"v_mfma_f32_32x32x16_bf16 a[32:47], \1, \2, a[48:63]"),                             # another block's sums
    (_MFMA, r"v_mfma_f32_32x32x16_bf16 a[34:49], \1, \2, a[34:49]"),                             # a block across two
    (_MFMA, r"v_mfma_f32_32x32x16_bf16 v[32:47], \1, \2, v[32:47]"),                             # the compiler's own accumulators
])
@pytest.mark.parametrize("src,kernel", _KERNELS)
def test_the_build_sees_a_foreign_use(src, kernel, pattern, instead):
    asm = _asm(src)
    (first, last) = [m.span() for m in re.finditer(r"^_ZN[^\n]*" + kernel + r"[^\n]*:.*?^\.Lfunc_end\d+:", asm, re.S | re.M)]
    for a, b in (first, last):
        body, n = re.subn(pattern, instead, asm[a:b], count=1)
        assert n == 1
        with pytest.raises(RuntimeError, match=kernel):
            B.check_named_accumulators(asm[:a] + body + asm[b:], kernel)
    with pytest.raises(RuntimeError, match="1 instantiations"):
        B.check_named_accumulators(asm[:last[0]], kernel)
