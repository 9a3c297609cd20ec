"""Generated-code checks of the kernels that mask by words (see test_codegen.py for the rules)."""
import pytest

from test_codegen import _asm, _blocks, _kernels


@pytest.mark.parametrize("D,loop_mfma", [(64, 64), (96, 96), (128, 128)])
def test_dkdv_words_loop_is_one_block(D, loop_mfma):
    for body in _kernels(_asm("lvx_bwd_dkdv_bf16.hip"), f"bwd_dkdv_bf16_kernelILi{D}ELb0ELb1ELb1E"):       # with and without parts
        loops = [b for b in _blocks(body) if b.count("v_mfma_f32_32x32x16_bf16") == loop_mfma]
        assert len(loops) == 1, "steady-state loop not found as one basic block"
        assert "v_accvgpr" not in loops[0] and "scratch_" not in loops[0]


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("src,kernel", [("lvx_fwd_bf16.hip", "fwd_bf16_kernelILi%dELi3EE"),
                                        ("lvx_bwd_dq_bf16.hip", "bwd_dq_bf16_kernelILi%dELb0ELi3EE")])
def test_tile_words_move_no_accumulator(src, kernel, D):
    (body,) = _kernels(_asm(src), kernel % D)
    n = 0
    for blk in _blocks(body):
        if "v_mfma_f32_32x32x16_bf16" in blk:
            n += 1
            assert "v_accvgpr" not in blk and "scratch_" not in blk
    assert n > 0
