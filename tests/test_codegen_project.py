"""The projection kernels whose accumulators are named registers (no GPU needed): nothing but its own statements may touch that
file, so the generated code must hold no other move into it and no spill."""
import re

import pytest

from test_codegen import _asm, _kernels


@pytest.mark.parametrize("src,kernel", [("lvx_project.hip", "project_run_bf16_kernel"),
                                        ("lvx_project_bwd.hip", "project_bwd_x_run_bf16_kernel")])
def test_named_accumulators_are_nobody_elses(src, kernel):
    for body in _kernels(_asm(src), kernel):
        assert "v_accvgpr_write" not in body and "v_accvgpr_mov" not in body and "scratch_" not in body
        # every read is one of the 256 of a tile's packing, which stands in the code twice
        assert len(re.findall(r"v_accvgpr_read", body)) == 512
        # no load lands there, and no matrix instruction takes an operand from there but its own block
        for line in re.findall(r"^\s+(?!v_mfma|v_accvgpr_read)\S+ .*\ba(?:\d+|\[[^\]]*\])(?:,|\s|$).*", body, re.M):
            raise AssertionError(f"the file is used elsewhere: {line.strip()}")
