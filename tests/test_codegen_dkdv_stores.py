"""dK and dV are written through the caches or past them, by their size (no GPU needed): the compiler makes one ordinary store of
the two forms if it can, so every kernel's code has to hold both."""
import re

import pytest

from test_codegen import _asm, _kernels


@pytest.mark.parametrize("src,kernel", [("lvx_bwd_dkdv_bf16.hip", "bwd_dkdv_bf16_kernel"),
                                        ("lvx_bwd_dkdv_short_bf16.hip", "bwd_dkdv_short_kernel")])
def test_both_kinds_of_stores(src, kernel):
    for body in _kernels(_asm(src), kernel):
        stores = re.findall(r"global_store_dwordx4 .*", body)
        past = sum(1 for s in stores if s.rstrip().endswith(" nt"))
        assert past >= 8 and len(stores) - past >= 8
