"""dK and dV are written through the caches or past them, by their size (no GPU needed): every kernel is there in both forms, and each
holds stores of its own kind only."""
import re

import pytest

from test_codegen import _asm, _kernels


@pytest.mark.parametrize("src,kernel", [("lvx_bwd_dkdv_bf16.hip", "bwd_dkdv_bf16_kernel"),
                                        ("lvx_bwd_dkdv_short_bf16.hip", "bwd_dkdv_short_kernel")])
def test_both_kinds_of_stores(src, kernel):
    kinds = {}
    for body in _kernels(_asm(src), kernel):
        name, past = re.match(r"_ZN\S*" + kernel + r"I(\S+)ELb([01])EEEv", body).groups()
        stores = re.findall(r"global_store_dwordx4 .*", body)
        nt = sum(1 for s in stores if s.rstrip().endswith(" nt"))
        sums = re.search(r"ELb1$", name) is not None and kernel == "bwd_dkdv_bf16_kernel"      # (of shared tiles, for the kernel that adds them)
        assert nt >= 8 and (sums or nt == len(stores)) if past == "1" else nt == 0 and len(stores) >= 8
        kinds.setdefault(name, set()).add(past)
    assert kinds and all(k == {"0", "1"} for k in kinds.values())
