"""dK and dV of up to 48 MB are written through the caches, larger ones past them.  A key's rows depend on no other key, so a
problem that ends just below the line and one that ends a key behind it have the same bits in the keys that both have, from both
kernels, dense and under masks, zeros of unseen keys among them; nothing is written behind the last key."""
import pytest
import torch

import plans

pytestmark = pytest.mark.gpu

_HEADS = 5
_AT_MOST = {64: 39321, 96: 26214, 128: 19660}        # keys of five heads in 48 MB


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("Sq", [40, 1700])           # few steps, and more than the kernel for few takes
@pytest.mark.parametrize("q_chunk,kv_block", [(0, 0), (32, 256), (5, 100)], ids=lambda x: str(x))
def test_same_bits_on_both_sides(D, Sq, q_chunk, kv_block):
    from paper_2502_02406_amd import binding as B
    n = _AT_MOST[D]
    assert _HEADS * n * D * 4 <= 48 << 20 < _HEADS * (n + 1) * D * 4
    shapes = [(1, _HEADS, _HEADS, Sq, keys, D) for keys in (n, n + 1)]
    assert len({plans.dkdv_parts(*s, masked=q_chunk > 0) for s in shapes}) == 1
    assert all(plans.dkdv_is_short(*s, q_chunk=q_chunk, kv_block=kv_block) == (Sq == 40) for s in shapes)
    g = torch.Generator(device="cuda").manual_seed(D + Sq + q_chunk)
    q, o, do = (torch.randn((1, _HEADS, Sq, D), generator=g, device="cuda").mul(0.5).bfloat16() for _ in range(3))
    k, v = (torch.randn((1, _HEADS, n + 2, D), generator=g, device="cuda").mul(0.5).bfloat16() for _ in range(2))
    lse = torch.full((1, _HEADS, Sq), 3.0, device="cuda")
    mask = None
    if q_chunk:
        allow = (torch.rand((-(-Sq // q_chunk), -(-n // kv_block)), generator=g, device="cuda") < 0.3).to(torch.uint8)
        allow[:, 3::4] = 0                           # keys that nobody sees
        mask = B.make_mask(allow, q_chunk, kv_block)
    out = []
    for keys in (n, n + 1):
        p = B.make_problem(q, k)
        p.Skv = keys
        ws = torch.empty(B.lvx_xattn_workspace_bytes(p, B.LVX_BF16, B.LVX_WS_BWD), dtype=torch.uint8, device="cuda")
        dq = torch.zeros((1, _HEADS, Sq, D), device="cuda")
        dk, dv = torch.full_like(k, -7.0), torch.full_like(v, -7.0)
        B.lvx_xattn_bwd(p, q, k, v, o, lse, do, mask, dq, dk, dv, ws, B.LVX_BWD_DELTA | B.LVX_BWD_DKDV)
        assert bool((dk[:, :, keys:] == -7.0).all()) and bool((dv[:, :, keys:] == -7.0).all())
        out.append((dk[:, :, :n], dv[:, :, :n]))
    for a, b in zip(*out):
        assert torch.equal(a, b) and bool(torch.isfinite(a).all()) and float(a.float().abs().max()) > 0
        assert bool((a != -7.0).any(-1).all())       # every row has been written
