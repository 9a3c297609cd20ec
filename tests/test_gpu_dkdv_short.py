"""dK and dV of key tiles of few steps (workgroups of 128 keys that share a compute unit), against the fp64 oracle: one step, the
most that a head width takes and one more (which the larger workgroups take), a short last step, keys that end inside a
wave, heads in a group; masks that select whole steps, masks by words, keys that nobody sees.  Tolerances: those of test_gpu_parity (bf16).
And the same bits as the larger workgroups.  Shared tiles go to the larger workgroups whatever their steps, so every shape is one that the
library's plan leaves whole."""
import numpy as np
import pytest
import torch

import plans
from test_gpu_parity import run_case, small

pytestmark = pytest.mark.gpu

_MOST = {64: 24, 96: 16, 128: 12}


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("Sq,Skv", [(32, 128), (32, 129), (33, 500), (63, 127), (64, 1), (95, 700), (97, 257)])
def test_few_steps(D, Sq, Skv):
    assert plans.dkdv_parts(1, 2, 1, Sq, Skv, D)[1] == 1 and plans.dkdv_is_short(1, 2, 1, Sq, Skv, D)
    run_case(small(f"short_{D}_{Sq}x{Skv}", D=D, Hq=2, Hkv=1, Sq=Sq, Skv=Skv))


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("over", [0, 1])
def test_most_steps(D, over):
    Sq = 32 * (_MOST[D] + over) - 5
    assert plans.dkdv_parts(2, 4, 4, Sq, 2000, D)[1] == 1 and plans.dkdv_is_short(2, 4, 4, Sq, 2000, D) == (over == 0)
    run_case(small(f"short_most_{D}_{over}", D=D, B=2, Hq=4, Hkv=4, Sq=Sq, Skv=2000))


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("q_chunk,kv_block", [(32, 256), (64, 256), (16, 64), (5, 100), (24, 729)], ids=lambda x: str(x))
def test_masks(D, q_chunk, kv_block):
    Sq, Skv = 190, 4 * kv_block + (0 if kv_block % 256 == 0 else 33)
    nq, nk = -(-Sq // q_chunk), -(-Skv // kv_block)
    assert plans.dkdv_parts(1, 2, 1, Sq, Skv, D, masked=True)[1] == 1 and plans.dkdv_is_short(1, 2, 1, Sq, Skv, D, q_chunk=q_chunk, kv_block=kv_block)
    allow = np.random.default_rng(q_chunk + kv_block).random((nq, nk)) < 0.5
    allow[:, nk // 2] = False                        # keys that nobody sees
    allow[:, 0] = True
    run_case(small(f"short_mask_{D}_{q_chunk}_{kv_block}", D=D, Hq=2, Hkv=1, Sq=Sq, Skv=Skv, q_chunk=q_chunk, kv_block=kv_block),
             allow=allow)


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("q_chunk,kv_block", [(0, 0), (32, 256), (5, 100)], ids=lambda x: str(x))
def test_same_bits_as_the_larger_workgroups(D, q_chunk, kv_block):
    """Rows of zeros behind the others add zeros to every sum and take the call beyond the limit."""
    from paper_2502_02406_amd import binding as B
    few, more, Skv = 64, 960, 8192 if q_chunk == 0 else 16384
    g = torch.Generator(device="cuda").manual_seed(D + q_chunk)
    k, v = (torch.randn((1, 8, Skv, D), generator=g, device="cuda").mul(0.5).bfloat16() for _ in range(2))
    rows = [torch.randn((1, 16, few, D), generator=g, device="cuda").mul(0.5).bfloat16() for _ in range(3)]
    lse = torch.rand((1, 16, few), generator=g, device="cuda") + 3
    mask = None
    if q_chunk:
        allow = (torch.rand((-(-more // q_chunk), -(-Skv // kv_block)), generator=g, device="cuda") < 0.4).to(torch.uint8)
        mask = B.make_mask(allow, q_chunk, kv_block)
    out = []
    for Sq in (few, more):
        shape = (1, 16, 8, Sq, Skv, D)
        assert plans.dkdv_parts(*shape, masked=q_chunk > 0)[1] == 1
        assert plans.dkdv_is_short(*shape, q_chunk=q_chunk, kv_block=kv_block) == (Sq == few)
        q, o, do = (torch.cat([r, r.new_zeros((1, 16, Sq - few, D))], 2) for r in rows)
        L = torch.cat([lse, lse.new_zeros((1, 16, Sq - few))], 2)
        p = B.make_problem(q, k)
        ws = torch.empty(B.lvx_xattn_workspace_bytes(p, B.LVX_BF16, B.LVX_WS_BWD), dtype=torch.uint8, device="cuda")
        dk, dv = torch.empty_like(k), torch.empty_like(v)
        B.lvx_xattn_bwd(p, q, k, v, o, L, do, mask, torch.zeros(q.shape, device="cuda"), dk, dv, ws, B.LVX_BWD_DELTA | B.LVX_BWD_DKDV)
        out.append((dk, dv))
    for a, b in zip(*out):
        assert torch.equal(a, b) and bool(torch.isfinite(a).all()) and float(a.float().abs().max()) > 0
