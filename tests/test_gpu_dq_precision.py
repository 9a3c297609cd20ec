"""dQ where scores are large, under masks that cut through tiles and on ragged key counts: the kernels
take Q as given there, so that nothing is rounded before the float32 scores.  What is left of bf16 is
the rounding of each dS and of the result, 2^-8 of either at most (8 significant bits), which with the float32 sums of
dP - delta (some 16 units in the last place of their terms) bounds every element:
    |error of dQ_ic| <= 2^-8 (scale sum_j |dS_ij K_jc| + |dQ_ic|) + 2^-20 scale sum_j p_ij t_ij |K_jc|,
    t_ij = sum_c |dO_ic V_jc| + |dO_ic O_ic|       (and 10 % of it all for float32 exponents up to some 2000)
against float64 from the same O and L.  A Q rounded to bf16 after scaling moves scores of hundreds by
several tenths and fails by an order of magnitude."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _check(Sq, Skv, D, q_chunk, kv_block, loud):
    """loud(j): keys that carry large scores (a tensor of truth values over the keys)"""
    from paper_2502_02406_amd.blockloop import BlockLoop, MediaMask
    g = torch.Generator().manual_seed(17)
    q, do = (torch.randn((1, 2, Sq, D), generator=g) for _ in range(2))
    k, v = (torch.randn((1, 1, Skv, D), generator=g) for _ in range(2))
    k *= torch.where(loud(torch.arange(Skv)), 16.0, 0.05)[:, None]
    q, k, v, do = (t.to(torch.bfloat16).cuda() for t in (q, k, v, do))
    mask, seen = None, torch.ones((Sq, Skv), dtype=torch.bool, device="cuda")
    if q_chunk:
        nq, nk = -(-Sq // q_chunk), -(-Skv // kv_block)
        allow = (torch.arange(nk)[None, :] <= torch.arange(nq)[:, None]).to(torch.uint8)
        mask = MediaMask(allow.cuda(), q_chunk, kv_block)
        seen = allow.bool().repeat_interleave(q_chunk, 0)[:Sq].repeat_interleave(kv_block, 1)[:, :Skv].cuda()
    loop = BlockLoop(tuple(q.shape), tuple(k.shape), torch.bfloat16, 1, mask)
    o, lse = loop.forward(q, k, v)
    dk, dv = torch.empty_like(k), torch.empty_like(v)
    dq = loop.backward(q, k, v, o, lse, do, dk, dv).double()
    qd, kd, vd, gd, od, L = (t.double() for t in (q, k, v, do, o, lse))
    scale = D ** -0.5
    p = torch.where(seen, torch.exp(qd @ kd.transpose(2, 3) * scale - L[..., None]), 0.0)
    ds = p * (gd @ vd.transpose(2, 3) - (gd * od).sum(-1, keepdim=True))
    ref, size = scale * ds @ kd, scale * ds.abs() @ kd.abs()
    t = gd.abs() @ vd.abs().transpose(2, 3) + (gd * od).abs().sum(-1, keepdim=True)
    bound = 2.0 ** -8 * (size + ref.abs()) + 2.0 ** -20 * scale * (p * t) @ kd.abs() + 1e-30
    worst = float(((dq - ref).abs() / bound).max())
    assert worst <= 1.1, f"an element of dQ is off by {worst:.2f} times its bound"


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("q_chunk,kv_block", [(48, 128), (64, 729), (2, 64)])
def test_masks_that_cut_tiles(D, q_chunk, kv_block):
    _check(300, 8 * kv_block, D, q_chunk, kv_block, lambda j: j % 61 == 0)


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("Skv", [100, 64 * 2 + 1, 64 * 5 + 50, 64 * 12 + 63])
def test_ragged_last_tile(D, Skv):
    # the keys with large scores are those past the last whole tile (of 100 keys: any)
    _check(300, Skv, D, 0, 0, lambda j: (j >= Skv // 64 * 64) | ((j % 13 == 0) & (Skv < 128)))
