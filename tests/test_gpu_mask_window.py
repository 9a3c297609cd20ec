"""General kernels whose window of the bitmap is copied to LDS and starts at a chunk or key block so far on that as many
bytes before the copy there is no LDS: late rows in chunks of a row (forward, dQ), late keys in blocks of one (dK/dV).
Against float64: O, P and dS are rounded to bf16 (2^-9 each, relative), 2^-7.5 of the norm bounds the results; L is a
float32 sum (1e-3)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,Sq,Skv,q_chunk,kv_block", [
    (64, 1064, 2640, 1, 16), (96, 1064, 2640, 1, 16), (128, 1064, 2640, 1, 16),      # forward and dQ: 1024 chunks x 165 blocks on
    (128, 1102, 2640, 1, 16),                                                        # dQ only (78 chunks x 165 blocks)
    (64, 256, 200000, 20, 1), (128, 256, 200000, 20, 1),                             # dK/dV: up to 199936 blocks on
])
def test_windows_that_start_late(D, Sq, Skv, q_chunk, kv_block):
    from paper_2502_02406_amd.blockloop import BlockLoop, MediaMask
    g = torch.Generator(device="cuda").manual_seed(16)
    q, do = (torch.randn((1, 1, Sq, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    k, v = (torch.randn((1, 1, Skv, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    nq, nk = -(-Sq // q_chunk), -(-Skv // kv_block)
    allow = (torch.rand((nq, nk), generator=g, device="cuda") < 0.3).to(torch.uint8)
    loop = BlockLoop(tuple(q.shape), tuple(k.shape), torch.bfloat16, 1, MediaMask(allow, q_chunk, kv_block))
    o, lse = loop.forward(q, k, v)
    dk, dv = torch.empty_like(k), torch.empty_like(v)
    dq = loop.backward(q, k, v, o, lse, do, dk, dv)
    seen = allow.bool().repeat_interleave(q_chunk, 0)[:Sq].repeat_interleave(kv_block, 1)[:, :Skv]
    qd, gd, od, kd, vd = (t[0, 0].double() for t in (q, do, o, k, v))
    s = torch.where(seen, qd @ kd.T * D ** -0.5, float("-inf"))
    L = torch.logsumexp(s, -1)
    p = torch.exp(s - L[:, None])
    ds = p * (gd @ vd.T - (gd * od).sum(-1, keepdim=True))
    assert float((lse[0, 0].double() - L).abs().max()) <= 1e-3
    for got, ref, name in ((o, p @ vd, "O"), (dq, ds @ kd * D ** -0.5, "dQ"), (dk, ds.T @ qd * D ** -0.5, "dK"), (dv, p.T @ gd, "dV")):
        assert float((got[0, 0].double() - ref).norm() / ref.norm()) <= 2.0 ** -7.5, name
