"""Row tiles of the dense forward and dQ kernels of which only those of the last round are split over the keys, and lists
shared by more workgroups than they have tiles, against float64.  O, P and dS are rounded to bf16 (2^-9 each,
relative), and so is the Q that dQ's scores are formed with: 2^-7.5 of the norm bounds O and 2^-7 dQ; L is a float32
sum (1e-3)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _case(B, Hq, Hkv, D, Sq, Skv, n_blocks=1, q_chunk=0, kv_block=0, made_for=0):
    from paper_2502_02406_amd.blockloop import BlockLoop, MediaMask
    g = torch.Generator(device="cuda").manual_seed(3)
    q, do = (torch.randn((B, Hq, Sq, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    k, v = (torch.randn((B, Hkv, Skv, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    mask, seen = None, torch.ones((Sq, Skv), dtype=torch.bool, device="cuda")
    if q_chunk:
        c, f = torch.arange(-(-Sq // q_chunk))[:, None], torch.arange(-(-Skv // kv_block))[None, :]
        allow = (f <= c).to(torch.uint8).cuda()
        mask = MediaMask(allow, q_chunk, kv_block)
        seen = allow.bool().repeat_interleave(q_chunk, 0)[:Sq].repeat_interleave(kv_block, 1)[:, :Skv]
    loop = BlockLoop(tuple(q.shape), (B, Hkv, made_for or Skv, D), torch.bfloat16, n_blocks, mask)
    o, lse = loop.forward(q, k, v)
    dq = loop.backward(q, k, v, o, lse, do, torch.empty_like(k), torch.empty_like(v))
    G = Hq // Hkv
    for b in range(B):
        for h in range(Hq):
            qd, gd, od, kd, vd = (t.double() for t in (q[b, h], do[b, h], o[b, h], k[b, h // G], v[b, h // G]))
            s = torch.where(seen, qd @ kd.T * D ** -0.5, float("-inf"))
            L = torch.logsumexp(s, -1)
            p = torch.exp(s - L[:, None])
            ref = p @ vd
            assert float((lse[b, h].double() - L).abs().max()) <= 1e-3, f"L of head {h}"
            assert float((od - ref).norm() / ref.norm()) <= 2.0 ** -7.5, f"O of head {h}"
            dref = p * (gd @ vd.T - (gd * od).sum(-1, keepdim=True)) @ kd * D ** -0.5
            assert float((dq[b, h].double() - dref).norm() / dref.norm()) <= 2.0 ** -7, f"dQ of head {h}"


@pytest.mark.parametrize("shape", [
    (1, 8, 8, 64, 33 * 256 - 5, 2000, 1),          # 32 of a head's 33 tiles whole, a ragged last one
    (1, 8, 8, 64, 33 * 256, 4032, 2),              # ... and merged with the running result
    (1, 12, 4, 128, 5600, 2100, 1),                # heads of a group in one list, four K/V heads: two XCDs each
    (1, 3, 3, 96, 90 * 256 + 1, 2048, 1),          # an odd number of heads
    (2, 8, 4, 128, 130, 700, 1),                   # fewer tiles than compute units, three key tiles a part
    (1, 4, 4, 64, 1024, 4096, 1),                  # 4096 rows of more than four parts, combined a workgroup a row,
    (1, 4, 4, 128, 1024, 4096, 2),
    (1, 4, 4, 64, 1025, 4096, 1),                  # ... and four rows more: a thread per 16 bytes
    (1, 4, 4, 128, 1025, 4096, 2),
], ids=lambda s: "x".join(map(str, s)))
def test_last_round(shape):
    _case(*shape)


@pytest.mark.parametrize("Sq,Skv", [(100, 6407), (300, 20000), (2000, 3000)])
def test_parts_are_runs_of_whole_tiles(Sq, Skv):
    """Part k holds tiles k t .. k t + t - 1 of 64 keys, t the same for all but the last: what P is rounded against, and so the bits
    of O, depends on nothing else about the split.  Seen in the parts' L, which follow the parts' O in the workspace."""
    from paper_2502_02406_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(7)
    D, Hq = 64, 2
    q = torch.randn((1, Hq, Sq, D), generator=g, device="cuda").bfloat16()
    k, v = (torch.randn((1, 1, Skv, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    p = B.make_problem(q, k)
    ws = torch.zeros(B.lvx_xattn_workspace_bytes(p, B.LVX_BF16, B.LVX_WS_FWD), dtype=torch.uint8, device="cuda")
    o, lse = torch.empty_like(q), torch.empty((1, Hq, Sq), device="cuda")
    B.lvx_xattn_fwd(p, q, k, v, None, o, lse, ws)
    rows, f = Hq * Sq, ws.view(torch.float32)
    for n in range(2, 65):
        at = (rows * D * n + 63) // 64 * 64
        if at + rows * n > f.numel():
            break
        part = f[at:at + rows * n].view(n, rows).double()
        if torch.allclose(torch.logsumexp(part, 0), lse.double().flatten(), rtol=0, atol=1e-3):
            break
    else:
        pytest.fail("no parts found")
    s = (q[0].reshape(rows, D).double() @ k[0, 0].double().T) * D ** -0.5
    t = -(-(-(-Skv // 64)) // n) * 64
    want = torch.stack([torch.logsumexp(s[:, i * t:(i + 1) * t], 1) for i in range(n)])
    assert float((part - want).abs().max()) <= 1e-3


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("mask", [(1, 4, 2, 300, 1900, 40, 729), (2, 2, 2, 80, 4096, 64, 256), (1, 8, 2, 64, 1088, 2, 64)],
                         ids=lambda m: "x".join(map(str, m)))
def test_short_lists(D, mask):
    B, Hq, Hkv, Sq, Skv, q_chunk, kv_block = mask
    _case(B, Hq, Hkv, D, Sq, Skv, 1, q_chunk, kv_block)


@pytest.mark.parametrize("shape", [(1, 128, 16, 64, 14, 1530, 1567), (2, 16, 2, 128, 29, 4982, 4996), (1, 4, 2, 96, 72, 23990, 29102),
                                   (1, 28, 4, 96, 1, 6369, 6597), (1, 7, 1, 128, 8, 4848, 4913)],
                         ids=lambda s: "x".join(map(str, s)))
def test_fewer_keys_than_the_workspace_was_made_for(shape):
    """... for which the plan of these keys would want more parts: they are split as far as there is room."""
    _case(*shape[:6], made_for=shape[6])
