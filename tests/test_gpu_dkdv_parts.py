"""Key tiles whose steps several dK/dV workgroups share: few keys, a last round of a few tiles, and lists of steps
under a media mask, against float64 from the same O and L.  P, dS and the results are bf16 (2^-9 each,
relative): 2^-7.5 of the norm bounds dK and dV; the parts' float32 sums add nothing to that.  The smallest workspace
that the library takes has no room for the parts and has to give the same up to the rounding of the results, and so
has one with room for some of them.  Whether a call has parts is seen in the workspace: nothing but their sums is written
behind that smallest size by a call without the dQ kernel."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _case(B, Hq, Hkv, D, Sq, Skv, q_chunk=0, kv_block=0, rule="causal", parts=True):
    from paper_2502_02406_amd import binding as L
    from paper_2502_02406_amd.blockloop import BlockLoop, MediaMask
    g = torch.Generator(device="cuda").manual_seed(5)
    q, do = (torch.randn((B, Hq, Sq, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    k, v = (torch.randn((B, Hkv, Skv, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    mask, seen = None, torch.ones((Sq, Skv), dtype=torch.bool, device="cuda")
    if q_chunk:
        c, f = torch.arange(-(-Sq // q_chunk))[:, None], torch.arange(-(-Skv // kv_block))[None, :]
        allow = (f <= c if rule == "causal" else f == c).to(torch.uint8).cuda()
        mask = MediaMask(allow, q_chunk, kv_block)
        seen = allow.bool().repeat_interleave(q_chunk, 0)[:Sq].repeat_interleave(kv_block, 1)[:, :Skv]
    loop = BlockLoop(tuple(q.shape), tuple(k.shape), torch.bfloat16, 1, mask)
    o, lse = loop.forward(q, k, v)
    out = []

    def backward(ws, stages):
        dk, dv = (torch.full_like(k, float("nan")) for _ in range(2))
        acc = torch.zeros(q.shape, dtype=torch.float32, device="cuda")
        L.lvx_xattn_bwd(L.make_problem(q, k), q, k, v, o, lse, do, loop._mask_for(0), acc, dk, dv, ws, stages)
        return dk, dv
    dk, dv = backward(loop.ws, L.LVX_BWD_ALL)
    for b in range(B):
        for h in range(Hkv):
            G = Hq // Hkv
            sl = slice(h * G, (h + 1) * G)
            qd, gd, od, ls = (t[b, sl].double() for t in (q, do, o, lse))
            kd, vd = k[b, h].double(), v[b, h].double()
            p = torch.where(seen, torch.exp(qd @ kd.T * D ** -0.5 - ls[..., None]), 0.0)
            ds = p * (gd @ vd.T - (gd * od).sum(-1, keepdim=True))
            for got, ref, name in ((dk[b, h], (ds.transpose(1, 2) @ qd).sum(0) * D ** -0.5, "dK"),
                                   (dv[b, h], (p.transpose(1, 2) @ gd).sum(0), "dV")):
                err = float((got.double() - ref).norm() / ref.norm())
                assert err <= 2.0 ** -7.5, f"{name} of batch {b}, head {h} is off by {err}"
    lo, hi = 0, loop.ws.numel() // 256               # the smallest workspace, in units of 256 bytes: found by what is refused
    while hi - lo > 1:
        mid = (lo + hi) // 2
        try:
            backward(loop.ws[:mid * 256], L.LVX_BWD_DELTA)
            hi = mid
        except L.LvxError:
            lo = mid
    ones = backward(loop.ws[:hi * 256], L.LVX_BWD_ALL)
    need = L.lvx_xattn_workspace_bytes(L.make_problem(q, k), L.LVX_BF16, L.LVX_WS_BWD)
    for size in (need, hi * 256 + 7 * (need - hi * 256) // 8):
        ws = torch.full_like(loop.ws[:size // 256 * 256], 0xa5)
        got = backward(ws, L.LVX_BWD_DELTA | L.LVX_BWD_DKDV)
        assert bool((ws[hi * 256:] != 0xa5).any()) == parts, f"parts or none in {size} bytes"
        for two, one in zip(got, ones):
            assert float((two.float() - one.float()).norm() / one.float().norm()) <= 2.0 ** -8


@pytest.mark.parametrize("shape", [(1, 8, 1, 64, 31, 700), (2, 8, 8, 64, 64, 16 * 256)], ids=lambda s: "x".join(map(str, s)))
def test_no_parts(shape):
    """Fewer rows than a step; a full round of tiles."""
    _case(*shape, parts=False)


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("shape", [(1, 2, 1, 700, 2), (2, 4, 2, 417, 700), (1, 8, 1, 1024, 256), (3, 5, 5, 1000, 513)],
                         ids=lambda s: "x".join(map(str, s)))
def test_few_keys(D, shape):
    B, Hq, Hkv, Sq, Skv = shape
    _case(B, Hq, Hkv, D, Sq, Skv)


@pytest.mark.parametrize("shape", [(1, 8, 8, 64, 2000, 33 * 256 + 5), (1, 4, 4, 64, 2048, 66 * 256), (1, 7, 1, 128, 417, 260 * 256 - 9)],
                         ids=lambda s: "x".join(map(str, s)))
def test_last_round(shape):
    _case(*shape)


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("mask", [(1, 8, 2, 600, 1200, 8, 64, "causal"), (2, 4, 2, 999, 4 * 729, 250, 729, "recent"),
                                  (1, 8, 2, 700, 1024, 64, 256, "causal"), (1, 8, 4, 1024, 2048, 256, 512, "recent")],
                         ids=lambda m: "x".join(map(str, m)))
def test_lists_of_steps(D, mask):
    B, Hq, Hkv, Sq, Skv, q_chunk, kv_block, rule = mask
    _case(B, Hq, Hkv, D, Sq, Skv, q_chunk, kv_block, rule)
