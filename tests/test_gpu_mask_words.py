"""Media masks that cut through tiles, against the fp64 oracle: the kernels that keep or drop
probabilities by one word per (32 query rows, key block) at the sizes where the words can go wrong --
chunks of one row, of an odd length, longer than a workgroup's rows; key blocks that straddle the
workgroups' keys, that several share, that one fills; a last step of rows that overlaps the one
before (Sq % 32), a last key block of a few keys, rows and keys that pair with nothing, a bitmap per
batch entry, several heads per K/V head.  Tolerances: those of test_gpu_parity (bf16)."""
import numpy as np
import pytest
import torch

from test_gpu_parity import run_case, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,kw,p_on", [
    ("mw_chunks_of_one", dict(D=64, Hq=2, Hkv=1, Sq=96, Skv=1024, q_chunk=1, kv_block=64), 0.3),
    ("mw_odd_chunks_729", dict(Hq=7, Hkv=1, Sq=333, Skv=2187 + 10, q_chunk=37, kv_block=729), 0.5),
    ("mw_recent_pairs", dict(D=64, Hq=2, Hkv=2, Sq=512, Skv=16384, q_chunk=2, kv_block=64), "recent"),
    ("mw_batch_ragged", dict(B=2, Hq=4, Hkv=2, Sq=65, Skv=1333, q_chunk=16, kv_block=100), 0.4),
    ("mw_causal_729", dict(Hq=4, Hkv=1, Sq=640, Skv=7290, q_chunk=64, kv_block=729), "causal"),
    ("mw_long_chunks_d96", dict(D=96, Hq=4, Hkv=2, Sq=700, Skv=1500, q_chunk=300, kv_block=450), 0.6),
    ("mw_sparse", dict(Hq=2, Sq=288, Skv=6000, q_chunk=9, kv_block=75), 0.03),
    ("mw_short_blocks", dict(Hq=2, Sq=70, Skv=700, q_chunk=33, kv_block=40), 0.5),
])
def test_masks_by_words(name, kw, p_on):
    w = small(name, **kw)
    nq, nk = -(-w.Sq // w.q_chunk), -(-w.Skv // w.kv_block)
    if p_on == "recent":
        allow = np.arange(nk)[None, :] == np.minimum(np.arange(nq)[:, None], nk - 1)
    elif p_on == "causal":
        allow = np.arange(nk)[None, :] <= np.arange(nq)[:, None]
    else:
        rng = np.random.Generator(np.random.Philox(99 + len(name)))
        allow = rng.random((w.B, nq, nk) if w.B > 1 else (nq, nk)) < p_on
    run_case(w, do_bwd=True, allow=allow)


@pytest.mark.parametrize("D", [64, 128])
def test_rows_whose_keys_score_far_below_the_first_tile(D):
    # Rows of chunk c see key block c only; the keys of block 0 are 40 times larger along one direction
    # that all queries share, so they score up to hundreds of units above everybody else's: a
    # reference taken from them leaves a row that does not see them no probability at all.
    import torch
    import oracle
    from paper_2502_02406_amd import workloads as W
    from paper_2502_02406_amd.blockloop import BlockLoop, MediaMask
    from test_gpu_parity import TOL, check_fwd
    w = small(f"mw_far_below_d{D}", D=D, Hq=2, Sq=128, Skv=1024, q_chunk=16, kv_block=128)
    x = W.make_inputs(w)
    x["q"][..., 0] = 4.0
    x["k"][:, :, :128, 0] = 800.0
    allow = torch.from_numpy((np.arange(8)[None, :] == np.arange(8)[:, None]).astype(np.uint8))
    loop = BlockLoop(tuple(x["q"].shape), tuple(x["k"].shape), torch.bfloat16, 1,
                     MediaMask(allow.cuda(), w.q_chunk, w.kv_block))
    O, L = loop.forward(*(x[n].cuda() for n in ("q", "k", "v")))
    torch.cuda.synchronize()
    Oref, Lref = oracle.fwd(*(W.as_f32_numpy(x[n]) for n in ("q", "k", "v")), mask=oracle.Mask(allow.numpy(), w.q_chunk, w.kv_block))
    check_fwd(O, L, Oref, Lref, TOL["bf16"], w.name)


def test_a_key_that_scores_far_above_the_rest_costs_nothing():
    # The first key of each frame scores 150 units of log2 above the others, which leaves one half-wave of every row without a sum
    # worth the name for good.  Asking such lanes again in every half took 2.1 times as long; the same run twice
    # differs by a few per cent.
    import torch
    from paper_2502_02406_amd.blockloop import BlockLoop, MediaMask
    g = torch.Generator(device="cuda").manual_seed(13)
    q = torch.randn((1, 16, 1024, 128), generator=g, device="cuda").bfloat16()
    k, v = (torch.randn((1, 16, 16384, 128), generator=g, device="cuda").bfloat16() for _ in range(2))
    q[..., 0] = 4.0
    loop = BlockLoop(tuple(q.shape), tuple(k.shape), torch.bfloat16, 1,
                     MediaMask(torch.ones((22, 16), dtype=torch.uint8, device="cuda"), 48, 1024))

    def ms():
        times = []
        for _ in range(8):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(5):
                loop.forward(q, k, v)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b) / 5)
        return min(times)

    even = ms()
    k[:, :, ::1024, 0] = 300.0       # (of every frame: every split of the keys has one)
    assert ms() <= 1.4 * even


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("q_chunk,kv_block", [(2, 64), (16, 64), (24, 100), (2, 729)])
def test_the_largest_probability_is_not_rounded(q_chunk, kv_block, D):
    # Every row sees one frame, in which one key (in any half of a tile) scores 40 above the rest and otherwise like
    # no other frame's: its probability is 1 and O its V.  Rounded to bf16 relative to some other reference it would
    # be off by up to 2^-9.  The float32 bound: the reference (64 .. 128 in units of log2) is rounded, by 2^-18 at most,
    # which the sum sees and the bf16 probability does not: 2^-18 ln 2 of O; as much again for the sum, its inverse and
    # the combine of the splits (some units of 2^-24), and the rest of the frame (e^-40).
    import torch
    from paper_2502_02406_amd import binding as B
    from paper_2502_02406_amd.blockloop import BlockLoop, MediaMask
    g = torch.Generator().manual_seed(14)
    Sq, nf = 24 * q_chunk, 24
    q = 0.1 * torch.randn((1, 2, Sq, D), generator=g)
    k, v = (0.1 * torch.randn((1, 1, nf * kv_block, D), generator=g) for _ in range(2))
    top = torch.arange(nf) * kv_block + torch.randint(0, kv_block, (nf,), generator=g)
    q[..., 0] = 1.0
    k[0, 0, top, 0] = D ** 0.5 * (42.0 + 3.0 * torch.rand(nf, generator=g))
    q, k, v = (t.bfloat16().cuda() for t in (q, k, v))
    loop = BlockLoop(tuple(q.shape), tuple(k.shape), torch.bfloat16, 1,
                     MediaMask(torch.eye(nf, dtype=torch.uint8).cuda(), q_chunk, kv_block))
    o = torch.empty(q.shape, dtype=torch.float32, device="cuda")
    B.lvx_xattn_fwd(B.make_problem(q, k, 0.0), q, k, v, loop._mask_for(0), o, loop.lse, loop.ws)
    want = v[0, 0, top.repeat_interleave(q_chunk).cuda()].float()
    assert ((o - want).abs() <= 2.0 ** -17 * 0.6932 * want.abs() + 1e-12).all()


@pytest.mark.parametrize("merge", [False, True])
def test_words_that_do_not_fit_the_workspace(merge):
    # 16 heads x 64 row tiles fill the chip without splits, so that the kernels that do without words need 256 bytes of
    # workspace: with less than the words take (35 KB) such a call runs on them.  Tolerances: those of bf16.
    import torch
    from paper_2502_02406_amd import binding as B
    from paper_2502_02406_amd.blockloop import BlockLoop, MediaMask
    g = torch.Generator().manual_seed(15)
    q = (0.5 * torch.randn((1, 16, 16384, 64), generator=g)).bfloat16().cuda()
    k, v = (0.5 * torch.randn((1, 16, 1024, 64), generator=g).bfloat16().cuda() for _ in range(2))
    allow = (torch.rand((4096, 16), generator=g) < 0.5).to(torch.uint8)
    loop = BlockLoop(tuple(q.shape), tuple(k.shape), torch.bfloat16, 1, MediaMask(allow.cuda(), 4, 64))
    p, m = B.make_problem(q, k, 0.0), loop._mask_for(0)
    call = B.lvx_xattn_fwd_merge if merge else B.lvx_xattn_fwd

    def run(ws):
        o, lse = torch.zeros(q.shape, device="cuda"), torch.full(q.shape[:3], float("-inf"), device="cuda")
        call(p, q, k, v, m, o, lse, ws)
        return o, lse

    o, lse = run(loop.ws)
    o2, lse2 = run(torch.empty(4096, dtype=torch.uint8, device="cuda"))
    seen = torch.isfinite(lse)
    assert torch.equal(seen, torch.isfinite(lse2)) and not o2[~seen].any()
    assert (o - o2).abs().max() <= 1e-2 and (lse - lse2)[seen].abs().max() <= 1e-3
    with pytest.raises(B.LvxError):
        run(torch.empty(128, dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("Hq,Sq,w", [(1, 256, 2036), (1, 256, 2000), (1, 512, 2038), (2, 100, 1000)])
def test_backward_of_one_head_has_room_for_the_words(Hq, Sq, w):
    """Key blocks of 64 whose words fill the place of a slice of dQ sums almost, or to the last byte: they are used (the place is
    written to by a call without the dQ kernel, as the general kernels would not), and the results are right."""
    from paper_2502_02406_amd import binding as L
    from paper_2502_02406_amd.blockloop import BlockLoop, MediaMask
    g = torch.Generator(device="cuda").manual_seed(15)
    D, Skv = 64, 64 * w
    q, do = (torch.randn((1, Hq, Sq, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    k, v = (torch.randn((1, 1, Skv, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    c, f = torch.arange(-(-Sq // 20))[:, None], torch.arange(w)[None, :]
    allow = ((f * 7 + c * 3) % 40 == 0).to(torch.uint8).cuda()
    loop = BlockLoop(tuple(q.shape), tuple(k.shape), torch.bfloat16, 1, MediaMask(allow, 20, 64))
    o, lse = (t.clone() for t in loop.forward(q, k, v))
    dk, dv = torch.empty_like(k), torch.empty_like(v)
    dq = loop.backward(q, k, v, o, lse, do, dk, dv)
    seen = allow.bool().repeat_interleave(20, 0)[:Sq].repeat_interleave(64, 1)
    kd, vd = k[0, 0].double(), v[0, 0].double()
    rk, rv = torch.zeros_like(kd), torch.zeros_like(vd)
    for h in range(Hq):
        qd, gd, od = q[0, h].double(), do[0, h].double(), o[0, h].double()
        p = torch.where(seen, torch.exp(qd @ kd.T * D ** -0.5 - lse[0, h].double()[:, None]), 0.0)
        ds = p * (gd @ vd.T - (gd * od).sum(-1, keepdim=True))
        rq = ds @ kd * D ** -0.5
        rk, rv = rk + ds.T @ qd * D ** -0.5, rv + p.T @ gd
        assert float((dq[0, h].double() - rq).norm() / rq.norm()) <= 2.0 ** -7.5
    assert float((dk[0, 0].double() - rk).norm() / rk.norm()) <= 2.0 ** -7.5
    assert float((dv[0, 0].double() - rv).norm() / rv.norm()) <= 2.0 ** -7.5
    loop.ws.fill_(0xa5)
    acc = torch.zeros(q.shape, device="cuda")
    L.lvx_xattn_bwd(L.make_problem(q, k), q, k, v, o, lse, do, loop._mask_for(0), acc, dk, dv, loop.ws, L.LVX_BWD_DELTA | L.LVX_BWD_DKDV)
    rows = (Sq + 31) // 32 * 32 * Hq
    at = -(-Hq * Sq * 4 // 256) * 256 + -(-(rows * 2 + (Hq * 64 if Sq % 32 else 0)) * 4 // 256) * 256
    assert bool((loop.ws[at:at + 32 * w] != 0xa5).any()), "no words"
