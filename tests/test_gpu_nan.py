"""Scores, values and gradients that are not finite.

A NaN in one key is a NaN in every result of the query rows that see it, and in no other: the float32
kernels (one block and a running state), the forward for few rows (one workgroup, splits with their
combine, a running state), whose combines leave out parts without keys but not parts without a value, and
the bf16 forward under masks by words.  Keys whose scores are -infinity have no weight.  What a tile repeats
or pads with (a ragged key or row count) adds nothing, be it infinite."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Skv", [100, 6000])
@pytest.mark.parametrize("dtype,Sq", [(torch.float32, 40), (torch.bfloat16, 1), (torch.bfloat16, 20)],
                         ids=["f32", "one_row", "rows"])
@pytest.mark.parametrize("n_blocks", [1, 2])
def test_nan_key(dtype, Sq, Skv, n_blocks):
    from paper_2502_02406_amd.blockloop import BlockLoop
    g = torch.Generator().manual_seed(5)
    q = torch.randn((1, 4, Sq, 64), generator=g).to(dtype).cuda()
    k, v = (torch.randn((1, 2, Skv, 64), generator=g).to(dtype).cuda() for _ in range(2))
    loop = BlockLoop(tuple(q.shape), tuple(k.shape), dtype, n_blocks)
    clean = loop.forward(q, k, v)[0].clone()
    for j in (0, Skv // 2 - 1, Skv - 1):
        bad = k.clone()
        bad[0, 1, j, 3] = float("nan")
        o = loop.forward(q, bad, v)[0]
        assert torch.isnan(o[:, 2:]).all(), f"key {j}: a row of the second K/V head has a value"
        assert torch.equal(o[:, :2], clean[:, :2]), f"key {j}: the first K/V head changed"


def test_infinite_gradient_of_a_row_without_keys():
    # float32: pairs that a mask leaves out add 0 to dQ whatever their dO says
    from paper_2502_02406_amd.blockloop import BlockLoop, MediaMask
    g = torch.Generator().manual_seed(6)
    q, do = (torch.randn((1, 2, 40, 64), generator=g).cuda() for _ in range(2))
    k, v = (torch.randn((1, 1, 100, 64), generator=g).cuda() for _ in range(2))
    allow = torch.ones((5, 4), dtype=torch.uint8)
    allow[2] = 0                                   # rows 16 .. 23 see no key
    loop = BlockLoop(tuple(q.shape), tuple(k.shape), torch.float32, 1, MediaMask(allow.cuda(), 8, 25))
    o, lse = loop.forward(q, k, v)
    dk, dv = torch.empty_like(k), torch.empty_like(v)
    clean = loop.backward(q, k, v, o, lse, do, dk, dv).clone()
    do[0, 1, 20] = float("inf")
    assert torch.equal(loop.backward(q, k, v, o, lse, do, dk, dv), clean)
    assert not clean[0, 1, 16:24].any()


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("q_chunk,kv_block", [(48, 128), (16, 100), (2, 64)])
def test_bad_key_in_a_frame_that_others_do_not_see(q_chunk, kv_block, D, bad):
    # chunk c sees the frames c and c + 1 (mod 12): O and L of the rows that do not see the bad key's frame
    # are as without it, but for the rounding of another reference: 2^-8 of a probability, 2^-9 of O
    from paper_2502_02406_amd.blockloop import BlockLoop, MediaMask
    g = torch.Generator().manual_seed(8)
    Sq, nf = 300, 12
    q = torch.randn((1, 2, Sq, D), generator=g).bfloat16().cuda()
    k, v = (torch.randn((1, 1, nf * kv_block, D), generator=g).bfloat16().cuda() for _ in range(2))
    chunk = torch.arange(-(-Sq // q_chunk))
    allow = torch.zeros((len(chunk), nf), dtype=torch.uint8)
    allow[chunk, chunk % nf] = allow[chunk, (chunk + 1) % nf] = 1
    loop = BlockLoop(tuple(q.shape), tuple(k.shape), torch.bfloat16, 1, MediaMask(allow.cuda(), q_chunk, kv_block))
    o0, l0 = (t.float() for t in loop.forward(q, k, v))
    for frame in (0, 3, nf - 1):
        for at in (0, kv_block - 1):
            k2 = k.clone()
            k2[0, 0, frame * kv_block + at, 5] = bad
            o, lse = (t.float() for t in loop.forward(q, k2, v))
            sees = allow[:, frame].bool().repeat_interleave(q_chunk)[:Sq].cuda()
            what = f"frame {frame} key {at}"
            assert ((lse - l0)[:, :, ~sees].abs() <= 2.0 ** -8).all(), what
            assert ((o - o0)[:, :, ~sees].abs() <= 2.0 ** -6 * o0.abs().max()).all(), what
            if bad != bad:
                assert torch.isnan(o[:, :, sees]).all(), what


@pytest.mark.parametrize("first,last", [(0, 40), (0, 5999), (32, 64), (100, 5000)])
@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("n_blocks", [1, 2])
def test_few_rows_against_keys_without_weight(n_blocks, D, first, last):
    from paper_2502_02406_amd.blockloop import BlockLoop
    g = torch.Generator().manual_seed(9)
    q = torch.randn((1, 4, 3, D), generator=g).bfloat16().cuda()
    k, v = (torch.randn((1, 2, 6000, D), generator=g).bfloat16().cuda() for _ in range(2))
    q[..., 3] = q[..., 3].abs() + 0.5
    q[:, :, 1, 3] = 0.5
    k[:, :, first:last, 3] = float("-inf")
    o, lse = BlockLoop(tuple(q.shape), tuple(k.shape), torch.bfloat16, n_blocks).forward(q, k, v)
    kd, vd = (t.double().repeat_interleave(2, 1) for t in (k, v))
    s = q.double() @ kd.transpose(2, 3) * D ** -0.5
    want = torch.softmax(s, -1) @ vd
    assert torch.allclose(o.double(), want, rtol=2e-2, atol=1e-2)
    assert torch.allclose(lse.double(), torch.logsumexp(s, -1), rtol=0, atol=1e-3)


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("Skv,j", [(100, 60), (64 * 3 + 20, 64 * 3 - 10), (64 * 40 + 1, 64 * 40 - 63), (64 * 12 + 63, 64 * 12 - 1)])
@pytest.mark.parametrize("masked", [False, True])
def test_infinite_value_of_a_key_that_the_last_tile_repeats(masked, Skv, j, D):
    from paper_2502_02406_amd.blockloop import BlockLoop, MediaMask
    g = torch.Generator().manual_seed(10)
    q = torch.randn((1, 4, 150, D), generator=g).bfloat16().cuda()
    k, v = (torch.randn((1, 2, Skv, D), generator=g).bfloat16().cuda() for _ in range(2))
    mask = None
    if masked:
        allow = torch.zeros((4, -(-Skv // 70)), dtype=torch.uint8)
        allow[:, -2:] = allow[:, j // 70:j // 70 + 1] = allow[1:, 0:1] = 1
        mask = MediaMask(allow.cuda(), 40, 70)
    loop = BlockLoop(tuple(q.shape), tuple(k.shape), torch.bfloat16, 1, mask)
    clean = loop.forward(q, k, v)[0].clone()
    v[0, 0, j, 7] = float("inf")
    o = loop.forward(q, k, v)[0]
    assert (o[:, :2, :, 7] == float("inf")).all()
    clean[:, :2, :, 7] = float("inf")
    assert torch.equal(o, clean)


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("Sq,Skv", [(40, 100), (7, 33), (33, 290)])
def test_infinities_in_the_last_key_and_row(Sq, Skv, D):
    # float32, no multiples of the 32-row tiles: an infinite V of the last key, an infinite dO of the last row
    from paper_2502_02406_amd.blockloop import BlockLoop
    g = torch.Generator().manual_seed(11)
    q, do = (torch.randn((1, 3, Sq, D), generator=g).cuda() for _ in range(2))
    k, v = (torch.randn((1, 1, Skv, D), generator=g).cuda() for _ in range(2))
    loop = BlockLoop(tuple(q.shape), tuple(k.shape), torch.float32, 1)
    o, lse = (t.clone() for t in loop.forward(q, k, v))
    dk, dv = torch.empty_like(k), torch.empty_like(v)
    loop.backward(q, k, v, o, lse, do, dk, dv)
    want = dv.clone()
    v2, do2 = v.clone(), do.clone()
    v2[0, 0, -1, 7] = do2[0, 2, -1, 3] = float("inf")
    o2 = loop.forward(q, k, v2)[0]
    o[..., 7] = want[..., 3] = float("inf")
    assert torch.equal(o2, o)
    loop.backward(q, k, v, o.nan_to_num(posinf=0.0), lse, do2, dk, dv)
    assert torch.equal(dv, want)


@pytest.mark.parametrize("blind", [0, 1])
def test_rows_that_see_nothing_of_a_block_with_a_bad_value(blind):
    # float32, two blocks: rows 0 .. 31 see nothing of block `blind`, whose V holds a NaN
    from paper_2502_02406_amd.blockloop import BlockLoop, MediaMask
    g = torch.Generator().manual_seed(12)
    q = torch.randn((1, 2, 64, 64), generator=g).cuda()
    k, v = (torch.randn((1, 1, 400, 64), generator=g).cuda() for _ in range(2))
    allow = torch.ones((2, 2), dtype=torch.uint8)
    allow[0, blind] = 0
    loop = BlockLoop(tuple(q.shape), tuple(k.shape), torch.float32, 2, MediaMask(allow.cuda(), 32, 200))
    clean, l0 = (t.clone() for t in loop.forward(q, k, v))
    v[0, 0, 200 * blind + 77, 4] = float("nan")
    o, lse = loop.forward(q, k, v)
    assert torch.equal(o[:, :, :32], clean[:, :, :32]) and torch.equal(lse, l0)
    assert torch.isnan(o[:, :, 32:, 4]).all()


@pytest.mark.parametrize("D,dtype,Hq,Hkv,Sq,Skv,q_chunk,kv_block", [
    (64, torch.bfloat16, 8, 8, 33 * 256 - 5, 2000, 0, 0),      # dense: row tiles left whole beside split ones
    (128, torch.bfloat16, 4, 2, 300, 150, 0, 0),               # ... not split
    (128, torch.bfloat16, 4, 2, 3, 60, 0, 0),                  # few rows
    (64, torch.bfloat16, 2, 1, 300, 320, 24, 64),              # words, streamed (not split)
    (64, torch.bfloat16, 2, 1, 300, 640, 256, 100),            # words, dense loop
    (64, torch.bfloat16, 2, 1, 300, 640, 256, 128),            # lists
    (96, torch.bfloat16, 2, 1, 300, 320, 24, 16),              # general kernel
    (64, torch.float32, 2, 1, 100, 320, 8, 32),
    (64, torch.float32, 2, 1, 100, 320, 0, 0),
])
def test_nan_key_is_a_nan_statistic(D, dtype, Hq, Hkv, Sq, Skv, q_chunk, kv_block):
    """L as well as O, by itself and merged with a running result of no keys or of some: an L of -infinity would be
    dropped by the next combine as that of rows without keys."""
    from paper_2502_02406_amd import binding as L
    g = torch.Generator().manual_seed(13)
    q = torch.randn((1, Hq, Sq, D), generator=g).to(dtype).cuda()
    k, v = (torch.randn((1, Hkv, Skv, D), generator=g).to(dtype).cuda() for _ in range(2))
    j = Skv // 3
    k[0, 0, j, 3] = float("nan")
    mask, sees = None, torch.ones(Sq, dtype=torch.bool, device="cuda")
    if q_chunk:
        c, f = torch.arange(-(-Sq // q_chunk))[:, None], torch.arange(-(-Skv // kv_block))[None, :]
        allow = ((f - c) % 5 == 0).to(torch.uint8).cuda()
        mask = L.make_mask(allow, q_chunk, kv_block)
        sees = allow[:, j // kv_block].bool().repeat_interleave(q_chunk)[:Sq]
    p = L.make_problem(q, k)
    n = max(L.lvx_xattn_workspace_bytes(p, L.dtype_code(dtype), w) for w in (L.LVX_WS_FWD, L.LVX_WS_FWD_MERGE))
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    o, lse = torch.empty_like(q), torch.empty((1, Hq, Sq), device="cuda")
    L.lvx_xattn_fwd(p, q, k, v, mask, o, lse, ws)
    heads = slice(0, Hq // Hkv)
    assert torch.isnan(o[0, heads][:, sees]).all() and torch.isnan(lse[0, heads][:, sees]).all()
    assert not torch.isnan(lse[0, Hq // Hkv:]).any()
    assert not torch.isnan(lse[:, :, ~sees]).any()
    for start in (float("-inf"), 1.0):
        acc, l_acc = torch.zeros(q.shape, device="cuda"), torch.full((1, Hq, Sq), start, device="cuda")
        L.lvx_xattn_fwd_merge(p, q, k, v, mask, acc, l_acc, ws)
        assert torch.isnan(acc[0, heads][:, sees]).all() and torch.isnan(l_acc[0, heads][:, sees]).all(), start
        L.lvx_xattn_merge([acc], [l_acc], o, l_acc)
        assert torch.isnan(o[0, heads][:, sees]).all(), start


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("kv_block", [66, 64 + 33])
def test_bad_keys_behind_a_streamed_frame(kv_block, D, bad):
    """Each row block sees a frame of its own (streamed); the keys behind the last of them, which nobody sees and no tile of
    64 keys holds together with one that is seen, are bad: a unit of 32 keys reaches into them."""
    from paper_2502_02406_amd.blockloop import BlockLoop, MediaMask
    g = torch.Generator().manual_seed(14)
    nf = 3 * 64
    end = next(f for f in range(8, nf) if f * kv_block % 64 == 0)
    q, do = (torch.randn((1, 2, 256, D), generator=g).bfloat16().cuda() for _ in range(2))
    k, v = (torch.randn((1, 1, nf * kv_block, D), generator=g).bfloat16().cuda() for _ in range(2))
    allow = torch.zeros((8, nf), dtype=torch.uint8)
    allow[torch.arange(8), end - 8 + torch.arange(8)] = 1
    loop = BlockLoop(tuple(q.shape), tuple(k.shape), torch.bfloat16, 1, MediaMask(allow.cuda(), 32, kv_block))
    out = []
    for fill in (None, bad):
        if fill is not None:
            k[:, :, end * kv_block:] = v[:, :, end * kv_block:] = fill
        dk, dv = torch.empty_like(k), torch.empty_like(v)
        o, lse = loop.forward(q, k, v)
        dq = loop.backward(q, k, v, o, lse, do, dk, dv)
        out.append([t.clone() for t in (o, lse, dq, dk[:, :, :end * kv_block], dv[:, :, :end * kv_block])])
    for name, a, b in zip(("O", "L", "dQ", "dK", "dV"), *out):
        assert torch.equal(a, b), name
