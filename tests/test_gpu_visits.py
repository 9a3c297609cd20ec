"""The block loop's first and last visits: nothing that the running buffers held before counts, and the last visit's
rounded result is what the separate conversion makes of the running one.  (The sums are formed in the same order
and rounded once either way: equal, but for a running 0 that is added.)"""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,n_blocks,Hq,Hkv,Sq,Skv,q_chunk,kv_block", [
    (torch.bfloat16, 1, 4, 2, 150, 700, 0, 0),             # one workgroup's rows split over the keys
    (torch.bfloat16, 2, 4, 2, 150, 1400, 0, 0),
    (torch.bfloat16, 3, 8, 8, 2000, 3 * 192, 0, 0),        # not split
    (torch.bfloat16, 2, 8, 2, 3, 4000, 0, 0),              # few rows
    (torch.bfloat16, 1, 4, 2, 100, 50, 0, 0),              # fewer keys than a tile: the general kernels
    (torch.bfloat16, 2, 4, 2, 256, 2048, 64, 128),         # masks by tile lists, by words (dense and streamed), in two launches
    (torch.bfloat16, 2, 4, 2, 300, 2 * 729, 48, 729),
    (torch.bfloat16, 2, 4, 2, 300, 2048, 2, 64),
    (torch.bfloat16, 2, 4, 2, 300, 2048, 24, 16),
    (torch.bfloat16, 2, 4, 2, 300, 600, 7, 20),
    (torch.float32, 2, 4, 2, 150, 300, 0, 0),
    (torch.float32, 2, 4, 2, 100, 320, 8, 32),
])
@pytest.mark.parametrize("D", [64, 96, 128])
def test_running_buffers(D, dtype, n_blocks, Hq, Hkv, Sq, Skv, q_chunk, kv_block):
    from paper_2502_02406_amd import binding as L
    from paper_2502_02406_amd.blockloop import BlockLoop, MediaMask
    g = torch.Generator(device="cuda").manual_seed(2)
    q, do = (torch.randn((1, Hq, Sq, D), generator=g, device="cuda").to(dtype) for _ in range(2))
    k, v = (torch.randn((1, Hkv, Skv, D), generator=g, device="cuda").to(dtype) for _ in range(2))
    mask = None
    if q_chunk:
        nq, nk = -(-Sq // q_chunk), -(-Skv // kv_block)
        f, c = torch.arange(nk)[None, :], torch.arange(nq)[:, None]
        mask = MediaMask(((f % nq == c) | (f == 0) & (c % 3 != 1)).to(torch.uint8).cuda(), q_chunk, kv_block)   # some rows see nothing of a block
    loop = BlockLoop(tuple(q.shape), tuple(k.shape), dtype, n_blocks, mask)
    for t in (loop.o, loop.lse, loop.dq_accum, loop.dq, loop.o_acc):
        if t is not None:
            t.fill_(float("nan"))
    o, lse = loop.forward(q, k, v)
    # the same visits, with the running result rounded by a call of its own
    p, step = loop._blocks(q, k, (v,))
    call = L.Calls(p, q.dtype, loop.ws)
    o_acc, l_acc = torch.zeros(q.shape, dtype=torch.float32, device="cuda"), torch.full(q.shape[:3], float("-inf"), device="cuda")
    a = [t.data_ptr() for t in (q, k, v)]
    for n in range(n_blocks):
        p.Skv = loop._keys_of(n, k)
        at = [a[1] + n * step, a[2] + n * step]
        if n == 0:
            call.fwd(a[0], *at, loop._mask_for(0), o_acc.data_ptr(), torch.float32, l_acc.data_ptr())
        else:
            call.fwd_merge(a[0], *at, loop._mask_for(n), o_acc.data_ptr(), l_acc.data_ptr())
    assert torch.equal(lse, l_acc) and torch.equal(o, o_acc.to(dtype))
    dk, dv = torch.empty_like(k), torch.empty_like(v)
    dq = loop.backward(q, k, v, o, lse, do, dk, dv)
    acc, dk2, dv2 = torch.zeros_like(o_acc), torch.empty_like(k), torch.empty_like(v)
    b = [t.data_ptr() for t in (o, lse, do)]
    for n in range(n_blocks):
        p.Skv = loop._keys_of(n, k)
        call.bwd(a[0], a[1] + n * step, a[2] + n * step, *b, loop._mask_for(n), acc.data_ptr(), dk2.data_ptr() + n * step,
                 dv2.data_ptr() + n * step, L.LVX_BWD_ALL if n == 0 else L.LVX_BWD_DKDV | L.LVX_BWD_DQ)
    assert torch.equal(dq, acc.to(dtype)) and torch.equal(dk, dk2) and torch.equal(dv, dv2)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_results_come_back_as_inputs(dtype):
    """O and dQ, buffers of the loop, as the next call's operands: the last visit writes them while others are still read."""
    from paper_2502_02406_amd.blockloop import BlockLoop
    g = torch.Generator(device="cuda").manual_seed(4)
    q, k, v, do = (torch.randn((1, 4, 640, 64), generator=g, device="cuda").to(dtype) for _ in range(4))
    loop = BlockLoop(tuple(q.shape), tuple(k.shape), dtype, 2)
    dk, dv = torch.empty_like(k), torch.empty_like(v)
    o, lse = (t.clone() for t in loop.forward(q, k, v))
    for back in ((q, loop.o, v), (q, k, loop.o), (loop.o, loop.o, loop.o)):
        loop.o.copy_(o)
        want = loop.forward(*(t.clone() for t in back))[0].clone()
        loop.o.copy_(o)
        assert torch.equal(loop.forward(*back)[0], want)
    x = loop.backward(q, k, v, o, lse, do, dk, dv).clone()
    for back in ((q, loop.dq, v, o, lse, do), (q, k, loop.dq, o, lse, do), (q, k, v, o, lse, loop.dq), (loop.dq, k, v, loop.dq, lse, loop.dq)):
        loop.dq.copy_(x)
        want = [t.clone() for t in (loop.backward(*(t.clone() for t in back), dk, dv), dk, dv)]
        loop.dq.copy_(x)
        assert all(torch.equal(a, b) for a, b in zip((loop.backward(*back, dk, dv), dk, dv), want))


@pytest.mark.parametrize("D,Hq,Hkv,Sq,Skv,q_chunk,kv_block", [
    (64, 8, 8, 33 * 256 - 5, 2000, 0, 0),                  # row tiles left whole beside split ones
    (128, 4, 2, 700, 150, 0, 0), (96, 8, 2, 3, 100, 0, 0), (64, 8, 2, 3, 4000, 0, 0), (128, 4, 2, 100, 50, 0, 0),
    (64, 4, 2, 500, 640, 64, 128), (64, 4, 2, 500, 320, 24, 64), (96, 4, 2, 500, 8 * 729, 48, 729), (64, 4, 2, 300, 640, 7, 20),
])
def test_last_visit_into_q_itself(D, Hq, Hkv, Sq, Skv, q_chunk, kv_block):
    from paper_2502_02406_amd import binding as L
    g = torch.Generator(device="cuda").manual_seed(8)
    q = torch.randn((2, Hq, Sq, D), generator=g, device="cuda").bfloat16()
    k, v = (torch.randn((2, Hkv, Skv, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    mask = None
    if q_chunk:
        c, f = torch.arange(-(-Sq // q_chunk))[:, None], torch.arange(-(-Skv // kv_block))[None, :]
        allow = ((f - c) % 3 == 0).to(torch.uint8).cuda()
        mask = L.make_mask(allow, q_chunk, kv_block)
    acc0, l0 = torch.randn(q.shape, generator=g, device="cuda"), torch.randn((2, Hq, Sq), generator=g, device="cuda")
    p = L.make_problem(q, k)
    ws = torch.empty(L.lvx_xattn_workspace_bytes(p, L.LVX_BF16, L.LVX_WS_FWD_MERGE), dtype=torch.uint8, device="cuda")
    out = []
    for o in (torch.full_like(q, float("nan")), q):
        acc, lse = acc0.clone(), l0.clone()
        L.lvx_xattn_fwd_merge_last(p, q, k, v, mask, acc, lse, o, ws)
        out.append((o.clone(), lse))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
