"""The backward of a call masked by words makes the words and the row statistics in one launch.  Asked for stage by stage it
makes them in two, from the same code: every result has the same bits, at sizes where the two parts of the grid or their last
workgroups can go wrong -- fewer rows than a workgroup's 32, rows that fill no tile of 256, a bitmap per batch entry or one for
all, one and several words of key blocks, and the kernels of the backward asked for one at a time."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,per_batch,Hq,Hkv,Sq,Skv,D,q_chunk,kv_block", [
    (1, False, 2, 1, 33, 700, 64, 5, 100),
    (2, True, 4, 2, 257, 1300, 96, 7, 64),
    (2, False, 3, 3, 300, 8300, 64, 2, 64),
    (3, True, 2, 2, 512, 2187, 128, 37, 729),
])
def test_words_and_statistics_in_one_launch(B, per_batch, Hq, Hkv, Sq, Skv, D, q_chunk, kv_block):
    from paper_2502_02406_amd import binding as Bi
    g = torch.Generator(device="cuda").manual_seed(Sq + Skv)
    q, do = (torch.randn((B, Hq, Sq, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    k, v = (torch.randn((B, Hkv, Skv, D), generator=g, device="cuda").bfloat16() for _ in range(2))
    shape = (-(-Sq // q_chunk), -(-Skv // kv_block))
    allow = (torch.rand((B, *shape) if per_batch else shape, generator=g, device="cuda") < 0.3).to(torch.uint8)
    mask = Bi.make_mask(allow, q_chunk, kv_block)
    p = Bi.make_problem(q, k)
    ws = torch.empty(max(Bi.lvx_xattn_workspace_bytes(p, Bi.dtype_code(torch.bfloat16), n) for n in (0, 1)), dtype=torch.uint8, device="cuda")
    o, lse = torch.empty_like(q), torch.empty((B, Hq, Sq), device="cuda")
    Bi.lvx_xattn_fwd(p, q, k, v, mask, o, lse, ws)

    def backward(calls):
        dq, dk, dv = torch.zeros((B, Hq, Sq, D), device="cuda"), torch.zeros_like(k), torch.zeros_like(v)
        ws.fill_(0xff)                              # what a call does not write itself is NaN
        for stages in calls:
            Bi.lvx_xattn_bwd(p, q, k, v, o, lse, do, mask, dq, dk, dv, ws, stages)
        torch.cuda.synchronize()
        return dq, dk, dv

    apart = backward([1, 2, 4])
    assert all(bool(torch.isfinite(x).all()) for x in apart) and all(float(x.abs().max()) > 0 for x in apart)
    for calls in ([7], [1, 6], [3, 4], [5, 2]):
        for x, y in zip(apart, backward(calls)):
            assert torch.equal(x, y), calls
