"""What the block loop hands to the library, with the library replaced by a recorder: no GPU needed."""
import pytest
import torch

from paper_2502_02406_amd import binding as B
from paper_2502_02406_amd.blockloop import BlockLoop


class Dev:
    """A host tensor that says it is on the device."""
    is_cuda = True

    def __init__(self, t):
        self.t = t

    def __getattr__(self, name):
        return getattr(self.t, name)


class Recorder:
    """The library's entry points: (name, keys of the problem passed, the addresses that follow it)."""

    def __init__(self):
        self.calls = []

    def lvx_xattn_workspace_bytes(self, p, dtype, which):
        return 256

    def __getattr__(self, name):
        def call(p, *a):
            self.calls.append((name, getattr(p, "_obj", p), getattr(getattr(p, "_obj", None), "Skv", None), a))
            return 0
        return call


@pytest.fixture
def lib(monkeypatch):
    r = Recorder()
    monkeypatch.setattr(torch.cuda, "is_available", lambda: True)
    monkeypatch.setattr(B, "load", lambda: r)
    monkeypatch.setattr(B, "_stream", lambda: 0)
    monkeypatch.setattr(B, "lvx_xattn_merge", lambda *a: None)
    monkeypatch.setattr(B, "lvx_xattn_dq_finalize", lambda *a: None)
    return r


def make(dtype=torch.bfloat16, Skv=2048, n_blocks=2):
    return BlockLoop((1, 4, 64, 64), (1, 2, Skv, 64), dtype, n_blocks, device="cpu")


def tensors(Skv, dtype=torch.bfloat16):
    q, o, do = (Dev(torch.zeros((1, 4, 64, 64), dtype=dtype)) for _ in range(3))
    k, v, dk, dv = (Dev(torch.zeros((1, 2, Skv, 64), dtype=dtype)) for _ in range(4))
    return q, k, v, o, torch.zeros((1, 4, 64)), do, dk, dv


@pytest.mark.parametrize("Skv,lengths", [(2048, [1024, 1024]), (1536, [1024, 512]), (1025, [1024, 1])])
def test_blocks_end_with_the_keys_that_are_given(lib, Skv, lengths):
    # a loop made for 2048 keys in two blocks: what it is called with decides how long the last one is
    q, k, v, o, lse, do, dk, dv = tensors(Skv)
    loop = make()
    loop.forward(q, k, v)
    starts = [0, 1024 * 64 * 2]
    fwd = [c for c in lib.calls if "fwd" in c[0]]
    assert [c[2] for c in fwd] == lengths
    assert [(c[3][2] - k.data_ptr(), c[3][3] - v.data_ptr()) for c in fwd] == [(s, s) for s in starts]
    lib.calls.clear()
    loop.backward(q, k, v, o, lse, do, dk, dv)
    assert [c[2] for c in lib.calls] == lengths
    for c, s in zip(lib.calls, starts):
        a = c[3]
        assert (a[2] - k.data_ptr(), a[3] - v.data_ptr(), a[9] - dk.data_ptr(), a[10] - dv.data_ptr()) == (s,) * 4


@pytest.mark.parametrize("n_blocks", [1, 2])
@pytest.mark.parametrize("short", ["v", "dk", "dv", "o", "do", "lse", "q"])
def test_tensors_that_the_kernels_would_leave_are_refused(lib, short, n_blocks):
    # an address is all that the library gets: a tensor smaller than K (or than Q; a Q larger than the
    # loop's results) would be read or written past its end
    t = dict(zip(("q", "k", "v", "o", "lse", "do", "dk", "dv"), tensors(2048)))
    if short == "q":
        t["q"] = t["o"] = t["do"] = Dev(torch.zeros((1, 4, 65, 64), dtype=torch.bfloat16))
        t["lse"] = torch.zeros((1, 4, 65))
    else:
        cut = t[short]
        cut = cut.t if isinstance(cut, Dev) else cut
        t[short] = Dev(cut[:, :, :-1]) if cut.dim() == 4 else cut[:, :, :-1].contiguous()
    loop = make(n_blocks=n_blocks)
    if short in ("v", "q"):
        with pytest.raises(ValueError):
            loop.forward(t["q"], t["k"], t["v"])
    with pytest.raises(ValueError):
        loop.backward(*(t[n] for n in ("q", "k", "v", "o", "lse", "do", "dk", "dv")))
    assert not lib.calls


def test_stride_of_a_single_batch_means_nothing(lib):
    # V as two of the five heads of a longer buffer: only its batch stride differs from K's
    q, k, v, o, lse, do, dk, dv = tensors(2048)
    v = Dev(torch.zeros((1, 5, 2048, 64), dtype=torch.bfloat16)[:, 1:3])
    assert v.stride()[1:] == k.stride()[1:] and v.stride(0) != k.stride(0)
    make().backward(q, k, v, o, lse, do, dk, dv)
    assert len(lib.calls) == 2
    with pytest.raises(AssertionError):          # (a head stride does mean something)
        make().backward(q, k, Dev(torch.zeros((1, 2, 2049, 64), dtype=torch.bfloat16)[:, :, :2048]), o, lse, do, dk, dv)


def test_float32_results_as_the_next_call_s_inputs(lib):
    # float32 results are the running state itself, which the first visit writes while the others still
    # read their inputs: what the library reads lies elsewhere
    f32 = torch.float32
    loop = make(f32)
    loop.o, loop.dq_accum = Dev(loop.o), Dev(loop.dq_accum)
    loop.o_acc, loop.dq = loop.o, loop.dq_accum
    q, k, v, o, lse, do, dk, dv = tensors(2048, f32)
    inside = lambda x, t: 0 <= x - t.data_ptr() < t.numel() * 4
    loop.forward(loop.forward(q, k, v)[0], k, v)
    reads = [a for c in lib.calls if "fwd" in c[0] for a in c[3][1:4]]
    assert len(reads) == 12 and not any(inside(a, loop.o) for a in reads)
    lib.calls.clear()
    loop.backward(q, k, v, o, lse, loop.backward(q, k, v, o, lse, do, dk, dv), dk, dv)
    reads = [a for c in lib.calls for a in c[3][1:7]]
    assert len(reads) == 24 and not any(inside(a, loop.dq_accum) for a in reads)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_results_as_inputs(dtype):
    # a result handed on as the next call's Q or dO is read whole, whatever the call writes first
    g = torch.Generator().manual_seed(4)
    q, do = (torch.randn((1, 4, 64, 64), generator=g).to(dtype).cuda() for _ in range(2))
    k, v = (torch.randn((1, 2, 256, 64), generator=g).to(dtype).cuda() for _ in range(2))
    a, b = (BlockLoop(tuple(q.shape), tuple(k.shape), dtype, 2) for _ in range(2))
    dk, dv = torch.empty_like(k), torch.empty_like(v)
    o, _ = a.forward(q, k, v)
    want = b.forward(o.clone(), k, v)[0].clone()
    assert torch.equal(a.forward(o, k, v)[0], want)
    o, lse = (t.clone() for t in b.forward(q, k, v))
    dq = a.backward(q, k, v, o, lse, do, dk, dv)
    want = [t.clone() for t in (b.backward(q, k, v, o, lse, dq.clone(), dk, dv), dk, dv)]
    assert all(torch.equal(x, y) for x, y in zip((a.backward(q, k, v, o, lse, dq, dk, dv), dk, dv), want))


def test_layer_refuses_gradients_that_are_not_laid_out_as_q(lib, monkeypatch):
    # what RecomputeLayer.backward is handed reaches the library by address: its type, shape and strides are looked at first
    from paper_2502_02406_amd import blockloop
    monkeypatch.setattr(B, "lvx_xattn_project", lambda *a, **k: None)
    monkeypatch.setattr(B, "lvx_xattn_project_bwd", lambda *a, **k: None)
    layer = blockloop.RecomputeLayer(1, 64, 256, 128, 4, 2, 64, torch.bfloat16, 2, device="cpu")
    layer.q = Dev(layer.q)
    x, y, good, lse = torch.zeros(1, 64, 128), torch.zeros(1, 256, 128), torch.zeros((1, 4, 64, 64), dtype=torch.bfloat16), torch.zeros(1, 4, 64)
    layer.backward(x, y, None, None, good, lse, good)
    assert [c[0] for c in lib.calls] == ["lvx_xattn_bwd_visit"] * 2
    for bad in (good.float(), good[:, :, :32], good.transpose(1, 2).contiguous().transpose(1, 2), good[:, :3]):
        for o, do in ((bad, good), (good, bad)):
            with pytest.raises(AssertionError):
                layer.backward(x, y, None, None, o, lse, do)
