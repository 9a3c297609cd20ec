"""The dense forward for 64-wide heads (two workgroups on a compute unit), against the fp64 oracle, where its loop can
go wrong: fewer key tiles than the ring has stages, one more, a ragged last tile that is the first or cuts either half,
rows that leave row blocks empty, references that have to be raised in either row block and half, parts beside whole row
tiles.  Tolerances: those of test_gpu_parity (bf16)."""
import pytest
import torch

import plans
from test_gpu_parity import run_case, small
from test_gpu_tail_split import _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Skv", [64, 65, 100, 128, 191, 192, 255, 256, 257, 320, 383, 449, 640])
def test_few_key_tiles(Skv):
    run_case(small(f"narrow_{Skv}", D=64, Hq=2, Hkv=1, Sq=97, Skv=Skv), do_bwd=False)


@pytest.mark.parametrize("Sq", [65, 96, 128, 129, 257])
def test_row_blocks_without_rows(Sq):
    run_case(small(f"narrow_rows_{Sq}", D=64, Hq=1, Hkv=1, Sq=Sq, Skv=500), do_bwd=False)


@pytest.mark.parametrize("key", [0, 31, 40, 64, 100, 133, 300, 511, 540])
@pytest.mark.parametrize("row", [3, 40])
def test_one_large_score_raises_the_reference(key, row):
    """Row `row` and key `key` point the same way, far longer than the rest: the row's softmax is that key, whose V its O is."""
    from paper_2502_02406_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn((1, 1, n, 64), generator=g, device="cuda") for n in (72, 541, 541))
    q[0, 0, row] = 3.0
    k[0, 0, key] = 4.0
    q, k, v = (t.bfloat16() for t in (q, k, v))
    o, lse = torch.empty_like(q), torch.empty((1, 1, 72), device="cuda")
    p = B.make_problem(q, k)
    ws = torch.empty(B.lvx_xattn_workspace_bytes(p, B.LVX_BF16, B.LVX_WS_FWD), dtype=torch.uint8, device="cuda")
    B.lvx_xattn_fwd(p, q, k, v, None, o, lse, ws)
    s = q[0, 0].double() @ k[0, 0].double().T * 0.125
    assert float((lse[0, 0].double() - torch.logsumexp(s, -1)).abs().max()) <= 1e-3
    ref = torch.softmax(s, -1) @ v[0, 0].double()
    assert float((o[0, 0].double() - ref).norm() / ref.norm()) <= 2.0 ** -7.5
    assert float((o[0, 0, row].double() - v[0, 0, key].double()).abs().max()) <= 2.0 ** -7 * float(v[0, 0, key].abs().max())


@pytest.mark.parametrize("shape,plan", [
    ((1, 8, 8, 64, 32 * 256 + 3, 900, 1), (32, 5)),             # a whole row tile for every compute unit, parts beside them
    ((1, 16, 16, 64, 17 * 256 + 3, 1100, 1), (16, 3)),          # ... of two heads on an XCD
    ((1, 8, 8, 64, 8 * 256, 2000, 2), (0, 4)),                  # parts of all, the second time merged with the running result
    ((1, 8, 8, 64, 70 * 256 - 1, 1100, 1), (64, 3)),            # two for every compute unit, then parts
    ((1, 2, 1, 64, 100, 6407, 1), (0, 26)),                     # a last part of one tile, which the tile before overlaps
], ids=lambda s: "x".join(map(str, s)))
def test_parts_beside_whole_row_tiles(shape, plan):
    B, Hq, Hkv, D, Sq, Skv, n_blocks = shape
    for n in range(n_blocks):                                   # (what the shape is here for)
        assert plans.fwd_plan(B, Hq, Hkv, Sq, Skv // n_blocks, D, running=n > 0) == plan
    _case(*shape)


def test_the_last_part_is_one_ragged_tile():
    tiles, parts = -(-6407 // 64), 26
    assert tiles - (parts - 1) * -(-tiles // parts) == 1 and 6407 % 64 != 0
