"""The projections' choices of tile height and of how dW's token parts meet, each at a small size, on
sampled tokens and columns against the fp64 oracle (bounds: those of test_gpu_project).  256-token tiles
need more than 192 of them (50000 tokens with one column tile, the last tile ragged); two and three parts
per dW tile take turns, four and more go through memory."""
import numpy as np
import pytest
import torch

from paper_2502_02406_amd import workloads as W
from test_gpu_project import check, check_bwd, run, run_bwd

pytestmark = pytest.mark.gpu


def _sample(S, N, k=12):
    rng = np.random.default_rng(S + N)
    rows = np.stack([np.zeros(k, dtype=np.int64), np.sort(rng.choice(S, k, replace=False))], axis=1)
    cols = np.sort(rng.choice(N, k, replace=False))
    rows[0, 1], rows[-1, 1], cols[0], cols[-1] = 0, S - 1, 0, N - 1
    return rows.astype(np.int32), cols.astype(np.int32)


@pytest.mark.parametrize("E,H,D,n_out", [(256, 2, 128, 1), (256, 8, 96, 1)])
def test_tall_token_tiles(E, H, D, n_out):
    S = 50001
    rows, cols = _sample(S, n_out * H * D)
    x, w, outs = run(1, S, E, H, D, n_out, "bf16", seed=3)
    check(x, w, outs, H, "bf16", "tall", rows=rows)
    x, w, gs, dx, dw = run_bwd(1, S, E, H, D, n_out, "bf16", seed=3)
    check_bwd(x, w, gs, dx, dw, H, "bf16", "tall", cols=cols, rows=rows)


@pytest.mark.parametrize("S,E,H,D", [(1090, 1536, 32, 128), (1600, 1280, 16, 256), (2100, 1024, 16, 256), (2111, 256, 4, 64)],
                         ids=["two_parts", "three_parts", "four_parts", "one_tile"])
def test_parts_of_dw(S, E, H, D):
    rows, cols = _sample(S, H * D)
    x, w, gs, dx, dw = run_bwd(1, S, E, H, D, 1, "bf16", seed=8)
    check_bwd(x, w, gs, dx, dw, H, "bf16", "parts", cols=cols, rows=rows)


@pytest.mark.parametrize("B,S,n_out", [(2, 832, 1), (3, 768, 2), (5, 640, 1), (4, 448, 2)],
                         ids=["three_parts", "four_parts", "six_parts", "three_parts_of_a_pair_of_outputs"])
def test_parts_of_dw_that_start_in_a_later_batch(B, S, n_out):
    # batches of whole pairs of 64 tokens, whose addresses run on from pair to pair
    rows, cols = _sample(S, n_out * 256)
    rows[:, 0] = np.arange(len(rows)) % B
    x, w, gs, dx, dw = run_bwd(B, S, 256, 4, 64, n_out, "bf16", seed=9)
    check_bwd(x, w, gs, dx, dw, 4, "bf16", "batches", cols=cols, rows=rows)


def test_infinity_in_the_last_part_of_dw():
    # An infinite gradient of the last token, which the last of five parts sums: the row of dW it reaches is
    # infinite with x's signs, not NaN, and every other row is finite.
    from paper_2502_02406_amd import binding as Bn
    S, E, H, D = 2600, 256, 2, 128
    inp = W.projection_inputs(1, S, E, H * D, "bf16", seed=4)
    g = W.projection_grad_inputs(1, S, H, D, 1, "bf16", seed=4)[0]
    x = inp["x"]
    x[0, -1] = torch.where(x[0, -1] < 0, -1.0, 1.0).to(x.dtype)
    g[0, 1, -1, 5] = float("inf")
    dw = torch.zeros((H * D, E), dtype=torch.float32, device="cuda")
    Bn.lvx_xattn_project_bwd(x.cuda(), inp["w"].cuda(), [g.cuda()], dw=dw)
    row = D + 5
    assert torch.equal(dw[row].cpu(), x[0, -1].float() * float("inf"))
    assert torch.isfinite(dw[:row]).all() and torch.isfinite(dw[row + 1:]).all()


@pytest.mark.parametrize("S,E,H", [(17958, 256, 8), (18100, 512, 4), (300, 256, 2), (1100, 768, 2)])
def test_odd_numbers_of_token_tiles(S, E, H):
    # 71 token tiles of 256 (the last one ragged), 141, 3 and 9 of 128: not a multiple of the XCDs, nor the tiles
    rows, cols = _sample(S, 2 * H * 128)
    x, w, outs = run(1, S, E, H, 128, 2, "bf16", seed=S)
    check(x, w, outs, H, "bf16", "odd", rows=rows)
    x, w, gs, dx, dw = run_bwd(1, S, E, H, 128, 2, "bf16", seed=S)
    check_bwd(x, w, gs, dx, dw, H, "bf16", "odd", cols=cols, rows=rows)
