"""The projection kernels whose workgroups take several tiles, outputs and gradients of the tokens, against float64: more tiles than compute units by a few, twice as
many and some, a last tile of few tokens (which a workgroup may have to write before it goes on), an odd number of tile
pairs, eight pairs and nine, tokens in several batches, every head width, results large enough to be written past the
caches; nothing is written beside the results.  bf16 products are exact in float32, their sum over E terms is off by at most
2^-20 A with A = sum |x| |w| up to E = 4096, and the result is rounded once: |out - ref| <= 2^-8 |ref| + 2^-20 A."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,S,E,H,D,n_out", [
    (1, 65 * 256, 512, 8, 64, 2),            # 260 tiles
    (1, 65 * 256 + 1, 512, 8, 64, 2),        # ... and four of one token
    (1, 130 * 256 - 3, 576, 8, 64, 2),       # nine pairs, the last tiles short
    (1, 17 * 256 + 40, 512, 48, 128, 2),     # 48 column tiles: a workgroup goes on after a short tile
    (3, 11000, 640, 4, 128, 2),              # tiles that lie in two batches
    (130, 256, 512, 8, 64, 1),               # a batch a tile
    (67, 300, 512, 16, 96, 1),
    (1, 40000, 1024, 16, 96, 1),
    (1, 77000, 512, 8, 64, 2),               # 150 MB of results
], ids=lambda x: str(x))
def test_runs_of_tiles(B, S, E, H, D, n_out):
    from paper_2502_02406_amd import binding as L
    g = torch.Generator(device="cuda").manual_seed(11)
    x = torch.randn((B, S, E), generator=g, device="cuda").bfloat16()
    w = (torch.randn((n_out * H * D, E), generator=g, device="cuda") * E ** -0.5).bfloat16()
    guard, n = 4096, B * H * S * D
    bufs = [torch.full((n + 2 * guard,), -7.0, dtype=torch.bfloat16, device="cuda") for _ in range(n_out)]
    outs = [t[guard:guard + n].view(B, H, S, D) for t in bufs]
    L.lvx_xattn_project(x, w, outs)
    for t in bufs:
        assert bool((t[:guard] == -7.0).all()) and bool((t[guard + n:] == -7.0).all()), "written beside the result"
    for first in range(0, n_out * H, 8):             # (heads in groups: float64 copies of all of them do not come for free)
        for b in range(B):
            for s0 in range(0, S, 20000):
                xd = x[b, s0:s0 + 20000].double()
                wd = w[first * D:(first + 8) * D].double()
                ref, most = xd @ wd.T, xd.abs() @ wd.abs().T
                got = torch.cat([outs[(first + i) // H][b, (first + i) % H, s0:s0 + 20000] for i in range(min(8, n_out * H - first))], 1)
                over = (got.double() - ref).abs() - (2.0 ** -8 * ref.abs() + 2.0 ** -20 * most)
                assert float(over.max()) <= 0, f"head {first} batch {b} token {s0}"


@pytest.mark.parametrize("B,S,E,H,D,n_out", [
    (1, 65 * 256, 1024, 4, 64, 2),           # 260 tiles of eight pairs
    (1, 65 * 256 + 1, 1024, 4, 64, 2),
    (1, 33 * 256 - 3, 2048, 12, 64, 1),      # twelve pairs, the last tiles short
    (1, 17 * 256 + 40, 12288, 8, 64, 1),     # 48 column tiles: a workgroup goes on after a short tile
    (3, 11001, 512, 4, 128, 2),              # batches that end inside tiles
    (130, 100, 2048, 8, 64, 1),              # several batches a tile
    (1, 40000, 768, 16, 96, 1),              # (96-wide heads: not by these kernels)
], ids=lambda x: str(x))
def test_runs_of_token_gradients(B, S, E, H, D, n_out):
    from paper_2502_02406_amd import binding as L
    g = torch.Generator(device="cuda").manual_seed(12)
    w = (torch.randn((n_out * H * D, E), generator=g, device="cuda") * (H * D) ** -0.5).bfloat16()
    gr = [torch.randn((B, H, S, D), generator=g, device="cuda").bfloat16() for _ in range(n_out)]
    guard, n = 4096, B * S * E
    buf = torch.full((n + 2 * guard,), -7.0, dtype=torch.bfloat16, device="cuda")
    dx = buf[guard:guard + n].view(B, S, E)
    L.lvx_xattn_project_bwd(torch.zeros((B, S, E), dtype=torch.bfloat16, device="cuda"), w, gr, dx=dx)
    assert bool((buf[:guard] == -7.0).all()) and bool((buf[guard + n:] == -7.0).all()), "written beside the result"
    wd = w.double()
    for b in range(B):
        for s0 in range(0, S, 10000):
            gd = torch.cat([t[b, :, s0:s0 + 10000].permute(1, 0, 2).reshape(-1, H * D) for t in gr], 1).double()
            over = (dx[b, s0:s0 + 10000].double() - gd @ wd).abs() - (2.0 ** -8 * (gd @ wd).abs() + 2.0 ** -20 * (gd.abs() @ wd.abs()))
            assert float(over.max()) <= 0, f"batch {b} token {s0}"
