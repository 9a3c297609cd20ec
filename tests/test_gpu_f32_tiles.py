"""The float32 kernels at the edges of their 32 x 32 tiles, against the fp64 oracle: one row and one key,
a tile and one more of each, head groups whose rows straddle tiles (shorter and longer than a tile),
more tiles than a workgroup has waves, a running state merged in the kernel, media masks that cut
through tiles and rows that see nothing.  Tolerances: those of test_gpu_parity (float32)."""
import numpy as np
import pytest

from test_gpu_parity import run_case, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("kw", [
    dict(Sq=2, Skv=3), dict(Sq=33, Skv=32), dict(Hq=6, Hkv=2, Sq=7, Skv=65), dict(Hq=4, Hkv=1, Sq=45, Skv=300),
    dict(B=2, Hq=4, Hkv=2, Sq=64, Skv=320), dict(Hq=4, Hkv=2, Sq=70, Skv=4 * 31, n_blocks=4),
], ids=lambda kw: f"{kw['Sq']}x{kw['Skv']}")
def test_f32_tiles(D, kw):
    run_case(small(f"f32t_d{D}_{kw['Sq']}x{kw['Skv']}", dtype="f32", std=1.0, D=D, **kw))


@pytest.mark.parametrize("D", [64, 128])
def test_f32_masks(D):
    w = small(f"f32t_mask_d{D}", dtype="f32", std=1.0, D=D, Hq=4, Hkv=2, Sq=75, Skv=210, q_chunk=10, kv_block=21)
    allow = np.random.Generator(np.random.Philox(7)).random((8, 10)) < 0.3
    allow[2] = False
    run_case(w, allow=allow)
