"""The float32 kernels with 16 and 32 stationary rows, at the edges of both and where one gives way to the other (one
32-row workgroup per compute unit, 256 of them), against the fp64 oracle.  Tolerances: those of test_gpu_parity
(float32)."""
import pytest

from test_gpu_parity import run_case, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("kw", [
    dict(Sq=15, Skv=17), dict(Sq=17, Skv=16), dict(Hq=4, Hkv=2, Sq=48, Skv=33, n_blocks=1),
    dict(B=8, Hq=8, Hkv=8, Sq=128, Skv=64),                # 256 workgroups of 32 rows: dQ narrow, dK/dV wide
    dict(B=8, Hq=8, Hkv=8, Sq=129, Skv=70, n_blocks=2),    # 320: all wide
    dict(B=3, Hq=4, Hkv=2, Sq=40, Skv=1300),               # few query rows, many keys: dQ narrow, dK/dV wide
], ids=lambda kw: f"{kw.get('B', 1)}x{kw['Sq']}x{kw['Skv']}")
def test_f32_widths(D, kw):
    run_case(small(f"f32w_d{D}_{kw.get('B', 1)}x{kw['Sq']}x{kw['Skv']}", dtype="f32", std=1.0, D=D, **kw))
