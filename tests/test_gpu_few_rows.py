"""The forward kernel for a few query rows per K/V head (a generated token) and the combine of many
parts of few rows, against the fp64 oracle: one row and one short of a block of 32 and of both
blocks, head groups that straddle the blocks, fewer keys than a unit of 32, a unit and one key more,
waves without a unit, splits of one unit per wave and of many, a running state merged in the
kernel and in the combine.  Tolerances: those of test_gpu_parity (bf16)."""
import pytest

from test_gpu_parity import run_case, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("kw", [
    dict(Hq=4, Hkv=2, Sq=1, Skv=5), dict(Hq=4, Hkv=1, Sq=8, Skv=33), dict(Hq=7, Hkv=1, Sq=9, Skv=700),
    dict(B=2, Hq=8, Hkv=2, Sq=16, Skv=129), dict(Hq=8, Hkv=2, Sq=1, Skv=5000), dict(Hq=1, Hkv=1, Sq=33, Skv=20001),
    dict(Hq=4, Hkv=1, Sq=1, Skv=2 * 4100, n_blocks=2), dict(B=8, Hq=64, Hkv=64, Sq=1, Skv=600, n_blocks=2),
], ids=lambda kw: f"{kw['Hq']}x{kw['Sq']}x{kw['Skv']}")
def test_few_rows(D, kw):
    run_case(small(f"few_d{D}_{kw['Hq']}x{kw['Sq']}x{kw['Skv']}", D=D, **kw), do_bwd=False)


@pytest.mark.parametrize("kw", [dict(Hq=4, Hkv=1, Sq=3, Skv=3000), dict(Hq=2, Hkv=1, Sq=30, Skv=3000, n_blocks=2)],
                         ids=["one_block", "two_blocks"])
def test_few_rows_rising_scores(kw):
    # key norms grow to 24-fold along the keys: every wave raises its references again and again
    run_case(small("few_rising", **kw), do_bwd=False, k_ramp=23.0)
