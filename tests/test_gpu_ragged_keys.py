"""Key counts that are no multiple of the 64-key tile, against the fp64 oracle: the dense kernels
move the last tile back to end with the last key and give the keys it shares with the tile before
it no weight.  One key over a tile and one short of it, a lone tile and a bit, long enough for the
pipelined loop, split over workgroups, several heads per K/V head, every head dim.  Tolerances:
those of test_gpu_parity (bf16)."""
import pytest

from test_gpu_parity import run_case, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("kw", [
    dict(Sq=40, Skv=65), dict(Sq=64, Skv=127), dict(Hq=8, Hkv=2, Sq=1, Skv=95),
    dict(Hq=4, Hkv=2, Sq=150, Skv=64 * 9 + 1), dict(Sq=33, Skv=64 * 80 + 31), dict(Hq=4, Hkv=1, Sq=100, Skv=64 * 40 + 33, n_blocks=1),
    dict(Hq=4, Hkv=2, Sq=64, Skv=2 * (64 * 7 + 50), n_blocks=2),
], ids=lambda kw: f"{kw['Sq']}x{kw['Skv']}")
def test_ragged_key_counts(D, kw):
    run_case(small(f"ragged_d{D}_{kw['Sq']}x{kw['Skv']}", D=D, **kw), do_bwd=True)


def test_rising_scores_into_a_ragged_tile():
    # key norms grow to 24-fold towards the end: the row maxima sit in the moved-back last tile
    run_case(small("ragged_rising", Hq=4, Hkv=2, Sq=96, Skv=64 * 12 + 20), do_bwd=False, k_ramp=23.0)
