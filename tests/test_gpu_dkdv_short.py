"""dK and dV of key tiles of few steps (workgroups of 128 keys that share a compute unit), against the fp64 oracle: one step, the
most that a head width takes and one more (which the larger workgroups take), a short last step, keys that end inside a
wave, heads in a group; masks that select whole steps, masks by words, keys that nobody sees.  Tolerances: those of test_gpu_parity (bf16)."""
import numpy as np
import pytest

from test_gpu_parity import run_case, small

pytestmark = pytest.mark.gpu

_MOST = {64: 24, 96: 16, 128: 12}


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("Sq,Skv", [(32, 128), (32, 129), (33, 500), (63, 127), (64, 1), (95, 700), (97, 257)])
def test_few_steps(D, Sq, Skv):
    run_case(small(f"short_{D}_{Sq}x{Skv}", D=D, Hq=2, Hkv=1, Sq=Sq, Skv=Skv))


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("over", [0, 1])
def test_most_steps(D, over):
    run_case(small(f"short_most_{D}_{over}", D=D, B=2, Hq=2, Hkv=2, Sq=32 * (_MOST[D] + over) - 5, Skv=300))


@pytest.mark.parametrize("D", [64, 96, 128])
@pytest.mark.parametrize("q_chunk,kv_block", [(32, 256), (64, 256), (16, 64), (5, 100), (24, 729)], ids=lambda x: str(x))
def test_masks(D, q_chunk, kv_block):
    Sq, Skv = 190, 4 * kv_block + (0 if kv_block % 256 == 0 else 33)
    nq, nk = -(-Sq // q_chunk), -(-Skv // kv_block)
    allow = np.random.default_rng(q_chunk + kv_block).random((nq, nk)) < 0.5
    allow[:, nk // 2] = False                        # keys that nobody sees
    allow[:, 0] = True
    run_case(small(f"short_mask_{D}_{q_chunk}_{kv_block}", D=D, Hq=2, Hkv=1, Sq=Sq, Skv=Skv, q_chunk=q_chunk, kv_block=kv_block),
             allow=allow)
