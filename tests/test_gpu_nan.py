"""A NaN in one key is a NaN in every result of the query rows that see it, and in no other: the float32
kernels (one block and a running state) and the forward for few rows (one workgroup, splits with their
combine, a running state), whose combines leave out parts without keys but not parts without a value."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Skv", [100, 6000])
@pytest.mark.parametrize("dtype,Sq", [(torch.float32, 40), (torch.bfloat16, 1), (torch.bfloat16, 20)],
                         ids=["f32", "one_row", "rows"])
@pytest.mark.parametrize("n_blocks", [1, 2])
def test_nan_key(dtype, Sq, Skv, n_blocks):
    from paper_2502_02406_amd.blockloop import BlockLoop
    g = torch.Generator().manual_seed(5)
    q = torch.randn((1, 4, Sq, 64), generator=g).to(dtype).cuda()
    k, v = (torch.randn((1, 2, Skv, 64), generator=g).to(dtype).cuda() for _ in range(2))
    loop = BlockLoop(tuple(q.shape), tuple(k.shape), dtype, n_blocks)
    clean = loop.forward(q, k, v)[0].clone()
    for j in (0, Skv // 2 - 1, Skv - 1):
        bad = k.clone()
        bad[0, 1, j, 3] = float("nan")
        o = loop.forward(q, bad, v)[0]
        assert torch.isnan(o[:, 2:]).all(), f"key {j}: a row of the second K/V head has a value"
        assert torch.equal(o[:, :2], clean[:, :2]), f"key {j}: the first K/V head changed"
