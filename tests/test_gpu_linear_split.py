"""The sign-batched linear layer on 32 x 32 tiles whose four waves share the contraction: five to 24 slabs (waves with one to
six of them), one row and 8 columns past a tile, the most tiles that the rule takes, each epilogue, both 16-bit types.
Every output element is compared, and a second call gives the same bits."""
import pytest
import torch

import paper_2507_03211_amd as zo_amd
import zo_inputs as zi
from test_gpu_linear_tiles import TDT, _inputs, test_linear_tiles as check_linear

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [zi.BF16, zi.FP16])
@pytest.mark.parametrize("epi", [0, 1, 2, 3])
@pytest.mark.parametrize("m_half,n,k", [(1, 8, 320), (32, 32, 320), (33, 40, 384), (31, 72, 448), (64, 24, 512), (65, 128, 576), (97, 264, 640), (20, 1000, 704), (130, 104, 768),
                                        (128, 1024, 320), (1, 4096, 384), (68, 384, 1536)])
def test_each_epilogue(m_half, n, k, epi, dtype):
    assert zo_amd.zo_kernel_linear_tile(m_half, n, k, epi) == (32, 32)
    check_linear(m_half, n, k, epi, dtype)


def test_the_same_bits_twice():
    _, x, w, b = _inputs(70, 200, 832, zi.BF16, 3)
    y = [torch.empty(140, 200, device=x.device, dtype=TDT[zi.BF16]) for _ in range(2)]
    for out in y:
        zo_amd.zo_kernel_linear_pm(x, w[0], w[1], b[0], b[1], out, zi.BF16, 70, 200, 832, 0)
    assert torch.equal(*y)


def test_rows_that_are_not_finite_stay_alone():
    _, x, w, b = _inputs(70, 200, 832, zi.BF16, 3)
    y = torch.empty(140, 200, device=x.device)
    zo_amd.zo_kernel_linear_pm(x, w[0], w[1], b[0], b[1], y, zi.BF16, 70, 200, 832, 3)
    x[5, 800], x[75, 1] = float("nan"), float("inf")
    bad = torch.empty_like(y)
    zo_amd.zo_kernel_linear_pm(x, w[0], w[1], b[0], b[1], bad, zi.BF16, 70, 200, 832, 3)
    keep = torch.ones(140, dtype=torch.bool)
    keep[[5, 75]] = False
    assert torch.equal(y[keep], bad[keep]) and bool((~torch.isfinite(bad[[5, 75]])).all())
