"""The plain attention of small heads: lengths at which a row's keys are dealt to groups of threads and at which the groups' partial
sums no longer fit beside the scores (one group), up to the longest that fits at all, against softmax in fp64 on some rows."""
import numpy as np
import pytest
import torch

import paper_2507_03211_amd as zo_amd
import zo_inputs as zi
from gpu_util import DEV, act_dtype

pytestmark = pytest.mark.gpu


# (seq + d_head + 16) scores of 8 bytes (4 for 16-bit types), and 128 partial sums with groups, of 32 KiB: 3936 and 3937, 8032 and
# 8033 lie on either side; 64 KiB without: 8160 (16-bit types: not reached here)
@pytest.mark.parametrize("dtype,seq,dh", [(zi.FP32, 1, 16), (zi.FP32, 130, 1), (zi.FP32, 130, 48), (zi.FP32, 5, 16), (zi.FP32, 9, 8),
                                          (zi.FP32, 130, 40), (zi.FP32, 3936, 16), (zi.FP32, 3937, 16), (zi.FP32, 8160, 16),
                                          (zi.BF16, 300, 8), (zi.BF16, 8032, 16), (zi.BF16, 8033, 16)])
def test_groups_of_keys_up_to_the_longest_sequence(dtype, seq, dh):
    heads = 2 if seq < 1000 else 1
    g = torch.Generator(device=DEV)
    g.manual_seed(seq)
    qkv = torch.randn(seq, 3 * heads * dh, device=DEV, generator=g, dtype=torch.float64).to(act_dtype(dtype))
    out = torch.full((seq + 1, heads * dh), 7.0, device=DEV, dtype=act_dtype(dtype))
    zo_amd.zo_kernel_attention(qkv, out, dtype, 1, seq, heads, dh)
    got, h = out.double().cpu().numpy(), qkv.double().cpu().numpy().reshape(seq, 3, heads, dh)
    assert np.all(got[seq] == 7.0)
    # fp64: sums of up to 8160 terms in 128 chains; bf16: fp32 probabilities and sums, one rounding of the output
    tol = 1e-13 * seq if dtype == zi.FP32 else 1.5 * 2.0**-8
    for t in sorted({0, min(1, seq - 1), seq // 3, seq - 1}):
        for a in range(heads):
            s = h[:t + 1, 1, a] @ h[t, 0, a] / np.sqrt(dh)
            p = np.exp(s - s.max())
            want = p @ h[:t + 1, 2, a] / p.sum()
            assert np.max(np.abs(got[t, a * dh:(a + 1) * dh] - want)) <= tol * (np.abs(want).max() + (1.0 if dtype == zi.FP32 else 1e-3)), (t, a)
