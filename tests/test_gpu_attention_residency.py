"""Causal attention, heads of 64 and 80 channels, on either side of the sizes where the number of workgroups a CU changes: every
sequence has the bits it gets alone, where all of its items are under way at once, and those match the oracle."""
import pytest
import torch

import zo_inputs as zi
from test_gpu_attention_items import _check, _qkv, _run

pytestmark = pytest.mark.gpu


# 64: short sequences that fit at once with four workgroups a CU and just don't (one tile each), from 6 tiles on, one group over 1.5 rounds of 16
# tiles; 80: all at once with three a CU, a second round that two a CU need too, rounds that favour three, 6 tiles over a little more than a
# round, 10 tiles that two a CU hold in two rounds
@pytest.mark.parametrize("dtype", [zi.BF16, zi.FP16])
@pytest.mark.parametrize("n_seq,seq,heads,dh", [(32, 70, 32, 64), (33, 70, 32, 64), (9, 641, 24, 64), (12, 1921, 8, 64), (24, 70, 32, 80), (25, 70, 32, 80), (8, 300, 50, 80),
                                               (9, 700, 16, 80), (4, 1211, 16, 80)])
def test_either_side_of_the_line(dtype, n_seq, seq, heads, dh):
    qkv = _qkv(n_seq, seq, heads, dh, dtype, seq)
    out = _run(qkv, n_seq, seq, heads, dh, dtype)
    for i in range(0, n_seq, max(1, n_seq // 4)):
        rows = slice(i * seq, (i + 1) * seq)
        assert torch.equal(out[rows], _run(qkv[rows].contiguous(), 1, seq, heads, dh, dtype))
    few = qkv.reshape(n_seq, seq, 3, heads, dh)[-1:, :, :, -2:].reshape(seq, 6 * dh).contiguous()     # the last sequence's last heads
    _check(out.reshape(n_seq, seq, heads, dh)[-1, :, -2:].reshape(seq, 2 * dh), few, 1, seq, 2, dh, dtype)
