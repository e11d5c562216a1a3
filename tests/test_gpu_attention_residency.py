"""Causal attention, heads of 64 and 80 channels, on either side of the sizes where the number of workgroups a CU or the way through the list
changes: every sequence has the bits it gets alone, where all of its items are under way at once, and those match the oracle."""
import pytest
import torch

import zo_inputs as zi
from test_gpu_attention_items import _check, _qkv, _run

pytestmark = pytest.mark.gpu


# sequences, tokens, heads, channels; the plan on 32 CUs an XCD (test_attention_residency.py asks for it): workgroups a CU, and "all" items at
# once, "persistent" workgroups, a workgroup per item with the pairs in "groups" or in "one" group
CASES = [(32, 70, 32, 64, 4, "all"), (33, 70, 32, 64, 3, "persistent"), (13, 1000, 8, 64, 3, "one"), (9, 641, 24, 64, 4, "one"), (12, 1921, 8, 64, 4, "one"),
         (40, 700, 8, 64, 3, "persistent"), (33, 1000, 8, 64, 4, "persistent"), (46, 800, 8, 64, 3, "groups"), (67, 700, 8, 64, 4, "groups"),
         (24, 70, 32, 80, 3, "all"), (25, 70, 32, 80, 2, "persistent"), (8, 300, 50, 80, 3, "persistent"), (9, 700, 16, 80, 3, "one"), (37, 600, 8, 80, 3, "groups"),
         (4, 1211, 16, 80, 2, "one")]


@pytest.mark.parametrize("dtype", [zi.BF16, zi.FP16])
@pytest.mark.parametrize("n_seq,seq,heads,dh", [c[:4] for c in CASES])
def test_either_side_of_the_line(dtype, n_seq, seq, heads, dh):
    qkv = _qkv(n_seq, seq, heads, dh, dtype, seq)
    out = _run(qkv, n_seq, seq, heads, dh, dtype)
    for i in range(0, n_seq, max(1, n_seq // 4)):
        rows = slice(i * seq, (i + 1) * seq)
        assert torch.equal(out[rows], _run(qkv[rows].contiguous(), 1, seq, heads, dh, dtype))
    few = qkv.reshape(n_seq, seq, 3, heads, dh)[-1:, :, :, -2:].reshape(seq, 6 * dh).contiguous()     # the last sequence's last heads
    _check(out.reshape(n_seq, seq, heads, dh)[-1, :, -2:].reshape(seq, 2 * dh), few, 1, seq, 2, dh, dtype)
