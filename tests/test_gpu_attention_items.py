"""Causal attention's work items: a workgroup per item (more items than resident workgroups, query tiles that do not divide
them) gives each sequence the bits it gets alone, from persistent workgroups, and those match the oracle; ragged ends that
leave one, two or three of a tile's four waves without a row; the diagonal's lane pattern at every length of a 32-row block."""
import numpy as np
import pytest
import torch

import paper_2507_03211_amd as zo_amd
import zo_inputs as zi
from oracle import zo_oracle as zo
from gpu_util import DEV

pytestmark = pytest.mark.gpu

TDT = {zi.BF16: torch.bfloat16, zi.FP16: torch.float16}
ULP = {zi.BF16: 2.0**-8, zi.FP16: 2.0**-11}


def _qkv(n_seq, seq, heads, dh, dtype, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.randn(n_seq * seq, 3 * heads * dh, device=DEV, generator=g).to(TDT[dtype])


def _run(qkv, n_seq, seq, heads, dh, dtype):
    out = torch.full((n_seq * seq + 1, heads * dh), 7.0, device=DEV, dtype=TDT[dtype])
    zo_amd.zo_kernel_attention(qkv, out, dtype, n_seq, seq, heads, dh)
    assert bool((out[-1] == 7.0).all())                                    # nothing behind the last row
    return out[:-1]


def _check(out, qkv, n_seq, seq, heads, dh, dtype):
    h = qkv.double().cpu().numpy().reshape(n_seq, seq, 3, heads * dh)
    want = zo.causal_attention(h[:, :, 0], h[:, :, 1], h[:, :, 2], heads).reshape(n_seq * seq, heads * dh)
    # three roundings (probabilities, values' product, output) on the output's scale
    assert np.max(np.abs(out.double().cpu().numpy() - want)) < 3 * ULP[dtype] * (1 + np.abs(want).max())


# Items of 128 rows, (sequence, head) pairs dealt to 8 XCDs; more items than an XCD holds at once in all of them (test_attention_residency.py
# asks for the plan): in groups of pairs, or all pairs in one group; the last one two whole groups
CASES = [(14, 600, 16, 64, 3, "one"), (32, 331, 32, 64, 3, "groups"), (7, 300, 31, 128, 2, "one"), (6, 257, 45, 80, 2, "groups"), (3, 1300, 16, 128, 2, "one"),
         (10, 600, 16, 128, 2, "groups"), (5, 1408, 16, 128, 2, "groups")]


@pytest.mark.parametrize("dtype", [zi.BF16, zi.FP16])
@pytest.mark.parametrize("n_seq,seq,heads,dh", [c[:4] for c in CASES])
def test_a_workgroup_per_item_gives_the_bits_of_persistent_ones(dtype, n_seq, seq, heads, dh):
    qkv = _qkv(n_seq, seq, heads, dh, dtype, seq)
    out = _run(qkv, n_seq, seq, heads, dh, dtype)
    for i in range(n_seq):
        rows = slice(i * seq, (i + 1) * seq)
        alone = _run(qkv[rows].contiguous(), 1, seq, heads, dh, dtype)
        assert torch.equal(out[rows], alone)
    few = qkv.reshape(n_seq, seq, 3, heads, dh)[-1:, :, :, -2:].reshape(seq, 6 * dh).contiguous()     # the last sequence's last heads
    _check(out.reshape(n_seq, seq, heads, dh)[-1, :, -2:].reshape(seq, 2 * dh), few, 1, seq, 2, dh, dtype)


@pytest.mark.parametrize("dh", [64, 80, 128])
@pytest.mark.parametrize("seq", [1, 2, 17, 31, 32, 33, 63, 65, 97, 127, 129, 159, 161, 193, 225, 257])
def test_ragged_ends(dh, seq):
    qkv = _qkv(2, seq, 3, dh, zi.BF16, seq + dh)
    _check(_run(qkv, 2, seq, 3, dh, zi.BF16), qkv, 2, seq, 3, dh, zi.BF16)


@pytest.mark.parametrize("seq", [40, 75, 140])
@pytest.mark.parametrize("n_seq,heads,dh", [(24, 40, 64), (24, 40, 128), (24, 30, 80)])
def test_sequences_of_nan_leave_their_neighbours_alone(seq, n_seq, heads, dh):
    # what a ragged tile holds past its sequence's end must not be what the workgroup's item before it left there
    qkv = _qkv(n_seq, seq, heads, dh, zi.BF16, seq)
    clean = _run(qkv, n_seq, seq, heads, dh, zi.BF16).reshape(n_seq, seq, heads * dh)
    bad = qkv.clone().reshape(n_seq, seq, 3 * heads * dh)
    bad[1::2] = float("nan")
    got = _run(bad.reshape(qkv.shape).contiguous(), n_seq, seq, heads, dh, zi.BF16).reshape(n_seq, seq, heads * dh)
    assert torch.equal(got[0::2], clean[0::2])
    assert bool(torch.isnan(got[1::2]).all())
