"""Causal attention on the matrix path for the head sizes between 64 and 128 whose last channel tile is padded or whose
number of contraction steps is odd (80, 96, 112), against the oracle: edges of the 32-key units, the 64-key tiles and the
128-row work items; every key weighed exactly once; values that are not finite behind a row's last visible key; where many
sequences of a few tokens leave the matrix path."""
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
    out = torch.full((n_seq * seq, heads * dh), 7.0, device=DEV, dtype=TDT[dtype])
    zo_amd.zo_kernel_attention(qkv, out, dtype, n_seq, seq, heads, dh)
    return out.double().cpu().numpy().reshape(n_seq, seq, heads, dh)


def _oracle(qkv, n_seq, seq, heads, dh):
    h = qkv.double().cpu().numpy().reshape(n_seq, seq, 3, heads * dh)
    return zo.causal_attention(h[:, :, 0], h[:, :, 1], h[:, :, 2], heads).reshape(n_seq, seq, heads, dh)


@pytest.mark.parametrize("dtype", [zi.BF16, zi.FP16])
@pytest.mark.parametrize("dh", [80, 96, 112])
@pytest.mark.parametrize("n_seq,seq,heads", [(1, 1, 1), (2, 31, 3), (1, 33, 2), (2, 64, 1), (1, 65, 9), (1, 128, 2), (3, 129, 1), (1, 331, 4)])
def test_head_sizes_against_the_oracle(dtype, dh, n_seq, seq, heads):
    qkv = _qkv(n_seq, seq, heads, dh, dtype, seq + dh)
    got, want = _run(qkv, n_seq, seq, heads, dh, dtype), _oracle(qkv, n_seq, seq, heads, dh)
    # three roundings (probabilities, values' product, output) on the output's scale, as for heads of 64 and 128
    assert np.max(np.abs(got - want)) < 3 * ULP[dtype] * (1 + np.abs(want).max())


@pytest.mark.parametrize("dh", [80, 96, 112])
def test_every_key_counts_once(dh):
    n_seq, seq, heads = 2, 700, 2
    qkv = torch.zeros(n_seq, seq, 3, heads, dh, device=DEV, dtype=torch.bfloat16)
    qkv[:, :, 1] = _qkv(n_seq, seq, heads, dh, zi.BF16, 3).reshape(n_seq, seq, 3, heads, dh)[:, :, 1]
    qkv[:, :, 2] = torch.nn.functional.one_hot(torch.arange(seq, device=DEV) % dh, dh).to(torch.bfloat16)[None, :, None]
    got = _run(qkv.contiguous(), n_seq, seq, heads, dh, zi.BF16)
    t, j = np.arange(seq)[:, None], np.arange(dh)[None, :]
    want = ((t >= j) * ((t - j) // dh + 1) / (t + 1.0))[None, :, None, :]
    assert np.all(np.abs(got - want) <= ULP[zi.BF16] * want + 1e-30)       # one rounding of the output


@pytest.mark.parametrize("dtype", [zi.BF16, zi.FP16])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
def test_values_behind_the_last_visible_key_do_not_matter(dtype, value):
    n_seq, seq, heads, dh, at = 1, 150, 2, 80, 70
    qkv = _qkv(n_seq, seq, heads, dh, dtype, 11)
    want = _oracle(qkv, n_seq, seq, heads, dh)
    bad = qkv.clone().reshape(n_seq, seq, 3, heads, dh)
    bad[0, at, 1:, 0] = value                       # key and value of one token, head 0
    got = _run(bad.reshape(qkv.shape).contiguous(), n_seq, seq, heads, dh, dtype)
    tol = 3 * ULP[dtype] * (1 + np.abs(want).max())
    assert np.max(np.abs(got[:, :at] - want[:, :at])) < tol and np.max(np.abs(got[:, :, 1] - want[:, :, 1])) < tol
    assert np.all(np.isnan(got[0, at, 0]))          # the token sees itself


def test_unaligned_buffers_still_run():
    n_seq, seq, heads, dh = 1, 40, 2, 80
    flat = _qkv(n_seq, seq + 1, heads, dh, zi.BF16, 5).reshape(-1)
    n = n_seq * seq * 3 * heads * dh
    qkv = flat[1:1 + n].reshape(n_seq * seq, 3 * heads * dh)               # 2 bytes past a 16-byte boundary
    want = _oracle(qkv, n_seq, seq, heads, dh)
    got = _run(qkv, n_seq, seq, heads, dh, zi.BF16)
    assert np.max(np.abs(got - want)) < 3 * ULP[zi.BF16] * (1 + np.abs(want).max())


@pytest.mark.parametrize("dh", [64, 80, 128])
@pytest.mark.parametrize("off_in,off_out", [(1, 0), (0, 1), (4, 4)])
def test_unaligned_buffers_of_any_head_size(dh, off_in, off_out):
    # off a 16-byte boundary by 2 and by 8 bytes: all head sizes leave the matrix path, bit for bit the same whichever buffer it is
    n_seq, seq, heads = 1, 40, 2
    flat = _qkv(n_seq, seq + 1, heads, dh, zi.BF16, 5).reshape(-1)
    n = n_seq * seq * 3 * heads * dh
    qkv = flat[1:1 + n].reshape(n_seq * seq, 3 * heads * dh)
    want = _oracle(qkv, n_seq, seq, heads, dh)
    src = torch.empty(n + 8, device=DEV, dtype=torch.bfloat16)[off_in:off_in + n].copy_(qkv.reshape(-1))
    out = torch.full((n // 3 + 8,), 7.0, device=DEV, dtype=torch.bfloat16)
    zo_amd.zo_kernel_attention(src, out[off_out:], zi.BF16, n_seq, seq, heads, dh)
    got = out[off_out:off_out + n // 3].double().cpu().numpy().reshape(want.shape)
    assert np.max(np.abs(got - want)) < 3 * ULP[zi.BF16] * (1 + np.abs(want).max())
    assert bool((out[:off_out] == 7.0).all()) and bool((out[off_out + n // 3:] == 7.0).all())
    other = torch.empty_like(out)
    zo_amd.zo_kernel_attention(qkv, other, zi.BF16, n_seq, seq, heads, dh)          # 2 bytes off, on the plain kernel
    assert torch.equal(other[:n // 3], out[off_out:off_out + n // 3])


@pytest.mark.parametrize("dtype", [zi.BF16, zi.FP16])
@pytest.mark.parametrize("n_seq,seq,heads,dh", [(40, 140, 9, 96), (1, 700, 3, 112), (2, 33, 2, 80),      # 720 items on 512 workgroups
                                               (4, 257, 45, 80), (10, 600, 17, 112)])                   # a workgroup per item: one group, groups of 12 pairs
def test_values_that_are_not_finite_reach_the_rows_that_see_them_and_no_other(dtype, n_seq, seq, heads, dh):
    qkv = _qkv(n_seq, seq, heads, dh, dtype, 21).reshape(n_seq, seq, 3, heads, dh)
    want = _oracle(qkv, n_seq, seq, heads, dh)
    rng = np.random.Generator(np.random.PCG64(seq))
    bad = np.zeros((n_seq, seq, heads, dh))
    for _ in range(max(3, n_seq * heads // 3)):
        at = (rng.integers(n_seq), rng.integers(seq), rng.integers(heads), rng.integers(dh))
        value = [np.inf, -np.inf, np.nan][rng.integers(3)]
        bad[at] = value
        qkv[at[0], at[1], 2, at[2], at[3]] = float(value)
    with np.errstate(invalid="ignore"):
        want = want + np.cumsum(bad, axis=1)          # a row's probabilities are positive: infinities stay, opposite ones meet as NaN
    got = _run(qkv.reshape(n_seq * seq, -1), n_seq, seq, heads, dh, dtype)
    fin = np.isfinite(want)
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
    assert np.max(np.abs(got[fin] - want[fin])) < 3 * ULP[dtype] * (1 + np.abs(want[fin]).max())


@pytest.mark.parametrize("dh", [80, 112])
@pytest.mark.parametrize("n_seq,seq", [(8, 64), (2, 1024)])
def test_rows_that_are_not_finite_cost_no_more_than_on_the_plain_kernel(n_seq, seq, dh):
    # buffers that are not 16-byte aligned take the plain kernel
    heads = 32
    n = n_seq * seq * 3 * heads * dh
    flat = torch.full((n + 8,), float("nan"), device=DEV, dtype=torch.bfloat16)
    out = torch.empty(n_seq * seq * heads * dh, device=DEV, dtype=torch.bfloat16)

    def us(qkv):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        best = 1e30
        for _ in range(5):
            ev[0].record()
            for _ in range(3):
                zo_amd.zo_kernel_attention(qkv, out, zi.BF16, n_seq, seq, heads, dh, torch.cuda.current_stream())
            ev[1].record()
            ev[1].synchronize()
            best = min(best, ev[0].elapsed_time(ev[1]) / 3 * 1000)
        return best

    plain, here = us(flat[1:1 + n]), us(flat[:n])
    assert bool(torch.isnan(out).all())
    assert here < 1.5 * plain, (here, plain)          # 16 times with a wavefront per row


@pytest.mark.parametrize("gap", [8.0, 17.0, 18.5, 20.0])
@pytest.mark.parametrize("dh", [80, 112])
def test_small_probabilities_count_in_fp16(dh, gap):
    # key 0 outweighs each of the others by e^gap, and its value is zero: a row is what the many small probabilities add up to
    n_seq, seq, heads = 1, 2000, 1
    qkv = torch.zeros(n_seq, seq, 3, heads, dh, device=DEV)
    qkv[:, :, 0, :, 0] = 16.0
    qkv[:, 0, 1, :, 0] = gap * dh**0.5 / 16.0
    qkv[:, 1:, 2] = 1000.0 * (1.0 + torch.arange(dh, device=DEV) / 128.0)
    qkv = qkv.half().reshape(n_seq * seq, -1)
    got, want = _run(qkv, n_seq, seq, heads, dh, zi.FP16), _oracle(qkv, n_seq, seq, heads, dh)
    # a small probability, 2^11 e^-gap, within half a unit of 2^-24; the output within half a unit of its own or of 2^-24
    bound = want * (2.0**-36 * np.exp(gap + 0.02) + 2.0**-10) + 2.0**-25
    assert np.all(np.abs(got - want) <= bound), np.max(np.abs(got - want) / np.maximum(want, 1e-9))


@pytest.mark.parametrize("dtype", [zi.BF16, zi.FP16])
@pytest.mark.parametrize("dh", [80, 96, 112])
@pytest.mark.parametrize("n_seq,seq,heads,plain", [(512, 1, 1, True), (511, 1, 1, False), (27, 2, 19, True), (256, 2, 2, False),
                                                   (171, 3, 3, True), (128, 3, 4, False), (129, 4, 4, True), (512, 4, 4, True), (2049, 4, 1, False),
                                                   (129, 5, 4, False)])
def test_many_sequences_of_a_few_tokens(dtype, dh, n_seq, seq, heads, plain):
    # both sides of the line: right on each, and beyond it bit for bit what a buffer off a 16-byte boundary gives (the plain kernel)
    qkv = _qkv(n_seq, seq, heads, dh, dtype, 6)
    want = _oracle(qkv, n_seq, seq, heads, dh)
    got = _run(qkv, n_seq, seq, heads, dh, dtype)
    assert np.max(np.abs(got - want)) < 3 * ULP[dtype] * (1 + np.abs(want).max())
    if plain:
        flat = torch.empty(qkv.numel() + 1, device=DEV, dtype=qkv.dtype)
        off = flat[1:].view_as(qkv).copy_(qkv)
        assert np.array_equal(got, _run(off, n_seq, seq, heads, dh, dtype))


# Scaled scores of 2^e and their neighbours a 64th apart: far enough that a row is the value of its largest key (or the mean of equal
# ones), and exact in fp32: equal channels of 7 bits, so that every partial sum has 14.
def _far(n_seq, seq, heads, dh, dtype, e, seed):
    sc = 1.4426950408889634 / dh ** 0.5
    a = int(np.round((e - np.log2(sc * dh)) / 2))                          # 2^a per channel of q, 2^b (1 .. 2) per channel of k
    b = int(np.round(e - np.log2(sc * dh))) - a
    qkv = torch.randn(n_seq, seq, 3, heads, dh, device=DEV, generator=torch.Generator(device=DEV).manual_seed(seed))
    j = torch.arange(n_seq * seq * heads, device=DEV).reshape(n_seq, seq, heads, 1)
    qkv[:, :, 0] = 2.0 ** a
    qkv[:, :, 1] = 2.0 ** b * (1 + (j * 37 % 64) / 64.0)
    return qkv.to(TDT[dtype]).reshape(n_seq * seq, 3 * heads * dh)


# Heads of 64 and 128: up to where the header says that they hold.
@pytest.mark.parametrize("dh,dtype,e", [(dh, zi.FP16, e) for dh in (80, 96, 112) for e in (16, 24, 27, 28, 29, 30, 31, 32)] +
                         [(dh, zi.BF16, e) for dh in (80, 96, 112) for e in (24, 29, 30, 31, 32, 33, 40, 60)] +
                         [(dh, zi.FP16, e) for dh in (64, 128) for e in (16, 24, 25)] + [(dh, zi.BF16, e) for dh in (64, 128) for e in (24, 28, 29)])
def test_scores_whose_reference_is_rounded_by_more_than_they_differ(dh, dtype, e):
    qkv = _far(2, 100, 3, dh, dtype, e, dh + e)
    want = _oracle(qkv, 2, 100, 3, dh)
    # e = 16: differences of 2^10 and more, so weights of 1 (of equal parts of it) throughout; one rounding of the output
    assert np.max(np.abs(_run(qkv, 2, 100, 3, dh, dtype) - want)) < ULP[dtype] * (1 + np.abs(want).max())


@pytest.mark.parametrize("dtype", [zi.BF16, zi.FP16])
@pytest.mark.parametrize("dh", [80, 112])
def test_such_sequences_among_others_over_several_rounds(dh, dtype):
    n_seq, seq, heads = 24, 70, 40                                          # 120 items an XCD: a workgroup works two
    qkv = _qkv(n_seq, seq, heads, dh, dtype, dh).reshape(n_seq, seq, -1)
    qkv[3::5] = _far(n_seq, seq, heads, dh, dtype, 31, dh).reshape(n_seq, seq, -1)[3::5]
    qkv = qkv.reshape(n_seq * seq, -1)
    got, want = _run(qkv, n_seq, seq, heads, dh, dtype), _oracle(qkv, n_seq, seq, heads, dh)
    # three roundings (probabilities, values' product, output) on the output's scale
    assert np.max(np.abs(got - want)) < 3 * ULP[dtype] * (1 + np.abs(want).max())
