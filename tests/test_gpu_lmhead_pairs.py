"""Merging a row's (maximum, sum) pairs: rows with fewer pairs than a wavefront has lanes, with as many as its lanes keep
in registers (512), the next count (514), and more than that, against the cross entropy in fp64."""
import numpy as np
import pytest
import torch

import paper_2507_03211_amd as zo_amd
import zo_inputs as zi
from gpu_util import DEV

pytestmark = pytest.mark.gpu


# strips of 64 columns with d 64: 2, 64, 128, 130, 250, 256, 258, 512, 514, 1024, 1026, 1100 pairs a row (2, 4 and 8 of a lane are kept);
# of 128 with d 192 from 32768 columns on: 256, 258, 512, 514, 550
@pytest.mark.parametrize("vocab", [40, 4096, 8192, 8200, 16000, 16384, 16392, 32768, 32776, 65536, 65544, 70400])
@pytest.mark.parametrize("d", [64, 192])
def test_pairs_of_a_row(vocab, d):
    m_half = 5
    g = torch.Generator(device=DEV)
    g.manual_seed(vocab + d)
    x = torch.randn(2 * m_half, d, device=DEV, generator=g).to(torch.bfloat16)
    ep, em = ((0.3 * torch.randn(vocab, d, device=DEV, generator=g)).to(torch.bfloat16) for _ in range(2))
    target = torch.randint(0, vocab, (2 * m_half,), device=DEV, dtype=torch.int32, generator=g)
    target[0], target[1], target[2] = 0, vocab - 1, -1
    loss = torch.full((2 * m_half,), 7.0, device=DEV, dtype=torch.float64)
    scratch = torch.empty(zo_amd.zo_kernel_lmhead_scratch_bytes(zi.BF16, m_half, vocab), device=DEV, dtype=torch.uint8)
    zo_amd.zo_kernel_lmhead_ce(x, ep, em, target, loss, scratch, zi.BF16, m_half, d, vocab, torch.cuda.current_stream())
    torch.cuda.synchronize()
    xs, tg, got = x.double().cpu().numpy(), target.cpu().numpy(), loss.cpu().numpy()
    for r in range(2 * m_half):
        logits = (ep if r < m_half else em).double().cpu().numpy() @ xs[r]
        mx = logits.max()
        want = mx + np.log(np.exp(logits - mx).sum()) - logits[tg[r]] if tg[r] >= 0 else 0.0
        # fp32 logits of size ~10 (a d-term dot product's accumulation order) and fp32 partial sums
        assert abs(got[r] - want) < 2e-4, (r, got[r], want)
