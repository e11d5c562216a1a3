"""Embedding rows four elements at a time: widths around a wavefront's 256, row counts that do not fill a
workgroup, position tables longer than the sequence or not (a pending update then rides on their staging), against the oracle and
between the two forms of the update."""
import numpy as np
import pytest

import paper_2507_03211_amd as zo_amd
import zo_inputs as zi
from oracle import zo_oracle as zo
from gpu_util import Model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,heads,batch,seq", [(8, 1, 1, 2), (40, 5, 3, 5), (72, 3, 1, 3), (248, 4, 1, 9), (256, 4, 3, 7), (264, 4, 1, 6), (520, 5, 1, 3)])
def test_losses(d, heads, batch, seq):
    mdl = Model(1, d, heads, 16, 40, seq + 1, zi.FP32, batch, seq, seed=d, plain_small=False, std=0.05)
    tok, tok_dev = mdl.tokens()
    lp, lm = zo_amd.zo_dual_forward(mdl.handle, tok_dev, batch, seq, 5, 1e-3)
    theta = [t.copy() for t in mdl.theta0]
    olp, olm, _ = zo.zo_step_fused(mdl.ocfg, theta, tok, 5, 1e-3, 0.0)
    assert abs(lp / olp - 1) < 1e-11 and abs(lm / olm - 1) < 1e-11        # summation order in fp64 alone
    mdl.close()


@pytest.mark.parametrize("dtype", [zi.FP32, zi.BF16, zi.FP16])
@pytest.mark.parametrize("seq,max_pos", [(24, 24), (24, 25), (7, 24)])
def test_a_pending_update_of_the_position_table(dtype, seq, max_pos):
    a, b = (Model(2, 64, 4, 128, 80, max_pos, dtype, 2, seq, seed=4, plain_small=False, std=0.05) for _ in range(2))
    _, tok_dev = a.tokens()
    zo_amd.zo_set_deferred_update(b.handle, True)
    got = [[zo_amd.zo_step(m.handle, tok_dev, 2, seq, seed, 1e-3, 1e-2) for seed in (1, 2, 3)] for m in (a, b)]
    assert got[0] == got[1]
    zo_amd.zo_flush_pending(b.handle)
    assert all(x.tobytes() == y.tobytes() for x, y in zip(a.theta(), b.theta()))
    a.close(); b.close()
