"""fp32 models (fp64 activations): layers that take their LayerNorm on the way, the lengths and counts at which they stop doing
so, and the plain attention's groups of keys, as whole forward passes against the oracle; the two routes against each other."""
import numpy as np
import pytest

import paper_2507_03211_amd as zo_amd
import zo_inputs as zi
from oracle import zo_oracle as zo
from gpu_util import Model

pytestmark = pytest.mark.gpu


# rows of 8, 40 (no multiple of the 16-deep pieces), 320 (the longest taken), 328, 512 and 520; 1440 rows a sign (32 x 32 tiles: two launches
# for QKV, one for a narrow layer); heads of 8, 16, 24, 64 and 68 channels (8, 8, 5, 1 and 1 groups of keys; one with 3 tokens), and of 104 and 128
@pytest.mark.parametrize("d,heads,ffn,vocab,batch,seq", [(8, 1, 8, 16, 1, 3), (40, 5, 40, 56, 3, 17), (72, 3, 40, 56, 2, 21), (64, 4, 64, 40, 16, 90),
                                                        (128, 2, 64, 64, 2, 33), (136, 2, 40, 24, 1, 20), (256, 4, 64, 72, 2, 19), (320, 4, 64, 72, 1, 19), (328, 4, 64, 72, 1, 9), (512, 4, 64, 72, 1, 19), (520, 5, 64, 24, 1, 9)])
def test_losses_of_fp32_models(d, heads, ffn, vocab, batch, seq):
    mdl = Model(2, d, heads, ffn, vocab, seq, zi.FP32, batch, seq, seed=d, plain_small=False, std=0.05)
    tok, tok_dev = mdl.tokens()
    theta = [t.copy() for t in mdl.theta0]
    lp, lm, g = zo_amd.zo_step(mdl.handle, tok_dev, batch, seq, 7, 1e-3, 1e-4)
    olp, olm, og = zo.zo_step_fused(mdl.ocfg, theta, tok, 7, 1e-3, 1e-4)
    assert abs(lp / olp - 1) < 1e-11 and abs(lm / olm - 1) < 1e-11        # summation order in fp64 alone
    assert abs(g - og) < 1e-6 * max(abs(og), 1.0)
    for a, b in zip(mdl.theta(), theta):
        assert np.all(np.abs(a.astype(np.float64) - b) <= 1e-4 * np.abs(b) + 1e-9)
    mdl.close()


def _losses_and_layernorms(mdl, tok_dev, batch, seq):
    zo_amd.zo_profile_begin(mdl.handle, 256)
    lp, lm = zo_amd.zo_dual_forward(mdl.handle, tok_dev, batch, seq, 7, 1e-3)
    prof = zo_amd.zo_profile_end(mdl.handle)
    return lp, lm, prof["norm"][1]


# LayerNorms of one block and the head that are launches of their own, for one sequence and for eight of them
@pytest.mark.parametrize("d,heads,ffn,vocab,seq,few,many", [(64, 4, 256, 512, 24, 0, 0), (256, 4, 1024, 1536, 24, 0, 3), (320, 5, 960, 640, 16, 0, 3), (320, 5, 128, 128, 24, 0, 1),
                                                           (512, 8, 128, 128, 8, 3, 3)])
def test_both_routes_give_the_same_losses(d, heads, ffn, vocab, seq, few, many):
    # eight copies of a sequence have the mean loss of one of them: other tile counts, so other routes, of the same layers
    mdl = Model(1, d, heads, ffn, vocab, seq, zi.FP32, 8, seq, seed=d, plain_small=False, std=0.05)
    _, one = mdl.tokens(batch=1)
    lp, lm, n = _losses_and_layernorms(mdl, one, 1, seq)
    lp8, lm8, n8 = _losses_and_layernorms(mdl, one.repeat(8, 1).contiguous(), 8, seq)
    mdl.close()
    assert (n, n8) == (few, many)
    assert abs(lp8 / lp - 1) < 1e-12 and abs(lm8 / lm - 1) < 1e-12        # rounding of fp64 sums of up to 512 terms, averaged
