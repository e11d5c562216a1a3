"""GPU parity: a resident model stages several blocks per launch, as many as fit beside the LM head's idle region.  The copies are the
same wherever they lie, so a step must give the bits of the streamed model, which stages block by block: one to six blocks (whole
groups, remainders), heads whose region holds none, one or more pairs of copies, the update at once and pending."""
import pytest

import paper_2507_03211_amd as zo_amd
import zo_inputs as zi
from gpu_util import Model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [zi.BF16, zi.FP32])
@pytest.mark.parametrize("deferred", [False, True])
@pytest.mark.parametrize("n_layers,vocab", [(1, 4096), (2, 4096), (3, 24), (3, 520), (4, 4096), (5, 520), (5, 1100), (6, 4096)])
def test_groups_of_blocks_leave_the_streamed_models_bits(n_layers, vocab, deferred, dtype):
    kw = dict(n_layers=n_layers, d_model=64, n_heads=2, d_ffn=136, vocab=vocab, max_pos=64, dtype=dtype, batch=2, seq=40, seed=3,
              plain_small=False, std=0.05)
    res, stm = Model(**kw), Model(**kw, streamed=True)
    if deferred:
        zo_amd.zo_set_deferred_update(res.handle, 1)
    _, tok = res.tokens()
    for seed in (0, 1, 2):
        assert zo_amd.zo_step(res.handle, tok, 2, 40, seed, 1e-3, 1e-2) == zo_amd.zo_step(stm.handle, tok, 2, 40, seed, 1e-3, 1e-2)
    for m in (res, stm):
        zo_amd.zo_flush_pending(m.handle)
    assert all(x.tobytes() == y.tobytes() for x, y in zip(res.theta(), stm.theta()))
    res.close(); stm.close()
