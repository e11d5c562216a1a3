"""GPU parity: a pending update and a position table longer than the prompts.  The rows beyond the prompt take the update along with the
staged ones while they are few, in a pass of their own beyond 16 MiB; both must leave the bits of the update applied at once."""
import pytest

import paper_2507_03211_amd as zo_amd
import zo_inputs as zi
from gpu_util import Model

pytestmark = pytest.mark.gpu


# (no row beyond the prompt; one; most of the table; 16 MiB beyond it, the last length that rides along; one row more)
@pytest.mark.parametrize("dtype,max_pos", [(zi.BF16, 24), (zi.BF16, 25), (zi.FP32, 25), (zi.FP16, 1000), (zi.FP32, 1000),
                                           (zi.BF16, 24 + 65536), (zi.BF16, 24 + 65537), (zi.FP32, 24 + 32768), (zi.FP32, 24 + 32769)])
def test_the_whole_table_takes_a_pending_update(dtype, max_pos):
    kw = dict(n_layers=2, d_model=128, n_heads=2, d_ffn=256, vocab=512, max_pos=max_pos, dtype=dtype, batch=2, seq=24, seed=3,
              plain_small=False, std=0.05)
    now, later = Model(**kw), Model(**kw)
    zo_amd.zo_set_deferred_update(later.handle, 1)
    _, tok = now.tokens()
    for seed in (0, 1, 2):
        assert zo_amd.zo_step(now.handle, tok, 2, 24, seed, 1e-3, 1e-2) == zo_amd.zo_step(later.handle, tok, 2, 24, seed, 1e-3, 1e-2)
    zo_amd.zo_flush_pending(later.handle)
    assert all(x.tobytes() == y.tobytes() for x, y in zip(now.theta(), later.theta()))
    now.close(); later.close()
