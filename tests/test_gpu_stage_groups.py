"""GPU parity: a resident model stages several blocks per launch, as many as fit beside the LM head's idle region.  The copies are the
same wherever they lie, so a step must give the bits of the streamed model, which stages block by block: one to six blocks (whole
groups, remainders), heads whose region holds none, one or more pairs of copies, the update at once and pending, rounded to nearest and
stochastically; the number of launches says that the groups are as large as meant."""
import pytest

import paper_2507_03211_amd as zo_amd
import zo_inputs as zi
from gpu_util import Model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [zi.BF16, zi.FP32])
@pytest.mark.parametrize("deferred", [False, True])
@pytest.mark.parametrize("n_layers,vocab", [(1, 4096), (2, 4096), (3, 24), (3, 520), (4, 4096), (5, 300), (5, 520), (5, 1100), (6, 4096)])
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


def _steps(model, rounding, deferred, batch, seq):
    if deferred:
        zo_amd.zo_set_deferred_update(model.handle, 1)
    zo_amd.zo_set_update_rounding(model.handle, rounding)
    _, tok = model.tokens()
    out = [zo_amd.zo_step(model.handle, tok, batch, seq, seed, 1e-3, 1e-2) for seed in (0, 1)]
    zo_amd.zo_profile_begin(model.handle, 4096)
    out.append(zo_amd.zo_step(model.handle, tok, batch, seq, 2, 1e-3, 1e-2))
    launches = zo_amd.zo_profile_end(model.handle)["stage"][1]
    zo_amd.zo_flush_pending(model.handle)
    return out, launches, model.theta()


# a pair of copies is 138240 bytes here, the head's region 160 rows of fp32 logits: room for none, one, two and more pairs
@pytest.mark.parametrize("n_layers,vocab,group", [(3, 24, 1), (5, 300, 2), (5, 520, 3), (6, 1100, 4)])
@pytest.mark.parametrize("rounding", [0, 1])
def test_groups_with_a_pending_update_in_either_rounding(n_layers, vocab, group, rounding):
    kw = dict(n_layers=n_layers, d_model=64, n_heads=2, d_ffn=136, vocab=vocab, max_pos=64, dtype=zi.BF16, batch=2, seq=40, seed=3,
              plain_small=False, std=0.05)
    res, stm = Model(**kw), Model(**kw, streamed=True)
    a, b = _steps(res, rounding, True, 2, 40), _steps(stm, rounding, False, 2, 40)
    assert a[1] == -(-n_layers // group)
    assert a[0] == b[0] and all(x.tobytes() == y.tobytes() for x, y in zip(a[2], b[2]))
    res.close(); stm.close()


def test_groups_end_where_their_copies_would_pass_the_cache():
    # 48 MiB a pair of copies and room for two beside the first: two blocks a launch, 96 MiB, not three
    kw = dict(n_layers=3, d_model=1024, n_heads=16, d_ffn=4096, vocab=24800, max_pos=64, dtype=zi.BF16, batch=16, seq=64, seed=3)
    res, stm = Model(**kw), Model(**kw, streamed=True)
    a, b = _steps(res, 0, True, 16, 64), _steps(stm, 0, False, 16, 64)
    assert a[1] == 2
    assert a[0] == b[0] and all(x.tobytes() == y.tobytes() for x, y in zip(a[2], b[2]))
    res.close(); stm.close()
