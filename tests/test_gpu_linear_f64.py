"""The fp32-parameter linear layer (fp64 activations and sums) on the matrix cores: both tile sizes, contractions shorter than
one piece, not a multiple of 16, and ragged in every direction, against the product in numpy's long double."""
import numpy as np
import pytest
import torch

import paper_2507_03211_amd as zo_amd
import zo_inputs as zi
from gpu_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("epi", [0, 1, 2, 3])
@pytest.mark.parametrize("m_half,n,k", [(1, 1, 4), (3, 17, 12), (16, 16, 16), (17, 33, 20), (64, 64, 256), (37, 130, 68), (31, 40, 7),
                                        (500, 515, 36), (512, 512, 64)])
def test_linear_f64(m_half, n, k, epi):
    rng = np.random.Generator(np.random.PCG64(m_half * n + k + epi))
    x = rng.standard_normal((2 * m_half, k))
    w = [rng.standard_normal((n, k)).astype(np.float32) for _ in range(2)]
    b = [rng.standard_normal(n).astype(np.float32) for _ in range(2)]
    y0 = rng.standard_normal((2 * m_half, n))
    y = torch.from_numpy(y0.copy()).to(DEV)
    dev = [torch.from_numpy(t).to(DEV) for t in (x, *w, *b)]
    zo_amd.zo_kernel_linear_pm(dev[0], dev[1], dev[2], dev[3], dev[4], y, zi.FP32, m_half, n, k, epi)
    got = y.cpu().numpy()
    for s in range(2):
        rows = slice(s * m_half, (s + 1) * m_half)
        xl, wl = x[rows].astype(np.longdouble), w[s].astype(np.longdouble)
        want, size = xl @ wl.T, np.abs(xl) @ np.abs(wl).T + 1.0
        if epi != 3:
            want = want + b[s]
        if epi == 1:
            want = np.maximum(want, 0)
        if epi == 2:
            want = want + y0[rows]
        # k + 3 additions, each within half a unit of 2^-52 of a partial sum that is at most `size`
        bound = (k + 4) * 2.0**-53 * (size + np.abs(b[s])[None] + np.abs(y0[rows]))
        assert np.all(np.abs(got[rows] - want) <= bound), (s, np.max(np.abs(got[rows] - want) / bound))
