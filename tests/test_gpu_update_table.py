"""The update pass over a table of tensors, in both orders of its chunks (runs per workgroup where the tensors are short, strided
where they are long), against the same pass over one tensor after the other: bit for bit."""
import pytest
import torch

import paper_2507_03211_amd as zo_amd
import zo_inputs as zi
from gpu_util import DEV, Model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [zi.BF16, zi.FP16, zi.FP32])
def test_table_equals_single_tensors(dtype):
    # some 3000 chunks in 132 tensors: one longer than the stride and many short ones, remainders, single chunks
    mdl = Model(8, 264, 3, 3000, 40008, 77, dtype, 1, 16)
    n_all = mdl.ocfg.n_tensors
    for first, n in ((0, n_all), (0, 1), (0, 2), (1, n_all - 1), (2, 16), (5, 37), (n_all - 2, 2)):
        before = [t.clone() for t in mdl.tensors]
        torch.cuda.synchronize()
        zo_amd.zo_perturb(mdl.handle, 11, 0.25, first, n)
        torch.cuda.synchronize()
        for i, (t, old) in enumerate(zip(mdl.tensors, before)):
            want = old.clone()
            if first <= i < first + n:
                zo_amd.zo_kernel_axpy_z(old, want, dtype, old.numel(), 11, i, 0.25)
            assert torch.equal(t.view(torch.uint8), want.view(torch.uint8)), (first, n, i)
    mdl.close()
