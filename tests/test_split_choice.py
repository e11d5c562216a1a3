"""Which linear layers take 32 x 32 tiles, on the host: up to one tile per CU from five slabs on, and against measured times of the other
small shapes."""
import pytest

import paper_2507_03211_amd as zo_amd


@pytest.mark.parametrize("m_half,n,k,small", [(128, 1024, 320, True), (129, 1024, 320, False), (128, 1032, 320, False), (128, 1024, 256, False), (32, 4096, 2048, True), (33, 4096, 2048, False),
                                              (1, 8, 320, True), (1, 8, 256, False)])
def test_where_the_line_lies(m_half, n, k, small):
    for epi in range(4):
        assert (zo_amd.zo_kernel_linear_tile(m_half, n, k, epi) == (32, 32)) == small


# m_half, n, k, epilogue, us with 64 x 64 tiles, with 32 x 32 ones (both signs, bf16, 256 CUs, operands far)
@pytest.mark.parametrize("m_half,n,k,epi,us64,us32", [(96, 1024, 4096, 2, 20.7, 12.2), (213, 576, 2304, 2, 11.3, 7.0), (68, 384, 1536, 2, 8.6, 5.4), (213, 576, 576, 2, 5.6, 4.3),
                                                      (536, 768, 3072, 2, 18.2, 23.6), (123, 2304, 2304, 2, 15.0, 17.4), (213, 1728, 576, 0, 5.3, 7.1), (96, 6144, 2048, 0, 19.6, 23.7)])
def test_against_measured_times(m_half, n, k, epi, us64, us32):
    assert (zo_amd.zo_kernel_linear_tile(m_half, n, k, epi) == (32, 32)) == (us32 < us64)
