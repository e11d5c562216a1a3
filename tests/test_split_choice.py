"""Which linear layers take 32 x 32 tiles, on the host: up to one tile per CU from five slabs on, and against measured times with 64 x 64
ones: where the rule takes them they are faster, where it does not they are slower or at most 1.3 times as fast."""
import pytest

import paper_2507_03211_amd as zo_amd


@pytest.mark.parametrize("m_half,n,k,small", [(128, 1024, 320, True), (129, 1024, 320, False), (128, 1032, 320, False), (128, 1024, 256, False), (32, 4096, 2048, True), (33, 4096, 2048, False),
                                              (1, 8, 320, True), (1, 8, 256, False)])
def test_where_the_line_lies(m_half, n, k, small):
    for epi in range(4):
        assert (zo_amd.zo_kernel_linear_tile(m_half, n, k, epi) == (32, 32)) == small


# m_half, n, k, epilogue, us with 64 x 64 tiles, with 32 x 32 ones (both signs, bf16, 256 CUs, operands far)
@pytest.mark.parametrize("m_half,n,k,epi,us64,us32", [(96, 1024, 4096, 2, 20.7, 12.2), (213, 576, 2304, 2, 11.3, 7.0), (68, 384, 1536, 2, 8.6, 5.4), (213, 576, 576, 2, 5.6, 4.3),
                                                      (536, 768, 3072, 2, 18.2, 23.6), (123, 2304, 2304, 2, 15.0, 17.4), (213, 1728, 576, 0, 5.3, 7.1), (96, 6144, 2048, 0, 19.6, 23.7),
                                                      (28, 4944, 5248, 3, 28.1, 30.5), (25, 4544, 384, 0, 4.7, 4.9), (536, 512, 2048, 2, 12.7, 13.1), (53, 4552, 4736, 2, 28.8, 33.0)])
def test_against_measured_times(m_half, n, k, epi, us64, us32):
    assert (zo_amd.zo_kernel_linear_tile(m_half, n, k, epi) == (32, 32)) == (us32 < us64)


# past the line and faster all the same, one to two tiles a CU or two to four slabs: what the rule leaves
@pytest.mark.parametrize("m_half,n,k,epi,us64,us32", [(250, 1024, 4096, 2, 21.6, 18.9), (250, 768, 3072, 2, 17.5, 15.1), (530, 296, 8320, 1, 36.4, 28.8), (401, 336, 640, 0, 5.7, 5.1),
                                                      (129, 1024, 320, 0, 4.1, 3.9), (54, 120, 128, 1, 3.2, 3.0), (33, 184, 256, 0, 4.0, 3.2), (186, 96, 192, 0, 3.5, 3.0)])
def test_what_the_rule_leaves(m_half, n, k, epi, us64, us32):
    assert zo_amd.zo_kernel_linear_tile(m_half, n, k, epi) != (32, 32) and us32 < us64 <= 1.3 * us32
