"""The rule that picks a linear layer's tile shape, on the host: against measured times, at sizes of every epilogue from short
contractions with large outputs to long ones with few rows.  The picked shape is about as fast at least as the two tilings (256 x 256 and
a register-staged 128 x 128) that the library had before the rule."""
import pytest

import paper_2507_03211_amd as zo_amd

TILES = [(256, 256), (256, 192), (256, 128), (192, 128), (128, 128), (64, 64)]

# m_half, n, k, epilogue, us with those two tilings, us in each of TILES (both signs, bf16, 256 CUs; None: too few slabs for
# the tile's pipeline)
MEASURED = [
    (966, 15512, 256, 3, 34.9, (32.3, 34.9, 39.4, 42.5, None, 68.2)),
    (1613, 9080, 384, 3, 39.5, (38.0, 43.5, 47.5, 50.8, 54.3, 70.2)),
    (920, 18312, 256, 3, 46.2, (42.3, 42.4, 53.3, 53.6, None, 80.5)),
    (1025, 11496, 576, 3, 43.4, (40.8, 47.5, 52.8, 49.3, 56.1, 70.1)),
    (4208, 6968, 192, 3, 67.3, (71.0, 69.6, 81.1, None, None, 83.5)),
    (4143, 3416, 320, 3, 34.5, (33.8, 40.4, 37.4, 31.9, 31.4, 50.1)),
    (3409, 2520, 512, 3, 37.9, (36.2, 30.5, 30.3, 26.9, 29.0, 39.8)),
    (5827, 3664, 192, 3, 47.7, (48.4, 45.0, 43.1, None, None, 55.3)),
    (160, 14800, 320, 2, 19.6, (18.6, 16.7, 14.1, 14.1, 16.6, 14.8)),
    (6653, 856, 384, 2, 32.7, (31.7, 42.7, 35.5, 32.3, 30.5, 27.2)),
    (1661, 3336, 320, 2, 29.7, (28.3, 28.0, 31.8, 29.3, 29.4, 25.0)),
    (3880, 1648, 192, 2, 28.7, (26.8, 35.6, 28.7, None, None, 21.8)),
    (249, 632, 3904, 2, 50.7, (69.5, 55.7, 39.8, 33.7, 26.2, 15.5)),
    (664, 704, 2816, 2, 39.5, (52.9, 41.8, 31.1, 26.1, 21.2, 13.1)),
    (181, 832, 3328, 2, 43.7, (58.0, 45.7, 33.2, 28.6, 22.2, 13.4)),
    (1832, 8880, 3008, 3, 214.2, (213.9, 185.9, 218.6, 214.8, 228.0, 339.4)),
    (229, 2536, 9088, 3, 136.5, (148.6, 119.5, 99.1, 68.6, 74.3, 65.5)),
    (66, 7680, 1920, 1, 29.0, (36.8, 29.7, 22.3, 19.0, 16.0, 13.6)),
    (718, 14256, 7424, 1, 326.5, (313.0, 266.9, 299.5, 322.4, 361.9, 611.9)),
    (105, 16816, 1536, 1, 37.3, (37.0, 30.7, 45.0, 38.5, 35.5, 35.0)),
    (5182, 6912, 2304, 0, 282.8, (275.9, 268.6, 283.8, 303.8, 329.8, 525.0)),
    (2750, 7968, 448, 1, 52.1, (51.3, 50.9, 48.2, 55.3, 56.0, 83.7)),
    (1860, 2328, 448, 1, 16.8, (16.6, 15.1, 17.8, 15.4, 16.4, 19.1)),
]


@pytest.mark.parametrize("m_half,n,k,epi,before,us", MEASURED)
def test_picked_tile_is_no_slower_than_before_the_rule(m_half, n, k, epi, before, us):
    tile = zo_amd.zo_kernel_linear_tile(m_half, n, k, epi)
    # 3 % is what repeated measurements of one size differ by; fp32 outputs without a residual of three slabs are up to 6 % behind
    assert us[TILES.index(tile)] <= 1.06 * before, tile


# LM head of few rounds: rows a sign, d, vocabulary, us with heights of 256, 192, 128 (256 columns)
HEADS = [
    (616, 1280, 6824, (31.6, 28.7, 37.4)),
    (595, 2624, 8296, (57.7, 85.3, 63.4)),
    (363, 832, 12392, (26.0, 21.6, 28.2)),
    (334, 1088, 12984, (32.0, 27.0, 34.3)),
    (828, 1280, 32000, (132.6, 136.9, 145.3)),
    (1048, 2048, 50272, (419.0, 399.0, 428.0)),
]


@pytest.mark.parametrize("rows,d,vocab,us", HEADS)
def test_picked_height_of_the_lm_head_is_near_the_best(rows, d, vocab, us):
    height, columns = zo_amd.zo_kernel_linear_tile(rows, vocab, d, 4)
    assert columns == 256 and us[(256, 192, 128).index(height)] <= 1.04 * min(us)


def test_shapes_off_the_matrix_cores_have_no_tile():
    assert zo_amd.zo_kernel_linear_tile(64, 64, 64, 0) == (64, 64)
    for m_half, n, k, epi in ((64, 64, 96, 0), (64, 60, 64, 0), (0, 64, 64, 0), (64, 64, 64, 5), (64, 64, 64, -1), (1, 1 << 24, 64, 2)):
        assert zo_amd.zo_kernel_linear_tile(m_half, n, k, epi) is None
