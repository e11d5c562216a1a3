"""The sign-batched linear layer over every tile shape its size rule picks (256 x 256, 256 x 192, 256 x 128, 192 x 128,
128 x 128, 64 x 64, 32 x 32): one row past a tile, ragged columns, contractions of one slab and up, each epilogue, both 16-bit types;
and the LM head over each of its tile heights and strip widths.  Every output element is compared."""
import pytest
import torch

import paper_2507_03211_amd as zo_amd
import zo_inputs as zi
from gpu_util import DEV

pytestmark = pytest.mark.gpu

TDT = {zi.BF16: torch.bfloat16, zi.FP16: torch.float16}
ULP = {zi.BF16: 2.0**-8, zi.FP16: 2.0**-11}

# m_half, n, k; the tile that the rule takes on 256 CUs is named for the reader (TILES below holds it to that)
SHAPES16 = [(3073, 4104, 192), (1537, 4104, 448),       # 256 x 256
            (769, 5128, 192), (1281, 3080, 192),        # 256 x 192
            (641, 4104, 192), (1281, 2056, 192),        # 256 x 128
            (385, 5128, 256), (641, 3080, 256),         # 192 x 128
            (257, 5128, 320), (641, 1544, 320),         # 128 x 128
            (1, 8, 64), (65, 72, 128), (257, 520, 192), (100, 1000, 1024),   # 64 x 64, the last 32 x 32
            (257, 520, 704), (129, 1032, 1024)]                              # 64 x 64
SHAPES32 = [(2561, 8200, 1024), (1025, 6152, 1024),     # 256 x 256; 128 x 128 and, without residual, 256 x 256
            (1281, 4104, 1024), (641, 5128, 2048),      # 192 x 128, 256 x 128
            (641, 3080, 768), (1281, 1544, 576),        # 192 x 128
            (385, 2568, 576), (641, 1544, 448),         # 64 x 64 and, without residual, 128 x 128
            (3, 16, 64), (64, 64, 64), (130, 520, 320)] # 64 x 64, the last 32 x 32
# LM head: rows a sign, d, vocabulary of each tile; its edges one row or 8 columns past where the rule allows it
HEADS = [((256, 256), 193, 320, 20008), ((256, 256), 769, 192, 20232), ((192, 256), 257, 192, 17000), ((192, 256), 385, 256, 8200),
         ((128, 256), 100, 320, 17000), ((128, 256), 300, 256, 17000), ((128, 256), 1, 256, 20232), ((128, 128), 65, 512, 1000),
         ((128, 128), 1, 320, 264), ((64, 128), 65, 256, 1032), ((64, 128), 3, 64, 520)]
# one row and 8 columns past whole tiles of the named shape: 16-bit outputs, fp32 outputs
TILES = {(256, 256): [(1537, 4104, 448), (1537, 4104, 1024)], (256, 192): [(1281, 3080, 192), (1281, 3080, 2048)],
         (256, 128): [(1281, 2056, 192), (1025, 3080, 2048)], (192, 128): [(385, 5128, 256), (769, 2568, 768)],
         (128, 128): [(257, 5128, 320), (513, 3080, 768)], (64, 64): [(257, 520, 704), (257, 520, 320)]}


def _inputs(m_half, n, k, dtype, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    x = torch.randn(2 * m_half, k, device=DEV, generator=g).to(TDT[dtype])
    w = [(0.05 * torch.randn(n, k, device=DEV, generator=g)).to(TDT[dtype]) for _ in range(2)]
    b = [torch.randn(n, device=DEV, generator=g).to(TDT[dtype]) for _ in range(2)]
    return g, x, w, b


@pytest.mark.parametrize("dtype", [zi.BF16, zi.FP16])
@pytest.mark.parametrize("m_half,n,k,epi", [s + (e,) for i, s in enumerate(SHAPES16) for e in ((0, 1) if i % 2 else (0,))] +
                         [s + (e,) for i, s in enumerate(SHAPES32) for e in ((2, 3) if i % 2 else (2,))])
def test_linear_tiles(m_half, n, k, epi, dtype):
    g, x, w, b = _inputs(m_half, n, k, dtype, m_half + n + k + epi)
    guard = 64                                  # values behind the result that must not change
    flat = torch.full((2 * m_half * n + guard,), 3.0, device=DEV, dtype=TDT[dtype] if epi < 2 else torch.float32)
    y = flat[:2 * m_half * n].view(2 * m_half, n)
    if epi == 2:
        y.normal_(generator=g)
    y0 = y.double()
    zo_amd.zo_kernel_linear_pm(x, w[0], w[1], b[0], b[1], y, dtype, m_half, n, k, epi)
    for s in range(2):
        rows = slice(s * m_half, (s + 1) * m_half)
        want = x[rows].double() @ w[s].double().t()
        size = x[rows].double().abs() @ w[s].double().abs().t() + 8.0
        if epi != 3:
            want = want + b[s].double()
        if epi == 1:
            want = want.clamp(min=0)
        if epi == 2:
            want = want + y0[rows]
        # fp32 sums of k terms (each partial sum rounded by half of 2^-23 of at most `size`, in pieces of 16 or more, so far
        # below this bound), then one rounding into the 16-bit type
        bound = size * (k + 4) * 2.0**-24 + (ULP[dtype] * want.abs() if epi < 2 else 0.0)
        assert bool(((y[rows].double() - want).abs() <= bound).all())
    assert bool((flat[2 * m_half * n:] == 3.0).all())


@pytest.mark.parametrize("dtype", [zi.BF16, zi.FP16])
@pytest.mark.parametrize("epi", [0, 1, 2, 3])
@pytest.mark.parametrize("tile", sorted(TILES))
def test_each_tile_with_each_epilogue(tile, epi, dtype):
    m_half, n, k = TILES[tile][epi // 2]
    assert zo_amd.zo_kernel_linear_tile(m_half, n, k, epi) == tile
    test_linear_tiles(m_half, n, k, epi, dtype)


@pytest.mark.parametrize("dtype", [zi.BF16, zi.FP16])
@pytest.mark.parametrize("m_half,d,vocab", [(257, 192, 17000), (520, 256, 8456), (100, 192, 17000), (193, 320, 20008),   # strips of 128
                                            (65, 512, 1000), (3, 64, 520), (130, 128, 2056)])                          # strips of 64
def test_lmhead_tiles(m_half, d, vocab, dtype):
    g, x, e, _ = _inputs(m_half, vocab, d, dtype, m_half + d)
    target = torch.randint(0, vocab, (2 * m_half,), device=DEV, dtype=torch.int32, generator=g)
    target[::7] = -1
    target[1] = vocab - 1
    loss = torch.empty(2 * m_half, device=DEV, dtype=torch.float64)
    scratch = torch.empty(zo_amd.zo_kernel_lmhead_scratch_bytes(dtype, m_half, vocab), device=DEV, dtype=torch.uint8)
    zo_amd.zo_kernel_lmhead_ce(x, e[0], e[1], target, loss, scratch, dtype, m_half, d, vocab)
    for s in range(2):
        rows = slice(s * m_half, (s + 1) * m_half)
        logits, tg = x[rows].double() @ e[s].double().t(), target[rows].long()
        want = torch.logsumexp(logits, 1) - logits.gather(1, tg.clamp(min=0)[:, None])[:, 0]
        want = torch.where(tg >= 0, want, torch.zeros_like(want))
        assert float((loss[rows] - want).abs().max()) < 2e-4          # fp32 logits: accumulation order only


@pytest.mark.parametrize("dtype", [zi.BF16, zi.FP16])
@pytest.mark.parametrize("tile,m_half,d,vocab", HEADS)
def test_each_lmhead_tile(tile, m_half, d, vocab, dtype):
    assert zo_amd.zo_kernel_linear_tile(m_half, vocab, d, 4) == tile
    test_lmhead_tiles(m_half, d, vocab, dtype)


@pytest.mark.parametrize("m_half,d,vocab", [(257, 192, 17000), (3, 64, 520)])     # a pipelined tile, the small one
def test_lmhead_of_logits_near_the_fp32_range(m_half, d, vocab):
    # one product per logit: the row's power of two times +- 1 (a target among equal largest ones, or as far below as it gets)
    x = torch.zeros(2 * m_half, d, device=DEV)
    x[:, 0] = torch.tensor([2.0**63, 2.0**61, -2.0**63, 1.0], device=DEV)[torch.arange(2 * m_half, device=DEV) % 4]
    e = torch.zeros(vocab, d, device=DEV)
    e[:, 0] = 2.0**63 * (1.0 - 2.0 * (torch.arange(vocab, device=DEV) % 2))
    target = torch.arange(2 * m_half, device=DEV, dtype=torch.int32) % vocab
    loss = torch.empty(2 * m_half, device=DEV, dtype=torch.float64)
    scratch = torch.empty(zo_amd.zo_kernel_lmhead_scratch_bytes(zi.BF16, m_half, vocab), device=DEV, dtype=torch.uint8)
    xb, eb = x.bfloat16(), e.bfloat16()
    zo_amd.zo_kernel_lmhead_ce(xb, eb, eb, target, loss, scratch, zi.BF16, m_half, d, vocab)
    logits = xb.double() @ eb.double().t()
    want = torch.logsumexp(logits, 1) - logits.gather(1, target.long()[:, None])[:, 0]
    # the products are exact; sums of equal terms in fp32 and one rounding of the pair's correction: a few 2^-24
    assert bool(((loss - want).abs() <= 1e-6 + 1e-6 * want.abs()).all())


@pytest.mark.parametrize("m_half,d,vocab", [(257, 192, 17000), (3, 64, 520)])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_lmhead_of_large_logits_with_full_mantissas(m_half, d, vocab, sign):
    # one product per logit, +-(1 + i / 128) 2^e times (1 + j / 128): 16 bits of mantissa, e from 20 up to the end of the fp32
    # range.  Every fourth column is of the row's own sign; with sign = -1 the last strips hold large negative logits only.
    rows, col = torch.arange(2 * m_half, device=DEV), torch.arange(vocab, device=DEV)
    x = torch.zeros(2 * m_half, d, device=DEV)
    x[:, 0] = (1.0 + (37 * rows % 128) / 128.0) * torch.exp2((rows * 107 // (2 * m_half) - 20).float())      # 2^-20 .. 2^86
    e = torch.zeros(vocab, d, device=DEV)
    e[:, 0] = (1.0 + (11 * col % 127) / 128.0) * 2.0**40 * torch.where((col % 4 == 0) & (col < vocab // 2), sign, -1.0)
    target = (rows * 61 % vocab).to(torch.int32)
    loss = torch.empty(2 * m_half, device=DEV, dtype=torch.float64)
    scratch = torch.empty(zo_amd.zo_kernel_lmhead_scratch_bytes(zi.BF16, m_half, vocab), device=DEV, dtype=torch.uint8)
    xb, eb = x.bfloat16(), e.bfloat16()
    zo_amd.zo_kernel_lmhead_ce(xb, eb, eb, target, loss, scratch, zi.BF16, m_half, d, vocab)
    logits = xb.double() @ eb.double().t()
    assert bool((logits == logits.float().double()).all())                  # so that what follows is the exact answer
    want = torch.logsumexp(logits, 1) - logits.gather(1, target.long()[:, None])[:, 0]
    # the products are exact; a sum of equal terms in fp32 and one rounding of the pair's correction, as above
    assert bool(((loss - want).abs() <= 1e-6 + 1e-6 * want.abs()).all())


@pytest.mark.parametrize("dtype", [zi.BF16, zi.FP16])
@pytest.mark.parametrize("epi", [0, 1, 2, 3])
@pytest.mark.parametrize("m_half,n", [(65, 128), (70, 136)])
@pytest.mark.parametrize("slabs", [1, 2, 3, 4, 5])
def test_small_tile_of_few_slabs(m_half, n, slabs, epi, dtype):
    # 64 x 64 tiles: a ring of as many stages as there are slabs, up to four; rows of whole cache lines and others, whose
    # 16-bit outputs of one or two slabs are stored another way; five slabs take 32 x 32 tiles
    assert zo_amd.zo_kernel_linear_tile(m_half, n, 64 * slabs, epi) == ((64, 64) if slabs < 5 else (32, 32))
    test_linear_tiles(m_half, n, 64 * slabs, epi, dtype)


@pytest.mark.parametrize("dtype", [zi.BF16, zi.FP16])
@pytest.mark.parametrize("epi", [0, 1, 2, 3])
@pytest.mark.parametrize("m_half,n,k", [(129, 1032, 320), (193, 776, 448), (257, 520, 576), (161, 1000, 1024)])
def test_small_tile_whose_ring_comes_round(m_half, n, k, epi, dtype):
    # 64 x 64 tiles of more slabs than their ring has stages: its first stage again once (5 slabs), all but one of them (7), two rounds
    # and one (9), whole rounds (16); one row past a tile of 32 or 64, ragged columns
    assert zo_amd.zo_kernel_linear_tile(m_half, n, k, epi) == (64, 64)
    test_linear_tiles(m_half, n, k, epi, dtype)
