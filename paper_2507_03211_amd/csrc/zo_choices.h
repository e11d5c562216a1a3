// Which route a call takes where its sizes decide: plain host arithmetic, no runtime call.
#pragma once

namespace zo {

inline long f64_tiles(int n_sign, int m_half, int n, int edge) { return (long)n_sign * ((m_half + edge - 1) / edge) * ((n + edge - 1) / edge); }

// fp64 linear layers: 32 x 32 tiles once they give every CU two workgroups, else 16 x 16 (times in us, both tilings):
// 256 x 384 x 128 (192 tiles) 5.0 / 5.3, 256 x 128 x 512 (64) 5.3 / 11.8, 512 x 768 x 768 (768) 50 / 33,
// 2048 x 768 x 3072 753 / 417
inline bool f64_tiles32(int n_sign, int m_half, int n) { return f64_tiles(n_sign, m_half, n, 32) >= 512; }

// The longest row that an fp64 layer takes its LayerNorm of, and the longest one of the two instances that holds fewer pieces.
constexpr int kNormRowMax = 320, kNormRowShort = 128;

// Does an fp64 layer take its LayerNorm on the way (one launch) or behind one (two)?  The launch costs 2 to 5 us, the more the
// more rows it has.  On the way every column tile normalises its rows over again: that costs with the tiles and, each tile's
// chain being longer and the rows leaving the L1, with more than the first power of the row's length.  In a step, where rows and
// weights are fresh from other kernels, one launch instead of two gains per layer (16 to 128 rows a sign) 3.2 us at 64, 2.6 at
// 128, 1.5 at 192, 0.8 at 256, 0.4 at 320 and loses 0.4 at 384, 1.5 at 448 and 1 - 2 at 512.  Below that limit: 16 x 16 tiles, and
// short rows or tiles x length^1.5 below a bound.  m_half x n x k, both signs, us, two launches / one, operands in the L2: 512 x 480 x
// 128 13.2 / 11.9, 250 x 976 x 104 10.1 / 10.1 (the last short rows before 32 x 32 tiles); 128 x 1024 x 192 10.2 / 9.4, 1280
// columns of 200 10.1 / 10.8; 128 x 512 x 320 10.1 / 9.2, 256 x 960 x 320 21.6 / 23.4.  A step of 4 layers, 256 rows a sign, d 192
// 304 / 294 (all layers on the way: 303).
inline bool norm_on_the_way(int n_sign, int m_half, int n, int k)
{
    if (k > kNormRowMax || f64_tiles32(n_sign, m_half, n)) return false;
    const long tiles = f64_tiles(n_sign, m_half, n, 16), rows = (long)n_sign * m_half;
    return k <= kNormRowShort || (tiles <= 1152 && (double)tiles * k * __builtin_sqrt(k / 300.0) <= 140000.0 + 150.0 * (double)(rows < 256 ? rows : 256));
}

// Pieces of 256 elements that a wavefront holds of a LayerNorm row of 16-bit models (three at least); 0: longer than 2048, a
// workgroup's.
inline int layernorm_pieces(int d) { return d > 2048 ? 0 : d <= 768 ? 3 : (d + 255) / 256; }

// Groups of d_head threads of the plain attention's 128 that a row's keys are dealt to; `room`: of the LDS for their partial sums.
// us, one group / as many as there are: fp64, 8 x 128 tokens, 8 heads of 8 channels (16 groups) 29.1 / 14.4, of 16 33.0 / 20.6, of
// 32 44.8 / 38.6, of 40 (3 groups) 50.4 / 48.7; two lose, their sums' loop waits for each product where that of one group is
// unrolled: of 48 55.4 / 63.3, of 64 66.4 / 69.3; bf16, 4 x 700 tokens, 2 heads of 48 74 / 86.  A group has two keys at least: 2
// sequences of 1 token 3.73 / 4.06 with 16 groups, of 6 3.91 / 4.06 (3: 3.87), of 9 4.08 / 4.09 (4: 4.04).
inline int plain_attention_groups(int seq, int d_head, bool room)
{
    const int groups = 128 / d_head;
    if (groups < 3 || !room) return 1;
    return seq >= 2 * groups ? groups : seq >= 4 ? seq / 2 : 1;
}

}  // namespace zo
