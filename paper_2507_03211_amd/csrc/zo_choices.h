// Which route a call takes where its sizes decide: plain host arithmetic, no runtime call.
#pragma once

namespace zo {

inline long f64_tiles(int n_sign, int m_half, int n, int edge) { return (long)n_sign * ((m_half + edge - 1) / edge) * ((n + edge - 1) / edge); }

// fp64 linear layers: 32 x 32 tiles once they give every CU two workgroups, else 16 x 16 (times in us, both tilings):
// 256 x 384 x 128 (192 tiles) 5.0 / 5.3, 256 x 128 x 512 (64) 5.3 / 11.8, 512 x 768 x 768 (768) 50 / 33,
// 2048 x 768 x 3072 753 / 417
inline bool f64_tiles32(int n_sign, int m_half, int n) { return f64_tiles(n_sign, m_half, n, 32) >= 512; }

// The longest row a lane group of the fp64 layer holds in registers for its LayerNorm, and the longest one of the two
// instances that holds fewer pieces.
constexpr int kNormRowMax = 512, kNormRowShort = 128;

// Does an fp64 layer take its LayerNorm on the way (one launch) or behind one (two)?  The launch costs 2 to 5 us, the more the
// more rows it has.  On the way every column tile normalises its rows over again: that costs with the tiles and, each tile's
// chain being longer and the rows leaving the L1, with more than the first power of the row's length.  So while the tiles
// are 16 x 16 and either the rows are short or tiles x length^1.5 stays below a bound.  m_half x n x k, both signs, us, two launches / one:
// 512 x 480 x 128 13.2 / 11.9, 250 x 976 x 104 10.1 / 10.1 (the last short rows before 32 x 32 tiles); 128 x 1024 x 192 10.2 / 9.4,
// 1280 columns of 200 10.1 / 10.8; 128 x 512 x 320 10.1 / 9.2, 512 x 128 x 352 12.5 / 13.2; 64 x 512 x 512 11.1 / 10.3, 640
// columns 12.0 / 12.3, 559 x 184 x 496 17.5 / 21.9.  Over 492 sizes of 136 to 512 none that is taken is more than 2 % slower than
// two launches; of the 193 left, 9 are 10 to 19 % faster on the way, 46 as much and more slower.
inline bool norm_on_the_way(int n_sign, int m_half, int n, int k)
{
    if (k > kNormRowMax || f64_tiles32(n_sign, m_half, n)) return false;
    const long tiles = f64_tiles(n_sign, m_half, n, 16), rows = (long)n_sign * m_half;
    return k <= kNormRowShort || (tiles <= 1152 && (double)tiles * k * __builtin_sqrt(k / 300.0) <= 140000.0 + 150.0 * (double)(rows < 256 ? rows : 256));
}

// Pieces of 256 elements that a wavefront holds of a LayerNorm row of 16-bit models (three at least); 0: longer than 2048, a
// workgroup's.
inline int layernorm_pieces(int d) { return d > 2048 ? 0 : d <= 768 ? 3 : (d + 255) / 256; }

}  // namespace zo
