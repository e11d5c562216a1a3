// Forward-pass kernels that are not matrix-core bound: embedding gather, LayerNorm, the
// cross-entropy reduction, the loss / projected-gradient scalars (DistZO2 Eq. 1), and the
// plain (non-MFMA) linear and attention kernels that serve the fp32-parameter precision,
// which runs with fp64 activations, and shapes the MFMA tilings do not cover.
//
// Row layout everywhere: row = sign * m_half + b * seq + t, sign 0 = theta + eps z,
// sign 1 = theta - eps z; each sign reads its own copy of every parameter.
#include "zo_choices.h"
#include "zo_kernels.h"
#include "zo_types.hip.h"

namespace zo {

// ------------------------------------------------------------------ embedding
// h[row, :] = E_sign[token] + Pos_sign[t];  target[row] = next token (or -1 at t = seq-1).
// A wavefront a row, four elements a lane and access (d is a multiple of 8, and tables and stream lie on 16 bytes).  In a step, 16384
// rows of 768, bf16, 28.9 us a workgroup a row and element by element, 22.3 so: 3.4 TB/s of what must reach memory (25 MB of token
// rows, 50 MB of the stream; the position rows stay in the caches), rows scattered by the tokens.
template <int DT>
__global__ __launch_bounds__(256) void embed_kernel(const int32_t *__restrict__ tokens, const void *e_p, const void *e_m,
                                                    const void *pos_p, const void *pos_m, void *resid,
                                                    int32_t *__restrict__ target, uint32_t *flags, int batch, int seq,
                                                    int d, int vocab, int rows)
{
    using P = Prec<DT>;
    const int m_half = batch * seq;
    const int row = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= rows) return;
    const int sign = row / m_half, bt = row % m_half, t = bt % seq;
    const int tok = tokens[bt];
    const bool ok = tok >= 0 && tok < vocab;
    if (lane == 0) {
        int tg = -1;
        if (t + 1 < seq) {
            tg = tokens[bt + 1];
            if (tg < 0 || tg >= vocab) { tg = -2; atomicOr(flags, 2u); }   // -2: poisons the row loss
        }
        target[row] = tg;
        if (!ok) atomicOr(flags, 2u);
    }
    using W = typename P::W;
    using R = typename P::R;
    const W *e = (const W *)(sign ? e_m : e_p) + (size_t)(ok ? tok : 0) * d;
    const W *p = (const W *)(sign ? pos_m : pos_p) + (size_t)t * d;
    R *h = (R *)resid + (size_t)row * d;
    const R bad = (R)__builtin_nanf("");
    struct alignas(4 * sizeof(W)) W4 { W v[4]; };
    struct alignas(16) R4 { R v[4]; };
#pragma unroll 2
    for (int c = 4 * lane; c < d; c += 256) {
        const W4 a = *(const W4 *)(e + c), b = *(const W4 *)(p + c);
        R4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o.v[i] = ok ? (R)P::w2f(a.v[i]) + (R)P::w2f(b.v[i]) : bad;
        *(R4 *)(h + c) = o;
    }
}

// ------------------------------------------------------------------ LayerNorm
// One workgroup per row; mean and (biased) variance by two passes over the row.
template <int DT>
__global__ __launch_bounds__(256) void layernorm_kernel(const void *resid, const void *g_p, const void *g_m,
                                                        const void *b_p, const void *b_m, void *y, int m_half, int d,
                                                        float eps)
{
    using P = Prec<DT>;
    using Acc = typename P::Acc;
    __shared__ Acc red[16];
    const int row = blockIdx.x;
    const int sign = row / m_half;
    const typename P::R *h = (const typename P::R *)resid + (size_t)row * d;
    const typename P::W *g = (const typename P::W *)(sign ? g_m : g_p);
    const typename P::W *b = (const typename P::W *)(sign ? b_m : b_p);
    typename P::A *out = (typename P::A *)y + (size_t)row * d;
    Acc s = 0;
    for (int c = threadIdx.x; c < d; c += blockDim.x) s += (Acc)h[c];
    const Acc mean = block_sum(s, red) / (Acc)d;
    Acc v = 0;
    for (int c = threadIdx.x; c < d; c += blockDim.x) { const Acc t = (Acc)h[c] - mean; v += t * t; }
    const Acc var = block_sum(v, red) / (Acc)d;
    Acc rstd;
    if constexpr (sizeof(Acc) == 8) rstd = 1.0 / __builtin_sqrt(var + (double)eps);
    else rstd = 1.0f / __builtin_sqrtf(var + eps);
    for (int c = threadIdx.x; c < d; c += blockDim.x) {
        const Acc t = ((Acc)h[c] - mean) * rstd * (Acc)P::w2f(g[c]) + (Acc)P::w2f(b[c]);
        out[c] = P::acc2a(t);
    }
}


// Fast path for 2-byte activations and rows of up to 2048 elements: one wavefront per row, the row held in registers
// (NV float4 per lane), so the residual stream is read once; statistics without LDS.  d % 4 == 0.
// What a wave waits for is latency: the row, twelve exchanges of the two sums, gain and bias.  Exchanges in the vector pipe and
// gain and bias loaded with the row, 16384 rows, us before / here: d 768 14.0 / 13.3, 1024 17.9 / 15.9 (6.3 TB/s), 2048 37.0 /
// 34.4.  As many pieces as the row has: with eight for all rows above 1024, 88 registers a lane (5 waves per SIMD) and loads of
// pieces that are not there, 4096 rows of 1280 8.7 us / 7.5 with five, of 1536 9.8 / 8.3 with six, of 1792 10.4 / 9.5 with seven.
template <int DT, int NV>
__global__ __launch_bounds__(256) void layernorm_wave_kernel(const float *__restrict__ resid, const uint16_t *__restrict__ g_p,
                                                             const uint16_t *__restrict__ g_m, const uint16_t *__restrict__ b_p,
                                                             const uint16_t *__restrict__ b_m, uint16_t *__restrict__ y, int rows,
                                                             int m_half, int d, float eps)
{
    using P = Prec<DT>;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= rows) return;
    const int sign = row / m_half;
    const float4 *h = (const float4 *)(resid + (size_t)row * d);
    const uint2 *g = (const uint2 *)(sign ? g_m : g_p), *b = (const uint2 *)(sign ? b_m : b_p);
    uint2 *out = (uint2 *)(y + (size_t)row * d);
    const int nvec = d >> 2;
    float4 v[NV];
    uint2 gv[NV], bv[NV];                       // on their way while the sums are taken
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int c = lane + 64 * i;
        v[i] = c < nvec ? h[c] : float4{0.0f, 0.0f, 0.0f, 0.0f};
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int c = lane + 64 * i < nvec ? lane + 64 * i : nvec - 1;
        gv[i] = g[c];
        bv[i] = b[c];
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
    const float mean = wave_sum(s) / (float)d;
    float q = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        if (lane + 64 * i < nvec) {
            const float a = v[i].x - mean, bb = v[i].y - mean, c = v[i].z - mean, dd = v[i].w - mean;
            q += (a * a + bb * bb) + (c * c + dd * dd);
        }
    }
    const float rstd = 1.0f / __builtin_sqrtf(wave_sum(q) / (float)d + eps);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int c = lane + 64 * i;
        if (c < nvec) {
            const uint2 gr = gv[i], br = bv[i];
            const float g0 = P::w2f((uint16_t)(gr.x & 0xffff)), g1 = P::w2f((uint16_t)(gr.x >> 16));
            const float g2 = P::w2f((uint16_t)(gr.y & 0xffff)), g3 = P::w2f((uint16_t)(gr.y >> 16));
            const float b0 = P::w2f((uint16_t)(br.x & 0xffff)), b1 = P::w2f((uint16_t)(br.x >> 16));
            const float b2 = P::w2f((uint16_t)(br.y & 0xffff)), b3 = P::w2f((uint16_t)(br.y >> 16));
            const float o0 = (v[i].x - mean) * rstd * g0 + b0, o1 = (v[i].y - mean) * rstd * g1 + b1;
            const float o2 = (v[i].z - mean) * rstd * g2 + b2, o3 = (v[i].w - mean) * rstd * g3 + b3;
            uint2 o;
            o.x = (uint32_t)P::acc2a(o0) | ((uint32_t)P::acc2a(o1) << 16);
            o.y = (uint32_t)P::acc2a(o2) | ((uint32_t)P::acc2a(o3) << 16);
            out[c] = o;
        }
    }
}

// The same for longer rows: one workgroup of 256 threads per row, NV float4 per thread, the two sums across the four
// wavefronts through LDS.  d % 4 == 0, d <= 1024 NV.  Measured against the wavefront-per-row kernel (8192 rows):
// 5.4 against 4.7 TB/s at d = 4096 and 5120, 5.5 against 2.7 at 12288 (48 float4 per lane leave a SIMD two waves),
// 5.5 against 5.9 at 2048, 4.3 against 5.6 at 1280: hence the switch at 2048.
template <int DT, int NV>
__global__ __launch_bounds__(256) void layernorm_block_kernel(const float *__restrict__ resid, const uint16_t *__restrict__ g_p,
                                                              const uint16_t *__restrict__ g_m, const uint16_t *__restrict__ b_p,
                                                              const uint16_t *__restrict__ b_m, uint16_t *__restrict__ y, int m_half,
                                                              int d, float eps)
{
    using P = Prec<DT>;
    __shared__ float red[16];
    const int row = blockIdx.x, tid = threadIdx.x;
    const int sign = row / m_half;
    const float4 *h = (const float4 *)(resid + (size_t)row * d);
    const uint2 *g = (const uint2 *)(sign ? g_m : g_p), *b = (const uint2 *)(sign ? b_m : b_p);
    uint2 *out = (uint2 *)(y + (size_t)row * d);
    const int nvec = d >> 2;
    float4 v[NV];
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int c = tid + 256 * i;
        v[i] = c < nvec ? h[c] : float4{0.0f, 0.0f, 0.0f, 0.0f};
        s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
    }
    const float mean = block_sum(s, red) / (float)d;
    float q = 0.0f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        if (tid + 256 * i < nvec) {
            const float a = v[i].x - mean, bb = v[i].y - mean, c = v[i].z - mean, dd = v[i].w - mean;
            q += (a * a + bb * bb) + (c * c + dd * dd);
        }
    }
    const float rstd = 1.0f / __builtin_sqrtf(block_sum(q, red) / (float)d + eps);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int c = tid + 256 * i;
        if (c < nvec) {
            const uint2 gr = g[c], br = b[c];
            const float g0 = P::w2f((uint16_t)(gr.x & 0xffff)), g1 = P::w2f((uint16_t)(gr.x >> 16));
            const float g2 = P::w2f((uint16_t)(gr.y & 0xffff)), g3 = P::w2f((uint16_t)(gr.y >> 16));
            const float b0 = P::w2f((uint16_t)(br.x & 0xffff)), b1 = P::w2f((uint16_t)(br.x >> 16));
            const float b2 = P::w2f((uint16_t)(br.y & 0xffff)), b3 = P::w2f((uint16_t)(br.y >> 16));
            const float o0 = (v[i].x - mean) * rstd * g0 + b0, o1 = (v[i].y - mean) * rstd * g1 + b1;
            const float o2 = (v[i].z - mean) * rstd * g2 + b2, o3 = (v[i].w - mean) * rstd * g3 + b3;
            uint2 o;
            o.x = (uint32_t)P::acc2a(o0) | ((uint32_t)P::acc2a(o1) << 16);
            o.y = (uint32_t)P::acc2a(o2) | ((uint32_t)P::acc2a(o3) << 16);
            out[c] = o;
        }
    }
}

// ------------------------------------------------------------------ plain linear layer
// (16-bit types whose k is not a multiple of 64, fp32 whose k is not a multiple of 4 or whose buffers are unaligned)
// y[row, n] = sum_k x[row, k] wt[n, k] (+ bias).  64 x 64 output tile, 16-deep LDS slabs,
// 4 x 4 outputs per thread.  blockIdx.z selects the sign.
template <int DT, int EPI>
__global__ __launch_bounds__(256) void linear_plain_kernel(const void *x, const void *wt_p, const void *wt_m,
                                                           const void *b_p, const void *b_m, void *y, int m_half, int n,
                                                           int k)
{
    using P = Prec<DT>;
    using Acc = typename P::Acc;
    constexpr int BM = 64, BN = 64, BK = 16;
    __shared__ Acc xs[BK][BM + 1];
    __shared__ Acc ws[BK][BN + 1];
    const int sign = blockIdx.z;
    const typename P::A *xa = (const typename P::A *)x + (size_t)sign * m_half * k;
    const typename P::W *wt = (const typename P::W *)(sign ? wt_m : wt_p);
    const typename P::W *bias = (const typename P::W *)(sign ? b_m : b_p);
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
    const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
    Acc acc[4][4] = {};
    for (int k0 = 0; k0 < k; k0 += BK) {
        // 64 rows x 16 k = 1024 values per operand, 4 per thread
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int idx = threadIdx.x + 256 * i;
            const int r = idx / BK, kk = idx % BK;
            const bool kin = k0 + kk < k;
            xs[kk][r] = (kin && m0 + r < m_half) ? P::a2acc(xa[(size_t)(m0 + r) * k + k0 + kk]) : (Acc)0;
            ws[kk][r] = (kin && n0 + r < n) ? (Acc)P::w2f(wt[(size_t)(n0 + r) * k + k0 + kk]) : (Acc)0;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < BK; ++kk) {
            Acc a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) { a[i] = xs[kk][ty * 4 + i]; b[i] = ws[kk][tx * 4 + i]; }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] += a[i] * b[j];
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = m0 + ty * 4 + i;
        if (r >= m_half) continue;
        const size_t row = (size_t)sign * m_half + r;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int c = n0 + tx * 4 + j;
            if (c >= n) continue;
            Acc v = acc[i][j];
            if constexpr (EPI != 3) v += (Acc)P::w2f(bias[c]);
            if constexpr (EPI == 0) ((typename P::A *)y)[row * n + c] = P::acc2a(v);
            if constexpr (EPI == 1) ((typename P::A *)y)[row * n + c] = P::acc2a(v > 0 ? v : (Acc)0);
            if constexpr (EPI == 2) ((typename P::R *)y)[row * n + c] += (typename P::R)v;
            if constexpr (EPI == 3) ((Acc *)y)[row * n + c] = v;
        }
    }
}

// ------------------------------------------------------------------ fp64 linear layer on the matrix cores
// The fp32-parameter precision (fp64 activations, fp64 sums).  Its models are tiny, so what a launch costs is the length
// of its dependent chain, not its work: a workgroup owns one 16 TB x 16 TB output tile, its four waves take every fourth
// 16-deep piece of the contraction straight from memory into v_mfma_f64_16x16x4 operands (no LDS slabs, no barrier in
// the loop), and the four partial sums meet once, in LDS, in a fixed order.  In a piece lane group g (16 lanes) holds
// k = 4 g .. 4 g + 3 of its row, which makes every load 16 or 32 contiguous bytes; the four multiplies of a piece take
// element 0, 1, 2, 3 of both operands.  Needs k % 4 == 0 and 16-byte aligned x and weights; other shapes stay on the
// plain kernel.  Both signs of m_half x n x k, plain kernel / here: 64 x 64 x 256 52 / 5.1 us, 64 x 192 x 64 16.6 / 5.0,
// 256 x 128 x 512 100 / 5.3, 512 x 768 x 768 202 / 33, 8192 x 768 x 768 985 / 430 (45 TFLOP/s; what bounds it there is
// L2 traffic, 5.3 flop a byte).
// NP > 0: x is the residual stream and the layer's input its LayerNorm, taken on the way: 16 lanes a row find mean and variance,
// the operands are normalised as they are loaded.  A lane holds its share of the row, NP pieces of 64 elements among the 16, in
// registers, loaded in one burst: read piece by piece, and again for the variance, a row of 320 waits for memory 10 times (9 rows
// a sign, 960 columns, 7.6 us / 7.2 in one burst; two launches take 8.8).  Two pieces where they do, with fewer registers.  Where
// this is taken: norm_on_the_way.
struct NormArgs { const float *g_p, *g_m, *b_p, *b_m; float eps; };
typedef double f64x4 __attribute__((ext_vector_type(4)));
template <int EPI, int TB, int NP>
__global__ __launch_bounds__(256) void linear_f64_mfma_kernel(const double *__restrict__ x, const float *__restrict__ wt_p,
                                                              const float *__restrict__ wt_m, const float *__restrict__ b_p,
                                                              const float *__restrict__ b_m, double *__restrict__ y, int m_half, int n,
                                                              int k, NormArgs norm)
{
    constexpr int BT = 16 * TB;
    constexpr bool NORM = NP > 0;
    __shared__ double part[4][BT][BT + 1];
    const int sign = blockIdx.z;
    const double *xa = x + (size_t)sign * m_half * k;
    const float *wt = sign ? wt_m : wt_p;
    const float *bias = sign ? b_m : b_p;
    const int m0 = blockIdx.y * BT, n0 = blockIdx.x * BT;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4;
    const double *xr[TB];
    const float *wr[TB];
#pragma unroll
    for (int t = 0; t < TB; ++t) {
        const int xi = m0 + 16 * t + r16, wi = n0 + 16 * t + r16;          // clamped: never stored
        xr[t] = xa + (size_t)(xi < m_half ? xi : m_half - 1) * k + 4 * g;
        wr[t] = wt + (size_t)(wi < n ? wi : n - 1) * k + 4 * g;
    }
    double mean[TB], rstd[TB];
    const float *gr = sign ? norm.g_m : norm.g_p, *br = sign ? norm.b_m : norm.b_p;
    if constexpr (NORM) {
        __shared__ double stats[BT][2];
        const int lane16 = threadIdx.x & 15;
        auto sum16 = [](double v) {
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
            return v;
        };
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            const int r = 16 * t + (int)(threadIdx.x >> 4), xi = m0 + r;
            const double *h = xa + (size_t)(xi < m_half ? xi : m_half - 1) * k;
            double2 p[NP][2];
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                if (64 * i >= k) break;
                const int c = 4 * lane16 + 64 * i < k ? 4 * lane16 + 64 * i : k - 4;                     // past the row: not counted
                p[i][0] = *(const double2 *)(h + c);
                p[i][1] = *(const double2 *)(h + c + 2);
            }
            double s = 0.0, v = 0.0;
#pragma unroll
            for (int i = 0; i < NP; ++i)
                if (4 * lane16 + 64 * i < k) s += (p[i][0].x + p[i][0].y) + (p[i][1].x + p[i][1].y);
            const double mu = sum16(s) / (double)k;
            auto square = [&](double q) { v += (q - mu) * (q - mu); };
#pragma unroll
            for (int i = 0; i < NP; ++i)
                if (4 * lane16 + 64 * i < k) {
                    square(p[i][0].x);
                    square(p[i][0].y);
                    square(p[i][1].x);
                    square(p[i][1].y);
                }
            const double var = sum16(v) / (double)k;
            if (lane16 == 0) { stats[r][0] = mu; stats[r][1] = 1.0 / __builtin_sqrt(var + (double)norm.eps); }
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < TB; ++t) { mean[t] = stats[16 * t + r16][0]; rstd[t] = stats[16 * t + r16][1]; }
    }
    f64x4 acc[TB][TB] = {};
#pragma unroll 4
    for (int k0 = 16 * wave; k0 < k; k0 += 64) {
        f64x4 xv[TB], wv[TB];
        const bool in = k0 + 4 * g < k;                                    // k % 4 == 0: a lane's four are all in or all out
        float4 gv = {}, bv = {};
        if constexpr (NORM) {
            if (in) { gv = *(const float4 *)(gr + k0 + 4 * g); bv = *(const float4 *)(br + k0 + 4 * g); }
        }
#pragma unroll
        for (int t = 0; t < TB; ++t) {
            const double2 a = in ? *(const double2 *)(xr[t] + k0) : double2{0.0, 0.0};
            const double2 b = in ? *(const double2 *)(xr[t] + k0 + 2) : double2{0.0, 0.0};
            const float4 w = in ? *(const float4 *)(wr[t] + k0) : float4{0.0f, 0.0f, 0.0f, 0.0f};
            xv[t] = f64x4{a.x, a.y, b.x, b.y};
            if constexpr (NORM) {
                xv[t] = f64x4{(a.x - mean[t]) * rstd[t] * (double)gv.x + (double)bv.x, (a.y - mean[t]) * rstd[t] * (double)gv.y + (double)bv.y,
                              (b.x - mean[t]) * rstd[t] * (double)gv.z + (double)bv.z, (b.y - mean[t]) * rstd[t] * (double)gv.w + (double)bv.w};
                if (!in) xv[t] = f64x4{0.0, 0.0, 0.0, 0.0};                // (weights are zero there: a row that is not finite stays out of it)
            }
            wv[t] = f64x4{(double)w.x, (double)w.y, (double)w.z, (double)w.w};
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < TB; ++i)
#pragma unroll
                for (int j = 0; j < TB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(xv[i][e], wv[j][e], acc[i][j], 0, 0, 0);
    }
    // element e of a lane's result: row 4 e + lane / 16, column lane % 16 of the 16 x 16 block
#pragma unroll
    for (int i = 0; i < TB; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) part[wave][16 * i + 4 * e + g][16 * j + r16] = acc[i][j][e];
    __syncthreads();
#pragma unroll
    for (int o = threadIdx.x; o < BT * BT; o += 256) {
        const int r = o / BT, c = o % BT;
        if (m0 + r >= m_half || n0 + c >= n) continue;
        double v = (part[0][r][c] + part[1][r][c]) + (part[2][r][c] + part[3][r][c]);
        if constexpr (EPI != 3) v += (double)bias[n0 + c];
        if constexpr (EPI == 1) v = v > 0.0 ? v : 0.0;
        double *p = y + ((size_t)sign * m_half + m0 + r) * n + n0 + c;
        if constexpr (EPI == 2) v += *p;
        *p = v;
    }
}

// ------------------------------------------------------------------ plain causal attention
// One workgroup per (query row, head, sequence): scores into LDS, softmax, then P V.
template <int DT>
__global__ __launch_bounds__(128) void attention_plain_kernel(const void *qkv_, void *out_, int seq, int n_heads,
                                                              int d_head, int groups)
{
    using P = Prec<DT>;
    using Acc = typename P::Acc;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    Acc *sc = (Acc *)smem_raw;          // [seq]
    Acc *qs = sc + seq;                 // [d_head]
    Acc *red = qs + d_head;             // [16]
    const int t = blockIdx.x, head = blockIdx.y, sq = blockIdx.z;
    const int d = n_heads * d_head;
    const typename P::A *qkv = (const typename P::A *)qkv_ + (size_t)sq * seq * 3 * d;
    const typename P::A *q = qkv + (size_t)t * 3 * d + head * d_head;
    for (int c = threadIdx.x; c < d_head; c += blockDim.x) qs[c] = P::a2acc(q[c]);
    __syncthreads();
    Acc scale;
    if constexpr (sizeof(Acc) == 8) scale = 1.0 / __builtin_sqrt((double)d_head);
    else scale = 1.0f / __builtin_sqrtf((float)d_head);
    Acc mx = -INFINITY;
    for (int j = threadIdx.x; j <= t; j += blockDim.x) {
        const typename P::A *kr = qkv + (size_t)j * 3 * d + d + head * d_head;
        Acc s = 0;
        for (int c = 0; c < d_head; ++c) s += qs[c] * P::a2acc(kr[c]);
        s *= scale;
        sc[j] = s;
        mx = s > mx ? s : mx;
    }
    mx = block_max(mx, red);
    Acc sum = 0;
    for (int j = threadIdx.x; j <= t; j += blockDim.x) {
        Acc e;
        if constexpr (sizeof(Acc) == 8) e = exp(sc[j] - mx); else e = __expf(sc[j] - mx);
        sc[j] = e;
        sum += e;
    }
    sum = block_sum(sum, red);
    __syncthreads();
    typename P::A *o = (typename P::A *)out_ + ((size_t)sq * seq + t) * d + head * d_head;
    const typename P::A *vr = qkv + 2 * d + head * d_head;
    // small heads: the keys are dealt to groups of d_head threads (plain_attention_groups)
    if (groups == 1) {
        for (int c = threadIdx.x; c < d_head; c += blockDim.x) {
            Acc a = 0;
            for (int j = 0; j <= t; ++j) a += sc[j] * P::a2acc(vr[(size_t)j * 3 * d + c]);
            o[c] = P::acc2a(a / sum);
        }
        return;
    }
    Acc *part = red + 16;               // [blockDim.x]
    const int c = (int)threadIdx.x % d_head, grp = (int)threadIdx.x / d_head;
    Acc a = 0;
    if (grp < groups)
        for (int j = grp; j <= t; j += groups) a += sc[j] * P::a2acc(vr[(size_t)j * 3 * d + c]);
    part[threadIdx.x] = a;
    __syncthreads();
    if (grp != 0) return;
    for (int i = 1; i < groups; ++i) a += part[i * d_head + c];
    o[c] = P::acc2a(a / sum);
}

// ------------------------------------------------------------------ cross entropy over stored logits
// row_loss[r] = logsumexp(logits[r, :]) - logits[r, target[r]]; 0 for target -1, NaN for -2.
template <typename Acc>
__global__ __launch_bounds__(256) void ce_rows_kernel(const Acc *__restrict__ logits, const int32_t *__restrict__ target,
                                                      double *__restrict__ row_loss, int vocab)
{
    __shared__ double red[16];
    const int r = blockIdx.x;
    const int tg = target[r];
    if (tg == -1) { if (threadIdx.x == 0) row_loss[r] = 0.0; return; }
    const Acc *lg = logits + (size_t)r * vocab;
    double mx = -INFINITY;
    for (int c = threadIdx.x; c < vocab; c += blockDim.x) { const double v = (double)lg[c]; mx = v > mx ? v : mx; }
    mx = block_max(mx, red);
    double s = 0;
    for (int c = threadIdx.x; c < vocab; c += blockDim.x) s += exp((double)lg[c] - mx);
    s = block_sum(s, red);
    if (threadIdx.x == 0) row_loss[r] = tg >= 0 ? (log(s) + mx - (double)lg[tg]) : (double)__builtin_nan("");
}

// Merge the (max, sum-exp) pairs the fused LM-head epilogue left for a row: one wavefront per row.
template <int KEEP>
__global__ __launch_bounds__(256) void ce_finish_kernel(const float2 *__restrict__ partials, int n_partial,
                                                        const float *__restrict__ target_logit,
                                                        const int32_t *__restrict__ target, double *__restrict__ row_loss,
                                                        int rows)
{
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (r >= rows) return;
    const int tg = target[r];
    if (tg == -1) { if (lane == 0) row_loss[r] = 0.0; return; }
    const float2 *p = partials + (size_t)r * n_partial;
    // A lane keeps its first KEEP pairs (8: 512 a row, 65536 columns in strips of 128, 32768 in strips of 64) in registers, so that
    // they are read once and all loads are under way together; what lies beyond is read again for the sum.  us, read twice / here:
    // 4192 rows of 394 pairs 7.8 / 7.1, 16352 rows 22.8 / 19.2 (the exponentials in 64 bits are most of it).  Each kept pair has an
    // exponential's code of its own, which short rows pay for without use (128 rows of 64 pairs, read twice / 2 / 4 / 8 kept: 3.24 /
    // 3.12 / 3.27 / 3.55; of 250 4.18 / 4.09 / 3.93 / 4.18): 2 up to 128 pairs, 4 up to 256.
    float2 v[KEEP];
#pragma unroll
    for (int i = 0; i < KEEP; ++i) v[i] = lane + 64 * i < n_partial ? p[lane + 64 * i] : float2{-INFINITY, 0.0f};
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < KEEP; ++i) mx = v[i].x > mx ? v[i].x : mx;
    for (int i = lane + 64 * KEEP; i < n_partial; i += 64) mx = p[i].x > mx ? p[i].x : mx;
    mx = wave_max(mx);
    double s = 0.0;
    auto add = [&](float2 q) {
        if (q.x > -INFINITY) s += (double)q.y * exp((double)q.x - (double)mx);
    };
#pragma unroll
    for (int i = 0; i < KEEP; ++i)
        if (64 * i < n_partial) add(v[i]);
    for (int i = lane + 64 * KEEP; i < n_partial; i += 64) add(p[i]);
    s = wave_sum(s);
    if (lane == 0) row_loss[r] = tg >= 0 ? (log(s) + (double)mx - (double)target_logit[r]) : (double)__builtin_nan("");
}

// Eq. 1 and the scalar of Eq. 2: g = (l+ - l-) / (2 eps), s = -(lr g) rounded once to fp32.
__device__ __forceinline__ void g_and_scalar(double lp, double lm, const GScalar &gs)
{
    const double g = (lp - lm) / (2.0 * (double)gs.eps);
    float s = (float)(-((double)gs.lr * g));
    if (!(g == g) || g - g != 0.0) { s = 0.0f; atomicOr(gs.flags, 1u); }
    *gs.g = g;
    *gs.s = s;
    if (gs.result) { gs.result[0] = lp; gs.result[1] = lm; gs.result[2] = g; }
}

// L+- = sum of the sign's row losses / count, in a fixed order (deterministic); 512 threads per sign.  One workgroup for
// both signs, so that g can follow in the same launch: a launch of its own costs 4.5 us for one thread's work.
__global__ __launch_bounds__(1024) void loss_reduce_kernel(const double *__restrict__ row_loss, int n_sign, int m_half, int count,
                                                           double *__restrict__ loss_pm, bool with_g, GScalar gs)
{
    __shared__ double red[16];
    const int sign = threadIdx.x >> 9, t = threadIdx.x & 511;
    double s = 0;
    if (sign < n_sign) {
        const double *r = row_loss + (size_t)sign * m_half;
        for (int i = t; i < m_half; i += 512) s += r[i];
    }
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x != 0) return;
    double l[2] = {0.0, 0.0};
    for (int k = 0; k < n_sign; ++k) {
        for (int w = 0; w < 8; ++w) l[k] += red[8 * k + w];
        l[k] /= (double)count;
        loss_pm[k] = l[k];
    }
    if (with_g) g_and_scalar(l[0], l[1], gs);
}

__global__ void g_scalar_kernel(const double *loss_pm, GScalar gs) { g_and_scalar(loss_pm[0], loss_pm[1], gs); }

// ------------------------------------------------------------------ launchers
#define ZO_DISPATCH_DT(dtype, CALL)                  \
    switch (dtype) {                                 \
    case kFP32: { constexpr int DT = kFP32; CALL; } break; \
    case kBF16: { constexpr int DT = kBF16; CALL; } break; \
    case kFP16: { constexpr int DT = kFP16; CALL; } break; \
    default: return hipErrorInvalidValue;            \
    }

hipError_t launch_embed(const int32_t *tokens, const void *e_p, const void *e_m, const void *pos_p, const void *pos_m,
                        void *resid, int32_t *target, uint32_t *flags, int dtype, int n_sign, int batch, int seq, int d,
                        int vocab, hipStream_t s)
{
    const int rows = n_sign * batch * seq;
    if (d % 4 != 0) return hipErrorInvalidValue;
    const dim3 grid((rows + 3) / 4), block(256);
    ZO_DISPATCH_DT(dtype, (embed_kernel<DT><<<grid, block, 0, s>>>(tokens, e_p, e_m, pos_p, pos_m, resid, target, flags, batch, seq, d, vocab, rows)));
    return hipGetLastError();
}

hipError_t launch_layernorm(const void *resid, const void *g_p, const void *g_m, const void *b_p, const void *b_m,
                            void *y, int dtype, int n_sign, int m_half, int d, float eps, hipStream_t s)
{
    const int rows = n_sign * m_half;
    if (dtype != kFP32 && d % 4 == 0 && d <= 12288) {
        const dim3 wgrid((rows + 3) / 4), wblock(256);
#define ZO_LNW(DT, NV)                                                                                                        \
    layernorm_wave_kernel<DT, NV><<<wgrid, wblock, 0, s>>>((const float *)resid, (const uint16_t *)g_p, (const uint16_t *)g_m, \
                                                           (const uint16_t *)b_p, (const uint16_t *)b_m, (uint16_t *)y, rows,   \
                                                           m_half, d, eps)
#define ZO_LNB(DT, NV)                                                                                                        \
    layernorm_block_kernel<DT, NV><<<dim3(rows), dim3(256), 0, s>>>((const float *)resid, (const uint16_t *)g_p,              \
                                                                    (const uint16_t *)g_m, (const uint16_t *)b_p,             \
                                                                    (const uint16_t *)b_m, (uint16_t *)y, m_half, d, eps)
#define ZO_LNW_D(DT)                          \
    switch (layernorm_pieces(d)) {            \
    case 3: ZO_LNW(DT, 3); break;             \
    case 4: ZO_LNW(DT, 4); break;             \
    case 5: ZO_LNW(DT, 5); break;             \
    case 6: ZO_LNW(DT, 6); break;             \
    case 7: ZO_LNW(DT, 7); break;             \
    case 8: ZO_LNW(DT, 8); break;             \
    default:                                  \
        if (d <= 4096) ZO_LNB(DT, 4);         \
        else if (d <= 5120) ZO_LNB(DT, 5);    \
        else if (d <= 8192) ZO_LNB(DT, 8);    \
        else ZO_LNB(DT, 12);                  \
    }
        if (dtype == kBF16) { ZO_LNW_D(kBF16) } else { ZO_LNW_D(kFP16) }
#undef ZO_LNB
#undef ZO_LNW_D
#undef ZO_LNW
        return hipGetLastError();
    }
    const dim3 grid(rows), block(256);
    ZO_DISPATCH_DT(dtype, (layernorm_kernel<DT><<<grid, block, 0, s>>>(resid, g_p, g_m, b_p, b_m, y, m_half, d, eps)));
    return hipGetLastError();
}

template <int DT>
static void linear_plain_launch(const void *x, const void *wt_p, const void *wt_m, const void *b_p, const void *b_m,
                                void *y, int n_sign, int m_half, int n, int k, int epi, hipStream_t s)
{
    const dim3 grid((n + 63) / 64, (m_half + 63) / 64, n_sign), block(256);
    switch (epi) {
    case 0: linear_plain_kernel<DT, 0><<<grid, block, 0, s>>>(x, wt_p, wt_m, b_p, b_m, y, m_half, n, k); break;
    case 1: linear_plain_kernel<DT, 1><<<grid, block, 0, s>>>(x, wt_p, wt_m, b_p, b_m, y, m_half, n, k); break;
    case 2: linear_plain_kernel<DT, 2><<<grid, block, 0, s>>>(x, wt_p, wt_m, b_p, b_m, y, m_half, n, k); break;
    default: linear_plain_kernel<DT, 3><<<grid, block, 0, s>>>(x, wt_p, wt_m, b_p, b_m, y, m_half, n, k); break;
    }
}

template <int TB, int NP>
static void linear_f64_launch(const void *x, const void *wt_p, const void *wt_m, const void *b_p, const void *b_m, void *y, int n_sign,
                              int m_half, int n, int k, int epi, const NormArgs &norm, hipStream_t s)
{
    const dim3 grid((n + 16 * TB - 1) / (16 * TB), (m_half + 16 * TB - 1) / (16 * TB), n_sign), block(256);
#define ZO_F64(E)                                                                                                       \
    linear_f64_mfma_kernel<E, TB, NP><<<grid, block, 0, s>>>((const double *)x, (const float *)wt_p, (const float *)wt_m,   \
                                                             (const float *)b_p, (const float *)b_m, (double *)y, m_half, n, k, norm)
    switch (epi) {
    case 0: ZO_F64(0); break;
    case 1: ZO_F64(1); break;
    case 2: if constexpr (NP == 0) ZO_F64(2); break;
    default: ZO_F64(3); break;
    }
#undef ZO_F64
}

bool norm_linear_fused(const void *resid, const void *g_p, const void *g_m, const void *lb_p, const void *lb_m, const void *wt_p,
                       const void *wt_m, int dtype, int n_sign, int m_half, int n, int k)
{
    auto off = [](const void *p) { return (uintptr_t)p % 16 != 0; };
    return dtype == kFP32 && k % 4 == 0 && norm_on_the_way(n_sign, m_half, n, k) && !off(resid) && !off(g_p) && !off(g_m) && !off(lb_p) &&
           !off(lb_m) && !off(wt_p) && !off(wt_m);
}

hipError_t launch_norm_linear(const void *resid, const void *g_p, const void *g_m, const void *lb_p, const void *lb_m, float eps,
                              const void *wt_p, const void *wt_m, const void *b_p, const void *b_m, void *y, int n_sign,
                              int m_half, int n, int k, int epilogue, hipStream_t s)
{
    if ((epilogue != 0 && epilogue != 1 && epilogue != 3) || k > kNormRowMax || k % 4 != 0) return hipErrorInvalidValue;
    const NormArgs norm{(const float *)g_p, (const float *)g_m, (const float *)lb_p, (const float *)lb_m, eps};
    if (k <= kNormRowShort) linear_f64_launch<1, kNormRowShort / 64>(resid, wt_p, wt_m, b_p, b_m, y, n_sign, m_half, n, k, epilogue, norm, s);
    else linear_f64_launch<1, kNormRowMax / 64>(resid, wt_p, wt_m, b_p, b_m, y, n_sign, m_half, n, k, epilogue, norm, s);
    return hipGetLastError();
}

hipError_t launch_linear(const void *x, const void *wt_p, const void *wt_m, const void *b_p, const void *b_m, void *y,
                         int dtype, int n_sign, int m_half, int n, int k, int epilogue, bool allow_mfma, hipStream_t s)
{
    if (allow_mfma && dtype != kFP32 && mfma_linear_supported(m_half, n, k))
        return launch_linear_mfma(x, wt_p, wt_m, b_p, b_m, y, dtype, n_sign, m_half, n, k, epilogue, s);
    if (dtype == kFP32 && k % 4 == 0 && (uintptr_t)x % 16 == 0 && (uintptr_t)wt_p % 16 == 0 && (uintptr_t)wt_m % 16 == 0) {
        if (f64_tiles32(n_sign, m_half, n)) linear_f64_launch<2, 0>(x, wt_p, wt_m, b_p, b_m, y, n_sign, m_half, n, k, epilogue, NormArgs{}, s);
        else linear_f64_launch<1, 0>(x, wt_p, wt_m, b_p, b_m, y, n_sign, m_half, n, k, epilogue, NormArgs{}, s);
        return hipGetLastError();
    }
    ZO_DISPATCH_DT(dtype, (linear_plain_launch<DT>(x, wt_p, wt_m, b_p, b_m, y, n_sign, m_half, n, k, epilogue, s)));
    return hipGetLastError();
}

hipError_t launch_attention(const void *qkv, void *out, int dtype, int n_seq, int seq, int n_heads, int d_head,
                            bool allow_mfma, hipStream_t s)
{
    // the matrix path reads and writes in pieces of 16 bytes
    const bool aligned = (uintptr_t)qkv % 16 == 0 && (uintptr_t)out % 16 == 0;
    // Sequences of one to four tokens with heads of 80 to 112 channels: an item of the matrix path is 128 query rows whatever the
    // length, and 512 are in flight; once they take a second round the plain kernel, one block a token, is done first, up to
    // 3 tokens or 2048 items.  bf16, heads of 80 channels, us plain / matrix: 1024 items of 1 token 5.8 / 8.4, 2 tokens 6.1 / 8.3,
    // 3 tokens 7.2 / 8.6, 4 tokens 8.0 / 8.5; 8192 items 14 / 51, 24 / 51, 42 / 52, 57 / 53; 512 items 5.2 / 5.5, 5.9 / 5.6,
    // 6.2 / 5.7, 6.3 / 5.7.  112 channels, 1024 items: 6.5 / 9.2, 6.7 / 9.2, 7.7 / 9.2, 8.6 / 9.7.
    const long items = (long)n_seq * n_heads;
    const bool tiny = d_head != 64 && d_head != 128 && items >= (seq == 1 ? 512 : 513) && (seq <= 3 || (seq == 4 && items <= 2048));
    if (allow_mfma && dtype != kFP32 && aligned && !tiny && mfma_attention_supported(seq, n_heads, d_head))
        return launch_attention_mfma(qkv, out, dtype, n_seq, seq, n_heads, d_head, s);
    const dim3 grid(seq, n_heads, n_seq), block(128);
    size_t smem = (size_t)(seq + d_head + 16) * acc_bytes(dtype);
    // (lengths near the LDS limit stay with one group)
    const int groups = plain_attention_groups(seq, d_head, smem + block.x * acc_bytes(dtype) <= 32768);
    if (groups > 1) smem += block.x * acc_bytes(dtype);
    ZO_DISPATCH_DT(dtype, (attention_plain_kernel<DT><<<grid, block, smem, s>>>(qkv, out, seq, n_heads, d_head, groups)));
    return hipGetLastError();
}

hipError_t launch_ce_rows(const void *logits, const int32_t *target, double *row_loss, int dtype, int rows, int vocab,
                          hipStream_t s)
{
    if (rows == 0) return hipSuccess;
    if (dtype == kFP32) ce_rows_kernel<double><<<dim3(rows), dim3(256), 0, s>>>((const double *)logits, target, row_loss, vocab);
    else ce_rows_kernel<float><<<dim3(rows), dim3(256), 0, s>>>((const float *)logits, target, row_loss, vocab);
    return hipGetLastError();
}

hipError_t launch_ce_finish(const void *partials, int n_partial, const float *target_logit, const int32_t *target,
                            double *row_loss, int rows, hipStream_t s)
{
    if (rows == 0) return hipSuccess;
#define ZO_CE(KEEP) \
    ce_finish_kernel<KEEP><<<dim3((rows + 3) / 4), dim3(256), 0, s>>>((const float2 *)partials, n_partial, target_logit, target, row_loss, rows)
    if (n_partial <= 128) ZO_CE(2);
    else if (n_partial <= 256) ZO_CE(4);
    else ZO_CE(8);
#undef ZO_CE
    return hipGetLastError();
}

hipError_t launch_loss_reduce(const double *row_loss, int n_sign, int m_half, int count_per_sign, double *loss_pm,
                              const GScalar *gs, hipStream_t s)
{
    if (n_sign < 1 || n_sign > 2 || (gs && n_sign != 2)) return hipErrorInvalidValue;
    loss_reduce_kernel<<<dim3(1), dim3(1024), 0, s>>>(row_loss, n_sign, m_half, count_per_sign, loss_pm, gs != nullptr, gs ? *gs : GScalar{});
    return hipGetLastError();
}

hipError_t launch_g_scalar(const double *loss_pm, const GScalar &gs, hipStream_t s)
{
    g_scalar_kernel<<<dim3(1), dim3(1), 0, s>>>(loss_pm, gs);
    return hipGetLastError();
}

}  // namespace zo
