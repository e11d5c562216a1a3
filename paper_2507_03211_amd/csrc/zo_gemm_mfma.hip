// Sign-batched linear layer on the matrix cores (bf16 / fp16 inputs, fp32 accumulate).
//
// This is where a ZO step spends its time: the paired forward passes of Eq. 1 (DistZO2,
// Preliminaries; PertP workflow Step 2 runs the two signs on two devices, here both signs are
// one launch on one device, rows [0, m_half) against W+ and rows [m_half, 2 m_half) against W-).
//
//   y[row, n] = sum_k x[row, k] wt[n, k]  (+ bias, ReLU, residual add)
//
// Both operands are K-contiguous ("TN"), which is what v_mfma_f32_32x32x16_{bf16,f16} wants:
// every lane feeds 8 consecutive k of one row.  The weight tile is the MFMA A operand and the
// activation tile the B operand, so a lane's 16 accumulators are 4 runs of 4 consecutive n of
// one output row, which makes the epilogue 8/16-byte stores.
//
// Three kernels (K a multiple of 64; others take the plain kernel):
//  * linear_mfma_pipe_kernel, for K of some slabs and more: one persistent workgroup of 2 x 2 waves per CU that walks its
//    XCD's share of the tile list, tiles of 256 x 256 down to 128 x 128 with slabs of 64 k.  Operand tiles go from global
//    memory straight into LDS (global_load_lds_dwordx4, no register staging), whole 128-byte lines per tile row, several
//    slabs ahead, and the pipeline runs on from one tile into the next.  16-byte chunks are XOR-swizzled on the global
//    side so that fragment reads are free of bank conflicts.  Tiles are numbered so that each XCD (its own L2) owns a
//    contiguous band of 8 tile-rows and walks it column by column.  Outputs leave through LDS as whole rows.
//  * linear_mfma_small_kernel, 64 x 64 tiles, one workgroup per tile and two or more of them per CU: any number of slabs,
//    and shapes so small that what counts is how many CUs take part.
//  * linear_mfma_split_kernel, 32 x 32 tiles whose waves share the contraction: shapes so small that each tile has a CU of its own.
// pick_tile() at the end chooses between the tile shapes.
#include "zo_device_once.h"
#include "zo_kernels.h"
#include "zo_types.hip.h"

namespace zo {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // native vector: arrays of it stay in registers
typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int BK = 64;                      // contraction slab; k is a multiple of it
constexpr int kMaxColumns = 1 << 24;        // 16 fp32 rows within 2^30 bytes: what an epilogue pass addresses with 32 bits

template <int DT> __device__ __forceinline__ f32x16 mfma32(const uint4 &a, const uint4 &b, const f32x16 &c)
{
    if constexpr (DT == kBF16)
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}


// Epilogue 4 (tied LM head fused with the cross-entropy reduction): nothing of the logits is stored.  A lane
// holds TN * 16 logits of one row (4 runs of 4 consecutive columns per MFMA tile); it reduces them to a
// (maximum, sum of exp) pair, merges with the other lane half (the remaining columns of the wave's range)
// and the wave writes one pair per row and per wave-column-range; the lane that holds the target column
// stores that logit.  A last small kernel merges the pairs of a row into logsumexp - target logit.
// Argument reuse for this epilogue: bias_p -> int32 target[rows], bias_m -> float target_logit[rows],
// y -> float2 partial[rows][n_partial].
template <int TN>
__device__ __forceinline__ void ce_partial_row(const f32x16 (&a)[TN], int col0, int fh, int n, bool live, int tg,
                                               float *tgt_logit_row, float2 *partial_slot)
{
    // `live` false: a row past the ragged end of the tile.  It takes part (the two halves of the wave exchange their
    // results below) and stores nothing; its pointers are those of the last valid row.
    //
    // A lane's 16 TN logits in register order k = 16 tn + i sit at columns col0 + 32 tn + 8 (i / 4) + 4 fh + i % 4,
    // which grow with k.  Nothing here keeps one compare result per element alive (64 of them, the same for every
    // row block, is what the compiler would hoist and then spill): the ragged strip of the vocabulary is masked by
    // arithmetic, the target logit is picked by a tree of selects on the bits of its register number.
    constexpr int NE = 16 * TN;
    float v[NE];
#pragma unroll
    for (int k = 0; k < NE; ++k) v[k] = a[k / 16][k % 16];
    if (col0 + 32 * TN > n) {                      // wave-uniform: only the last strip of the vocabulary
        // number of this lane's registers that lie inside the vocabulary
        int kmax = 0;
#pragma unroll
        for (int g = 0; g < 4 * TN; ++g) {         // runs of 4 columns: col0 + 32 (g / 4) + 8 (g % 4) + 4 fh + 0..3
            const int c0 = col0 + 32 * (g / 4) + 8 * (g % 4) + 4 * fh, left = n - c0;
            kmax += left < 0 ? 0 : left > 4 ? 4 : left;
        }
        const float kf = (float)kmax - 0.5f;
#pragma unroll
        for (int k = 0; k < NE; ++k) {
            // (kf - k) * inf is +inf for registers inside, -inf outside (never 0 * inf); min(., 0) makes it 0 or -inf
            const float pen = __builtin_fminf((kf - (float)k) * INFINITY, 0.0f);
            v[k] += pen;
        }
    }
    // (two maxima and four sums side by side: with one wave per SIMD an instruction that waits for the one before it issues
    // after 8 cycles instead of 5, and 64 additions in a row are half of such waits.  With the row targets loaded together, see
    // the caller: LM head of 50272 columns, us before / here: 8176 rows a sign, d 768, 1048 / 1022; 1048 rows, d 2048, 389 / 384)
    float mx2[2] = {v[0], v[1]};
#pragma unroll
    for (int k = 2; k < NE; k += 4) {
        mx2[0] = __builtin_fmaxf(__builtin_fmaxf(v[k], v[k + 1]), mx2[0]);
        if (k + 2 < NE) mx2[1] = __builtin_fmaxf(__builtin_fmaxf(v[k + 2], v[k + 3]), mx2[1]);
    }
    const float mx = __builtin_fmaxf(mx2[0], mx2[1]);
    // exp(v - mx) as 2^(v L - c), c = rn(mx L): one fma and one exponential per logit, where subtracting first and scaling
    // then takes one instruction more of some six.  c's rounding is taken out of the sum again (the fma that finds it is
    // exact), so that the pair belongs to mx itself.  That holds while 2^(c's rounding) is an fp32 number: up to |mx| = 2^30
    // half a unit of c is at most 64.  Beyond, two logits are equal or at least 64 apart, where an exponential to any base
    // from 2 up is lost in the sum, and base 2 needs no scale: c = mx, differences exact.
    // LM head of 50272 columns, before -> after in us: 8176 rows a sign, d 768, 1071 -> 1056; 2048 rows 286 -> 279; 1048
    // rows, d 2048, 391 -> 387.  Error against fp64 unchanged (rms 2.6e-7 at logits of about 1, 3.4e-6 at 8).
    const float ms = mx > -INFINITY ? mx : 0.0f;      // a strip that lies wholly past the vocabulary: 2^(-inf - 0) = 0
    const float L = __builtin_fabsf(ms) > 0x1p30f ? 1.0f : 1.44269504f, c = ms * L;
    float sum4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < NE; ++k) sum4[k & 3] += __builtin_amdgcn_exp2f(__builtin_fmaf(v[k], L, -c));
    float sum = (sum4[0] + sum4[1]) + (sum4[2] + sum4[3]);
    sum *= __builtin_amdgcn_exp2f(-__builtin_fmaf(ms, L, -c));
    // the target column, if it is one of this lane's: register 16 (rel / 32) + 4 (rel / 8 % 4) + rel % 4 of the lane
    // half rel / 4 % 2
    const int rel = tg - col0;
    const bool mine = rel >= 0 && rel < 32 * TN && ((rel >> 2) & 1) == fh;
    const int which = (rel >> 5) * 16 + ((rel >> 3) & 3) * 4 + (rel & 3);
    if (__builtin_amdgcn_ballot_w64(mine) != 0) {        // of 50272 columns a wave holds 128: one wave in twelve
        float t[NE];
#pragma unroll
        for (int k = 0; k < NE; ++k) t[k] = v[k];
#pragma unroll
        for (int bit = 0, cnt = NE; cnt > 1; ++bit, cnt >>= 1) {
            const bool odd = (which >> bit) & 1;
#pragma unroll
            for (int k = 0; k < cnt / 2; ++k) t[k] = odd ? t[2 * k + 1] : t[2 * k];
        }
        if (live && mine) *tgt_logit_row = t[0];
    }
    const float mo = __shfl_xor(mx, 32, 64), so = __shfl_xor(sum, 32, 64);
    const float m2 = mx > mo ? mx : mo;
    const float s2 = (mx > -INFINITY ? sum * __expf(mx - m2) : 0.0f) + (mo > -INFINITY ? so * __expf(mo - m2) : 0.0f);
    if (live && fh == 0) *partial_slot = float2{m2, s2};
}

constexpr int kGroupM = 8;                      // tile-rows per band

// 16 bytes per lane from global memory straight into LDS: lane L lands at lds_off + 16 L.
// Issued from asm so that the waits are ours: the compiler would otherwise drain every
// outstanding load before the next LDS read, which defeats the overlap.
// The address is a wave-uniform 64-bit base (scalar registers: the k advance of the pipeline costs no vector
// instruction) plus a 32-bit per-lane byte offset that stays the same for the whole tile.
__device__ __forceinline__ void gload_lds16(uint64_t base, uint32_t lane_off, uint32_t lds_off)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_off), "s"(base), "s"(lds_off) : "memory", "m0");
}
__device__ __forceinline__ uint64_t uniform64(uint64_t v)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Tile `lin` of the list -> sign, first row, tile column.  The list runs through the signs, in each through bands of 8
// tile-rows, in a band column by column: what an XCD works on at one time shares operand slabs in its L2, and a band
// never mixes the two signs, which share no weights.
__device__ __forceinline__ void tile_at(int lin, int tiles_m, int tiles_n, int &sign, int &trow, int &tcol)
{
    const int per_sign = tiles_m * tiles_n;
    sign = lin / per_sign;
    const int in_sign = lin % per_sign, band = in_sign / (kGroupM * tiles_n), rem = in_sign % (kGroupM * tiles_n);
    const int band_rows = tiles_m - band * kGroupM < kGroupM ? tiles_m - band * kGroupM : kGroupM;
    trow = band * kGroupM + rem % band_rows;
    tcol = rem / band_rows;
}

// Epilogues 0 - 3 of a wave's 32 TM x 32 TN outputs (rows m0 + wm 32 TM .., columns n0 + wn 32 TN .. of sign `sign`).
// `stage`: kTileStageBytes<TN> bytes of LDS that are this wave's alone.  NT: non-temporal accesses (see launch_small).
template <int TN> constexpr int kTileStageBytes = (TN & (TN - 1)) ? 2048 * TN + 512 : 2048 * TN;
template <int DT, int EPI, int TM, int TN, bool NT>
__device__ __forceinline__ void store_tile(const f32x16 (&acc)[TN][TM], char *stage, const uint16_t *__restrict__ bias, void *__restrict__ y,
                                           int sign, int m_half, int n, int m0, int n0, int wm, int wn, int lane)
{
    const int fr = lane & 31, fh = lane >> 5;
    // Output through LDS so that global stores are whole rows: in the MFMA layout a lane holds runs of 4
    // consecutive columns of ONE row and a wave instruction would touch 32 rows with 16 or 32 bytes each.
    // A wave stages 2 KiB x TN at a time (32 rows of two-byte columns, or 16 rows of fp32).  No workgroup barrier.  Rows whose
    // length is a power of two are XOR-swizzled by the row: the run-wise writes and the row-wise 16-byte reads are free of
    // bank conflicts (16-bit rows of one tile apart, see chunk16 below).  Others have 16 bytes of padding, which leaves two
    // lanes per bank in the writes (15 % of the LDS cycles of a 12-slab launch of 256 x 192 tiles).
    constexpr bool kOut16 = (EPI == 0 || EPI == 1);              // 2-byte outputs; else fp32
    constexpr int RP = kOut16 ? 32 : 16;                         // rows per pass
    constexpr int NPASS = 32 * TM / RP;
    constexpr int RB = (kOut16 ? 64 : 128) * TN;                 // bytes per row
    constexpr bool kXor = (TN & (TN - 1)) == 0;
    constexpr int PITCH = kXor ? RB : RB + 16;
    constexpr int NRUN = 8 * TN, LPR = RB / 16;                  // runs of 4 columns, 16-byte pieces per row
    constexpr int NIO = RP * LPR / 64;                           // pieces per lane and pass
    static_assert(RP * PITCH <= kTileStageBytes<TN>, "a pass fits the wave's staging area");
    const int ncol0 = n0 + wn * 32 * TN;
    // Bias: 2-byte outputs take it before the rounding, so per run of the MFMA layout (the same 16 runs
    // for every row block); fp32 outputs take it after the LDS pass, where a lane always holds the same
    // 4 columns.
    // They come through the scalar cache (a wave-uniform address in the constant address space: 16 bytes
    // = the 8 columns of a run pair, of which the lane half keeps its 4): a vector load here would make
    // the compiler wait for every outstanding vector memory operation, the next tile's loads included.
    float bvals[kOut16 ? TN : 1][4][4];
    if constexpr (kOut16) {
        typedef const __attribute__((address_space(4))) u32x4 *cptr;
        const uint64_t bbase = uniform64((uint64_t)(uintptr_t)bias);
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                int c8 = ncol0 + tn * 32 + 8 * g;               // wave-uniform; clamped: columns >= n are never stored
                c8 = c8 + 8 <= n ? c8 : n - 8;
                const u32x4 raw = *(cptr)(uintptr_t)(bbase + 2u * (uint32_t)c8);
                const uint32_t lo = fh ? raw.z : raw.x, hi = fh ? raw.w : raw.y;
                bvals[tn][g][0] = Prec<DT>::w2f((uint16_t)(lo & 0xffff));
                bvals[tn][g][1] = Prec<DT>::w2f((uint16_t)(lo >> 16));
                bvals[tn][g][2] = Prec<DT>::w2f((uint16_t)(hi & 0xffff));
                bvals[tn][g][3] = Prec<DT>::w2f((uint16_t)(hi >> 16));
            }
    }
    // Addresses: a wave-uniform base for the pass (scalar registers) plus a per-lane offset that is worked out once.  With a
    // 64-bit address and both bounds worked out per row the epilogue was 1650 (16-bit outputs) / 2980 (residual)
    // instructions per wave and 256 x 256 tile instead of 1390 / 2150.
    // 16-bit outputs: a row mask of one compare with a constant.  fp32: buffer accesses, which drop (or read as zero) what
    // lies past the pass's last row, and lanes whose columns lie past the end point behind any buffer.  With a branch
    // around each piece the compiler cannot count what is under way and lets every piece of the residual epilogue wait for
    // all memory operations before it, the stores of the piece before included: us, m_half x n x k, code with both bounds
    // per row / branches / here, residual: 8192 x 4096 x 1024 184 / 188 / 175, 2794 x 16304 x 512 193 / 205 / 185, 8192 x
    // 5120 x 5120 670 / 680 / 656.  (16-bit outputs wait for nothing here; as buffer stores they were up to 6 % slower.)
    constexpr int ES = kOut16 ? 2 : 4;
    constexpr int NBV = 64 % LPR == 0 ? 1 : 3;                   // a lane's column and row step repeat after this many pieces
    constexpr int RSTEP = 64 * NBV / LPR;                        // rows between those
    static_assert(64 * NBV % LPR == 0 && NIO % NBV == 0, "pieces repeat");
    const int row0 = m0 + wm * 32 * TM;
    const uint64_t ybase = uniform64((uint64_t)(uintptr_t)y + (((uint64_t)sign * m_half + row0) * n + ncol0) * ES);
    constexpr uint32_t kOutside = 0xc0000000u;                   // with a pass's offsets on top still below 2^32 (kMaxColumns)
    uint32_t voff[NBV];
    int rows_left[NBV];          // rows from the lane's first one to the end of the output; none where its columns lie past the end
#pragma unroll
    for (int v = 0; v < NBV; ++v) {
        const int r = (64 * v + lane) / LPR, c = (64 * v + lane) % LPR;
        const bool in = ncol0 + c * (16 / ES) < n;
        rows_left[v] = in ? m_half - row0 - r : 0;
        voff[v] = kOut16 || in ? (uint32_t)r * (uint32_t)n * ES + (uint32_t)c * 16u : kOutside;
    }
    const uint32_t step = (uint32_t)RSTEP * (uint32_t)n * ES;
    // 16-bit: piece i of the pass that starts at the wave-uniform address `at`, which moves on with every NBV pieces
    typedef __attribute__((address_space(1))) f32x4 *out4;
    auto piece = [&](uint64_t at, int i) { return (out4)((__attribute__((address_space(1))) char *)(uintptr_t)at + voff[i % NBV]); };
    auto valid = [&](int pass, int i) { return pass * RP + i / NBV * RSTEP < rows_left[i % NBV]; };
    uint64_t at_store = ybase;
    // fp32: the rows of a pass that exist, up to the last one's last column, and piece i's offset in them
    auto pass_rows = [&](int pass) {
        const int left = m_half - row0 - pass * RP, rows = left < RP ? left : RP;
        const uint32_t bytes = left > 0 && ncol0 < n ? ((uint32_t)(rows - 1) * (uint32_t)n + (uint32_t)(n - ncol0)) * ES : 0u;
        const uint64_t first = ybase + (uint64_t)pass * RP * (uint32_t)n * ES;
        return __builtin_amdgcn_make_buffer_rsrc((void *)(uintptr_t)first, 0, __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000);
    };
    auto offset = [&](int i) { return voff[i % NBV] + (uint32_t)(i / NBV) * step; };
    constexpr int kPolicy = NT && EPI == 2 ? 2 : 0;              // of a buffer access: non-temporal or not
    // Residual epilogue: the reads of the running sum that a pass needs are all issued one pass ahead
    // (a load may not overtake an earlier store that the compiler cannot tell apart from it).  Reading
    // further ahead (two passes, which is what the registers allow) changes nothing: what the tile waits
    // for is the bandwidth of all workgroups' read-modify-write bursts arriving together, not one latency.
    f32x4 hres[2][EPI == 2 ? NIO : 1];
    auto load_res = [&](int pass, f32x4 (&h)[EPI == 2 ? NIO : 1]) {
        // read once, written once: neither the running sum nor any output is worth an L2 line that
        // an operand slab could keep (non-temporal loads and stores)
        const auto rows = pass_rows(pass);
#pragma unroll
        for (int i = 0; i < NIO; ++i) h[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rows, offset(i), 0, kPolicy));
    };
    float bias4[EPI == 2 ? NBV : 1][4] = {};
    if constexpr (EPI == 2) {
        load_res(0, hres[0]);
#pragma unroll
        for (int v = 0; v < NBV; ++v) {
            const int nc = ncol0 + (64 * v + lane) % LPR * 4;
            if (nc < n) {
                const uint2 braw = *(const uint2 *)(bias + nc);
                bias4[v][0] = Prec<DT>::w2f((uint16_t)(braw.x & 0xffff));
                bias4[v][1] = Prec<DT>::w2f((uint16_t)(braw.x >> 16));
                bias4[v][2] = Prec<DT>::w2f((uint16_t)(braw.y & 0xffff));
                bias4[v][3] = Prec<DT>::w2f((uint16_t)(braw.y >> 16));
            }
        }
    }
    // 16-bit rows that are a power of two long: the chunk (two runs) is XORed by row bits, and the half within it flips with
    // row bit kFlip, a whole piece's rows at a time on the way out.  Written runs are 8 bytes of 32 rows (lanes): they spread
    // over all 64 banks, and those of 16 rows over the 32 that an access of 8 bytes a lane reaches in one go.  (TN == 1 has
    // no row bit to flip by that is one value per piece and within 16 rows: two lanes per bank there.)
    constexpr int kFlip = TN == 1 ? 4 : 3;
    auto chunk16 = [](int r) {
        return TN == 4 ? (r & 7) | ((r >> 4) & 1) << 3 : TN == 2 ? ((r >> 1) & 3) | ((r ^ (r >> 4)) & 1) << 2 : ((r >> 2) & 3);
    };
#pragma unroll
    for (int pass = 0; pass < NPASS; ++pass) {
        const int tm = pass * RP / 32;                          // MFMA row block of this pass
        if constexpr (EPI == 2) {
            if (pass + 1 < NPASS) load_res(pass + 1, hres[(pass + 1) & 1]);
        }
        // fp32: the pass covers rows 16 (pass % 2) .. + 15 of the block, held by the lanes with that fr / 16
        if (kOut16 || (fr >> 4) == (pass & 1)) {
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        v[e] = acc[tn][tm][4 * g + e];
                        if constexpr (kOut16) v[e] += bvals[tn][g][e];
                        if constexpr (EPI == 1) v[e] = v[e] > 0.0f ? v[e] : 0.0f;
                    }
                    const int run = tn * 8 + 2 * g + fh;         // which run of 4 columns of the row
                    if constexpr (kOut16) {
                        // two outputs per conversion instruction (round to nearest even, as the single one does)
                        auto pack2 = [](float lo, float hi) {
                            const f32x2 pr = {lo, hi};
                            if constexpr (DT == kBF16) return __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2));
                            else return __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, f16x2));
                        };
                        const uint2 o = {pack2(v[0], v[1]), pack2(v[2], v[3])};
                        const int slot = kXor ? (((tn * 4 + g) ^ chunk16(fr)) << 1) + (fh ^ ((fr >> kFlip) & 1)) : run;
                        *(uint2 *)(stage + fr * PITCH + (slot << 3)) = o;
                    } else {
                        *(float4 *)(stage + (fr & 15) * PITCH + ((kXor ? run ^ (fr & 15 & (NRUN - 1)) : run) << 4)) = float4{v[0], v[1], v[2], v[3]};
                    }
                }
        }
        asm volatile("" ::: "memory");      // the wave's LDS operations execute in order; keep the compiler to it too
        if constexpr (kOut16) {
#pragma unroll
            for (int i = 0; i < NIO; ++i) {
                const int r = (64 * i + lane) / LPR, c = (64 * i + lane) % LPR;
                u32x4 q = *(const u32x4 *)(stage + r * PITCH + ((kXor ? c ^ chunk16(r) : c) << 4));
                if (kXor && ((i * 64 / LPR) >> kFlip & 1)) q = u32x4{q.z, q.w, q.x, q.y};
                if (valid(pass, i)) {
                    if constexpr (NT) __builtin_nontemporal_store(__builtin_bit_cast(f32x4, q), piece(at_store, i));
                    else *piece(at_store, i) = __builtin_bit_cast(f32x4, q);
                }
                if (i % NBV == NBV - 1) at_store = uniform64(at_store + step);
            }
        } else {
            const auto rows = pass_rows(pass);
#pragma unroll
            for (int i = 0; i < NIO; ++i) {
                const int r = (64 * i + lane) / LPR, c = (64 * i + lane) % LPR;
                f32x4 q = *(const f32x4 *)(stage + r * PITCH + ((kXor ? c ^ (r & (NRUN - 1)) : c) << 4));
                if constexpr (EPI == 2) {
                    const f32x4 h = hres[pass & 1][i];
                    const float *b4 = bias4[i % NBV];
                    q = f32x4{h.x + (q.x + b4[0]), h.y + (q.y + b4[1]), h.z + (q.z + b4[2]), h.w + (q.w + b4[3])};
                }
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, q), rows, offset(i), 0, kPolicy);
            }
        }
        asm volatile("" ::: "memory");
    }
}

// ------------------------------------------------------------------ pipelined tiles
// What a tile shape is made of: 2 x 2 waves, each with TM x TN matrix tiles of 32 x 32; loads run A slabs ahead.
template <int TM_, int TN_, int A_> struct Shape {
    static constexpr int TM = TM_, TN = TN_, A = A_;
    static constexpr int BM = 64 * TM, BN = 64 * TN;
    static constexpr int STX = A + 1, STW = A;                   // LDS stages of the activation tile / of the weight tile
    static constexpr int XU4 = BM * (BK / 8), WU4 = BN * (BK / 8);   // uint4 per stage
    static constexpr int kLdsBytes = (STX * XU4 + STW * WU4) * 16;
    static constexpr int LX = 2 * TM, LW = 2 * TN, NM = TM * TN, R = TM + TN;   // loads per wave and slab; multiplies and fragments per quarter
    static_assert(NM % 2 == 0 && R <= NM, "the schedules below");
    // Fragment reads that have gone out before multiply j of quarter q, for the quarter after it.
    static constexpr int reads(int q, int j)
    {
        const int c = q == 3 ? j : q == 2 ? (NM >= 8 ? 2 : 4) * j : NM == 2 * R ? j / 2 : (R * j + NM - 2) / (NM - 1);
        return c > R ? R : c;
    }
    // Activation loads that have gone out before slot s of the 2 NM + NM / 2 multiplies ahead of the barrier; weight loads
    // before slot s of the NM / 2 + NM behind it.
    static constexpr int xloads(int s)
    {
        if (TM == 4 && TN == 4) return s <= 0 ? 0 : s <= 6 ? 1 : s <= 12 ? 2 : s <= 16 ? 3 : s <= 22 ? 4 : s <= 28 ? 5 : s <= 36 ? 6 : s <= 38 ? 7 : 8;
        const int P = 2 * NM + NM / 2, c = (LX * s + P - 1) / P;
        return c > LX ? LX : c;
    }
    static constexpr int wloads(int s)
    {
        const int P = NM / 2 + NM, c = (LW * s + P - 1) / P;
        return c > LW ? LW : c;
    }
    // everything goes out exactly once, and the last fragments of a slab ahead of its barrier
    static_assert(reads(0, 0) == 0 && reads(0, NM) == R && reads(2, 0) == 0 && reads(2, NM / 2) == R && reads(3, 0) == 0 && reads(3, NM) == R, "");
    static_assert(xloads(0) == 0 && xloads(2 * NM + NM / 2) == LX && wloads(0) == 0 && wloads(NM / 2 + NM) == LW, "");
};

template <int DT, int EPI, class SH>
__global__ __launch_bounds__(256) void linear_mfma_pipe_kernel(const uint16_t *__restrict__ x, const uint16_t *__restrict__ wt_p,
                                                             const uint16_t *__restrict__ wt_m, const uint16_t *__restrict__ b_p,
                                                             const uint16_t *__restrict__ b_m, void *__restrict__ y, int m_half,
                                                             int n, int k, int tiles_m, int tiles_n, int total)
{
    constexpr int TM = SH::TM, TN = SH::TN, A = SH::A, BM = SH::BM, BN = SH::BN, LX = SH::LX, LW = SH::LW, NM = SH::NM;
    extern __shared__ __attribute__((aligned(16))) uint4 smem[];
    // Persistent workgroups, one per CU: the hardware deals consecutive workgroup ids round-robin to the 8 XCDs,
    // so workgroup b sits on XCD b % 8 and is that XCD's slot b / 8; it walks the XCD's contiguous share of the
    // tile list, slot, slot + slots, ...  The software pipeline does not stop between tiles: while the last two
    // slabs of a tile are multiplied the first two slabs of the next tile are already being loaded, and they land
    // during the epilogue.
    const int per_xcd = (total + 7) / 8, slots = (int)gridDim.x / 8;
    const int xcd = (int)blockIdx.x % 8, slot0 = (int)blockIdx.x / 8;
    auto tile_lin = [&](int it) {                                   // -1: no such tile
        const int sl = slot0 + slots * it, lin = xcd * per_xcd + sl;
        return (sl < per_xcd && lin < total) ? lin : -1;
    };
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    // Load assignment: one wave instruction moves 8 tile rows x 128 bytes (whole cache lines); wave w,
    // instruction i of n covers rows (n w + i) * 8 .. + 7; lane -> (row, 16-byte slot).  The slot holds logical
    // chunk slot ^ (row / 2 mod 8): 16 consecutive rows of one logical chunk then sit on 16 distinct
    // 16-byte positions of the 64-bank (256-byte wide) LDS, so fragment reads are conflict-free.
    const int lrow = lane >> 3, lslot = lane & 7;
    struct Tile {
        int sign, m0, n0, tcol;
        uint64_t xbase, wbase;          // first row of the tile in x / in the sign's weights (wave-uniform)
        uint32_t xg[LX], wg[LW];        // byte offsets of this lane's loads from those (clamped at ragged edges)
    };
    auto setup = [&](int lin, Tile &t) {
        int trow;
        tile_at(lin, tiles_m, tiles_n, t.sign, trow, t.tcol);
        t.m0 = trow * BM;
        t.n0 = t.tcol * BN;
        const uint16_t *xa = x + (size_t)t.sign * m_half * k;
        const uint16_t *wt = t.sign ? wt_m : wt_p;
        t.xbase = uniform64((uint64_t)(uintptr_t)(xa + (size_t)t.m0 * k));
        t.wbase = uniform64((uint64_t)(uintptr_t)(wt + (size_t)t.n0 * k));
#pragma unroll
        for (int i = 0; i < LX; ++i) {
            const int row = (wave * LX + i) * 8 + lrow;
            int xr = t.m0 + row; xr = xr < m_half ? xr : m_half - 1;       // clamp: masked at the store
            t.xg[i] = ((uint32_t)(xr - t.m0) * (uint32_t)k + (lslot ^ ((row >> 1) & 7)) * 8) * 2u;
        }
#pragma unroll
        for (int i = 0; i < LW; ++i) {
            const int row = (wave * LW + i) * 8 + lrow;
            int wr = t.n0 + row; wr = wr < n ? wr : n - 1;
            t.wg[i] = ((uint32_t)(wr - t.n0) * (uint32_t)k + (lslot ^ ((row >> 1) & 7)) * 8) * 2u;
        }
    };
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint4 *)smem;
    const int nk = k / BK;                              // > A (the launcher sees to it)
    // Slabs are numbered through all the tiles of this workgroup.  x slab g lives in x stage g % (A + 1), w slab g in w
    // stage g % A (after the x stages).  Kept as rotating scalars (uint4 index into smem): the stages of slabs g and
    // g + 1, and the x stage of slab g - 1, which x slab g + A will go into.
    constexpr uint32_t kXEnd = SH::STX * SH::XU4, kWEnd = kXEnd + SH::STW * SH::WU4;
    auto next_x = [](uint32_t st) { st += SH::XU4; return st == kXEnd ? 0u : st; };
    auto next_w = [](uint32_t st) { st += SH::WU4; return st == kWEnd ? kXEnd : st; };
    uint32_t xs0 = 0, xs1 = next_x(0), xfree = kXEnd - SH::XU4;
    uint32_t ws0 = kXEnd, ws1 = next_w(kXEnd);
    auto lds_x = [&](uint32_t stage) { return lds_base + stage * 16u + (uint32_t)(wave * LX) * 1024u; };   // this wave's slice
    auto lds_w = [&](uint32_t stage) { return lds_base + stage * 16u + (uint32_t)(wave * LW) * 1024u; };

    f32x16 acc[TN][TM];
    const int fr = lane & 31, fh = lane >> 5, sw = (fr >> 1) & 7;
    const int xrow = (wm * 32 * TM + fr) * 8, wrow = (wn * 32 * TN + fr) * 8;     // uint4 index of the lane's first rows
    uint4 wfa[TN], xfa[TM], wfb[TN], xfb[TM];                             // two fragment sets: one multiplies while one loads
    // One fragment of set (wf, xf) for k-step ks of the slab in stages (xst, wst), in the order the multiplies need them:
    // wf0, xf0 .. , wf1 ..
    auto frag1 = [&](uint32_t xst, uint32_t wst, int ks, int idx, uint4 (&wf)[TN], uint4 (&xf)[TM]) {
        const uint4 *xs = smem + xst;
        const uint4 *ws = smem + wst;
        const int slot = (2 * ks + fh) ^ sw;
        if (idx == 0) wf[0] = ws[wrow + slot];
        else if (idx <= TM) xf[idx - 1] = xs[xrow + (idx - 1) * 256 + slot];
        else wf[idx - TM] = ws[wrow + (idx - TM) * 256 + slot];
    };
    // Multiplies j0 .. j1-1 of the TM x TN fragment product of set (wf, xf), quarter q of the slab.  Before multiply j go
    // out: the fragment reads that SH::reads has due there, of set (nwf, nxf) for k-step nks of the slab in stages (nxst,
    // nwst); the global->LDS load that SH::xloads / SH::wloads has due at slot s0 + j, into LDS at `st`.
    //  `first`: the product starts the accumulators (first quarter of a tile's first slab) instead of adding to them.
    auto mma_rl = [&](const uint4 (&wf)[TN], const uint4 (&xf)[TM], int q, int j0, int j1, uint4 (&nwf)[TN], uint4 (&nxf)[TM],
                      uint32_t nxst, uint32_t nwst, int nks, const auto &offs, uint64_t gbase, uint32_t st, bool is_x, int s0,
                      bool first = false) {
#pragma unroll
        for (int j = j0; j < j1; ++j) {
            const int r0 = SH::reads(q, j), r1 = SH::reads(q, j + 1);
            if (r1 > r0) {
#pragma unroll
                for (int r = r0; r < r1; ++r) frag1(nxst, nwst, nks, r, nwf, nxf);
                __builtin_amdgcn_sched_barrier(0);
            }
            const int l0 = is_x ? SH::xloads(s0 + j) : SH::wloads(s0 + j), l1 = is_x ? SH::xloads(s0 + j + 1) : SH::wloads(s0 + j + 1);
            if (l1 > l0) {
#pragma unroll
                for (int l = l0; l < l1; ++l) gload_lds16(gbase, offs[l], st + l * 1024u);
                __builtin_amdgcn_sched_barrier(0);
            }
            // back and forth over the activation fragments, so that one operand changes from one multiply to
            // the next, not both (a little less switching on a chip whose clock is set by its power)
            const int wi = j / TM, xi = (wi & 1) ? TM - 1 - j % TM : j % TM;
            if (first) {
                f32x16 zero;
#pragma unroll
                for (int i = 0; i < 16; ++i) zero[i] = 0.0f;
                acc[wi][xi] = mfma32<DT>(wf[wi], xf[xi], zero);
            } else {
                acc[wi][xi] = mfma32<DT>(wf[wi], xf[xi], acc[wi][xi]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // Software pipeline (in brackets: the 256 x 256 tile).  The LDS holds A + 1 [3] stages of the activation tile and A [2]
    // of the weight tile, so the activation half of every slab's loads is issued A slab-times ahead and the weight half
    // nearly so: with a single slab of lookahead for everything the multiplies wait on memory latency.  One wave per SIMD
    // means nothing else hides an instruction that is slow to issue, so neither the global->LDS loads nor the
    // LDS fragment reads come in bursts: each sits alone between two multiplies and issues while the matrix
    // pipe works on the one before.  The fragments of a quarter slab (TM TN [16] multiplies) are read during the quarter
    // before it, into the set of registers the quarter before that used.  The barrier sits in the middle of
    // the third quarter, once this wave's last LDS reads of slab g are in registers.
    // sched_barrier(0) pins the order (the compiler would sink each LDS read down to its first use).
    //
    // One slab: multiplies slab g (fragment set A holds its first quarter), loads slab g + A from (xb, wb) with
    // the lane offsets (xo, wo).  x(g+A) goes into the activation stage that slab g-1 left at the previous barrier:
    // its loads sit under the multiplies before this slab's barrier; w(g+A) can only follow the barrier: its
    // loads sit under the multiplies after it.
    auto slab = [&](uint64_t xb, uint64_t wb, const uint32_t (&xo)[LX], const uint32_t (&wo)[LW], bool first) {
        const uint32_t stx = lds_x(xfree), stw = lds_w(ws0);
        constexpr int NB = NM / 2;
        mma_rl(wfa, xfa, 0, 0, NM, wfb, xfb, xs0, ws0, 1, xo, xb, stx, true, 0, first);
        mma_rl(wfb, xfb, 1, 0, NM, wfa, xfa, xs0, ws0, 2, xo, xb, stx, true, NM);
        // the last fragments of slab g, several reads at a time, so that they have landed when the barrier's wait comes
        mma_rl(wfa, xfa, 2, 0, NB, wfb, xfb, xs0, ws0, 3, xo, xb, stx, true, 2 * NM);
        // slab g+1 landed (what was loaded after it may still be out); slab g fully in registers
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((A - 1) * LX + (A - 2) * LW) : "memory");
        __builtin_amdgcn_s_barrier();
        mma_rl(wfa, xfa, 2, NB, NM, wfb, xfb, xs0, ws0, 3, wo, wb, stw, false, -NB);
        // the first fragments of slab g+1 early in the quarter: the loop's back edge waits for all LDS reads
        mma_rl(wfb, xfb, 3, 0, NM, wfa, xfa, xs1, ws1, 0, wo, wb, stw, false, NM - NB);
        if constexpr (A == 2) {                 // three and two stages: moves alone
            const uint32_t tx = xfree, tw = ws0;
            xfree = xs0; xs0 = xs1; xs1 = tx;
            ws0 = ws1; ws1 = tw;
        } else {
            xfree = xs0;
            xs0 = xs1; xs1 = next_x(xs1);
            ws0 = ws1; ws1 = next_w(ws1);
        }
    };

    Tile cur, nxt;
    int lin = tile_lin(0);
    if (lin < 0) return;
    setup(lin, cur);
    int it = 0;                                         // tile number of this workgroup
    // prologue of the first tile only: slabs 0 .. A - 1, fragments of the first quarter
    {
        uint32_t px = xs0, pw = ws0;
#pragma unroll
        for (int g = 0; g < A; ++g) {
#pragma unroll
            for (int i = 0; i < LX; ++i) gload_lds16(cur.xbase + 2u * (uint32_t)(g * BK), cur.xg[i], lds_x(px) + i * 1024u);
#pragma unroll
            for (int i = 0; i < LW; ++i) gload_lds16(cur.wbase + 2u * (uint32_t)(g * BK), cur.wg[i], lds_w(pw) + i * 1024u);
            px = next_x(px); pw = next_w(pw);
        }
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((A - 1) * (LX + LW)) : "memory");               // slab 0 landed
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int idx = 0; idx < SH::R; ++idx) frag1(xs0, ws0, 0, idx, wfa, xfa);

    for (;;) {
        const int lin_next = tile_lin(it + 1);
        const bool has_next = lin_next >= 0;
        if (has_next) {
            setup(lin_next, nxt);
        } else {
            // no successor: the A slabs loaded ahead are this tile's last over again, which nothing reads
            nxt = cur;
            nxt.xbase += 2u * (uint32_t)((nk - A) * BK);
            nxt.wbase += 2u * (uint32_t)((nk - A) * BK);
        }
        // all slabs but the last A load A slabs ahead in this tile; the first one starts the accumulators
        slab(cur.xbase + 2u * (uint32_t)(A * BK), cur.wbase + 2u * (uint32_t)(A * BK), cur.xg, cur.wg, true);
        for (int kt = 1; kt < nk - A; ++kt)
            slab(cur.xbase + 2u * (uint32_t)((kt + A) * BK), cur.wbase + 2u * (uint32_t)((kt + A) * BK), cur.xg, cur.wg, false);
        // the last A load the first A slabs of the next tile
#pragma unroll
        for (int g = 0; g < A; ++g)
            slab(nxt.xbase + 2u * (uint32_t)(g * BK), nxt.wbase + 2u * (uint32_t)(g * BK), nxt.xg, nxt.wg, false);

        // ---- epilogue of tile `cur`
        const int sign = cur.sign, m0 = cur.m0, n0 = cur.n0;
        const uint16_t *bias = sign ? b_m : b_p;
        if constexpr (EPI == 4) {
            const int n_partial = 2 * tiles_n;
            // the rows' targets all at once: one by one, each would wait for its load and for the stores of the row block before
            int target[TM];
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                const int mr = m0 + wm * 32 * TM + tm * 32 + fr;
                target[tm] = ((const int32_t *)b_p)[(size_t)sign * m_half + (mr < m_half ? mr : m_half - 1)];
            }
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) asm volatile("" : "+v"(target[tm]));
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                const int mr = m0 + wm * 32 * TM + tm * 32 + fr;
                const size_t row = (size_t)sign * m_half + (mr < m_half ? mr : m_half - 1);
                f32x16 a[TN];
#pragma unroll
                for (int t = 0; t < TN; ++t) a[t] = acc[t][tm];
                ce_partial_row<TN>(a, n0 + wn * 32 * TN, fh, n, mr < m_half, target[tm], (float *)b_m + row, (float2 *)y + row * n_partial + (cur.tcol * 2 + wn));
            }
        } else {
            // staged in the wave's own slice of the activation stage that the tile's last slab has just left (every wave
            // finished reading that stage before the slab's barrier, and the next loads into the slice are this wave's
            // own, issued after the epilogue)
            static_assert(kTileStageBytes<TN> <= 1024 * LX, "a pass fits the slice");
            char *stage = (char *)(smem + xfree) + wave * (1024 * LX);
            store_tile<DT, EPI, TM, TN, true>(acc, stage, bias, y, sign, m_half, n, m0, n0, wm, wn, lane);
        }
        if (!has_next) break;
        cur = nxt;
        ++it;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                 // the tail loads land before LDS is released
}


// ------------------------------------------------------------------ small tiles
// One output tile of 64 x (64 TN) per workgroup of 2 x 2 waves, each with 1 x TN matrix tiles; slabs of 64 k through a ring
// of up to ST LDS stages, one barrier per slab, and a second workgroup on the CU to work while this one waits.  For shapes
// with few tiles: a slab of a larger tile is loaded at about 58 bytes a nanosecond and CU whatever the shape (what the
// in-order return of loads that partly miss the L2 allows), so the more CUs take part, the sooner the operands are in.
// m_half 160, n 2560, k 10240: 155 us on 128 x 128 register-staged tiles, 95 on pipelined 128 x 128, 50 here (240 CUs).
constexpr int kSmallStages = 4;
template <int TN> constexpr int kSmallStageBytes = (64 + 64 * TN) * BK * 2;
template <int DT, int EPI, int TN, bool NT>
__global__ __launch_bounds__(256, 2) void linear_mfma_small_kernel(
    const uint16_t *__restrict__ x, const uint16_t *__restrict__ wt_p, const uint16_t *__restrict__ wt_m, const uint16_t *__restrict__ b_p,
    const uint16_t *__restrict__ b_m, void *__restrict__ y, int m_half, int n, int k, int tiles_m, int tiles_n, int total)
{
    constexpr int ST = kSmallStages, BM = 64, BN = 64 * TN, LX = 2, LW = 2 * TN, L = LX + LW, CPR = BK / 8;
    constexpr uint32_t kStageBytes = kSmallStageBytes<TN>;
    extern __shared__ __attribute__((aligned(16))) uint4 smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int fr = lane & 31, fh = lane >> 5;

    // consecutive workgroup ids go round-robin to the 8 XCDs; each takes a contiguous share of the tile list
    const int per_xcd = (total + 7) / 8;
    const int lin = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
    if (((int)blockIdx.x >> 3) >= per_xcd || lin >= total) return;
    int sign, trow, tcol;
    tile_at(lin, tiles_m, tiles_n, sign, trow, tcol);
    const int m0 = trow * BM, n0 = tcol * BN;
    const uint64_t xbase = uniform64((uint64_t)(uintptr_t)(x + ((size_t)sign * m_half + m0) * k));
    const uint64_t wbase = uniform64((uint64_t)(uintptr_t)((sign ? wt_m : wt_p) + (size_t)n0 * k));

    // one wave instruction loads 8 tile rows of 128 bytes; chunk c of row r sits at slot c ^ (r / 2 mod 8)
    auto swz = [](int r) { return (r >> 1) & 7; };
    uint32_t off[L];                            // LX loads of x, LW of w
#pragma unroll
    for (int i = 0; i < L; ++i) {
        const int row = (i < LX ? wave * LX + i : wave * LW + i - LX) * 8 + (lane >> 3);
        const int first = i < LX ? m0 : n0, end = i < LX ? m_half : n;
        int r = first + row; r = r < end ? r : end - 1;                      // clamped: never stored
        off[i] = ((uint32_t)(r - first) * (uint32_t)k + ((lane & 7) ^ swz(row)) * 8) * 2u;
    }
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint4 *)smem;
    auto load_slab = [&](int slab, uint32_t stage) {
        const uint32_t st = lds_base + stage * kStageBytes, adv = (uint32_t)slab * (BK * 2);
#pragma unroll
        for (int i = 0; i < L; ++i)
            gload_lds16((i < LX ? xbase : wbase) + adv, off[i], st + (i < LX ? (uint32_t)(wave * LX + i) : (uint32_t)(BM / 8 + wave * LW + i - LX)) * 1024u);
    };

    f32x16 acc[TN][1] = {};
    const int xrow = (wm * 32 + fr) * CPR, wrow = (BM + wn * 32 * TN + fr) * CPR;
    auto mult_slab = [&](uint32_t stage) {
        const uint4 *st = smem + stage * (kStageBytes / 16);
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            const int slot = (2 * ks + fh) ^ swz(fr);
            uint4 wf[TN];
            const uint4 xf = st[xrow + slot];
#pragma unroll
            for (int t = 0; t < TN; ++t) wf[t] = st[wrow + t * 32 * CPR + slot];
#pragma unroll
            for (int t = 0; t < TN; ++t) acc[t][0] = mfma32<DT>(wf[t], xf, acc[t][0]);
        }
    };
    const int nk = k / BK;
#pragma unroll
    for (int s = 0; s < ST - 1; ++s)
        if (s < nk) load_slab(s, s);
    uint32_t rd = 0, wr = ST - 1;
    int kt = 0;
    for (; kt < nk - (ST - 2); ++kt) {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((ST - 2) * L) : "memory");   // slab kt landed (this wave's part)
        __builtin_amdgcn_s_barrier();
        if (kt + ST - 1 < nk) load_slab(kt + ST - 1, wr);
        mult_slab(rd);
        rd = rd + 1 == ST ? 0 : rd + 1;
        wr = wr + 1 == ST ? 0 : wr + 1;
    }
    for (; kt < nk; ++kt) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        mult_slab(rd);
        rd = rd + 1 == ST ? 0 : rd + 1;
    }

    // ---- epilogue
    if constexpr (EPI == 4) {
        const int n_partial = 2 * tiles_n, mr = m0 + wm * 32 + fr;
        const size_t row = (size_t)sign * m_half + (mr < m_half ? mr : m_half - 1);
        f32x16 a[TN];
#pragma unroll
        for (int t = 0; t < TN; ++t) a[t] = acc[t][0];
        ce_partial_row<TN>(a, n0 + wn * 32 * TN, fh, n, mr < m_half, ((const int32_t *)b_p)[row], (float *)b_m + row,
                           (float2 *)y + row * n_partial + (tcol * 2 + wn));
    } else {
        static_assert(4 * kTileStageBytes<TN> <= (int)kStageBytes, "the staging areas fit the ring, of one stage at least");
        __syncthreads();                                          // every wave is done with the ring
        store_tile<DT, EPI, 1, TN, NT>(acc, (char *)smem + wave * kTileStageBytes<TN>, sign ? b_m : b_p, y, sign, m_half, n, m0, n0, wm, wn, lane);
    }
}

// ------------------------------------------------------------------ few tiles, deep contractions
// One output tile of 32 x 32 per workgroup; its four waves take every fourth slab of the contraction each, through rings of
// their own (kSplitStages slabs of 32 rows of x and of the weights), so that nothing waits for another wave until the four
// partial sums meet in LDS, in a fixed order.  For shapes whose tiles leave most CUs idle at 64 x 64: four times as many take part, a
// CU loads half as much a slab, and the chain of slabs is a fourth as long.  What bounds it is a CU's loads: 32 KB of lines under way at
// most, 55 B/ns from far memory and 110 from the L2.  Two stages are as fast as three (a second workgroup fits besides).
// The other tilings add up a contraction slab by slab; here every fourth slab, then the four sums.  The error is no larger, but a row's last
// bits depend on which tiling its launch takes, and so on how many rows and signs share the launch.
// Both signs of m_half x n x k, us, operands far / near, 64 x 64 tiles -> here: 96 x 1024 x 4096 20.7 / 15.5 -> 12.2 / 7.1, 213 x 576 x
// 2304 11.3 / 10.0 -> 7.0 / 5.4, 68 x 384 x 1536 8.6 / 7.6 -> 5.4 / 4.5, 213 x 576 x 576 5.6 / 4.9 -> 4.3 / 3.7.
constexpr int kSplitStages = 2, kSplitBytes = 4 * kSplitStages * 64 * BK * 2;
template <int DT, int EPI>
__global__ __launch_bounds__(256, 2) void linear_mfma_split_kernel(
    const uint16_t *__restrict__ x, const uint16_t *__restrict__ wt_p, const uint16_t *__restrict__ wt_m, const uint16_t *__restrict__ b_p,
    const uint16_t *__restrict__ b_m, void *__restrict__ y, int m_half, int n, int k, int tiles_m, int tiles_n, int total)
{
    constexpr int ST = kSplitStages, BM = 32, BN = 32, L = 8, CPR = BK / 8;      // L: loads of a slab, four of x and four of w
    extern __shared__ __attribute__((aligned(16))) uint4 smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 31, fh = lane >> 5;
    const int per_xcd = (total + 7) / 8;
    const int lin = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
    if (((int)blockIdx.x >> 3) >= per_xcd || lin >= total) return;
    int sign, trow, tcol;
    tile_at(lin, tiles_m, tiles_n, sign, trow, tcol);
    const int m0 = trow * BM, n0 = tcol * BN;
    const uint64_t xbase = uniform64((uint64_t)(uintptr_t)(x + ((size_t)sign * m_half + m0) * k));
    const uint64_t wbase = uniform64((uint64_t)(uintptr_t)((sign ? wt_m : wt_p) + (size_t)n0 * k));
    auto swz = [](int r) { return (r >> 1) & 7; };              // chunk c of row r sits at slot c ^ swz(r)
    uint32_t off[L];
#pragma unroll
    for (int i = 0; i < L; ++i) {
        const int row = (i & 3) * 8 + (lane >> 3), first = i < 4 ? m0 : n0, end = i < 4 ? m_half : n;
        int r = first + row; r = r < end ? r : end - 1;                      // clamped: never stored
        off[i] = ((uint32_t)(r - first) * (uint32_t)k + ((lane & 7) ^ swz(row)) * 8) * 2u;
    }
    // the epilogue's operands of this thread: row tid / 8, columns 4 (tid % 8) ..
    const int er = m0 + (tid >> 3), ec = n0 + 4 * (tid & 7);
    const bool live = er < m_half && ec < n;
    const size_t eo = ((size_t)sign * m_half + (er < m_half ? er : m_half - 1)) * n + (ec < n ? ec : n - 4);
    const uint32_t ring = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint4 *)smem + (uint32_t)wave * (ST * 8192u);
    auto load_slab = [&](int slab, uint32_t stage) {
        const uint32_t adv = (uint32_t)slab * (BK * 2);
#pragma unroll
        for (int i = 0; i < L; ++i) gload_lds16((i < 4 ? xbase : wbase) + adv, off[i], ring + stage * 8192u + (uint32_t)i * 1024u);
    };
    f32x16 acc = {};
    const int nk = k / BK, mine = (nk - wave + 3) / 4;                        // slabs wave, wave + 4, ..
#pragma unroll
    for (int s = 0; s < ST; ++s)
        if (s < mine) load_slab(wave + 4 * s, s);
    uint32_t rd = 0;
    for (int i = 0; i < mine; ++i) {
        if (i + ST - 1 < mine) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((ST - 1) * L) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const uint4 *st = smem + (wave * ST + rd) * 512;
        uint4 xf[4], wf[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int slot = (2 * ks + fh) ^ swz(fr);
            xf[ks] = st[fr * CPR + slot];
            wf[ks] = st[256 + fr * CPR + slot];
        }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) acc = mfma32<DT>(wf[ks], xf[ks], acc);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                       // the stage's reads are in registers
        if (i + ST < mine) load_slab(wave + 4 * (i + ST), rd);
        rd = rd + 1 == ST ? 0 : rd + 1;
    }
    // the four partial sums meet in LDS: row fr, runs of four columns 8 g + 4 fh
    __syncthreads();
    float *part = (float *)smem;
    constexpr int PITCH = 36;
#pragma unroll
    for (int g = 0; g < 4; ++g)
        *(float4 *)(part + (wave * 32 + fr) * PITCH + 8 * g + 4 * fh) = float4{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
    __syncthreads();
    float v[4];
    {
        const float *q = part + (tid >> 3) * PITCH + 4 * (tid & 7);
        const f32x4 a = *(const f32x4 *)q, b = *(const f32x4 *)(q + 32 * PITCH), c = *(const f32x4 *)(q + 64 * PITCH), d = *(const f32x4 *)(q + 96 * PITCH);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (a[e] + b[e]) + (c[e] + d[e]);
    }
    if (!live) return;
    if constexpr (EPI != 3) {
        const uint2 raw = *(const uint2 *)((sign ? b_m : b_p) + ec);
        const float bias[4] = {Prec<DT>::w2f((uint16_t)(raw.x & 0xffff)), Prec<DT>::w2f((uint16_t)(raw.x >> 16)), Prec<DT>::w2f((uint16_t)(raw.y & 0xffff)), Prec<DT>::w2f((uint16_t)(raw.y >> 16))};
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] += bias[e];
    }
    if constexpr (EPI < 2) {
        if constexpr (EPI == 1) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.0f ? v[e] : 0.0f;
        }
        uint2 o;
        o.x = (uint32_t)Prec<DT>::acc2a(v[0]) | ((uint32_t)Prec<DT>::acc2a(v[1]) << 16);
        o.y = (uint32_t)Prec<DT>::acc2a(v[2]) | ((uint32_t)Prec<DT>::acc2a(v[3]) << 16);
        *(uint2 *)((uint16_t *)y + eo) = o;
    } else {
        f32x4 *p = (f32x4 *)((float *)y + eo);
        f32x4 o = {v[0], v[1], v[2], v[3]};
        if constexpr (EPI == 2) { const f32x4 h = *p; o = f32x4{h.x + o.x, h.y + o.y, h.z + o.z, h.w + o.w}; }
        *p = o;
    }
}

// ------------------------------------------------------------------ launchers
// CUs of the current device, rounded down to whole XCDs' worth; 0 when the runtime does not say
int cu_count()
{
    static int n_cu = 0;
    if (n_cu == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        n_cu = v >= 8 ? v / 8 * 8 : 8;
    }
    return n_cu;
}

struct Args {
    const void *x, *wt_p, *wt_m, *b_p, *b_m;
    void *y;
    int n_sign, m_half, n, k;
    hipStream_t s;
};

template <int DT, int EPI, class SH> hipError_t launch_pipe(const Args &a)
{
    const int tiles_m = (a.m_half + SH::BM - 1) / SH::BM, tiles_n = (a.n + SH::BN - 1) / SH::BN;
    const int total = a.n_sign * tiles_m * tiles_n, n_cu = cu_count();
    if (n_cu == 0 || a.k / BK <= SH::A) return hipErrorInvalidValue;
    // persistent workgroups: one per CU (their LDS allows no second one), a multiple of the 8 XCDs
    const int want = (total + 7) / 8 * 8;
    const dim3 grid(want < n_cu ? want : n_cu), block(256);
    auto kern = linear_mfma_pipe_kernel<DT, EPI, SH>;
    static std::atomic<uint64_t> lds_allowed{0};
    const hipError_t e = once_per_device(lds_allowed, [&] {
        return hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, SH::kLdsBytes);
    });
    if (e != hipSuccess) return e;
    kern<<<grid, block, SH::kLdsBytes, a.s>>>((const uint16_t *)a.x, (const uint16_t *)a.wt_p, (const uint16_t *)a.wt_m, (const uint16_t *)a.b_p,
                                                   (const uint16_t *)a.b_m, a.y, a.m_half, a.n, a.k, tiles_m, tiles_n, total);
    return hipGetLastError();
}

template <int DT, int EPI, int TN, bool NT> hipError_t launch_small_t(const Args &a)
{
    const int tiles_m = (a.m_half + 63) / 64, tiles_n = (a.n + 64 * TN - 1) / (64 * TN), total = a.n_sign * tiles_m * tiles_n;
    auto kern = linear_mfma_small_kernel<DT, EPI, TN, NT>;
    static std::atomic<uint64_t> lds_allowed{0};
    const hipError_t e = once_per_device(lds_allowed, [&] {
        return hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kSmallStages * kSmallStageBytes<TN>);
    });
    if (e != hipSuccess) return e;
    // no more stages than there are slabs: with one or two, 8 or 5 workgroups fit a CU instead of 2, and what such a shape
    // takes is the workgroups' latency (both signs 6217 x 6320 x 64, 16-bit outputs: 70 -> 41 us)
    const int stages = a.k / BK < kSmallStages ? a.k / BK : kSmallStages;
    kern<<<dim3((total + 7) / 8 * 8), dim3(256), stages * kSmallStageBytes<TN>, a.s>>>((const uint16_t *)a.x, (const uint16_t *)a.wt_p,
                                                                                       (const uint16_t *)a.wt_m, (const uint16_t *)a.b_p,
                                                                                       (const uint16_t *)a.b_m, a.y, a.m_half, a.n, a.k,
                                                                                       tiles_m, tiles_n, total);
    return hipGetLastError();
}

// A wave's rows of a 64 x 64 tile are 64 (16-bit) or 128 bytes long: parts of cache lines, all of them when n is not a
// multiple of 64.  Written past the L2 each part is a memory transaction of its own, left there it meets the rest of its
// line.  fp32 read-modify-write: always left in the L2 (median 1.02 - 1.2 times as fast, 0.87 - 1.6, the more the shorter the
// contraction).  16-bit: left there where one or two slabs make the outputs most of the traffic and rows share lines (5740 x
// 4592 x 64 57 -> 26 us, 6217 x 6320 x 128 76 -> 57); past it otherwise, where operands want the room (2 % from 512 on; whole
// lines 4096 x 16384 x 64 70 -> 58).
template <int DT, int EPI, int TN> hipError_t launch_small(const Args &a)
{
    if constexpr (EPI < 2) {
        if (a.k >= 3 * BK || a.n % 64 == 0) return launch_small_t<DT, EPI, TN, true>(a);
    }
    return launch_small_t<DT, EPI, TN, false>(a);
}

template <int DT, int EPI> hipError_t launch_split(const Args &a)
{
    const int tiles_m = (a.m_half + 31) / 32, tiles_n = (a.n + 31) / 32, total = a.n_sign * tiles_m * tiles_n;
    auto kern = linear_mfma_split_kernel<DT, EPI>;
    static std::atomic<uint64_t> lds_allowed{0};
    const hipError_t e = once_per_device(lds_allowed, [&] {
        return hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kSplitBytes);
    });
    if (e != hipSuccess) return e;
    kern<<<dim3((total + 7) / 8 * 8), dim3(256), kSplitBytes, a.s>>>((const uint16_t *)a.x, (const uint16_t *)a.wt_p, (const uint16_t *)a.wt_m,
                                                                         (const uint16_t *)a.b_p, (const uint16_t *)a.b_m, a.y, a.m_half, a.n, a.k,
                                                                         tiles_m, tiles_n, total);
    return hipGetLastError();
}

enum Tile { T256x256, T256x192, T256x128, T192x128, T128x128, T64x64, T32x32, kTiles };
constexpr int kTileRows[kTiles] = {256, 256, 256, 192, 128, 64, 32}, kTileColumns[kTiles] = {256, 192, 128, 128, 128, 64, 32};
template <int DT, int EPI> hipError_t launch_tile(Tile t, const Args &a)
{
    switch (t) {
    case T256x256: return launch_pipe<DT, EPI, Shape<4, 4, 2>>(a);
    case T256x192: return launch_pipe<DT, EPI, Shape<4, 3, 2>>(a);
    case T256x128: return launch_pipe<DT, EPI, Shape<4, 2, 2>>(a);
    case T192x128: return launch_pipe<DT, EPI, Shape<3, 2, 3>>(a);
    case T128x128: return launch_pipe<DT, EPI, Shape<2, 2, 4>>(a);
    case T64x64: return launch_small<DT, EPI, 1>(a);
    default: return launch_split<DT, EPI>(a);
    }
}

// Do the 32 x 32 tiles get a CU each, and five slabs at least?  They are then faster than any other shape: over 159 shapes (24 - 870 rows
// a sign, n 80 - 5120, k 320 - 14592, all epilogues) 1.52 times in the geometric mean, 1.19 at least, operands far; over 30 others
// far 1.57 (1.18 - 2.05), near 1.74 (1.20 - 2.49).
// The line is short of where they stop gaining.  From one to two tiles a CU they gain 1.12 far, 1.18 near in the mean (39 shapes), up to
// 1.26 and 1.33, but lose up to 8 and 12 % where a sign has few rows and many columns (28 x 4944 x 5248 28.1 -> 30.5 us, 25 x 4544 x 384
// 4.7 -> 4.9); past two they lose (536 x 512 x 2048 12.7 -> 13.1, 642 x 400 x 9280 39.9 -> 47.3).  With two to four slabs they gain 1.15
// (1.07 - 1.27, 0.3 - 0.6 us of a launch's 3.5; 30 shapes of up to a tile a CU).  Both are left to 64 x 64 tiles, with the bits they have there.
bool one_small_tile_a_cu(int n_sign, int m_half, int n, int k)
{
    const long tiles = (long)n_sign * ((m_half + 31) / 32) * ((n + 31) / 32);
    return k >= 5 * BK && tiles <= (cu_count() ? cu_count() : 256);
}

// The tile shape with the least estimated time in us: start + rounds (slabs slab + epilogue), where a round of tiles that
// fills more than half of the CUs also pays slabs busy b, b = 0 .. 1 from half full to full (a full chip clocks lower and
// shares the fabric).  fp32 outputs are paid for by the rounds' share of the chip (their bursts share the memory), with and
// without the running sum read, the first round at a price of its own: the caches take part of it, and of what a 64 x 64
// tile writes nearly all, while from the second round on it pays most per byte (half lines).
// Constants: least squares over 90 shapes (m_half 96 .. 8192, n and k 512 .. 19200) timed with every tile shape; those of
// fp32 outputs over 973 shapes (m_half 64 .. 8192, n 240 .. 20000, k from 64): one price for both fp32 epilogues and all
// rounds, from shapes of k >= 512 alone, had sent short contractions with large outputs to 64 x 64 tiles, up to twice the
// time of the code before the rule (us, that / one price / here: 1374 x 14048 x 384 fp32 57 / 92 / 55, 2185 x 15512 x 512
// residual 168 / 230 / 170).  Over 1688 shapes of more than 11 us, all epilogues: on average 1.2 % slower than the best tile
// of each; 12 more than 5 % slower than the code before, the worst 12 %.
// The 256 x 256 tile gets 3 % credit: near a tie it is the one that long contractions lose least with.  In us, picked
// here / the former choice between 256 x 256 and a register-staged 128 x 128 kernel, m_half x n x k: 536 x 2304 x 768
// 9.0 / 17.1, 692 x 5120 x 5120 84 / 115, 1028 x 1024 x 4096 30 / 53, 391 x 704 x 2816 13 / 39, 8192 x 2304 x 768 61 / 70.
Tile pick_tile(int n_sign, int m_half, int n, int k, int epi)
{
    struct Out { float first, more; };
    static const struct { int min_slabs; float start, slab, busy, out16; Out rmw, out32; } kCost[T32x32] = {
        {3, 4.9f, 1.00f, 0.52f, 3.5f, {26.1f, 21.3f}, {9.0f, 11.4f}}, {3, 3.6f, 0.79f, 0.38f, 3.1f, {20.9f, 16.7f}, {7.0f, 9.0f}},
        {3, 3.6f, 0.59f, 0.28f, 1.6f, {12.0f, 11.4f}, {2.7f, 7.0f}},  {4, 4.1f, 0.49f, 0.21f, 0.9f, {7.9f, 7.6f}, {1.2f, 5.0f}},
        {5, 4.1f, 0.38f, 0.16f, 0.3f, {4.3f, 4.5f}, {0.0f, 3.1f}},    {1, 2.6f, 0.21f, 0.41f, 0.4f, {0.5f, 2.5f}, {0.0f, 1.3f}}};
    if (one_small_tile_a_cu(n_sign, m_half, n, k)) return T32x32;
    const float n_cu = cu_count() ? (float)cu_count() : 256.0f, slabs = (float)(k / BK);
    Tile best = kTiles;
    float best_us = 0.0f;
    for (int t = 0; t < T32x32; ++t) {
        const auto &c = kCost[t];
        if (k / BK < c.min_slabs) continue;
        const float tiles = (float)n_sign * (float)((m_half + kTileRows[t] - 1) / kTileRows[t]) * (float)((n + kTileColumns[t] - 1) / kTileColumns[t]);
        const float slots = t == T64x64 ? 2 * n_cu : n_cu;        // workgroups at a time
        const float full = __builtin_floorf(tiles / slots), part = tiles / slots - full, rounds = full + (part > 0 ? 1.0f : 0.0f);
        float us = c.start;
        if (t == T64x64) {
            // two workgroups per CU: `slab` for one alone, `busy` for the two together
            const float lone = part > 0 && part <= 0.5f ? 1.0f : 0.0f;
            us += slabs * ((rounds - lone) * c.busy + lone * c.slab);
        } else {
            us += slabs * (rounds * c.slab + (full + (part > 0.5f ? 2 * part - 1 : 0.0f)) * c.busy);
        }
        const Out &o = epi == 2 ? c.rmw : c.out32;
        us += epi < 2 ? c.out16 * rounds : full + part < 1 ? o.first * part : o.first + o.more * (full + part - 1);
        if (t == T256x256) us *= 0.97f;
        if (best == kTiles || us < best_us) { best = (Tile)t; best_us = us; }
    }
    return best;
}

// LM head (epilogue 4): strips of 128 columns per (max, sum-exp) pair when tiles 256 columns wide fill half the CUs, else
// strips of 64.  The callers' scratch is sized for either.
bool wide_strips(int n_sign, int m_half, int n, int k)
{
    if (k < 3 * BK) return false;
    const long tiles = (long)n_sign * ((m_half + 255) / 256) * ((n + 255) / 256);
    return tiles >= 128;
}

// Its tile.  256 columns wide: the height of least estimated time in us, start + slabs (rounds slab + r share) + rounds out +
// r out_share, with r the rounds and the last one's fraction.  Constants: least squares over 1100 shapes (40 - 4500 rows a
// sign, vocabularies 2 k - 64 k and OPT's 50272, d 192 - 2700) timed with each height; the picked one is on average 0.15 %
// slower than the best.  (By padded rows alone, from one vocabulary, shorter tiles were taken where they need a round more:
// 616 rows, d 1280, 6824 columns 31.8 us at 256, 37.4 at 128.)  In us, heights 256 / 192 / 128, vocabulary 50272: 1048
// rows, d 2048, 419 / 399 / 428; 700 rows, d 1024, 148 / 159 / 161; 536 rows, d 768, 118 / 98 / 109; 300 rows 92 / 83 /
// 76; 100 rows 54 / 51 / 46.  (These last while the epilogue spent one instruction more per logit, 1 - 2 % of each.)
enum HeadTile { H256x256, H192x256, H128x256, H128x128, H64x128 };
HeadTile pick_head(int n_sign, int m_half, int n, int k)
{
    if (!wide_strips(n_sign, m_half, n, k)) return k / BK > 4 ? H128x128 : H64x128;
    static const struct { int rows, min_slabs; float start, slab, share, out, out_share; } kCost[3] = {
        {256, 3, 9.2f, 0.99f, 0.44f, 3.6f, 0.0f}, {192, 3, 9.0f, 1.13f, 0.0f, 2.4f, 0.4f}, {128, 4, 9.2f, 0.86f, 0.0f, 1.3f, 0.3f}};
    const float n_cu = cu_count() ? (float)cu_count() : 256.0f, slabs = (float)(k / BK);
    HeadTile best = H256x256;
    float best_us = 0.0f;
    for (int t = 0; t < 3; ++t) {
        const auto &c = kCost[t];
        if (k / BK < c.min_slabs) continue;
        const float r = (float)n_sign * (float)((m_half + c.rows - 1) / c.rows) * (float)((n + 255) / 256) / n_cu;
        const float us = c.start + slabs * (__builtin_ceilf(r) * c.slab + r * c.share) + __builtin_ceilf(r) * c.out + r * c.out_share;
        if (t == 0 || us < best_us) { best = (HeadTile)t; best_us = us; }
    }
    return best;
}

template <int DT> hipError_t launch_ce(const Args &a)
{
    switch (pick_head(a.n_sign, a.m_half, a.n, a.k)) {
    case H256x256: return launch_pipe<DT, 4, Shape<4, 4, 2>>(a);
    case H192x256: return launch_pipe<DT, 4, Shape<3, 4, 2>>(a);
    case H128x256: return launch_pipe<DT, 4, Shape<2, 4, 3>>(a);
    case H128x128: return launch_pipe<DT, 4, Shape<2, 2, 4>>(a);
    default: return launch_small<DT, 4, 2>(a);
    }
}

template <int DT> hipError_t launch_t(const Args &a, int epi)
{
    const Tile t = epi == 4 ? kTiles : pick_tile(a.n_sign, a.m_half, a.n, a.k, epi);
    switch (epi) {
    case 0: return launch_tile<DT, 0>(t, a);
    case 1: return launch_tile<DT, 1>(t, a);
    case 2: return launch_tile<DT, 2>(t, a);
    case 3: return launch_tile<DT, 3>(t, a);
    default: return launch_ce<DT>(a);
    }
}

}  // namespace

int mfma_linear_tile(int n_sign, int m_half, int n, int k, int epilogue)
{
    if (!mfma_linear_supported(m_half, n, k)) return 0;
    if (epilogue == 4) {
        static const int kHead[] = {256 << 16 | 256, 192 << 16 | 256, 128 << 16 | 256, 128 << 16 | 128, 64 << 16 | 128};
        return kHead[pick_head(n_sign, m_half, n, k)];
    }
    const Tile t = pick_tile(n_sign, m_half, n, k, epilogue);
    return kTileRows[t] << 16 | kTileColumns[t];
}

int mfma_ce_partials(int n_sign, int m_half, int n, int k) { return wide_strips(n_sign, m_half, n, k) ? 2 * ((n + 255) / 256) : 2 * ((n + 127) / 128); }

bool mfma_linear_supported(int m_half, int n, int k) { return m_half >= 1 && n >= 8 && n < kMaxColumns && n % 8 == 0 && k >= BK && k % BK == 0; }

hipError_t launch_linear_mfma(const void *x, const void *wt_p, const void *wt_m, const void *b_p, const void *b_m, void *y,
                              int dtype, int n_sign, int m_half, int n, int k, int epilogue, hipStream_t s)
{
    if (!mfma_linear_supported(m_half, n, k) || (dtype != kBF16 && dtype != kFP16)) return hipErrorInvalidValue;
    // 16-byte pieces everywhere (operand loads, row-wise stores, bias through the scalar cache)
    if ((uintptr_t)x % 16 || (uintptr_t)wt_p % 16 || (uintptr_t)wt_m % 16 || (uintptr_t)y % 16) return hipErrorInvalidValue;
    if (epilogue != 3 && epilogue != 4 && ((uintptr_t)b_p % 16 || (uintptr_t)b_m % 16)) return hipErrorInvalidValue;
    const Args a{x, wt_p, wt_m, b_p, b_m, y, n_sign, m_half, n, k, s};
    return dtype == kBF16 ? launch_t<kBF16>(a, epilogue) : launch_t<kFP16>(a, epilogue);
}

}  // namespace zo
