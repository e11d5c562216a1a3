// Causal multi-head attention on the matrix cores (bf16 / fp16 in, fp32 softmax statistics),
// part of the paired forward passes of Eq. 1 (DistZO2, Preliminaries).  Both signs are just
// more sequences: the kernel sees n_seq = 2 * batch independent sequences.
//
// One work item = (128 query rows, one head, one sequence); 4 waves x 32 query rows.  Workgroups walk a per-XCD item list,
// as many as the chip holds at once or one per item (zo_attn_items.h).  Key / value tiles of 64 keys stream through LDS.
// Everything is computed transposed so that a lane owns one query row:
//     S^T[key, q] = K Q^T        (MFMA A = K rows, B = Q rows; lane: column q, 16 keys)
//     O^T[c, q]  += V^T P^T      (MFMA A = V^T rows, B = P^T; lane: column q, 16 channels)
// so the online-softmax reference maximum, normaliser and the rescaling of O are per-lane scalars.  The contraction
// order of the P V product follows the accumulator layout of S^T (keys 16s + 4h + {0..3}, 16s + 8 + 4h + {0..3} for
// lane half h), which V^T is read with as well, so P never leaves registers.  V stays row-major in LDS; its
// transposed fragments come from the LDS transposing read of gfx950.  The key loop is software-pipelined in units of
// 32 keys: the vector arithmetic of one unit's softmax is issued between the matrix instructions of the next
// unit's scores and of its own P V product.
#include "zo_attn_items.h"
#include "zo_kernels.h"
#include "zo_types.hip.h"
#include <type_traits>

namespace zo {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

namespace {

constexpr int BQ = kAttnRows, BKV = 64;

template <int DT> __device__ __forceinline__ f32x16 mfma32(const uint4 &a, const uint4 &b, const f32x16 &c)
{
    if constexpr (DT == kBF16)
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// Two probabilities into one register, round-to-nearest-even: one packed conversion instead of two
// single ones and a merge.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
template <int DT> __device__ __forceinline__ uint32_t pack2(float a, float b)
{
    const f32x2 v = {a, b};
    if constexpr (DT == kBF16) return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
    else return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2));
}

// The value that the lane 32 places away holds, taken with the register swap between the two halves of a
// wave (no trip through LDS as a shuffle would make): after the swap of two copies of x, one result holds
// x of lanes 0..31 in both halves and the other x of lanes 32..63, so one of the two is the lane's own value
// and the other its partner's; sum and maximum take both and do not care which is which.
__device__ __forceinline__ void swap_halves(float x, float &a, float &b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}

// The query rows q0 .. q0 + 31 that `rows` marks, the plain way, by a whole wavefront: scores of keys 0 .. t only, in fp32.
// The matrix path multiplies the zero probability of a future key with that key's value, which is not a number when the
// value is infinite or not a number; rows that come out as such are worked again here, from the keys they may see.
// A row belongs to the two lanes fr, fr + 32, each with half of its channels (those of the matrix path's fragments), so
// that a key or value row is read once for all 32 query rows, 16 bytes at a time and from one address per half wave.
// A diverged model has all its rows here.  32 heads of 80, not a number throughout, plain kernel / a wavefront per row /
// here: 2 sequences of 2048 keys 6.4 / 77 / 2.5 ms, 8 of 64 keys 53 / 694 / 58 us.
template <int DT, int DH>
__device__ __forceinline__ void attention_rows(const uint16_t *base, uint16_t *out, int ld, int d, int q0, uint32_t rows)
{
    constexpr int KS = DH / 16;
    const int lane = threadIdx.x & 63, fr = lane & 31, fh = lane >> 5, t = q0 + fr;
    const bool mine = (rows >> fr) & 1u;
    const int last = q0 + 31 - __builtin_clz(rows);                // of the marked rows
    const float scale = 1.0f / __builtin_sqrtf((float)DH);
    auto piece = [&](int row, int what, int s) { return *(const uint4 *)(base + (size_t)row * ld + what * d + 16 * s + 8 * fh); };
    auto elem = [](const uint4 &v, int e) {
        const uint32_t w = e < 2 ? v.x : e < 4 ? v.y : e < 6 ? v.z : v.w;
        return Prec<DT>::a2acc((uint16_t)(e & 1 ? w >> 16 : w & 0xffffu));
    };
    uint4 q[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) q[s] = mine ? piece(t, 0, s) : uint4{0u, 0u, 0u, 0u};
    // f(j, score) for the keys j = 0 .. last; a key is on its way while the one before it is worked
    auto keys = [&](auto &&f) {
        uint4 k[KS], next[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) k[s] = piece(0, 1, s);
        for (int j = 0; j <= last; ++j) {
            const int jn = j < last ? j + 1 : last;
#pragma unroll
            for (int s = 0; s < KS; ++s) next[s] = piece(jn, 1, s);
            float part[2] = {0.0f, 0.0f}, a, b;
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int e = 0; e < 8; ++e) part[e & 1] = __builtin_fmaf(elem(q[s], e), elem(k[s], e), part[e & 1]);
            swap_halves(part[0] + part[1], a, b);
            f(j, (a + b) * scale);
#pragma unroll
            for (int s = 0; s < KS; ++s) k[s] = next[s];
        }
    };
    float mx = -INFINITY, sum = 0.0f, acc[8 * KS] = {};
    keys([&](int j, float s) { if (j <= t) mx = __builtin_fmaxf(mx, s); });
    keys([&](int j, float s) {
        if (j > t) return;
        const float p = __expf(s - mx);
        sum += p;
#pragma unroll
        for (int i = 0; i < KS; ++i) {
            const uint4 v = piece(j, 2, i);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[8 * i + e] = __builtin_fmaf(p, elem(v, e), acc[8 * i + e]);
        }
    });
    if (!mine) return;
    const float inv = 1.0f / sum;
    uint16_t *o = out + (size_t)t * d + 8 * fh;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        auto two = [&](int e) { return pack2<DT>(acc[8 * s + e] * inv, acc[8 * s + e + 1] * inv); };
        *(uint4 *)(o + 16 * s) = uint4{two(0), two(2), two(4), two(6)};
    }
}

template <int LO, int HI, class F> __device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (LO < HI) {
        f(std::integral_constant<int, LO>{});
        static_for<LO + 1, HI>(f);
    }
}

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // native vector: stays in registers across the loop

// Workgroups a CU: four with 64 channels and three with 80, two with more.  A wave waits (for its item's first tiles, for LDS, for
// its workgroup at a tile's barrier) more than it works, so a further workgroup is worth two K fragments less in flight (a ring of
// two, 128 registers at 64 channels) and LDS rows without padding (80 channels: 50 KiB a workgroup, 162 registers).  us, a
// workgroup less / so, launches back to back: 64 channels, 2048 tokens x 256 (head, sequence) pairs 188 / 170, 277 x 288 17.9 / 14.8; 80,
// 2048 x 128 164.5 / 148.9 (as single calls of a program 162.6 / 156.9), 847 x 128 44.9 / 37.7.  Bit for bit the same.  Registers spilled to
// memory cost more than the workgroup gains (138 registers held to 128: 277 x 288 16.5, 512 x 384 32 -> 37).  Launches that keep three a CU
// with 64 channels (zo_attn_items.h) run this instance too, held to three by LDS: one with a ring of four in 138 registers is no
// faster there (46 sizes of 70 - 640 tokens: 1.001 of its time, 0.993 - 1.011).
template <int DH> constexpr int kAttnPerCu = DH == 64 ? 4 : DH == 80 ? 3 : 2;
template <int DT, int DH>
__global__ __launch_bounds__(256, kAttnPerCu<DH>) void attn_mfma_kernel(const uint16_t *__restrict__ qkv, uint16_t *__restrict__ out, int seq,
                                                        int n_heads, int n_seq, int fill)
{
    constexpr int KS = DH / 16, CT = (DH + 31) / 32;   // contraction steps of K Q^T, channel tiles of O^T
    constexpr int CHD = DH / 8;           // 16-byte chunks per K / V row in memory
    // 16-byte chunks per K / V row in LDS: whole channel tiles, so that the row pitch is 128, 192 or 256 bytes.  The
    // chunks past a row's end hold its chunk two (of four) places before over again; what the last channel tile of O^T makes of
    // them lies in the channels past DH and is not stored.  Without padding (TIGHT) it reads the first chunks of the next row
    // there, two chunks behind the tile for the last one: whatever they hold stays in those channels too.
    constexpr bool TIGHT = DH == 80;
    constexpr int CH = TIGHT ? CHD : 4 * CT;
    constexpr int TILE = BKV * CH;        // 16-byte chunks per K / V tile
    // Head sizes that the plain kernel served before this one: there a probability is an fp32 number.  Here it enters the
    // P V product as the sum of two 16-bit numbers (p rounded, and what the rounding left), two multiplies instead of one:
    // 16 bits of it in bf16, up to 22 in fp16, instead of 24.  The error against 64 bits is the plain kernel's, 1.61e-3
    // (bf16) and 2.01e-4 (fp16) at 2048 keys; with one number it was 2.1e-3 (bf16).
    constexpr bool SPLIT = DH != 64 && DH != 128;
    constexpr bool kRedo = SPLIT;         // rows that are not finite are worked again (see the end)
    constexpr int KR = DH <= 80 ? 2 : KS % 4 == 0 ? 4 : KS;   // depth of the K fragment ring (it divides 2 KS: a fragment's slot is the same in every other unit)
    // K and V tiles, both [key][channel] as they sit in memory, 16-byte chunks XOR-swizzled per key so that
    // the MFMA fragment reads of K (32 keys, one chunk) and the transposing reads of V (4 keys x 32 bytes
    // per 16 lanes) are free of conflicts on the 64-bank LDS (but for V's with 80 channels, below).
    // Three K and two V buffers: tiles arrive (global memory straight into LDS) while earlier ones are multiplied.
    __shared__ u32x4 ks3[3][TILE];
    __shared__ u32x4 vs2[2 * TILE + 4 * CT - CH];
    // (pitch 192 bytes: 4 consecutive rows start on 4 different quarters of the 64 banks, which is all the reads of V
    // need; K's 16 rows per read are told apart by the row bits above.  Pitch 160: 8 consecutive rows start on the 8 multiples of
    // 8 banks, and K's other 8 rows have their chunks swapped in pairs; V's second 16 channels meet the first ones of the row three
    // before on 8 banks, a third of the LDS cycles counted)
    auto kswz = [](int r) { return TIGHT ? ((r >> 3) & 1) : CH == 16 ? (r & 15) : CH == 12 ? ((r >> 2) & 3) : ((r >> 1) & 7); };
    auto vswz = [](int r) { return CH == 16 ? ((r & 3) << 2) : CH == 12 || TIGHT ? 0 : (((r >> 1) & 1) << 2); };
    auto in_row = [](int chunk) { return chunk < CHD ? chunk : chunk - 2; };

    const int d = n_heads * DH, ld = 3 * d;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // wave-uniform, and known to be: it feeds scalar operands
    const int fr = lane & 31, fh = lane >> 5;
    // of the work item in hand (see the item loop at the end): its query tile, first query row of this wave, this
    // lane's query row, its first element in qkv as a pointer and as a wave-uniform address
    int q0 = 0, qrow = 0;
    const uint16_t *base = qkv;
    uint64_t gbase0 = 0;

    uint4 qf[KS];                                    // Q fragments: B operand, lane = (row fr, k half fh), all k-steps
    f32x16 oacc[CT];
    // reference maximum of the raw scores (see the key loop); l_lane: this lane's share of the normaliser (the keys
    // its half of the wave holds; the two halves are added once, at the end); sc = log2(e)/sqrt(d_head)
    const float sc = 1.4426950408889634f / __builtin_sqrtf((float)DH);
    // The reference is raised when a raw score passes it by 2^kRaise after scaling; probabilities carry a factor 2^kShift,
    // which the normaliser has too.  bf16 reaches as far down as fp32 does.  Two parts in fp16 end at 2^-25 however large
    // the rest: 2^15 at most leaves 40 binary places below the largest one (25 with 2^8 and no factor, where 2000 keys 18
    // below the maximum, 3e-5 of a row's weight, came to nothing).  4 x 2048 tokens, 32 heads of 80, scores of deviation 1:
    // 164 us / 167 (one box, alternated); of deviation 6, where the reference rises more often, 166 / 173.
    // A probability is 2^(m sc - rn(m sc)) off, the same for all of a row, which the normaliser cancels while both are numbers: heads of 64 and
    // 128 below scaled scores of 2^26 in fp16 (half a unit: 2^2; 2^-14 is the least normal number) and 2^30 in bf16.  To work such rows again
    // as the other heads do (see the end) cost 0.04 - 0.08 us a launch of 3.5 us, and 2 % of all sizes with 64 channels where it spilled.
    constexpr bool kHalf = SPLIT && DT == kFP16;
    constexpr float kRaise = kHalf ? 4.0f : 8.0f, kShift = kHalf ? 11.0f : 0.0f;
    const float lazy = kRaise / sc;
    float m_run = -INFINITY, l_lane = 0.0f, moff = 0.0f, thr = -INFINITY;   // (set per work item)

    // global -> LDS for a K/V tile, without passing through registers: one wave instruction moves 64 x 16
    // bytes and lane L's piece lands at the instruction's LDS base + 16 L.  Piece p = 64 load_no + L of a tile
    // is slot p % CH of key row p / CH; the slot holds logical chunk slot ^ swizzle(row), so the
    // swizzle is applied on the global side (still whole 16-byte pieces of one row per lane).  The lane part
    // of the address does not change from tile to tile: the key advance goes into a scalar base.
    constexpr int NLD = (TILE + 255) / 256;       // instructions per wave and operand, at most
    // a wave's i-th instruction of K (which = 0) or V (1): where they are no multiple of four, two waves load three of K's and two of
    // V's, the others the other way round
    auto load_no = [&](int which, int i) { return TIGHT ? ((wave + 2 * which) & 3) + 4 * i : NLD * wave + i; };
    auto load_is = [&](int which, int i) { return 256 * (i + 1) <= TILE || load_no(which, i) < TILE / 64; };
    uint32_t kgo[NLD], vgo[NLD];          // byte offsets from the tile's first key row
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
        const int pk = 64 * load_no(0, i) + lane, rk = pk / CH, sk = pk % CH, pv = 64 * load_no(1, i) + lane, rv = pv / CH, sv = pv % CH;
        kgo[i] = (uint32_t)(rk * ld + d + in_row(sk ^ kswz(rk)) * 8) * 2u;
        vgo[i] = (uint32_t)(rv * ld + 2 * d + in_row(sv ^ vswz(rv)) * 8) * 2u;
    }
    const uint32_t ks_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)&ks3[0][0];
    const uint32_t vs_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)&vs2[0];
    // Buffer accesses, the buffer as long as what exists of the tile: rows past the end of the sequence come as zeros (masked
    // as future keys) without a branch or a comparison.  Offsets are from the tile's first row: from the sequence's they would
    // not fit 32 bits for long sequences.
    auto dma16 = [](u32x4 rows, uint32_t lane_off, uint32_t lds_off) {
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds" ::"v"(lane_off), "s"(rows), "s"(lds_off) : "memory", "m0");
    };
    // this wave's pieces of K (which = 0) or V (which = 1) rows k0 .. k0 + 63, into buffer `buf` of that operand
    auto issue = [&](int which, int k0, int buf) {
        const uint32_t dst = (which ? vs_lds : ks_lds) + (uint32_t)buf * (TILE * 16);
        const uint64_t gb = gbase0 + (uint64_t)k0 * (uint64_t)ld * 2u;
        const int left = seq - k0 < BKV ? seq - k0 : BKV;
        const u32x4 rows = {(uint32_t)gb, (uint32_t)(gb >> 32), (uint32_t)left * (uint32_t)ld * 2u, 0x00020000u};
#pragma unroll
        for (int i = 0; i < NLD; ++i)
            if (load_is(which, i)) dma16(rows, which ? vgo[i] : kgo[i], dst + (uint32_t)load_no(which, i) * 1024u);
    };
    // Transposing LDS read (ds_read_b64_tr_b16): in every group of 16 lanes, lane j hands in the address of
    // four consecutive 16-bit elements ("row j") and lane i gets back element i%4 of rows i/4, i/4+4, i/4+8,
    // i/4+12.  With lane j pointing at key kb + j/4, channels cb + 4 (j%4) .. + 3, lane i receives channel
    // cb + i for the four keys kb .. kb+3: a V^T fragment straight from row-major V.
    const int tj = lane & 15;
    const int tr_key = tj >> 2;                                  // + key base
    const int tr_chan = 16 * ((lane >> 4) & 1) + 4 * (tj & 3);   // + 32 * channel tile
    // Everything of an LDS address that depends on the lane is worked out once, here: the key bases of the
    // loop are multiples of 4 (V) and 16 or 32 (K), which the swizzles do not see, so inside the loop an
    // address is one of these plus a compile-time constant.
    int voff[CT];                                                // element offset of (key tr_key + 4 fh, channel tile c)
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const int key = 4 * fh + tr_key, chan = c * 32 + tr_chan;
        voff[c] = (key * CH + ((chan >> 3) ^ vswz(key))) * 8 + (chan & 7);
    }
    auto vt_frag = [&](const u32x4 *vs, int kb16, int ctile) {   // keys kb16 + 4 fh + tr_key, kb16 a multiple of 8
        const uint16_t *p = (const uint16_t *)vs + (TIGHT ? voff[0] + 32 * ctile : voff[ctile]) + kb16 * CH * 8;
        return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16 *)p);
    };
    int koff[KS];                                                // u32x4 index of (key fr, k-step s)
#pragma unroll
    for (int s = 0; s < KS; ++s) koff[s] = fr * CH + ((2 * s + fh) ^ kswz(fr));

    // The keys are worked in units of 32 (one 32 x 32 score block; a tile holds two), software-pipelined so that
    // the vector arithmetic of a unit's softmax is issued in the shadow of matrix instructions that do not depend
    // on it.  Step s of a wave:
    //     phase A   S(s+1) = K Q^T of the next unit          |  exponentials of the first 16 keys of unit s
    //     phase B   O^T += V^T P^T of unit s (first its 16   |  exponentials of its last 16 keys, then the
    //               keys done in phase A, then the rest)     |  maximum (and causal mask) of S(s+1)
    // A vector instruction issued right after a matrix instruction of the same wave runs beside it, so a step
    // costs about its 16 matrix instructions when the vector work (4 to 5 instructions per slot) fits under
    // them.  K fragments run through a ring that is refilled as it drains and runs on into the next unit;
    // V^T fragments are read one 16-key step ahead.  The sched_barriers pin the order written here.
    //
    // Tiles in LDS: K of tiles T, T+1 and the arriving T+2 (the pipeline reads K one unit ahead of V), V of tiles
    // T and the arriving T+1.  One barrier per tile: after it tile T+1's K and tile T's V have landed for
    // everybody (each wave waits for its own pieces first) and everybody is done with the buffers that the
    // loads issued next overwrite.  Those loads (K of tile T+2, V of tile T+1) go out together right after the
    // barrier: spread over the slots of a step they cost more, a wave that waits for the memory pipeline to accept
    // a load issues no multiplies either.
    int n_tiles = 0, u_last = 0;                     // of the work item: tiles of the workgroup, last unit of this wave
    int kb0 = 0, kb1 = 1, kb2 = 2;                   // K buffers of tiles T, T+1, T+2
    auto sync_tile = [&](int T) {                    // on entry to tile T
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (T + 2 < n_tiles) issue(0, (T + 2) * BKV, kb2);
        if (T + 1 < n_tiles) issue(1, (T + 1) * BKV, (T + 1) & 1);
    };

    f32x16 S[2];                                     // raw scores: S[s & 1] of unit s, the other of unit s + 1
    u32x4 kf[KR];                                    // K fragment ring
    v4i16 vf[CT][2];                                 // V^T fragments of one 16-key step
    uint4 pf[2];                                     // probabilities of the unit's two 16-key steps, packed
    uint4 pl[SPLIT ? 2 : 1];                         // what rounding left of them
    float tmax;                                      // this lane's maximum over S of the unit about to be exponentiated
    auto k_frag = [&](int buf, int half, int f) { return ks3[buf][half * 32 * CH + (TIGHT ? koff[0] + 2 * f : koff[f])]; };
    auto unit_max = [&](const f32x16 &x) {
        float t = __builtin_fmaxf(__builtin_fmaxf(x[0], x[1]), x[2]);
#pragma unroll
        for (int i = 3; i < 15; i += 2) t = __builtin_fmaxf(__builtin_fmaxf(x[i], x[i + 1]), t);
        return __builtin_fmaxf(t, x[15]);
    };
    // Future keys (key > query) of the unit on a wave's diagonal: its first key is the wave's first row, so which lanes a
    // register loses is the same for every wave and item, a constant: one select per register and scalar moves beside it,
    // where comparing keys and rows takes a vector comparison each that the select has to wait for.  (In a step a score's last
    // product lies a channel tile's multiplies and half the softmax, 26 instructions and more, ahead of this.)
    auto causal_mask = [&](f32x16 &x) {
        const float none = -INFINITY;
        static_for<0, 16>([&](auto ic) {
            constexpr int key = 8 * (decltype(ic)::value >> 2) + (decltype(ic)::value & 3);      // + 4 fh
            float v = x[decltype(ic)::value];
            asm("s_mov_b32 vcc_lo, %2\n\ts_mov_b32 vcc_hi, %3\n\tv_cndmask_b32 %0, %0, %1, vcc" : "+v"(v) : "v"(none), "i"((1u << key) - 1), "i"((1u << (key + 4)) - 1) : "vcc");
            x[decltype(ic)::value] = v;
        });
    };
    // scores of unit u from K buffer `buf`, half `half`, into dst; the ring then holds the first fragments of the
    // unit after it (buffer nbuf, half nhalf).  `odd`: u's lowest bit, a constant.  `between(i)`: what to issue after the i-th multiply.
    auto qk_unit = [&](auto odd, f32x16 &dst, int buf, int half, int nbuf, int nhalf, auto &&between) {
        constexpr int R0 = decltype(odd)::value * KS;
#pragma unroll
        for (int i = 0; i < KS; ++i) {
            if (i == 0) {
                const f32x16 zero = {};
                dst = mfma32<DT>(__builtin_bit_cast(uint4, kf[R0 % KR]), qf[0], zero);
            } else {
                dst = mfma32<DT>(__builtin_bit_cast(uint4, kf[(R0 + i) % KR]), qf[i], dst);
            }
            __builtin_amdgcn_sched_barrier(0);       // the refill goes out after the multiply that frees its slot
            kf[(R0 + i) % KR] = i + KR < KS ? k_frag(buf, half, i + KR) : k_frag(nbuf, nhalf, i + KR - KS);
            between(i);
        }
    };
    // m_run is the reference the exponentials are taken against, not the exact running maximum: it is raised (and
    // O and the normaliser rescaled) only when some row's raw scores pass it by more than 2^kRaise after scaling, so
    // after the first units almost no step pays for the rescaling.  Probabilities then reach 2^(kRaise + kShift) at most; the
    // final division by the normaliser, taken against the same reference, cancels it.  A lane tests its own 16
    // keys; the two halves of the wave agree on the new reference only when one of them asks for it.
    // First unit: m_run = -inf and every row moves (key 0 is never masked, so the row maximum is finite).
    auto step = [&](auto hc, int s) {
        constexpr int H = decltype(hc)::value;       // s & 1: unit s is half H of tile T
        f32x16 &Sc = S[H], &Sn = S[H ^ 1];
        if (__builtin_amdgcn_ballot_w64(tmax > thr) != 0) {
            float ha, hb;
            swap_halves(tmax, ha, hb);
            const float m_new = __builtin_fmaxf(__builtin_fmaxf(ha, hb), m_run);
            const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * sc);
            l_lane *= alpha;
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int i = 0; i < 16; ++i) oacc[c][i] *= alpha;
            m_run = m_new;
            moff = kHalf ? __builtin_fmaf(-m_new, sc, kShift) : -m_new * sc;
            thr = m_new + lazy;
        }
        auto pre = [&](int e) { Sc[e] = __builtin_fmaf(Sc[e], sc, moff); };
        auto ex = [&](int e) {
            const float pe = __builtin_amdgcn_exp2f(Sc[e]);
            Sc[e] = pe;
            l_lane += pe;
            // (pinned here by the empty asm: left alone the compiler gathers the sixteen additions of a unit in one
            // place, a serial chain with no multiply to hide behind.  The addition itself stays the compiler's: it
            // has to keep the distance that a transcendental result needs before its first use.)
            asm volatile("" : "+v"(l_lane));
        };
        auto cvt = [&](int e) {                      // after elements e - 1 and e (e odd) are done
            const uint32_t w = pack2<DT>(Sc[e - 1], Sc[e]);
            const int r = (e & 7) >> 1;
            auto put = [r](uint4 &dst, uint32_t v) {
                if (r == 0) dst.x = v;
                else if (r == 1) dst.y = v;
                else if (r == 2) dst.z = v;
                else dst.w = v;
            };
            put(pf[e >> 3], w);
            if constexpr (SPLIT)
                put(pl[e >> 3], pack2<DT>(Sc[e - 1] - Prec<DT>::a2acc((uint16_t)(w & 0xffffu)), Sc[e] - Prec<DT>::a2acc((uint16_t)(w >> 16))));
        };
        __builtin_amdgcn_sched_barrier(0);
        // phase A.  K of unit s + 1: H = 0: tile T, second half; H = 1: tile T + 1, first half.  Unit s + 2 is
        // tile T + 1 either way.
        qk_unit(std::integral_constant<int, H ^ 1>{}, Sn, H == 0 ? kb0 : kb1, H == 0 ? 1 : 0, kb1, H == 0 ? 0 : 1, [&](int i) {
            if (i < CT) {                            // V^T fragments of this unit's first 16 keys
                vf[i][0] = vt_frag(vs2 + ((s >> 1) & 1) * TILE, 32 * H, i);
                vf[i][1] = vt_frag(vs2 + ((s >> 1) & 1) * TILE, 32 * H + 8, i);
            }
            __builtin_amdgcn_sched_barrier(0);
            // a KS-th of the elements of each 16-key step per slot
#pragma unroll
            for (int e = 8 * i / KS; e < 8 * (i + 1) / KS; ++e) {
                pre(e);
                ex(e);
                if (e & 1) cvt(e);
            }
#pragma unroll
            for (int e = 8 + 8 * i / KS; e < 8 + 8 * (i + 1) / KS; ++e) pre(e);
            __builtin_amdgcn_sched_barrier(0);
        });
        // phase B
#pragma unroll
        for (int j = 0; j < 2 * CT; ++j) {
            const int kstep = j / CT, c = j % CT;
            const uint2 lo2 = __builtin_bit_cast(uint2, vf[c][0]), hi2 = __builtin_bit_cast(uint2, vf[c][1]);
            oacc[c] = mfma32<DT>(uint4{lo2.x, lo2.y, hi2.x, hi2.y}, pf[kstep], oacc[c]);
            if constexpr (SPLIT) oacc[c] = mfma32<DT>(uint4{lo2.x, lo2.y, hi2.x, hi2.y}, pl[kstep], oacc[c]);
            if (kstep == 0) {                        // the slot's fragments are in the matrix pipe: read the next step's
                vf[c][0] = vt_frag(vs2 + ((s >> 1) & 1) * TILE, 32 * H + 16, c);
                vf[c][1] = vt_frag(vs2 + ((s >> 1) & 1) * TILE, 32 * H + 24, c);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (kstep == 0) {
#pragma unroll
                for (int e = 8 + 8 * c / CT; e < 8 + 8 * (c + 1) / CT; ++e) {
                    ex(e);
                    if (e & 1) cvt(e);
                }
            } else if (c == 0) {
                if (s + 1 == u_last) causal_mask(Sn);
            } else if (c == 1) {
                tmax = unit_max(Sn);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    const int slots = (int)gridDim.x >> 3, slot = (int)blockIdx.x >> 3, xcd = (int)blockIdx.x & 7;
    const AttnItems list(seq, n_heads, n_seq, fill);
    auto lin_of = [&](int round) { return round * slots + ((round & 1) ? slots - 1 - slot : slot); };
    uint64_t again = 0;                              // rounds (mod 64) in which a row of this wave came out not finite
    for (int round = 0; round * slots < list.n_lin; ++round) {
        int qt;
        const int pair = list.pair_at(lin_of(round), xcd, qt);
        if (pair < 0) continue;
        const int head = pair % n_heads, sq = pair / n_heads;
        base = qkv + (size_t)sq * seq * ld + head * DH;
        // (the halves go through unsigned 32-bit variables: readfirstlane returns a signed int, which would
        // sign-extend into the upper half)
        const uint32_t gb_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)base);
        const uint32_t gb_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uintptr_t)base >> 32));
        gbase0 = ((uint64_t)gb_hi << 32) | (uint64_t)gb_lo;
        q0 = qt * BQ + wave * 32;
        qrow = q0 + fr;
        const int qload = qrow < seq ? qrow : seq - 1;
        const int q_hi = qt * BQ + BQ - 1 < seq - 1 ? qt * BQ + BQ - 1 : seq - 1;   // last query row of the workgroup
        n_tiles = q_hi / BKV + 1;
        // last unit this wave needs (the one on its diagonal); none where its rows all lie past a ragged end: it takes its
        // share of the loads and leaves the CU's issue slots to the others
        u_last = q0 < seq ? q0 / 32 : -1;
        kb0 = 0, kb1 = 1, kb2 = 2;
        m_run = -INFINITY, l_lane = 0.0f, moff = 0.0f, thr = -INFINITY;
        // everybody is done with the LDS tiles of the previous item: the first tiles of this one go out, then Q is
        // read while they fly
        __syncthreads();
        issue(0, 0, 0);
        issue(1, 0, 0);
        if (n_tiles > 1) issue(0, BKV, 1);
#pragma unroll
        for (int s = 0; s < KS; ++s) qf[s] = *(const uint4 *)(base + (size_t)qload * ld + s * 16 + fh * 8);
        // The Q loads are made to land here, before the key loop.  Otherwise the compiler waits for them where the
        // loop first uses them, by counting outstanding memory operations, and inside the loop that count also
        // holds the next tile's global->LDS loads (issued from asm, unknown to the compiler): every tile would
        // wait for its successor's data.
#pragma unroll
        for (int s = 0; s < KS; ++s) asm volatile("" ::"v"(qf[s].x), "v"(qf[s].y), "v"(qf[s].z), "v"(qf[s].w));
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int i = 0; i < 16; ++i) oacc[c][i] = 0.0f;
        sync_tile(0);

        // prologue: scores of unit 0, nothing to overlap them with
    #pragma unroll
        for (int r = 0; r < KR; ++r) kf[r] = k_frag(0, 0, r);
        qk_unit(std::integral_constant<int, 0>{}, S[0], 0, 0, 0, 1, [](int) { __builtin_amdgcn_sched_barrier(0); });
        if (u_last == 0) {
            // (the select is written out, so the distance that a product needs before its first use is ours to keep)
            asm volatile("s_nop 15\n\ts_nop 3" : "+v"(S[0]));
            causal_mask(S[0]);
        }
        tmax = unit_max(S[0]);


        for (int T = 0; T < n_tiles; ++T) {
            if (2 * T <= u_last) step(std::integral_constant<int, 0>{}, 2 * T);
            if (2 * T + 1 <= u_last) step(std::integral_constant<int, 1>{}, 2 * T + 1);
            if (T + 1 < n_tiles) {
                const int k = kb0;                       // tile T's K buffer takes tile T + 3
                kb0 = kb1;
                kb1 = kb2;
                kb2 = k;
                sync_tile(T + 1);
            }
        }
        auto store_row = [&](float inv) {
            uint16_t *o = out + ((size_t)sq * seq + qrow) * d + head * DH;   // (rows past the end store nothing)
            // A lane holds four channels of each run of eight, its partner half a wave away the other four: of two runs the
            // lower lane takes the first whole and the upper one the second, 16 bytes a store instead of 8.
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int g = 0; g < 4; g += 2) {
                    if (c * 32 + 8 * g >= DH) continue;          // the padding of the last channel tile
                    auto two = [&](int e) { return pack2<DT>(oacc[c][e] * inv, oacc[c][e + 1] * inv); };
                    const auto lo = __builtin_amdgcn_permlane32_swap(two(4 * g), two(4 * g + 4), false, false);
                    const auto hi = __builtin_amdgcn_permlane32_swap(two(4 * g + 2), two(4 * g + 6), false, false);
                    if (qrow < seq) *(uint4 *)(o + c * 32 + 8 * g + 8 * fh) = uint4{lo[0], hi[0], lo[1], hi[1]};
                }
        };
        float l_run;
        {
            float ha, hb;
            swap_halves(l_lane, ha, hb);
            l_run = ha + hb;
        }

        // Head sizes that ran on the plain kernel before this one took them keep its answer where a later token's value
        // is not finite (64 and 128 have always multiplied it with zero here): 20 instructions per work item.  And where the
        // scores are so large that rounding the reference moves it by places: the key that set it has a probability of 2^kShift,
        // so a normaliser below that means that they sank, below what fp16 holds from 2^29 on (scaled scores) and to nothing
        // from 2^31.  (Upwards they overflow, and the row is not finite.)
        float inv = 1.0f / l_run;
        if constexpr (kRedo) {
            constexpr float least = kHalf ? 128.0f : 5.42101086e-20f;     // 2^(kShift - 4); 2^-64
            if (!(l_run >= least)) inv = __builtin_nanf("");
            float probe = 0.0f;                                  // x times 0 is 0 for every finite x
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (c * 32 + 8 * (i >> 2) < DH) probe = __builtin_fmaf(oacc[c][i], 0.0f, probe);
            if (__builtin_amdgcn_ballot_w64(qrow < seq && !(probe == 0.0f && l_run >= least)) != 0) again |= 1ull << (round & 63);
        }
        store_row(inv);
    }
    // The rows that came out not finite, once more the plain way, after all items: nothing of the loop above is live any
    // more, and a register that this needs is not missing there.  A lane finds its half of its row's state in what it has stored
    // itself; the row is worked again if either half is not finite.
    if constexpr (kRedo) {
        if (again == 0) return;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // this wave's own stores lie behind the ones that follow
        for (int round = 0; round * slots < list.n_lin; ++round) {
            int qt;
            const int pair = (again >> (round & 63)) & 1 ? list.pair_at(lin_of(round), xcd, qt) : -1;
            if (pair < 0) continue;
            const int head = pair % n_heads, sq = pair / n_heads;
            q0 = qt * BQ + wave * 32;
            qrow = q0 + fr;
            uint16_t *rows0 = out + (size_t)sq * seq * d + head * DH;
            bool bad = false;
            if (qrow < seq) {
#pragma unroll
                for (int s = 0; s < KS; ++s) {                   // the pieces that store_row wrote from this lane
                    const uint4 v = *(const uint4 *)(rows0 + (size_t)qrow * d + 16 * s + 8 * fh);
                    auto not_finite = [](uint32_t w) {           // either half's exponent is all ones
                        const uint32_t e = DT == kBF16 ? 0x7f80u : 0x7c00u;
                        return (w & e) == e || ((w >> 16) & e) == e;
                    };
                    bad = bad || not_finite(v.x) || not_finite(v.y) || not_finite(v.z) || not_finite(v.w);
                }
            }
            const uint64_t lanes = __builtin_amdgcn_ballot_w64(bad);
            if (lanes != 0)
                attention_rows<DT, DH>(qkv + (size_t)sq * seq * ld + head * DH, rows0, ld, d, q0, (uint32_t)lanes | (uint32_t)(lanes >> 32));
        }
    }
}
}  // namespace

// Head sizes from 64 to 128 in steps of the matrix instruction's contraction (16).  Smaller heads (the test models'),
// odd multiples of 8 and buffers that are not 16-byte aligned take the plain kernel.  Measured at 4 x 2048 tokens, 32
// heads of 80, bf16: 12.7 ms on the plain kernel (a workgroup per query row, K and V re-read per row), 0.165 ms here
// (0.130 with probabilities rounded to 16 bits).
// Any length; the offsets inside a tile of 64 keys are 32-bit.
bool mfma_attention_supported(int seq, int n_heads, int d_head)
{
    return seq >= 1 && d_head >= 64 && d_head <= 128 && d_head % 16 == 0 && 3LL * BKV * n_heads * d_head < 0x7fffffffLL;
}

hipError_t launch_attention_mfma(const void *qkv, void *out, int dtype, int n_seq, int seq, int n_heads, int d_head,
                                 hipStream_t s)
{
    if (!mfma_attention_supported(seq, n_heads, d_head) || (dtype != kBF16 && dtype != kFP16)) return hipErrorInvalidValue;
    if (n_heads < 1 || n_seq < 1) return hipErrorInvalidValue;
    static int n_cu = 0;
    if (n_cu == 0) {
        int dev = 0, v = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        n_cu = v >= 8 ? v / 8 * 8 : 8;
    }
    const int n_qt = (seq + BQ - 1) / BQ;
    const long long pairs = (long long)n_heads * n_seq;
    if ((pairs + 7) / 8 * n_qt > 0x7fffffffLL / 64) return hipErrorInvalidValue;      // the kernel's item indices are ints
    const AttnPlan plan = attention_plan_on(pairs, n_qt, n_cu / 8, d_head);
    const int fill = plan.fill;
    // a workgroup less a CU: by LDS that nobody uses
    const size_t spare = (d_head == 64 && plan.per_cu == 3) || (d_head == 80 && plan.per_cu == 2) ? 12 * 1024 : 0;
    const dim3 grid(8u * (unsigned)plan.slots), block(256);
    const uint16_t *q = (const uint16_t *)qkv;
    uint16_t *o = (uint16_t *)out;
#define ZO_ATTN(DH)                                                                                       \
    case DH:                                                                                              \
        if (dtype == kBF16) attn_mfma_kernel<kBF16, DH><<<grid, block, spare, s>>>(q, o, seq, n_heads, n_seq, fill); \
        else attn_mfma_kernel<kFP16, DH><<<grid, block, spare, s>>>(q, o, seq, n_heads, n_seq, fill);                \
        break;
    switch (d_head) {
    ZO_ATTN(64) ZO_ATTN(80) ZO_ATTN(96) ZO_ATTN(112) ZO_ATTN(128)
    default: return hipErrorInvalidValue;
    }
#undef ZO_ATTN
    return hipGetLastError();
}

}  // namespace zo
