// Attention logits against a paged cache of quantized keys, for decoding, on
// the integer matrix cores: groups of two or more query heads per key head
// (grouped-query attention), and single heads where the lookup tables of
// isoq_scores.h are slower (see score_by_tables).
//
// A key stored by isoq_kv_append is x_hat = rho T^{-1}(c[idx]) with T the
// block rotation of its head.  T is orthogonal (Prop. 1), so for a query q
//     <q, x_hat> = rho <T q, c[idx]>:
// the query is rotated once and the keys are never inverse-rotated.  What is
// left, <T q, c[idx]> for every key of the context, is a product of the index
// matrix, mapped through the codebook, with the group's rotated queries.
//
// Arithmetic.  Both factors are held as fixed-point integers cut into 8-bit
// digits, and the digits meet in v_mfma_i32_16x16x64_i8, whose int32 sums are
// exact:
//   level  c_k   = 2^exp quantum (256^2 d_0 + 256 d_1 + d_2),   3 balanced digits
//   query  T q   = 2^-e (256^3 l_0 + ... + l_3),          4 balanced digits
// (4 bits: c_k = quantum (int + (1 + 256 + 256^2) / 2), so that a level's
// mirror image is the complement of its digits).  The quantum is searched so
// that the integers hit the levels (build_level_digits); a codebook that one
// set of digits does not hold to 2^-23 of each level, or whose smallest level is
// far below the largest, is `wide` (MP): every digit product, and passes over
// the residual levels.  Against 64 bits the logits are off by 7e-8 to 8e-8 of
// their rms (d = 128 and 512, 2 to 4 bits, with and without the sketch); the
// fp32 lookup tables that this replaces were off by 1.2e-7 to 1.7e-7 at d = 128
// and 2.2e-7 to 3.0e-7 at d = 512.
//
// Why digits.  A level digit is a byte picked by a 3-bit index, which is what
// v_perm_b32 does for four coordinates at once: a quad of coordinates costs
// one instruction per digit plus four to spread its index bits into selector
// bytes, whatever the number of query heads, and all products are matrix
// work.  Lookup tables of the query (one LDS read, shift, and-or and add per
// two coordinates and query head) are bound by LDS reads and VALU issue in
// proportion to the heads of a group.  What bounds this kernel is VALU issue
// too (counters, preparation included: 422 instructions per 64 keys at d = 128,
// 3 bits, 4 heads, 24 of them matrix instructions; the matrix cores are busy an
// eighth of the time), but once per key.  Measured at 8 sequences x 32,768 keys
// x 8 key heads, d = 128, tables -> digits: 4 heads, 2 / 3 / 4 bits 45 / 88 / 83
// -> 28 / 34 / 43 us, with 128 sketch bits 109 / 156 / 161 -> 44 / 50 / 57 us; 8
// heads (4 key heads), 3 bits 125 -> 26 us; 2 heads (16 key heads, 16,384 keys),
// 3 bits 43 -> 31 us.
//
// Lane layout.  A lane loads one key of the wave's 64 (its record's pieces,
// norm and sketch: consecutive lanes read consecutive bytes of the piece-major
// cache).  The matrix instruction wants lane l to hold key l mod 16 of a group
// of 16 and a quarter (l / 16) of its coordinates, so the record is cut into
// four chunks of d/4 coordinates and a 4 x 4 transposition over the wave's
// 16-lane rows (two v_permlane32_swap and two v_permlane16_swap per word of a
// chunk) hands chunk l / 16 of key 16 r + l mod 16 to lane l for r = 0 .. 3.
// The rows of A are the digits of the query heads (4 rows per head): lane l
// then receives the four digit sums of one head for key l mod 16, and combines
// them by itself.  HT heads share an instruction: HT = 4 gives each quarter of
// the result a head; with HT = 2 the rows of two copies of A are zero in one
// half, so that two 16-key groups land in the two halves of one accumulator.
// NT = 2: two tiles (8 heads) per pass over the digits; larger groups loop.
//
// With the stage-2 sketch (QM > 0 sign bits per key, Sec. 8) each logit also
// gets the residual correction sqrt(pi/2)/m gamma <S q, 2 z - 1>: the sign
// bits are 0/1 bytes (a shift and a mask per four) against the digits of
// 2 S q, minus the constant sum of S q.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "isoq_device.h"
#include "isoq_internal.h"

namespace isoq {
namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));

template <int D, int BITS, int QM>
struct ScoreMShape {
    static constexpr int K = 1 << BITS;
    static constexpr int RW = (D * BITS + 31) / 32;   // record words (the last one partial at 3 bits, d = 80)
    static constexpr int RH = D * BITS / 16;          // record half-words
    static_assert(RH * 16 == D * BITS, "records are a whole number of half-words");
    // words per record load: 16, 8 or 4 bytes, the largest that divides the
    // record; 0: a record of an odd number of half-words
    static constexpr int LW = RW * 32 != D * BITS ? 0 : RW % 4 == 0 ? 4 : RW % 2 == 0 ? 2 : 1;
    static constexpr int CP = cache_piece(D * BITS / 8);
    static constexpr int CC = D / 4;                  // coordinates per chunk
    static constexpr int CB = CC * BITS;              // index bits per chunk
    static constexpr int WC = (CB + 31) / 32;         // words per chunk
    static constexpr int NQ = 2 * ((CC + 7) / 8);     // quads of coordinates per chunk (zero query digits past CC)
    static constexpr int SW = QM / 32;                // sketch words per key
    static constexpr int SQ = QM / 16;                // sketch quads per chunk
    static constexpr int SC = QM > 0 ? QM / 4 : 1;    // sign bits per chunk
    // LDS words per digit row of a head: 4 chunks of NQ quads, padded so
    // that the rows of an A read start on different banks
    static constexpr int ROWW = 4 * NQ + 4;
    static constexpr int SROWW = 4 * SQ + 4;
    // LDS words per head: rotated query, digits and digit sums, largest
    // magnitude; with the sketch also the raw query, S q, its digits, sums
    // and largest magnitude
    static constexpr int head_words() { return D + 4 * ROWW + 8 + (QM ? D + QM + 4 * SROWW + 8 : 0); }
    // chunk coordinate of byte b of quad q
    static constexpr int coord(int q, int b)
    {
        if (BITS == 2 && 4 * (q / 4) + 4 <= CC / 4)     // a full word of 16 fields
            return 16 * (q / 4) + 4 * b + q % 4;
        return 8 * (q / 2) + 2 * b + q % 2;
    }
};

// Balanced base-256 digits of v, most significant first.
__device__ __forceinline__ void digits4(int v, int out[4])
{
#pragma unroll
    for (int j = 3; j > 0; j--) {
        const int d = (int)(int8_t)(v & 255);
        out[j] = d;
        v = (v - d) >> 8;
    }
    out[0] = v;
}

// v as an integer below 2^p, given the largest magnitude mx of its head
// (mx < 2^E: v 2^(p - E)); the head's values times 2^-(p - E) are restored by
// one ldexp.
__device__ __forceinline__ int head_exponent(float mx, int p)
{
    return mx > 0.f ? p - __builtin_amdgcn_frexp_expf(mx) : 0;
}

__device__ __forceinline__ int to_fixed(float v, int e) { return (int)__builtin_rintf(__builtin_amdgcn_ldexpf(v, e)); }

// mask ? a : b, bit by bit, in one instruction.
__device__ __forceinline__ uint32_t bit_select(uint32_t mask, uint32_t a, uint32_t b)
{
    return __builtin_amdgcn_bitop3_b32(mask, a, b, 0xCA);
}

// A constant kept in a vector register: a scalar operand halves the rate of
// the instructions that read it.
__device__ __forceinline__ uint32_t vector_const(uint32_t k)
{
    asm("" : "+v"(k));
    return k;
}

// Selector bytes of quads 4 ks .. 4 ks + n - 1 of a chunk (its words y): one
// index per byte, other bits clear.
template <class S, int BITS, int NS>
__device__ __forceinline__ void selectors(const uint32_t *y, int q0, uint32_t *sel)
{
    if constexpr (BITS == 2) {
        if (4 * (q0 / 4) + 4 <= S::CC / 4) {   // a full word: 16 fields
            const uint32_t w = y[q0 / 4];
#pragma unroll
            for (int j = 0; j < NS; j++)
                sel[j] = (w >> (2 * j)) & 0x03030303u;
            return;
        }
    }
    // An octet's bits end at the top of x (3 bits; below them the previous
    // octet's) or fill or start it, so that the spreading needs right shifts
    // and bit selects only, which issue at twice the rate of left shifts and
    // of v_bfi.
#pragma unroll
    for (int o = 0; o < NS / 2; o++) {
        const int u = q0 / 2 + o, bit = 8 * u * BITS + (BITS == 3 ? -8 : 0), k = bit >> 5, sh = bit & 31;
        uint32_t x;
        if (k < 0)
            x = y[0] << 8;
        else if (sh == 0)
            x = y[k];
        else if (sh + 8 * BITS + (BITS == 3 ? 8 : 0) > 32)
            x = __builtin_amdgcn_alignbit(k + 1 < S::WC ? y[k + 1] : 0u, y[k], sh);
        else
            x = y[k] >> sh;
        if constexpr (BITS == 4) {
            sel[2 * o] = x & 0x0F0F0F0Fu;
            sel[2 * o + 1] = (x >> 4) & 0x0F0F0F0Fu;
        } else if constexpr (BITS == 3) {
            // 24 bits to the upper six bits of four bytes, two fields each
            const uint32_t t = bit_select(vector_const(0xFFF00000u), x, x >> 4);
            const uint32_t v = bit_select(vector_const(0xFC00FC00u), t, t >> 2);
            sel[2 * o] = (v >> 2) & 0x07070707u;
            sel[2 * o + 1] = (v >> 5) & 0x07070707u;
        } else {
            const uint32_t t = bit_select(vector_const(0x000000FFu), x, x << 8);
            const uint32_t v = bit_select(vector_const(0x000F000Fu), t, t << 4);
            sel[2 * o] = v & 0x03030303u;
            sel[2 * o + 1] = (v >> 2) & 0x03030303u;
        }
    }
}

// 4 x 4 transposition over the wave's 16-lane rows: on return x[r] of lane
// 16 c + i is what x[c] of lane 16 r + i was.
__device__ __forceinline__ void transpose_rows(uint32_t &x0, uint32_t &x1, uint32_t &x2, uint32_t &x3)
{
    const auto a = __builtin_amdgcn_permlane32_swap(x0, x2, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(x1, x3, false, false);
    const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
    const auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
    x0 = c[0];
    x1 = c[1];
    x2 = d[0];
    x3 = d[1];
}

// acc += A B over one k-step of 4 (K = 64) or 2 (K = 32) quads.
template <int NS>
__device__ __forceinline__ i32x4 digit_mfma(const uint32_t *a, const uint32_t *b, i32x4 acc)
{
    if constexpr (NS == 4) {
        const i32x4 av = {(int)a[0], (int)a[1], (int)a[2], (int)a[3]}, bv = {(int)b[0], (int)b[1], (int)b[2], (int)b[3]};
        return __builtin_amdgcn_mfma_i32_16x16x64_i8(av, bv, acc, 0, 0, 0);
    } else {
        const long av = (long)(((uint64_t)a[1] << 32) | a[0]), bv = (long)(((uint64_t)b[1] << 32) | b[0]);
        return __builtin_amdgcn_mfma_i32_16x16x32_i8(av, bv, acc, 0, 0, 0);
    }
}

// Whether a magnitude (its bits) is infinite or NaN.
__device__ __forceinline__ bool nonfinite(uint32_t bits) { return bits >= 0x7F800000u; }

// Rotate the group's queries (scale folded in): qt[g][D], the raw rows to
// qraw (if wanted), the largest magnitude of each head to mx and a flag to odd
// where one is infinite or NaN.
template <int VAR, int D>
__device__ __forceinline__ void rotate_queries(const SMArgs &a, int s, int h, int set, int G, float *qt, float *qraw,
                                               uint32_t *mx, uint32_t *odd)
{
    constexpr int LPQ = D / kCoordsPerLane, PL = kLanePL<VAR>;   // chunks per query, parameters per chunk
    for (int i = threadIdx.x; i < G * LPQ; i += blockDim.x) {
        const int g = i / LPQ, l = i - g * LPQ;
        const int64_t row = (int64_t)s * a.n_q_heads + (int64_t)h * G + g;
        float x[8], y[8], P[VAR == VAR_BLOCK8 ? 8 : PL];
        if (a.q_f16) {
            Raw<true> r;
            load_row_chunk<true>(static_cast<const char *>(a.q) + row * D * 2 + l * 16, r);
            unpack<true>(r, x);
        } else {
            Raw<false> r;
            load_row_chunk<false>(static_cast<const char *>(a.q) + row * D * 4 + l * 32, r);
            unpack<false>(r, x);
        }
        const float *par = a.params + ((int64_t)set * LPQ + l) * PL;
        if constexpr (VAR == VAR_BLOCK8) {
            // row by row (all 64 parameters at once would set the kernel's registers)
#pragma unroll
            for (int r = 0; r < 8; r++) {
                load_params<8>(par + 8 * r, P);
                y[r] = P[0] * x[0];
#pragma unroll
                for (int c = 1; c < 8; c++)
                    y[r] = fmaf(P[c], x[c], y[r]);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            load_params<PL>(par, P);
            rotate_forward<VAR>(P, x, y);
        }
        uint32_t m = 0;
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const float v = y[k] * a.scale;
            qt[g * D + 8 * l + k] = v;
            m = max(m, __float_as_uint(fabsf(v)));   // ordered as the magnitudes; NaN above all
            if (qraw)
                qraw[g * D + 8 * l + k] = x[k];
        }
        atomicMax(mx + 8 * g, m);
        if (nonfinite(m))
            *odd = 1u;
    }
}

// A value where it is infinite or NaN, zero where it is not.
__device__ __forceinline__ float nonfinite_part(float v) { return fabsf(v) < INFINITY ? 0.f : v; }

// What the kernel leaves in the first kOddWords words of its LDS for
// nonfinite_logits.
enum { kOddFlag, kOddArgs, kOddX = kOddArgs + 2, kOddY, kOddZ, kOddWords = 8 };

// The workgroup's logits of every head whose query (or S q) is infinite or NaN
// somewhere, which no digit holds: each is infinite or NaN, by IEEE rules from
// the signs of the key's levels at those coordinates and of its sketch.  Rare
// and not tuned; it starts over from what the kernel left in LDS, so that the
// kernel holds no register for it (the scalar ones are all in use), and every
// wave goes over all of the positions.
template <int D, int BITS, int QM>
__device__ __forceinline__ void nonfinite_logits(const uint32_t *smem)
{
    using S = ScoreMShape<D, BITS, QM>;
    typedef const __attribute__((address_space(4))) SMArgs KernArgs;
    auto word = [&](int i) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)smem[i]); };
    KernArgs &a = *(KernArgs *)((uint64_t)word(kOddArgs + 1) << 32 | word(kOddArgs));
    constexpr int64_t RB = (int64_t)D * BITS / 8;
    const int h = (int)xcd_head(word(kOddX), (uint32_t)a.n_kv_heads, a.block_size * RB % 128 != 0);
    const int s = (int)word(kOddZ), G = a.group, t0 = (int)word(kOddY) * a.chunk;
    const int len = (int)min((int64_t)a.seq_lens[s], min(a.max_len, (int64_t)a.max_blocks * a.block_size));
    const float *qt = reinterpret_cast<const float *>(smem + kOddWords), *sqv = qt + 2 * G * D;
    const uint32_t *mx = smem + kOddWords + G * (D + 4 * S::ROWW + (QM ? D + QM + 4 * S::SROWW : 0)) + 4;
    const FastDiv by_block = {a.div_block.m, a.div_block.s1, a.div_block.s2};
    const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
#pragma unroll 1
    for (int g = 0; g < G; g++) {
        if (!nonfinite(mx[8 * g]) && !(QM > 0 && nonfinite(mx[8 * (G + g)])))
            continue;
        float *out = a.scores + ((int64_t)s * a.n_q_heads + (int64_t)h * G + g) * a.max_len;
#pragma unroll 1
        for (int t = t0 + lane; t < min(t0 + a.chunk, len); t += 64) {
            const uint32_t bi = fast_div((uint32_t)t, by_block);
            const int32_t blk = a.block_table[(int64_t)s * a.max_blocks + bi];
            if (blk < 0 || blk >= a.n_blocks)
                continue;
            const int pos = (int)((uint32_t)t - bi * a.block_size);
            const int64_t krow = ((int64_t)blk * a.n_kv_heads + h) * a.block_size + pos;
            const uint8_t *rec = a.k_idx + (krow - pos) * RB + (int64_t)pos * S::CP;
            float acc = 0.f;
#pragma unroll 1
            for (int c = 0; c < D; c++) {
                const int bit = c * BITS + BITS - 1, i = bit >> 3;   // an index's top bit: a positive level
                const uint32_t byte = rec[(int64_t)(i / S::CP) * a.block_size * S::CP + i % S::CP];
                const float x = nonfinite_part(qt[g * D + c]);
                acc += (byte >> (bit & 7)) & 1 ? x : -x;
            }
            float v = a.k_rho[krow] * acc;
            if constexpr (QM > 0) {
                float acc2 = 0.f;
#pragma unroll 1
                for (int r = 0; r < QM; r++) {
                    const float x = nonfinite_part(sqv[g * QM + r]);
                    acc2 += (a.k_signs[krow * (QM / 8) + (r >> 3)] >> (r & 7)) & 1 ? x : -x;
                }
                v = fmaf(a.k_gamma[krow], acc2, v);
            }
            out[t] = v;
        }
    }
}

template <int D, int BITS, int QM, int HT, int NT, bool LOOP, bool MP>
__global__ __launch_bounds__(256) void score_m_kernel(const SMArgs a)
{
    using S = ScoreMShape<D, BITS, QM>;
    constexpr int64_t RB = (int64_t)D * BITS / 8;    // record bytes
    static_assert(HT == 2 || HT == 4, "heads per instruction");
    constexpr int RG = 4 / HT;                       // 16-key groups per accumulator
    constexpr int HPS = HT * NT;                     // heads per pass over a batch's digits
    constexpr int QP = BITS == 4 ? 29 : 30;          // query integers below 2^QP (4 bits: digits of twice them)
    extern __shared__ __align__(16) uint32_t smem[];

    // a head's records of one cache block: block_size records of RB bytes
    const int h = (int)xcd_head(blockIdx.x, (uint32_t)a.n_kv_heads, a.block_size * RB % 128 != 0);
    const int s = blockIdx.z;
    const int G = a.group;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // positions fit 31 bits (the host checks max_blocks * block_size)
    const int len = (int)min((int64_t)a.seq_lens[s], min(a.max_len, (int64_t)a.max_blocks * a.block_size));
    const int t0 = (int)blockIdx.y * a.chunk;
    const int tend = a.fill ? (int)min((int64_t)t0 + a.chunk, a.max_len) : min(t0 + a.chunk, len);
    float *const out = a.scores + ((int64_t)s * a.n_q_heads + (int64_t)h * G) * a.max_len;
    if (t0 >= len) {
        // nothing to compute (block-uniform: the whole workgroup leaves before
        // any barrier)
        for (int t = t0 + (int)threadIdx.x; t < tend; t += 256)
            for (int g = 0; g < G; g++)
                out[(int64_t)g * a.max_len + t] = -INFINITY;
        return;
    }
    // LDS: kOddWords words for nonfinite_logits, then per head rotated query |
    // raw query | S q, then digit rows, digit sums and largest magnitudes
    float *qt = reinterpret_cast<float *>(smem + kOddWords);
    float *qraw = qt + G * D;
    float *sqv = qraw + (QM ? G * D : 0);
    uint32_t *dig = smem + kOddWords + G * (D + (QM ? D + QM : 0));
    uint32_t *sdig = dig + G * 4 * S::ROWW;
    int *sums = reinterpret_cast<int *>(sdig + (QM ? G * 4 * S::SROWW : 0));   // [G][8]: 4 digit sums, largest magnitude
    int *ssums = sums + G * 8;
    uint32_t *mx = reinterpret_cast<uint32_t *>(sums) + 4, *smx = reinterpret_cast<uint32_t *>(ssums) + 4;
    const int set = a.n_sets == 1 ? 0 : h;

    // 0. the wave's keys: batch b holds keys t0 + 256 b + 64 w + lane.  A
    //    record's address depends on its block-table entry, which is loaded
    //    two batches ahead; the record itself one batch ahead, into the
    //    registers that the transposition has just emptied (the first batch's
    //    while the query digits are built).
    const int32_t *table = a.block_table + (int64_t)s * a.max_blocks;
    struct Place {
        int32_t blk, pos;   // cache block and position in it
    };
    struct Batch {
        uint32_t w[S::RW];
        uint32_t z[S::SW > 0 ? S::SW : 1];
        float rho, gam;
        uint64_t ok;   // lanes holding a key
    };
    const int tw = t0 + 64 * w + lane;
    auto place = [&](int b) {
        const uint32_t tt = (uint32_t)min(tw + 256 * b, len - 1);
        const uint32_t bi = fast_div(tt, a.div_block);
        return Place{table[bi], (int)(tt - bi * a.block_size)};
    };
    // the head's share of the cache: rows (and bytes) from one cache block to
    // the next, and the head's first row
    const uint64_t rstride = (uint64_t)a.n_kv_heads * a.block_size, row0 = (uint64_t)h * a.block_size;
    const uint64_t bstride = rstride * RB;
    const uint8_t *const idx_h = a.k_idx + row0 * RB;
    auto times = [](uint32_t blk, uint64_t stride, uint32_t add) {   // one multiply unless the stride needs 33 bits
        uint64_t o = (uint64_t)blk * (uint32_t)stride + add;
        if (stride >> 32)
            o += (uint64_t)(blk * (uint32_t)(stride >> 32)) << 32;
        return o;
    };
    auto issue = [&](int b, const Place &pl, Batch &k) {
        const bool ok = tw + 256 * b < len && pl.blk >= 0 && pl.blk < a.n_blocks;
        k.ok = __builtin_amdgcn_ballot_w64(ok);
        // an invalid key reads position 0 of the head in block 0 (always present) and is not stored
        const uint32_t blk = ok ? (uint32_t)pl.blk : 0u, pos = ok ? (uint32_t)pl.pos : 0u;
        // piece v of the record (piece-major: consecutive keys' pieces are adjacent)
        const uint8_t *pc0 = idx_h + times(blk, bstride, 0) + (uint64_t)pos * S::CP;
        const int64_t pstep = (int64_t)a.block_size * S::CP;
        const uint64_t krow = row0 + times(blk, rstride, pos);
        if constexpr (S::LW == 4) {
#pragma unroll
            for (int v = 0; v < S::RW / 4; v++) {
                const u32x4 q4 = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(pc0 + v * pstep));
#pragma unroll
                for (int c = 0; c < 4; c++) {
                    const uint32_t e = q4[c];
                    k.w[4 * v + c] = e;
                }
            }
        } else if constexpr (S::LW == 2) {
            static_assert(S::LW != 2 || S::CP == 8, "one load per piece");
#pragma unroll
            for (int v = 0; v < S::RW / 2; v++) {
                const u32x2 q2 = __builtin_nontemporal_load(reinterpret_cast<const u32x2 *>(pc0 + v * pstep));
                const uint32_t e0 = q2[0], e1 = q2[1];
                k.w[2 * v] = e0;
                k.w[2 * v + 1] = e1;
            }
        } else if constexpr (S::LW == 1) {
            // records stored whole, an odd number of words: ordinary 4-byte
            // loads (the second and later ones of a line hit L1)
#pragma unroll
            for (int v = 0; v < S::RW; v++)
                k.w[v] = reinterpret_cast<const uint32_t *>(pc0)[v];
        } else {
            // an odd number of half-words (records stored whole): an odd row
            // starts in the middle of a word, so the aligned words of the
            // record and the half-word before or after them
            const bool odd = krow & 1;
            const uint32_t *al = reinterpret_cast<const uint32_t *>(pc0 + (odd ? 2 : 0));
            const uint32_t half = *reinterpret_cast<const uint16_t *>(pc0 + (odd ? 0 : RB - 2));
            uint32_t r[S::RW - 1];
#pragma unroll
            for (int v = 0; v < S::RW - 1; v++)
                r[v] = al[v];
            // odd: word v is (upper half of r[v - 1], lower half of r[v])
            const uint32_t sh = odd ? 16u : 0u;
            k.w[0] = odd ? (r[0] << 16) | half : r[0];
#pragma unroll
            for (int v = 1; v < S::RW - 1; v++)
                k.w[v] = odd ? __builtin_amdgcn_alignbit(r[v], r[v - 1], 16) : r[v];
            k.w[S::RW - 1] = odd ? r[S::RW - 2] >> sh : half;
        }
        k.rho = a.k_rho[krow];
        if constexpr (QM > 0) {
            const uint32_t *zp = reinterpret_cast<const uint32_t *>(a.k_signs + krow * (QM / 8));
#pragma unroll
            for (int c = 0; c < S::SW; c++)
                k.z[c] = zp[c];
            k.gam = a.k_gamma[krow];
        }
    };
    const int nb = (min(tend, len) - t0 + 255) / 256;   // batches with keys
    Batch k;
    issue(0, place(0), k);
    Place next = place(1);

    // 1. rotated queries q~_g = scale T_h q_g
    for (int i = threadIdx.x; i < G * 8; i += 256) {
        sums[i] = 0;
        if constexpr (QM > 0)
            ssums[i] = 0;
    }
    if (threadIdx.x == 255) {   // (a wave with less to do)
        const uint64_t ka = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
        smem[kOddFlag] = 0u;
        smem[kOddArgs] = (uint32_t)ka;
        smem[kOddArgs + 1] = (uint32_t)(ka >> 32);
        smem[kOddX] = blockIdx.x;
        smem[kOddY] = blockIdx.y;
        smem[kOddZ] = blockIdx.z;
    }
    __syncthreads();
    float *const raw_to = QM ? qraw : nullptr;
    switch (a.variant) {
    case VAR_FULL: rotate_queries<VAR_FULL, D>(a, s, h, set, G, qt, raw_to, mx, smem + kOddFlag); break;
    case VAR_FAST: rotate_queries<VAR_FAST, D>(a, s, h, set, G, qt, raw_to, mx, smem + kOddFlag); break;
    case VAR_PLANAR2D: rotate_queries<VAR_PLANAR2D, D>(a, s, h, set, G, qt, raw_to, mx, smem + kOddFlag); break;
    default: rotate_queries<VAR_BLOCK8, D>(a, s, h, set, G, qt, raw_to, mx, smem + kOddFlag); break;
    }
    __syncthreads();

    // 2. their digits, [head][digit][chunk][quad] (4 bits: of twice the
    //    integer, with the integers' digit sums for the levels' half offset)
    for (int i = threadIdx.x; i < G * 4 * S::NQ; i += 256) {
        const int g = i / (4 * S::NQ), cq = i - g * (4 * S::NQ);
        const int c = cq / S::NQ, q = cq - c * S::NQ;
        const int e = head_exponent(__uint_as_float(mx[8 * g]), QP);
        uint32_t word[4] = {0u, 0u, 0u, 0u};
        int sum[4] = {0, 0, 0, 0};
#pragma unroll
        for (int b = 0; b < 4; b++) {
            // S::coord(q, b), q at run time
            const bool full = BITS == 2 && 4 * (q / 4) + 4 <= S::CC / 4;
            const int ci = full ? 16 * (q / 4) + 4 * b + q % 4 : 8 * (q / 2) + 2 * b + q % 2;
            const int v = ci < S::CC ? to_fixed(qt[g * D + c * S::CC + ci], e) : 0;
            int d[4];
            if constexpr (BITS == 4) {
                digits4(v, d);
#pragma unroll
                for (int j = 0; j < 4; j++)
                    sum[j] += d[j];
            }
            digits4(BITS == 4 ? 2 * v : v, d);
#pragma unroll
            for (int j = 0; j < 4; j++)
                word[j] |= (uint32_t)(d[j] & 255) << (8 * b);
        }
#pragma unroll
        for (int j = 0; j < 4; j++) {
            dig[(g * 4 + j) * S::ROWW + cq] = word[j];
            if constexpr (BITS == 4)
                atomicAdd(sums + 8 * g + j, sum[j]);
        }
    }
    if constexpr (QM > 0) {
        // (S q_g)_r for every query head of the group, S fp32 [QM][D]: 8 lanes
        // per row, so that a load covers consecutive bytes
        for (int i = threadIdx.x; i < G * QM * 8; i += 256) {
            const int gr = i >> 3, g = gr / QM, r = gr - g * QM, l8 = i & 7;
            const float4 *srow = reinterpret_cast<const float4 *>(a.qjl_S + (int64_t)r * D);
            const float4 *qv = reinterpret_cast<const float4 *>(qraw + g * D);
            float acc = 0.f;
#pragma unroll
            for (int j = 0; j < (D / 4 + 7) / 8; j++) {
                const int jj = 8 * j + l8;
                if (D % 32 == 0 || jj < D / 4) {
                    const float4 sv = srow[jj], q4 = qv[jj];
                    acc = fmaf(sv.x, q4.x, acc);
                    acc = fmaf(sv.y, q4.y, acc);
                    acc = fmaf(sv.z, q4.z, acc);
                    acc = fmaf(sv.w, q4.w, acc);
                }
            }
            acc = row_sum<8>(acc) * a.qjl_scale;
            if (l8 == 0) {
                sqv[g * QM + r] = acc;
                atomicMax(smx + 8 * g, __float_as_uint(fabsf(acc)));
            }
        }
        __syncthreads();
        // digits of 2 S q, [head][digit][chunk][quad], and of -sum S q: sign
        // bit 8 b + j (m = 128) or 4 b + j (m = 64) of a chunk is byte b of quad j
        for (int i = threadIdx.x; i < G * 4 * S::SQ; i += 256) {
            const int g = i / (4 * S::SQ), cq = i - g * (4 * S::SQ);
            const int c = cq / S::SQ, q = cq - c * S::SQ;
            const int e = head_exponent(__uint_as_float(smx[8 * g]), 29);
            if (nonfinite(smx[8 * g]))
                smem[kOddFlag] = 1u;
            uint32_t word[4] = {0u, 0u, 0u, 0u};
            int sum[4] = {0, 0, 0, 0};
#pragma unroll
            for (int b = 0; b < 4; b++) {
                const int v = to_fixed(sqv[g * QM + c * S::SC + S::SQ * b + q], e);
                int d[4];
                digits4(v, d);
#pragma unroll
                for (int j = 0; j < 4; j++)
                    sum[j] += d[j];
                digits4(2 * v, d);
#pragma unroll
                for (int j = 0; j < 4; j++)
                    word[j] |= (uint32_t)(d[j] & 255) << (8 * b);
            }
#pragma unroll
            for (int j = 0; j < 4; j++) {
                sdig[(g * 4 + j) * S::SROWW + cq] = word[j];
                atomicAdd(ssums + 8 * g + j, -sum[j]);
            }
        }
    }
    __syncthreads();

    // 3. batches.  Lane l: column l mod 16 (key), digit rows 4 (l / 16) .. + 3
    //    of the result; row l mod 16 of A, chunk l / 16.
    const int col = lane & 15, kq = lane >> 4;
    const int hh = kq % HT, rgl = kq / HT;   // the lane's head of a tile, its 16-key group of an accumulator
    struct Head {
        // the copies of A (and of the sketch's) for the 16-key groups of an
        // accumulator: zero where the row belongs to another group
        uint32_t A[RG][S::NQ];
        uint32_t Z[RG][S::SQ > 0 ? S::SQ : 1];
        i32x4 sum, ssum;                     // constant terms of the lane's result rows
        float f1, f2;                        // 2^-e (with the quantum) of the digits, in two factors;
        float s1, s2;                        // the sketch's
    };
    auto load_head = [&](int g0, Head &t) {
        // A: row `col` is digit col mod 4 of head g0 + (col / 4) mod HT
        const int ga = g0 + (col >> 2) % HT, gr = g0 + hh, grp = (col >> 2) / HT;
        const uint32_t *row = dig + ((ga < G ? ga : 0) * 4 + (col & 3)) * S::ROWW + kq * S::NQ;
#pragma unroll
        for (int q = 0; q < S::NQ; q += 2) {
            const u32x2 v = *reinterpret_cast<const u32x2 *>(row + q);
            const uint32_t v0 = v[0], v1 = v[1];
#pragma unroll
            for (int rr = 0; rr < RG; rr++) {
                t.A[rr][q] = ga < G && grp == rr ? v0 : 0u;
                t.A[rr][q + 1] = ga < G && grp == rr ? v1 : 0u;
            }
        }
        const int gi = gr < G ? gr : 0;
        const float m = __uint_as_float(mx[8 * gi]);
        const int e = head_exponent(m, QP) - a.lv.exp;
        t.f1 = __builtin_amdgcn_ldexpf(1.f, -(e / 2));
        t.f2 = __builtin_amdgcn_ldexpf(1.f, e / 2 - e);
        if constexpr (!MP)
            t.f1 *= a.lv.quantum;
        t.sum = i32x4{0, 0, 0, 0};
        if constexpr (BITS == 4)
            t.sum = *reinterpret_cast<const i32x4 *>(sums + 8 * gi);
        if constexpr (QM > 0) {
            const uint32_t *srow = sdig + ((ga < G ? ga : 0) * 4 + (col & 3)) * S::SROWW + kq * S::SQ;
#pragma unroll
            for (int q = 0; q < S::SQ; q++) {
                const uint32_t v = srow[q];
#pragma unroll
                for (int rr = 0; rr < RG; rr++)
                    t.Z[rr][q] = ga < G && grp == rr ? v : 0u;
            }
            const float sm = __uint_as_float(smx[8 * gi]);
            const int se = head_exponent(sm, 29);
            t.s1 = __builtin_amdgcn_ldexpf(1.f, -(se / 2));
            t.s2 = __builtin_amdgcn_ldexpf(1.f, se / 2 - se);
            t.ssum = *reinterpret_cast<const i32x4 *>(ssums + 8 * gi);
        }
    };
    Head hd[NT];
    if constexpr (!LOOP) {
#pragma unroll
        for (int nt = 0; nt < NT; nt++)
            load_head(nt * HT, hd[nt]);
    }

    float *const out_lane = out + (int64_t)hh * a.max_len + 16 * rgl + col;

    for (int b = 0; b < nb; b++) {
        const int tb = t0 + 256 * b + 64 * w;   // the wave's first key
        const uint64_t ok_mask = k.ok;
        const bool all = ok_mask == ~0ull;
        const float rho_own = k.rho, gam_own = QM > 0 ? k.gam : 0.f;
        // chunks of the record, then 16-key group r's in y[r]
        uint32_t y[4][S::WC];
#pragma unroll
        for (int v = 0; v < S::WC; v++) {
#pragma unroll
            for (int c = 0; c < 4; c++) {
                const int o = c * S::CB + 32 * v, i = o >> 5, sh = o & 31;
                if (i >= S::RW)
                    y[c][v] = 0u;
                else if (sh == 0)
                    y[c][v] = k.w[i];
                else
                    y[c][v] = __builtin_amdgcn_alignbit(i + 1 < S::RW ? k.w[i + 1] : 0u, k.w[i], sh);
            }
            transpose_rows(y[0][v], y[1][v], y[2][v], y[3][v]);
        }
        uint32_t z[4] = {0u, 0u, 0u, 0u};
        if constexpr (QM == 128) {
#pragma unroll
            for (int c = 0; c < 4; c++)
                z[c] = k.z[c];
            transpose_rows(z[0], z[1], z[2], z[3]);
        } else if constexpr (QM == 64) {
            // 16 bits per chunk, spread to four bytes of four bits
#pragma unroll
            for (int c = 0; c < 4; c++)
                z[c] = c & 1 ? k.z[c >> 1] >> 16 : k.z[c >> 1];
            transpose_rows(z[0], z[1], z[2], z[3]);
#pragma unroll
            for (int c = 0; c < 4; c++) {
                const uint32_t t = bit_select(vector_const(0x000000FFu), z[c], z[c] << 8);
                z[c] = bit_select(vector_const(0x000F000Fu), t, t << 4);
            }
        }
        // the batch is in y and z: the next one's loads go out now
        __builtin_amdgcn_sched_barrier(0);
        if (b + 1 < nb) {
            issue(b + 1, next, k);
            next = place(b + 2);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (ok_mask == 0 && !a.fill)
            continue;
        for (int g0 = 0; g0 < G; g0 += HPS) {
            if constexpr (LOOP) {
#pragma unroll
                for (int nt = 0; nt < NT; nt++)
                    load_head(g0 + nt * HT, hd[nt]);
                // the chunks look modified per pass: the selectors are not
                // hoisted out of the loop and held in registers
#pragma unroll
                for (int r = 0; r < 4; r++) {
#pragma unroll
                    for (int v = 0; v < S::WC; v++)
                        asm volatile("" : "+v"(y[r][v]));
                    asm volatile("" : "+v"(z[r]));
                }
            }
#pragma unroll
            for (int st = 0; st < HT; st++) {   // accumulator st: 16-key groups RG st .. RG st + RG - 1
                float val[NT];
                uint32_t tab[3][2];
#pragma unroll
                for (int t = 0; t < 3; t++) {
                    tab[t][0] = a.lv.tab[t][0];
                    tab[t][1] = a.lv.tab[t][1];
                }
                float quantum = a.lv.quantum;
                for (int pass = 0;;) {
                    i32x4 acc[NT][3];
#pragma unroll
                    for (int nt = 0; nt < NT; nt++)
#pragma unroll
                        for (int t = 0; t < 3; t++)
                            acc[nt][t] = hd[nt].sum;
#pragma unroll
                    for (int rr = 0; rr < RG; rr++) {
                        const uint32_t *yr = y[RG * st + rr];
                        auto step = [&](auto nsc, int q0) {
                            constexpr int NS = decltype(nsc)::value;
                            uint32_t sel[NS], inv[NS], p[NS];
                            selectors<S, BITS, NS>(yr, q0, sel);
                            if constexpr (BITS == 4) {
                                // index 8 + m: magnitude m; 7 - m: its mirror
                                // image, the complement of its digits
#pragma unroll
                                for (int j = 0; j < NS; j++) {
                                    const uint32_t neg = 0x0D0D0D0Du - ((sel[j] >> 3) & 0x01010101u);
                                    inv[j] = __builtin_amdgcn_perm(0u, 0u, neg);   // 0xFF where the index is below 8
                                    sel[j] = (sel[j] ^ inv[j]) & 0x07070707u;
                                }
                            }
#pragma unroll
                            for (int t = 0; t < 3; t++) {
#pragma unroll
                                for (int j = 0; j < NS; j++) {
                                    p[j] = __builtin_amdgcn_perm(tab[t][1], tab[t][0], sel[j]);
                                    if constexpr (BITS == 4)
                                        p[j] ^= inv[j];
                                }
#pragma unroll
                                for (int nt = 0; nt < NT; nt++)
                                    acc[nt][t] = digit_mfma<NS>(hd[nt].A[rr] + q0, p, acc[nt][t]);
                            }
                        };
#pragma unroll
                        for (int q0 = 0; q0 + 4 <= S::NQ; q0 += 4)
                            step(std::integral_constant<int, 4>{}, q0);
                        if constexpr (S::NQ % 4 != 0)
                            step(std::integral_constant<int, 2>{}, S::NQ - 2);
                        // one 16-key group's selectors and digits at a time
                        __builtin_amdgcn_sched_barrier(0);
                    }
#pragma unroll
                    for (int nt = 0; nt < NT; nt++) {
                        // sum of 256^(5 - t - j) acc[t][j], in units of 256^2.
                        // (The terms below them are left out: 128.25 per
                        // coordinate at most, 2^-28 of the largest product,
                        // 30 in the root mean square; with wide codebooks they
                        // are all that some levels have.)
                        const i32x4 *d = acc[nt];
                        const int w01 = (d[0][0] << 8) + d[0][1] + d[1][0];
                        const int w2 = d[0][2] + d[1][1] + d[2][0];
                        const int w3 = d[0][3] + d[1][2] + d[2][1];
                        float f = (float)w3;
                        if constexpr (MP)
                            f += fmaf((float)(d[1][3] + d[2][2]), 0x1p-8f, (float)d[2][3] * 0x1p-16f);
                        f = fmaf((float)w01, 65536.f, fmaf((float)w2, 256.f, f));
                        val[nt] = !MP ? f : pass == 0 ? f * quantum : fmaf(f, quantum, val[nt]);
                    }
                    if (!MP || ++pass >= a.n_pass)   // uniform
                        break;
                    const LevelDigits &lv = a.lv_more[pass - 1];
#pragma unroll
                    for (int t = 0; t < 3; t++) {
                        tab[t][0] = lv.tab[t][0];
                        tab[t][1] = lv.tab[t][1];
                    }
                    quantum = lv.quantum;
                }
                // the lane's key: 16 (RG st + rgl) + col of the wave's 64
                const int kk = 16 * (RG * st + rgl) + col;
                const float rho = __int_as_float(__builtin_amdgcn_ds_bpermute(4 * kk, __float_as_int(rho_own)));
                float gam = 0.f;
                if constexpr (QM > 0)
                    gam = __int_as_float(__builtin_amdgcn_ds_bpermute(4 * kk, __float_as_int(gam_own)));
                const int t = tb + kk;
#pragma unroll
                for (int nt = 0; nt < NT; nt++) {
                    float v = (val[nt] * hd[nt].f1) * (rho * hd[nt].f2);
                    if constexpr (QM > 0) {
                        i32x4 acc = hd[nt].ssum;
#pragma unroll
                        for (int rr = 0; rr < RG; rr++) {
#pragma unroll
                            for (int q0 = 0; q0 < S::SQ; q0 += 4) {
                                uint32_t bz[4];
#pragma unroll
                                for (int j = 0; j < 4; j++)
                                    bz[j] = (z[RG * st + rr] >> (q0 + j)) & 0x01010101u;
                                acc = digit_mfma<4>(hd[nt].Z[rr] + q0, bz, acc);
                            }
                        }
                        const float f = fmaf((float)((acc[0] << 8) + acc[1]), 65536.f, (float)((acc[2] << 8) + acc[3]));
                        v = fmaf(f * hd[nt].s1, gam * hd[nt].s2, v);
                    }
                    const int g = g0 + nt * HT + hh;
                    float *const dst = out_lane + (int64_t)((g0 + nt * HT) * a.max_len) + (tb + 16 * RG * st);
                    if (all) {
                        if (g < G)
                            *dst = v;
                    } else {
                        const bool ok = (ok_mask >> kk) & 1;
                        if (g < G && (ok || (a.fill && t < tend)))
                            *dst = ok ? v : -INFINITY;
                    }
                }
            }
            if constexpr (!LOOP)
                break;
        }
    }
    // 4. heads that no digit holds, again
    if (__builtin_expect(__builtin_amdgcn_readfirstlane((int)smem[kOddFlag]) != 0, 0)) {
        __syncthreads();   // the other waves' stores of step 3 to the same positions
        nonfinite_logits<D, BITS, QM>(smem);
    }
    // positions of the chunk past the last batch (fill only)
    for (int t = t0 + 256 * nb + (int)threadIdx.x; t < tend; t += 256)
        for (int g = 0; g < G; g++)
            out[(int64_t)g * a.max_len + t] = -INFINITY;
}

}  // namespace
}  // namespace isoq
