// Decode attention with little work (any cache type, gfx950).  Short contexts: final results by one launch, no partial results and no merge.
//
// What bounds a call over short contexts is not its bytes but what has to happen in turn: lengths, schedule, tiles, partial results, the end of a
// kernel, the start of the next, merge; about 10 us before anything counts.  So a workgroup computes 16 * NH heads and 256 / DS output dims of one
// row (a query token of a sequence) over ALL of its tokens, and needs nobody else.  The 4 / NH * DS workgroups of a row read the same keys; they run on
// one die, so memory is read once and the rest comes from its L2.  How many there are depends on the rows (brief_parts in mfa_kernel_choice.hpp, with
// both sides measured): us per call 2 x 256 bf16 9.8 -> 6.6, 64 x 1024 4 bit 20.4 -> 13.9, 8 bit, four tokens, 16 x 1024 41.2 -> 15.2.
//
// The waves take the 32-token units of the row in turn (wave w: units w, w + kWaves, ..), each with LDS of its own for one unit, its own
// softmax state, and no barrier until the waves' results are added up at the end.  The first unit of every wave is requested before the sequence's
// length is known: its rows lie below the hint, i.e. in memory the caller has vouched for, and so does its entry of a block table, whose page is clamped into the pool.  (Waiting
// for the length over a paged cache: 8 bit, 7 x 65 4.6 -> 5.5 us, 5 x 1500 bf16 11.3 -> 11.8.)  Rows at or past the length may hold anything: their
// weights are 0 and their value rows are cleared in LDS.  A unit's keys are requested as soon as those before it have been multiplied, its values
// likewise; two units of LDS per wave instead: the same within 2 % (the issue of the two waves of a SIMD is the limit, then a compute unit's way to
// L2: 107 GB/s of it at 16 parts and bf16).  Two head groups per wave with less of the dims each instead of one: 10 .. 50 % slower.
//
// Weights (times value scales) meet the values as two bf16 terms, 16 significant bits: the error against 64 bits is about 2e-6 of a result in the 2-norm (1.8 .. 2.4e-6 in calls of 1 .. 128 rows), 3 .. 6e-6 of a
// row's largest in single elements, where weights rounded once leave 1.2 .. 1.7e-3.  It costs up to 8 %: 64 x 1024 bf16, taken uncut, 19.7 -> 21.7 us, now, with the loads unrolled by eight, 18.3.
// The second term may be negative or zero, which an infinite value (or value scale) would turn into NaN.  So where a sum is not finite the workgroup
// works its tokens off once more, with terms that are both positive (two_terms); every other call pays a vote of the waves at its end, 0.1 us, 0.4 with two parts (75 x 72 8 bit 9.6 -> 10.0).
// The body stands in the code twice for that: a branch in its loop instead costs 8-bit calls 5 .. 8 %.
//
// MFMA shapes as in mfa_attn_core.hpp (v_mfma_f32_16x16x32_bf16; lane = 16*g + n): scores S^T[token, head], two blocks of 16 tokens; a lane's eight weights,
// tokens 16*tb + 4*g + i, are its operand of O^T[d, head] += V^T . P^T.  8-bit and 4-bit codes are expanded to bf16 (exactly) between LDS and the matrix
// cores; a key's scale multiplies its score, a value's scale its weight.
#pragma once
#include "mfa_attn_core.hpp"

namespace mfa {

template <int BITS, int NH, int DS>
struct BriefShape {
    static constexpr int kParts = 4 / NH * DS;                          // workgroups per row
    static constexpr int kDimBlocks = 16 / DS;                          // 16-dim blocks of a workgroup
    static constexpr int kKRow = kHeadDim * BITS / 8;                    // bytes of a cached row
    static constexpr int kVRow = kKRow / DS;                             // ... of the part of a value row that is needed
    static constexpr int kKLoads = kUnitTokens * kKRow / 1024;          // direct loads of a unit
    static constexpr int kVLoads = kUnitTokens * kVRow >= 1024 ? kUnitTokens * kVRow / 1024 : 1;
    static constexpr int kKBytes = kUnitTokens * kKRow;
    static constexpr int kVBytes = 1024 * kVLoads;
    static constexpr int kScales = kKBytes + kVBytes;                   // key scales, value scales (256 bytes each, the second half a repetition)
    static constexpr int kSlotBytes = kScales + (BITS == 16 ? 0 : 512);
    // Eight waves, each with a unit of its own, where registers (256 a wave) and LDS allow it: not with NH = 2 (four), nor over bf16 caches with 8 parts (six) and 4 (five, on four SIMDs)
    static constexpr int kLds = 160 * 1024;
    static constexpr int kMostWaves = NH == 1 ? 8 : 4;
    static constexpr int kWaves = kMostWaves * kSlotBytes <= kLds ? kMostWaves : kLds / kSlotBytes;
    static constexpr int kThreads = 64 * kWaves;
    static constexpr int kAccBytes = kDimBlocks * 1024;                 // a wave's result for 16 heads ...
    static constexpr int kMlBase = kWaves * kAccBytes;                  // ... and (m, l) per head, over the dead units
    static constexpr int kVote = kMlBase + kWaves * 128;                // whether a sum is not finite
    static constexpr int kMergeBytes = kVote + 16;
    static constexpr int kLdsBytes = kWaves * kSlotBytes > kMergeBytes ? kWaves * kSlotBytes : kMergeBytes;
    static_assert(kLdsBytes <= kLds, "LDS of a compute unit");
    // Where 16-byte chunk c of row r of a unit lies within its row.  Keys: operand reads (16 rows x one chunk) touch every bank once.  Values: the
    // chunks of a transposing read (bf16 32 bytes, 8 bit 16, 4 bit 8 of 16 dims) spread over the banks as far as the row is wide.
    __host__ __device__ static constexpr int key_chunk(int c, int r) { return BITS == 4 ? c ^ ((r >> 1) & 7) : c ^ (r & 15); }
    __host__ __device__ static constexpr int value_chunk(int c, int r)
    {
        constexpr int kChunks = kVRow / 16;
        constexpr int kRows = kChunks < 16 ? 16 / kChunks : 1;          // rows that span the banks
        return BITS == 16 ? c ^ 2 * (r / kRows & (kChunks / 2 - 1)) : c ^ (r / kRows & (kChunks - 1));
    }
};

// A weight as the sum of two bf16 terms.  The nearest one and what it leaves: 2^-17 of the weight at most is lost.  Or (BOTH_POSITIVE) the largest one
// below the weight and what that leaves, 2^-16: of a weight above zero neither term is zero or negative then, so infinite values stay infinite.
template <bool BOTH_POSITIVE>
__device__ __forceinline__ void two_terms(float w, __bf16& first, __bf16& rest)
{
    if constexpr (BOTH_POSITIVE) {
        const uint32_t bits = __float_as_uint(w);
        first = __builtin_bit_cast(__bf16, (uint16_t)((bits - ((bits << 1) != 0 ? 1u : 0u)) >> 16));
    } else {
        first = (__bf16)w;
    }
    rest = (__bf16)(w - (float)first);
}

// CUT: few rows of longer contexts leave most of the chip idle so.  Then a row's units are dealt out to a.n_splits runs (of kParts workgroups; run s has units
// s, s + n_splits, ..: as even as it can be for every length, and the first units still lie where the hint alone says), which leave partial results;
// merge_splits_kernel adds those up in the order of the runs.  Against the streaming kernels, where a compute unit takes all heads of a
// range: a quarter as many ranges, so a quarter of the partial results to write and merge.  (Eight waves over 8-bit and 4-bit caches, five over a bf16 one.)  us per call, 64 runs of
// 1 x 32768 bf16 22.0 -> 16.5, 8 bit 22.3 -> 15.0; 12 of 5 x 4096 bf16 18.6 -> 14.8; 16 of four tokens, 1 x 8192 8 bit 41.0 -> 15.5 (two passes before).  Runs of
// consecutive tokens, cut by the hint, take the same at its length, but no less wherever a length fills the first of them.
//
// Returns whether a sum is not finite (never with BOTH_POSITIVE).
template <bool PAGED, int BITS, int NH, int DS, bool CUT, bool BOTH_POSITIVE>
__device__ __forceinline__ bool brief_attn(const AttnArgs& a, lds_ptr_t lds_base)
{
    using S = BriefShape<BITS, NH, DS>;
    int thread = threadIdx.x;
    asm volatile("" : "+v"(thread));                                    // (nothing computed from it is kept for the second time)
    const int lane = thread & 63;
    const int wave = __builtin_amdgcn_readfirstlane(thread >> 6);
    const int n = lane & 15, g = lane >> 4;

    // workgroup i runs on die i % 8 (only speed depends on it): the workgroups of a row (of a run of it) follow each other on one die
    const int rows = a.B * a.q_len, runs = CUT ? a.n_splits : 1;
    const int place = (int)(blockIdx.x >> 3);
    const int item = place / S::kParts * 8 + (int)(blockIdx.x & 7);
    if (item >= rows * runs) return false;
    const int row = CUT ? item / runs : item, run = CUT ? item - row * runs : 0;
    const int part = place % S::kParts;
    const int head0 = part / DS * 16 * NH, block0 = part % DS * S::kDimBlocks;
    static_assert(kMaxQueryTokens == 4, "the division by q_len");
    const int b = a.q_len == 3 ? (int)((unsigned)row / 3u) : row >> (a.q_len >> 1), qtok = row - b * a.q_len;

    const uint32_t lds_addr0 = (uint32_t)(uintptr_t)lds_base;
    const int slot = wave * S::kSlotBytes;                              // LDS offset of the wave's unit
    auto row_of = [&](int unit) {
        const int t0 = unit * kUnitTokens;
        return tile_row0<PAGED>(a, b, t0, lookup_page<PAGED>(a, b, t0)) + (PAGED ? t0 & (kPage - 1) : 0);
    };
    // The direct loads of the unit whose first row is row0.  Rows at or past `left` re-read the last one before it.  From one load to
    // the next a lane's row moves by a constant, and its chunk by an exclusive or with one.  (Unrolled by eight: wholly, the first ones cost 0.2 .. 0.5 us, since
    // code that runs once comes cold from the instruction cache, about 100 cycles per 64 bytes; not at all, 64 x 1024, taken uncut, takes 21.5 us in place of 18.3.)
    auto request = [&](int64_t row0, int left, auto value) {
        constexpr bool V = decltype(value)::value;
        constexpr int kRow = S::kKRow, kChunks = (V ? S::kVRow : kRow) / 16, kRowStep = 64 / kChunks, kLoads = V ? S::kVLoads : S::kKLoads;
        auto chunk = [](int c, int r) { return V ? S::value_chunk(c, r) : S::key_chunk(c, r); };
        const int last = left - 1;
        int lane_now = lane;
        asm volatile("" : "+v"(lane_now));
        const int p = lane_now & (kChunks - 1), r0 = lane_now / kChunks & (kUnitTokens - 1);
        const unsigned char* src = (const unsigned char*)(V ? a.v : a.k) + row0 * kRow + (V ? block0 * (kRow / 16) : 0);
        uint32_t dst = lds_addr0 + slot + (V ? S::kKBytes : 0);
        if (left >= kUnitTokens) {
            const uint32_t off = (uint32_t)(r0 * kRow + chunk(p, r0) * 16);
#pragma unroll 8
            for (int r = 0; r < kLoads * kRowStep; r += kRowStep, src += kRowStep * kRow, dst += 1024)
                load_to_lds_16B_keep(src, off ^ (uint32_t)(chunk(0, r) * 16), dst);
        } else {
#pragma unroll 1
            for (int u = 0; u < kLoads; ++u) {
                const int r = r0 + u * kRowStep;
                load_to_lds_16B_keep(src, (uint32_t)((r < last ? r : last) * kRow + chunk(p, r) * 16), dst + u * 1024);
            }
        }
        if (BITS != 16) {
            const int r = lane_now & (kUnitTokens - 1);
            load_to_lds_4B((V ? a.v_scale : a.k_scale) + row0, (uint32_t)(4 * (r < last ? r : last)), lds_addr0 + slot + S::kScales + (V ? 256 : 0));
        }
    };

    int unit = run + runs * wave;
    const int stride = runs * S::kWaves;
    if (unit * kUnitTokens < a.max_seq_len_hint) {
        const int64_t row0 = row_of(unit);
        request(row0, a.max_seq_len_hint - unit * kUnitTokens, std::false_type{});
        request(row0, a.max_seq_len_hint - unit * kUnitTokens, std::true_type{});
    }
    // Query operands: k step ks of a lane holds dims 32*ks + 8*g.. against bf16 keys; against codes a lane reads 16 bytes of a key row at a time, so its
    // k steps are the consecutive dims of such a piece.
    bf16x8 q[NH][8];
#pragma unroll
    for (int j = 0; j < NH; ++j) {
        const bf16x8* src = (const bf16x8*)((const uint16_t*)a.q + ((size_t)row * kHeads + head0 + 16 * j + n) * kHeadDim);
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) q[j][ks] = src[BITS == 16 ? 4 * ks + g : BITS == 8 ? 8 * (ks >> 1) + 2 * g + (ks & 1) : 16 * (ks >> 2) + 4 * g + (ks & 3)];
    }
    const int len = clamped_len(a, b), end = len - (a.q_len - 1 - qtok);   // tokens this row attends to
    if (CUT && run > 0 && run * kUnitTokens >= len) {                   // no partial result is expected of this run
        wait_vmem_but<0>();                                             // (no load may still be on its way into LDS that others get next)
        return false;
    }

    f32x4 acc[NH][S::kDimBlocks];
    float m[NH], l[NH];
#pragma unroll
    for (int j = 0; j < NH; ++j) {
        m[j] = -INFINITY;
        l[j] = 0.f;
#pragma unroll
        for (int i = 0; i < S::kDimBlocks; ++i) acc[j][i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    union Bf16s { bf16x8 v; bf16x2 p[4]; s16x4 h[2]; };
    typedef int i32x2 __attribute__((ext_vector_type(2)));
    // eight codes (two words, or one at 4 bit) -> bf16
    auto expand = [](uint32_t w0, uint32_t w1) {
        Bf16s x;
        if constexpr (BITS == 8) {
            x.p[0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)w0, 1.0f, false);
            x.p[1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)w0, 1.0f, true);
            x.p[2] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)w1, 1.0f, false);
            x.p[3] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)w1, 1.0f, true);
        } else {
            x.p[0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4((int)w0, 1.0f, 0);
            x.p[1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4((int)w0, 1.0f, 1);
            x.p[2] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4((int)w0, 1.0f, 2);
            x.p[3] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4((int)w0, 1.0f, 3);
        }
        return x.v;
    };

    const float c = BITS == 16 ? a.scale_log2e : 1.0f;
    for (; unit * kUnitTokens < end; unit += stride) {
        const int left = end - unit * kUnitTokens;                      // tokens of this unit that count
        const bool whole = left >= kUnitTokens;
        const int left_next = left - stride * kUnitTokens;              // of the unit that takes this one's place
        const int64_t row_next = left_next > 0 ? row_of(unit + stride) : 0;
        wait_vmem_but<0>();
        // ---- scores
        f32x4 s[NH][2];
#pragma unroll
        for (int j = 0; j < NH; ++j) s[j][0] = s[j][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
            const int r = 16 * tb + n, at = slot + r * S::kKRow;
#pragma unroll
            for (int c = 0; c < S::kKRow / 64; ++c) {                   // 16-byte pieces of a lane: 4*c + g
                const u32x4 x = *LDS_AT(u32x4, lds_base, at + 16 * S::key_chunk(4 * c + g, r));
                constexpr int kSteps = 16 / BITS;                       // k steps of a piece
#pragma unroll
                for (int i = 0; i < kSteps; ++i) {
                    const bf16x8 k = BITS == 16 ? __builtin_bit_cast(bf16x8, x) : BITS == 8 ? expand(x[(2 * i) & 3], x[(2 * i + 1) & 3]) : expand(x[i], 0);
#pragma unroll
                    for (int j = 0; j < NH; ++j) s[j][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k, q[j][kSteps * c + i], s[j][tb], 0, 0, 0);
                }
            }
        }
        // ---- scales, and what lies past the end
        f32x4 ks[2], vs[2];
        if (BITS != 16) {
#pragma unroll
            for (int tb = 0; tb < 2; ++tb) {
                ks[tb] = *LDS_AT(f32x4, lds_base, slot + S::kScales + 64 * tb + 16 * g);
                vs[tb] = *LDS_AT(f32x4, lds_base, slot + S::kScales + 256 + 64 * tb + 16 * g);
            }
        }
        if (!whole) {
#pragma unroll
            for (int tb = 0; tb < 2; ++tb)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (16 * tb + 4 * g + i < left) continue;
                    if (BITS != 16) ks[tb][i] = 1.f, vs[tb][i] = 0.f;
#pragma unroll
                    for (int j = 0; j < NH; ++j) s[j][tb][i] = -INFINITY;
                }
            for (int at = left * S::kVRow + lane * 16; at < kUnitTokens * S::kVRow; at += 1024)
                *LDS_AT(u32x4, lds_base, slot + S::kKBytes + at) = (u32x4){0, 0, 0, 0};
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");              // the keys and scales have been read, the value rows cleared
        if (left_next > 0) request(row_next, left_next, std::false_type{});
        // ---- softmax
        bf16x8 p[NH], p_rest[NH];
#pragma unroll
        for (int j = 0; j < NH; ++j) {
            // Reference and exponents, in units of c: raw scores (bf16; their differences are exact where it matters, and a sequence of one token is its
            // value row to the bit, infinities included) or scores in the log2 domain (codes)
            float factor[8], top = -INFINITY;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                factor[t] = BITS == 16 ? 1.0f : a.scale_log2e * ks[t >> 2][t & 3];
                top = fmaxf(top, s[j][t >> 2][t & 3] * factor[t]);
            }
            // (the reference moves when the maximum is more than 2^kLag ahead of it: weights up to that, and few rescales)
            constexpr float kLag = 8.0f;
            const float seen = head_max(fmaxf(m[j], top));
            const float m_new = (seen - m[j]) * c > kLag ? seen : m[j], m_safe = m_new == -INFINITY ? 0.f : m_new;
            const float keep = fast_exp2((m[j] - m_safe) * c);
            m[j] = m_new;
            if (__any(keep != 1.0f)) {
                l[j] *= keep;
#pragma unroll
                for (int i = 0; i < S::kDimBlocks; ++i) acc[j][i] *= keep;
            }
            // weights (times value scales) as two bf16 terms
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const float w = fast_exp2(BITS == 16 ? (s[j][t >> 2][t & 3] - m_safe) * c : __builtin_fmaf(s[j][t >> 2][t & 3], factor[t], -m_safe));
                l[j] += w;
                __bf16 first, rest;
                two_terms<BOTH_POSITIVE>(BITS == 16 ? w : w * vs[t >> 2][t & 3], first, rest);
                p[j][t] = first;
                p_rest[j][t] = rest;
            }
        }
        // ---- weighted sum
        const int vb = slot + S::kKBytes;
        // Two blocks at a time: the two instructions on the same sums are not neighbours
#pragma unroll
        for (int i = 0; i < S::kDimBlocks; i += 2) {
            bf16x8 v[2];
            if constexpr (BITS == 4) {
                // sixteen "rows" of eight bytes: the eight tokens in dims of block i, then in those of block i + 1
                const int r = 4 * g + (n & 3) + 16 * ((n >> 2) & 1);
                const int at = vb + r * S::kVRow + 16 * S::value_chunk(i >> 1, r) + 8 * (n >> 3);
                const i32x2 x = __builtin_amdgcn_ds_read_tr4_b64_v2i32(LDS_AT(i32x2, lds_base, at));
                v[0] = expand((uint32_t)x[0], 0);
                v[1] = expand((uint32_t)x[1], 0);
            } else {
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    if constexpr (BITS == 16) {
                        Bf16s both;
#pragma unroll
                        for (int tb = 0; tb < 2; ++tb) {
                            const int r = 16 * tb + 4 * g + (n >> 2);   // (a lane names eight of a row's 32 bytes)
                            const int at = vb + r * S::kVRow + 16 * S::value_chunk(2 * (i + k), r) + 8 * (n & 3);
                            both.h[tb] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_AT(s16x4, lds_base, at));
                        }
                        v[k] = both.v;
                    } else {
                        const int r = 4 * g + ((n >> 1) & 3) + 16 * (n >> 3);   // (eight rows, eight of a row's 16 bytes)
                        const int at = vb + r * S::kVRow + 16 * S::value_chunk(i + k, r) + 8 * (n & 1);
                        const i32x2 x = __builtin_amdgcn_ds_read_tr8_b64_v2i32(LDS_AT(i32x2, lds_base, at));
                        v[k] = expand((uint32_t)x[0], (uint32_t)x[1]);
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < NH; ++j) {
#pragma unroll
                for (int k = 0; k < 2; ++k) acc[j][i + k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v[k], p_rest[j], acc[j][i + k], 0, 0, 0);
#pragma unroll
                for (int k = 0; k < 2; ++k) acc[j][i + k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v[k], p[j], acc[j][i + k], 0, 0, 0);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");              // the values have been read
        if (left_next > 0) request(row_next, left_next, std::true_type{});
    }

    // ---- the waves' results added up
    wait_vmem_but<0>();                                                 // (a unit asked for ahead of a shorter length)
    const int units = end > 0 ? (end + kUnitTokens - 1) / kUnitTokens : 0;
    const int mine = CUT ? (units - run + runs - 1) / runs : units, n_active = mine < S::kWaves ? mine : S::kWaves;   // (below 1: no tokens)
    const bool partial = CUT && len > 0;                                // (an empty sequence: zeros by its first run, and nothing is merged)
    const size_t slot_out = CUT ? ((size_t)b * runs + run) * a.q_len + qtok : 0;
    float finite = 0.f;                                                 // NaN once a sum is not
#pragma unroll
    for (int j = 0; j < NH; ++j) {
        __syncthreads();                                                // nobody reads a unit, or the results of the heads before, any more
        l[j] = head_sum(l[j]);
        if (!BOTH_POSITIVE && j == 0 && thread == 0) *LDS_AT(int, lds_base, S::kVote) = 0;
#pragma unroll
        for (int i = 0; i < S::kDimBlocks; ++i) *LDS_AT(f32x4, lds_base, wave * S::kAccBytes + i * 1024 + lane * 16) = acc[j][i];
        const int ml = S::kMlBase + n * 4;
        if (g == 0) {
            *LDS_AT(float, lds_base, ml + wave * 128) = m[j];
            *LDS_AT(float, lds_base, ml + wave * 128 + 64) = l[j];
        }
        __syncthreads();
        float top = -INFINITY, l_sum = 0.f;
        for (int w = 0; w < n_active; ++w) top = fmaxf(top, *LDS_AT(float, lds_base, ml + w * 128));
        const float m_safe = top == -INFINITY ? 0.f : top;
        f32x4 sum[(S::kDimBlocks + S::kWaves - 1) / S::kWaves];         // of blocks wave, wave + kWaves, ..
        for (int w = 0; w < n_active; ++w) {
            const float weight = fast_exp2((*LDS_AT(float, lds_base, ml + w * 128) - m_safe) * c);
            l_sum += weight * *LDS_AT(float, lds_base, ml + w * 128 + 64);
#pragma unroll
            for (int i = 0, block = wave; i * S::kWaves < S::kDimBlocks; ++i, block += S::kWaves) {
                if (block >= S::kDimBlocks) break;
                const f32x4 part = *LDS_AT(f32x4, lds_base, w * S::kAccBytes + block * 1024 + lane * 16);
                sum[i] = w == 0 ? weight * part : sum[i] + weight * part;
            }
        }
        // (a row without tokens is zero; one of nothing but -inf scores is not)
        const float inv = partial ? 1.0f : 1.0f / l_sum;
        if (partial && wave == 0 && block0 == 0 && g == 0) *(float2*)(a.ws_ml + (slot_out * kHeads + head0 + 16 * j + n) * 2) = make_float2(top * c, l_sum);
#pragma unroll
        for (int i = 0, block = wave; i * S::kWaves < S::kDimBlocks; ++i, block += S::kWaves) {
            if (block >= S::kDimBlocks) break;
            if (!BOTH_POSITIVE && n_active > 0)
#pragma unroll
                for (int k = 0; k < 4; ++k) finite = __builtin_fmaf(sum[i][k], 0.f, finite);
            const f32x4 result = n_active > 0 ? sum[i] * inv : (f32x4){0.f, 0.f, 0.f, 0.f};
            if (partial) ((f32x4*)a.ws_acc)[(slot_out * (kHeads / 16) + (head0 / 16 + j)) * 1024 + (block0 + block) * 64 + lane] = result;
            else *(f32x4*)(a.out + ((size_t)row * kHeads + head0 + 16 * j + n) * kHeadDim + 16 * (block0 + block) + 4 * g) = result;
        }
    }
    if constexpr (BOTH_POSITIVE) return false;
    if (__any(!(finite == 0.f))) *LDS_AT(int, lds_base, S::kVote) = 1;
    __syncthreads();
    return *LDS_AT(int, lds_base, S::kVote) != 0;
}

template <bool PAGED, int BITS, int NH, int DS, bool CUT>
__global__ __launch_bounds__((BriefShape<BITS, NH, DS>::kThreads)) __attribute__((amdgpu_waves_per_eu(NH == 2 ? 1 : 2, NH == 2 ? 1 : 2))) void brief_attn_kernel(AttnArgs a)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const lds_ptr_t lds_base = (lds_ptr_t)smem;
    if (!brief_attn<PAGED, BITS, NH, DS, CUT, false>(a, lds_base)) return;
    __syncthreads();                                                    // everyone has read the vote; units may come in
    brief_attn<PAGED, BITS, NH, DS, CUT, true>(a, lds_base);
}

}  // namespace mfa
