// Decode attention over the 8-bit and the 4-bit cache for little work per workgroup (the rule is short_lowbit_work() in mfa_attn.hip).
//
// Eight waves of 16 heads, 64-token tiles, scores on the 16x16x128 fp8/fp4 matrix instruction and the weighted sum on the
// bf16 one from values converted once per tile.  Per tile it takes about 1.15 (8 bit) to 1.25 times (4 bit) what decode_lowbit_kernel takes,
// but a segment begins and ends in less: its query fragments (64 values per lane) are converted straight from registers, two waves per SIMD
// cover each other's waits, and there is no pipeline to fill.
#pragma once
#include "mfa_lowbit.hpp"

namespace mfa {
namespace few {

// A lane's query operands: q * 2^e = hi + lo as in decode_lowbit_kernel.
//   8 bit: head n, d = 128*c + 32*g + j (j = 0..31, one byte each, in register order)
//   4 bit: the keys are e2m1 operands (16 bytes per lane and 128 elements).  Measured on the device with one-hot operands: with an
//          e2m1 A and an e4m3 B operand, element j of A's lane group g multiplies byte 16*(g >> 1) + (j & 15) of B's lane
//          group 2*(g & 1) + (j >> 4).  The keys keep the plain order (a lane holds d = 128*c + 32*g + j, one
//          16-byte read), so the query takes the matching one: d = 128*c + 64*(j >> 4) + 16*g + (j & 15).
struct Query { i32x8 hi[2]; i32x8 lo[2]; float inv_scale; };

template <int BITS>
__device__ __forceinline__ void load_split_q(Query& q, const void* qptr, int b, int head, int g)
{
    const bf16x8* qp = (const bf16x8*)((const uint16_t*)qptr + ((size_t)b * kHeads + head) * kHeadDim + (BITS == 8 ? 32 : 16) * g);
    bf16x8 qf[2][4];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) qf[c][i] = qp[c * 16 + (BITS == 8 ? i : 8 * (i >> 1) + (i & 1))];
    float amax = 0.f;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) amax = fmaxf(amax, fabsf((float)qf[c][i][j]));
    amax = head_max(amax);
    int e = (int)((__float_as_uint(amax) >> 23) & 0xFFu);          // biased exponent of the largest element
    e = e < 24 ? 24 : e;                                           // (all-zero or vanishing heads: any scale will do)
    const float scale = __uint_as_float((uint32_t)(261 - e) << 23);   // amax * scale in [128, 256)
    q.inv_scale = __uint_as_float((uint32_t)(e - 7) << 23);
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                float x[4], r[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) x[j] = (float)qf[c][i][4 * w + j] * scale;
                int h = __builtin_amdgcn_cvt_pk_fp8_f32(x[0], x[1], 0, false);
                h = __builtin_amdgcn_cvt_pk_fp8_f32(x[2], x[3], h, true);
                const auto h01 = __builtin_amdgcn_cvt_pk_f32_fp8(h, false);
                const auto h23 = __builtin_amdgcn_cvt_pk_f32_fp8(h, true);
                r[0] = x[0] - h01[0]; r[1] = x[1] - h01[1]; r[2] = x[2] - h23[0]; r[3] = x[3] - h23[1];
                int l = __builtin_amdgcn_cvt_pk_fp8_f32(r[0], r[1], 0, false);
                l = __builtin_amdgcn_cvt_pk_fp8_f32(r[2], r[3], l, true);
                q.hi[c][2 * i + w] = h;
                q.lo[c][2 * i + w] = l;
            }
}

// One 32-token unit: scores, online softmax, weighted sum.
//   kbase      LDS byte offset of the unit's keys:
//                8 bit: 32 rows of 256 B of e4m3 codes, 16-byte chunk c of row r at c ^ (r & 15)
//                4 bit: 32 rows of 128 B of packed e2m1 codes, 16-byte chunk c of row r at c ^ ((r >> 1) & 7)
//   vbase      LDS byte offset of the unit's values in bf16 (the codes expanded, unscaled); layout at pv_unit
//   unit_t0    index (within the sequence) of the unit's first token; tokens >= t1 are masked
//   kscale_off, vscale_off   the fp32 per-token scales of the unit's 32 tokens
template <int BITS>
__device__ __forceinline__ RawScores qk_unit(const Query& q, lds_ptr_t lds_base, int kbase, int n, int g)
{
    f32x4 s[2] = {(f32x4){0.f, 0.f, 0.f, 0.f}, (f32x4){0.f, 0.f, 0.f, 0.f}};
    if constexpr (BITS == 4) {
        // e2m1 keys x e4m3 query terms with unit block scales (E8M0 exponent 127)
        constexpr int kOne = 0x7F7F7F7F;
        // both query terms go into one accumulator per 16-token block: two independent chains keep the MFMA
        // pipe fed, and the small term is added first
#pragma unroll
        for (int c = 0; c < 2; ++c) {
#pragma unroll
            for (int tb = 0; tb < 2; ++tb) {
                const int row = kbase + tb * 2048 + n * 128;
                const u32x4 k4 = *LDS_AT(u32x4, lds_base, row + (((4 * c + g) ^ ((n >> 1) & 7)) << 4));
                const i32x8 kf = {(int)k4[0], (int)k4[1], (int)k4[2], (int)k4[3], 0, 0, 0, 0};
                s[tb] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(kf, q.lo[c], s[tb], 4, 0, 0, kOne, 0, kOne);
                s[tb] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(kf, q.hi[c], s[tb], 4, 0, 0, kOne, 0, kOne);
            }
        }
    } else {
        // e4m3 x e4m3 with unit block scales (E8M0 exponent 127)
        constexpr int kOne = 0x7F7F7F7F;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
#pragma unroll
            for (int tb = 0; tb < 2; ++tb) {
                const int row = kbase + tb * 4096 + n * 256;
                const int m = 8 * c + 2 * g;                       // first of this lane's two 16-byte chunks
                union { i32x8 v; u32x4 h[2]; } kf;
                kf.h[0] = *LDS_AT(u32x4, lds_base, row + ((m ^ n) << 4));
                kf.h[1] = *LDS_AT(u32x4, lds_base, row + (((m + 1) ^ n) << 4));
                s[tb] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(kf.v, q.lo[c], s[tb], 0, 0, 0, kOne, 0, kOne);
                s[tb] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(kf.v, q.hi[c], s[tb], 0, 0, 0, kOne, 0, kOne);
            }
        }
    }
    RawScores r;
    r.s[0] = s[0];
    r.s[1] = s[1];
    return r;
}
// Online softmax of a unit from its raw scores, and the rescale of what has been accumulated so far. Returns the
// attention weights as the B operand of the weighted sum (8 tokens of this lane's head).
__device__ __forceinline__ bf16x8 softmax_unit(WaveState& st, const Query& q, const RawScores& raw, lds_ptr_t lds_base,
                                               int unit_t0, int t1, float scale_log2e, int g, int kscale_off, int vscale_off)
{
    f32x4 s[2] = {raw.s[0], raw.s[1]};
    scale_log2e *= q.inv_scale;
    f32x4 vsc[2];
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
        const f32x4 ksc = *LDS_AT(f32x4, lds_base, kscale_off + (16 * tb + 4 * g) * 4);
        vsc[tb] = *LDS_AT(f32x4, lds_base, vscale_off + (16 * tb + 4 * g) * 4);
        s[tb] *= ksc;
    }

    // ---- online softmax in the log2 domain.  The raw scores are compared first and scaled inside the
    // exponent's fused multiply-add (the scale is positive); only a unit that reaches past t1, the last
    // of a sequence at most, spends instructions on masking.
    float sv[8];
    float m_raw = -INFINITY;
    if (unit_t0 + kUnitTokens <= t1) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            sv[j] = s[j >> 2][j & 3];
            m_raw = fmaxf(m_raw, sv[j]);
        }
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int tok = unit_t0 + 16 * (j >> 2) + 4 * g + (j & 3);
            sv[j] = tok < t1 ? s[j >> 2][j & 3] : -INFINITY;
            m_raw = fmaxf(m_raw, sv[j]);
        }
    }
    // The reference exponent st.m follows the running maximum lazily: it moves only when the maximum
    // has run ahead of it by more than kRescaleLag, so weights reach at most 2^kRescaleLag (harmless in
    // bf16 and fp32) and the 64 accumulator registers are rescaled a few times per sequence instead of
    // whenever some head of the wave sees a new maximum.  The normalisation at the end is unaffected.
    constexpr float kRescaleLag = 8.0f;
    const float m_seen = head_max(fmaxf(st.m, m_raw * scale_log2e));
    const float m_new = m_seen > st.m + kRescaleLag ? m_seen : st.m;   // (-inf + lag = -inf: the first token always moves it)
    const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
    const float alpha = fast_exp2(st.m - m_safe);      // 1 when unmoved; 0 while nothing has been accumulated
    st.m = m_new;

    bf16x8 pf;
    float psum = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        // the value scale rides on the weight; the normaliser sums the unscaled weight
        const float p = fast_exp2(__builtin_fmaf(sv[j], scale_log2e, -m_safe));
        pf[j] = (__bf16)(p * vsc[j >> 2][j & 3]);
        psum += p;
    }
    st.l = st.l * alpha + psum;

    if (__any(alpha != 1.0f)) {
#pragma unroll
        for (int db = 0; db < 16; ++db) st.acc[db] *= alpha;
    }
    return pf;
}

// Second half of a unit: O^T += V^T P^T over the unit's 32 tokens.  Value rows are kPaddedVRow = 544 bytes apart: the 32 bytes of padding
// shift consecutive rows by eight banks, which spreads a transposing read (4 rows x 32 bytes per 16 lanes, 8 rows per
// half wave) over all 64 banks, and every operand address is one lane register plus a compile-time offset.
// Within a row the 16-byte pieces are placed so that the lanes of one 16-byte store instruction (store_tile) spread over the
// banks whether the hardware takes them 8 or 16 at a time; in the plain order they collide two by two:
//   8 bit: a thread owns the 32-byte chunk c of a row; its two 16-byte halves are swapped when bits 2 and 3 of c
//          differ (chunks 4..11);
//   4 bit: a thread owns the 64-byte group c of four pieces; piece w sits at position (w + (c >> 1)) & 3 of the group.
// A reader knows the chunk (db) at compile time, so undoing this costs it lane registers and no instruction.
constexpr int kPaddedVRow = 544;
constexpr int kPaddedVUnitBytes = kUnitTokens * kPaddedVRow;      // 17408
__host__ __device__ constexpr bool padded_v_halves_swapped(int chunk32) { return (((chunk32 >> 2) ^ (chunk32 >> 3)) & 1) != 0; }
__host__ __device__ constexpr int padded_v_rotation(int group64) { return (group64 >> 1) & 3; }
template <int BITS>
__device__ __forceinline__ void pv_unit(WaveState& st, lds_ptr_t lds_base, int vbase, const bf16x8& pf, int n, int g)
{
    const int v_row = 4 * g + (n >> 2);                 // V: row within a 16-token block (= swizzle key)
    const int piece = n & 3;                            // which 8 bytes of the 32-byte chunk this lane supplies
    const int v_lane_off = v_row * kPaddedVRow + (piece << 3);
    // 8 bit: [1] = halves swapped.  4 bit: [k] = the chunk's first piece sits at position k of its 64-byte group
    // (offsets relative to the group).
    int v_lane_alt[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        v_lane_alt[k] = BITS == 8 ? (k == 1 ? v_lane_off ^ 16 : v_lane_off)
                                  : v_row * kPaddedVRow + 16 * ((k + (piece >> 1)) & 3) + 8 * (piece & 1);
    union VFrag { bf16x8 v; s16x4 h[2]; };
    auto read_v = [&](VFrag& f, int db) {
        int lane_off = v_lane_off, place = db << 5;
        if (BITS == 8) lane_off = v_lane_alt[padded_v_halves_swapped(db) ? 1 : 0];
        if (BITS == 4) {
            lane_off = v_lane_alt[(2 * (db & 1) + padded_v_rotation(db >> 1)) & 3];
            place = (db >> 1) << 6;
        }
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
            const int off = vbase + tb * 16 * kPaddedVRow + lane_off + place;
            f.h[tb] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_AT(s16x4, lds_base, off));
        }
    };
    // The operands of kAhead output blocks are on their way while one block is multiplied: an LDS read takes
    // several times as long as the MFMA it feeds, and a wave has only one other wave on its SIMD to hide it.
    constexpr int kAhead = 4;
    VFrag f[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) read_v(f[i], i);
#pragma unroll
    for (int db = 0; db < 16; ++db) {
        __builtin_amdgcn_sched_barrier(0);
        st.acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[db % kAhead].v, pf, st.acc[db], 0, 0, 0);
        if (db + kAhead < 16) read_v(f[db % kAhead], db + kAhead);
    }
    __builtin_amdgcn_sched_barrier(0);
}

// Keys stay codes all the way: each tile's rows go by direct loads into a ring of three LDS slots.  Values: every thread carries 32
// bytes (8 bit: two 16-byte pieces; 4 bit: one) and one per-token scale in registers from HBM, converts them (exactly: every
// e4m3 and e2m1 value is a bf16 value) and writes the bf16 rows into one of two value images.
//
// LDS: value image P (P = tile & 1) at P*34 KB, its unit g at + g*17 KB; key slot k (tile % 3) at 68 KB + k*16 KB (4 bit: the
// first 8 KB of it); scale set P at 116 KB + P*512 B (64 key scales, then 64 value scales).
constexpr int kLbVImageBytes = 2 * kPaddedVUnitBytes;    // two units of 32 padded bf16 rows
constexpr int kLbKBase = 2 * kLbVImageBytes;
constexpr int kLbKSlotBytes = kTile * 256;
constexpr int kLbKSlots = 3;
constexpr int kLbScaleBase = kLbKBase + kLbKSlots * kLbKSlotBytes;
constexpr int kLbLdsBytes = kLbScaleBase + 2 * 512;
static_assert(kLbLdsBytes <= kBf16SchedOffset, "the schedule lives where that of the bf16 kernels does, behind the exchange area");

struct LowbitTileRegs {
    u32x4 piece[2];       // 8 bit: V rows prow and prow + 32, 16-byte chunk pchunk; 4 bit: piece[0] only,
                          // V row tid / 8, 16-byte chunk tid % 8 (32 elements)
    float scale;          // threads 0..63: key scale of token tid; 64..127: value scale of token tid - 64
};
// Every step of the pipeline issues, per wave and in this order, the register loads of a tile
// (8 bit: two pieces and a scale; 4 bit: one piece and a scale) and the direct loads of a key tile
// (8 bit: two; 4 bit: one).  They are inline assembly, awaited with an explicit vmcnt that leaves
// exactly the youngest step's loads in flight: left to the compiler, the wait would be widened to
// vmcnt(0) at the loop's control-flow joins and drain the pipeline every tile.  The registers pass
// through the waiting statement, so no use of them can be scheduled before it.
template <int BITS> constexpr int kLowbitOpsPerStep = BITS == 8 ? 5 : 3;
// (address = wave-uniform base in scalar registers + 32-bit byte offset per lane; non-temporal: read once)
__device__ __forceinline__ void load_regs_16B(u32x4& dst, const void* sbase, uint32_t voff)
{
    asm volatile("global_load_dwordx4 %0, %1, %2 nt" : "=&v"(dst) : "v"(voff), "s"(sbase) : "memory");
}
__device__ __forceinline__ void load_regs_4B(float& dst, const void* sbase, uint32_t voff)
{
    asm volatile("global_load_dword %0, %1, %2 nt" : "=&v"(dst) : "v"(voff), "s"(sbase) : "memory");
}
template <int BITS>
__device__ __forceinline__ void wait_all_but_youngest_step(LowbitTileRegs& t)
{
    if constexpr (BITS == 8) {
        static_assert(kLowbitOpsPerStep<8> == 5, "the wait below leaves 5 operations in flight");
        asm volatile("s_waitcnt vmcnt(5)" : "+v"(t.piece[0]), "+v"(t.piece[1]), "+v"(t.scale) :: "memory");
    } else {
        static_assert(kLowbitOpsPerStep<4> == 3, "the wait below leaves 3 operations in flight");
        asm volatile("s_waitcnt vmcnt(3)" : "+v"(t.piece[0]), "+v"(t.scale) :: "memory");
    }
}
// Wait for every load in flight while both register sets are still owned by the pipeline: no
// register of theirs may be handed to other code before its load has landed.
template <int BITS>
__device__ __forceinline__ void drain_tiles(LowbitTileRegs& t, LowbitTileRegs& u)
{
    if constexpr (BITS == 8)
        asm volatile("s_waitcnt vmcnt(0)"
                     : "+v"(t.piece[0]), "+v"(t.piece[1]), "+v"(t.scale), "+v"(u.piece[0]), "+v"(u.piece[1]), "+v"(u.scale)
                     :: "memory");
    else
        asm volatile("s_waitcnt vmcnt(0)" : "+v"(t.piece[0]), "+v"(t.scale), "+v"(u.piece[0]), "+v"(u.scale) :: "memory");
}

}  // namespace few

template <bool PAGED, int QL, int BITS>
__global__ __launch_bounds__(kAttnThreads) void short_lowbit_kernel(AttnArgs a)
{
    using namespace few;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const lds_ptr_t lds_base = (lds_ptr_t)smem;
    const uint32_t lds_addr0 = (uint32_t)(uintptr_t)lds_base;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wq = wave & 3;
    const int grp = wave >> 2;
    const int n = lane & 15;
    const int g = lane >> 4;

    stage_lengths(a, lds_base, kBf16SchedOffset);
    await_lengths<0>(a, false);
    Schedule sched = schedule_begin<kAttnThreads>(a, lds_base, kBf16SchedOffset, kShortLowbitSwitch);
    Segment r;
    bool first_segment = true;
    while (schedule_next<kAttnThreads>(a, sched, r)) {
        if (!first_segment) __syncthreads();          // the previous segment's exchange area is the tile memory
        first_segment = false;

        // Tiles past the end of the segment repeat its last tile (never consumed), so that every step
        // issues the same number of loads.  Rows at or past t1 re-read the last valid token.
        constexpr int kRowBytes = BITS == 8 ? 256 : 128;                   // one cached row of K or V
        const int prow = BITS == 8 ? threadIdx.x >> 4 : threadIdx.x >> 3;  // 8 bit: 0..31 (and + 32); 4 bit: 0..63
        const int pchunk = BITS == 8 ? threadIdx.x & 15 : threadIdx.x & 7; // 16-byte chunk of the row
        auto tile_origin = [&](int tile, int& tile_t0, int64_t& row0, int& last) {
            if (tile >= r.n_tiles) tile = r.n_tiles - 1;
            tile = __builtin_amdgcn_readfirstlane(tile);                   // keeps the page lookup a scalar load
            tile_t0 = r.t0 + tile * kTile;
            row0 = tile_row0<PAGED>(a, r.b, tile_t0, lookup_page<PAGED>(a, r.b, tile_t0));
            last = r.t1 - 1 - tile_t0;                                    // last valid row of this tile (>= 0)
        };
        auto load_tile = [&](LowbitTileRegs& t, int tile) {
            int tile_t0, last; int64_t row0;
            tile_origin(tile, tile_t0, row0, last);
#pragma unroll
            for (int i = 0; i < (BITS == 8 ? 2 : 1); ++i) {
                const int row = prow + 32 * i;
                const int in_tile = row > last ? last : row;
                load_regs_16B(t.piece[i], (const unsigned char*)a.v + row0 * kRowBytes, (uint32_t)(in_tile * kRowBytes + pchunk * 16));
            }
            const int tok = lane;                                          // waves 2.. repeat those of waves 0 and 1
            const int in_tile = tok > last ? last : tok;
            load_regs_4B(t.scale, ((wave & 1) ? a.v_scale : a.k_scale) + row0, (uint32_t)(in_tile * 4));
        };
        // Keys of a tile.  8 bit: 16 direct loads of 4 rows, wave w issues loads 2w and 2w + 1, 16-byte
        // chunk c of row r lands at c ^ (r & 15).  4 bit: 8 direct loads of 8 rows, one per wave, chunk c
        // of row r lands at c ^ ((r >> 1) & 7): 16 consecutive rows then spread one chunk column over all
        // 64 banks.
        auto issue_keys = [&](int tile, int kslot) {
            int tile_t0, last; int64_t row0;
            tile_origin(tile, tile_t0, row0, last);
            if constexpr (BITS == 8) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int first_row = 4 * (2 * wave + i);                     // wave-uniform
                    const int row = first_row + (lane >> 4);
                    const int in_tile = row > last ? last : row;
                    const int c16 = (lane & 15) ^ (row & 15);
                    load_to_lds_16B((const unsigned char*)a.k + row0 * 256, (uint32_t)(in_tile * 256 + c16 * 16),
                                    lds_addr0 + kLbKBase + kslot * kLbKSlotBytes + first_row * 256);
                }
            } else {
                const int first_row = 8 * wave;                                   // wave-uniform
                const int row = first_row + (lane >> 3);
                const int in_tile = row > last ? last : row;
                const int c16 = (lane & 7) ^ ((row >> 1) & 7);
                load_to_lds_16B((const unsigned char*)a.k + row0 * 128, (uint32_t)(in_tile * 128 + c16 * 16),
                                lds_addr0 + kLbKBase + kslot * kLbKSlotBytes + first_row * 128);
            }
        };
        // Convert a tile's value codes to bf16 and write them into image `image`; the scales go beside it.
        auto store_tile = [&](const LowbitTileRegs& t, int image) {
            if constexpr (BITS == 8) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    bf16x8 half[2];
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
                        const bf16x2 p01 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(t.piece[i][w], 1.0f, false);
                        const bf16x2 p23 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(t.piece[i][w], 1.0f, true);
                        half[w >> 1][4 * (w & 1) + 0] = p01[0];
                        half[w >> 1][4 * (w & 1) + 1] = p01[1];
                        half[w >> 1][4 * (w & 1) + 2] = p23[0];
                        half[w >> 1][4 * (w & 1) + 3] = p23[1];
                    }
                    // (halves swapped in some chunks: see pv_unit)
                    const int off = image * kLbVImageBytes + i * kPaddedVUnitBytes + prow * kPaddedVRow + (pchunk << 5) + (padded_v_halves_swapped(pchunk) ? 16 : 0);
                    *LDS_AT(bf16x8, lds_base, off) = half[0];
                    *LDS_AT(bf16x8, lds_base, off ^ 16) = half[1];
                }
            } else {
                // 32 elements = bf16 chunks 2*pchunk and 2*pchunk + 1 (32 bytes each) of row prow
                const int row_off = image * kLbVImageBytes + (prow >> 5) * kPaddedVUnitBytes + (prow & 31) * kPaddedVRow;
#pragma unroll
                for (int w = 0; w < 4; ++w) {                                  // word w: elements 8w .. 8w + 7
                    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
                    const bf16x2 p0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(t.piece[0][w], 1.0f, 0);
                    const bf16x2 p1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(t.piece[0][w], 1.0f, 1);
                    const bf16x2 p2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(t.piece[0][w], 1.0f, 2);
                    const bf16x2 p3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(t.piece[0][w], 1.0f, 3);
                    const bf16x8 eight = {p0[0], p0[1], p1[0], p1[1], p2[0], p2[1], p3[0], p3[1]};
                    // piece w of this thread's 64-byte group, rotated within the group (see pv_unit)
                    *LDS_AT(bf16x8, lds_base, row_off + (pchunk << 6) + (((w + padded_v_rotation(pchunk)) & 3) << 4)) = eight;
                }
            }
            if (threadIdx.x < 128) *LDS_AT(float, lds_base, kLbScaleBase + image * 512 + threadIdx.x * 4) = t.scale;
        };

        WaveState st;
        init_state(st);

        // Step t consumes tile t (value image t & 1, key slot t % 3) while it converts the values of
        // tile t+1 into the other image and has the registers of tiles t+2, t+3 and the keys of tiles
        // t+1, t+2 in flight.  Prologue: what steps -2 and -1 would have issued.
        LowbitTileRegs regs[2];
        load_tile(regs[0], 0);
        load_tile(regs[1], 1);
        issue_keys(0, 0);
        // The query fragments are loaded by ordinary loads: the compiler completes them, and with them
        // everything above, right here instead of inside the loop.
        Query q;
        load_split_q<BITS>(q, a.q, QL == 2 ? a.q_len * r.b + a.q0 + grp : r.b, 16 * wq + n, g);
        const int end_mine = r.len - (a.q_len - 1 - a.q0 - grp);      // QL == 2: grp = query token of the pair
        const int t1_mine = QL == 2 ? (r.t1 < end_mine ? r.t1 : end_mine) : r.t1;
        asm volatile("" : "+v"(q.hi[0]), "+v"(q.hi[1]), "+v"(q.lo[0]), "+v"(q.lo[1]));
        drain_tiles<BITS>(regs[0], regs[1]);
        store_tile(regs[0], 0);
        load_tile(regs[0], 2);
        issue_keys(1, 1);
        schedule_record(a, sched, r);

        int kslot = 0;                                                     // t % 3
        auto step = [&](auto parity_c, int t) {
            constexpr int P = decltype(parity_c)::value;                    // t & 1
            wait_all_but_youngest_step<BITS>(regs[P ^ 1]);       // registers of tile t+1 and keys of tile t have landed
            __syncthreads();                               // ... for every wave; everyone is done with tile t-1
            const int kb = kLbKBase + kslot * kLbKSlotBytes;
            const int vb = P * kLbVImageBytes;
            const int scales = kLbScaleBase + P * 512;
            // The score products of this wave's (first) unit are issued ahead of the conversion of the next tile's
            // values: the MFMA pipe and the LDS work while the vector ALU converts (4 % on the 8-bit workload,
            // compared on one device).
            const int u0 = QL == 2 ? 0 : grp;
            const RawScores raw0 = few::qk_unit<BITS>(q, lds_base, kb + u0 * kUnitTokens * kRowBytes, n, g);
            store_tile(regs[P ^ 1], P ^ 1);                                 // values of tile t+1
            load_tile(regs[P ^ 1], t + 3);
            issue_keys(t + 2, kslot == 0 ? 2 : kslot - 1);                  // (t + 2) % 3, the slot tile t-1 has left
            {
                const bf16x8 pf = few::softmax_unit(st, q, raw0, lds_base, r.t0 + t * kTile + u0 * kUnitTokens, t1_mine,
                                               a.scale_log2e, g, scales + u0 * kUnitTokens * 4, scales + 256 + u0 * kUnitTokens * 4);
                few::pv_unit<BITS>(st, lds_base, vb + u0 * kPaddedVUnitBytes, pf, n, g);
            }
            if (QL == 2) {
                const RawScores raw1 = few::qk_unit<BITS>(q, lds_base, kb + kUnitTokens * kRowBytes, n, g);
                const bf16x8 pf = few::softmax_unit(st, q, raw1, lds_base, r.t0 + t * kTile + kUnitTokens, t1_mine, a.scale_log2e, g,
                                               scales + kUnitTokens * 4, scales + 256 + kUnitTokens * 4);
                few::pv_unit<BITS>(st, lds_base, vb + kPaddedVUnitBytes, pf, n, g);
            }
            kslot = kslot == 2 ? 0 : kslot + 1;
        };
        for (int t = 0; t < r.n_tiles; t += 2) {
            step(std::integral_constant<int, 0>{}, t);
            if (t + 1 >= r.n_tiles) break;
            step(std::integral_constant<int, 1>{}, t + 1);
        }
        drain_tiles<BITS>(regs[0], regs[1]);  // the repeats of the last tile issued past the end
        if (QL == 2) finish_segment_two(st, a, r, grp, wq, lane);
        else         finish_segment(st, lds_base, 0, a, r, wq, grp, lane);
    }
}

}  // namespace mfa
