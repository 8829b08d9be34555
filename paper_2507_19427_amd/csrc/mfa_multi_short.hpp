// Three query tokens per sequence over a bf16 cache, for little work per workgroup (the rule is short_multi_work() in mfa_attn.hip).  Products, softmax and
// weighted sum of a unit follow one another, so a unit takes longer than in decode_bf16_multi_kernel, but a segment has no pipeline to
// fill and all four waves compute.
#pragma once
#include "mfa_multi.hpp"

namespace mfa {

constexpr int kThree = 3;                             // query tokens

// ---- One 32-token unit for three query tokens held by one wave (short_bf16_multi_kernel): every key fragment read from LDS
// feeds three score products and every value fragment three weighted-sum
// products, so the LDS traffic is that of a single token; the three accumulator chains are independent, which
// keeps the MFMA pipe busy from one wave.
//
// Registers.  3 x 64 accumulator registers and 3 x 32 of query fragments leave a wave (the only one on its
// SIMD) some 220 of its 512 registers for everything else, and only if the accumulators sit in the accumulation
// half of the file (where just MFMAs reach them) and nothing else does:
//   * the score products are written out as instructions with ordinary destination registers (the compiler gives
//     every MFMA of such a kernel an accumulation-register destination, which oversubscribes
//     that half); the wait states between the last of them and the first read of a score are inserted by hand;
//   * the accumulators are never rescaled: the reference exponent of a head is set by its first unit with a token
//     (or handed in) and then stays, and the weights of later tokens may grow to 2^kFixedReferenceLag relative to
//     it, harmless in bf16 and fp32.  A unit that would exceed that changes nothing and reports the exponents it
//     would need; the caller starts the segment again with them (short_bf16_multi_kernel).
__device__ __forceinline__ void mfma_bf16_into_vgprs(f32x4& acc, const bf16x8& a, const bf16x8& b)
{
    asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ bool process_unit_three(WaveState (&st)[kThree], const QFrags (&q)[kThree], lds_ptr_t lds_base, int kbase,
                                                   int vbase, int unit_t0, const int (&t1)[kThree], float scale_log2e, int n, int g,
                                                   float (&m_wanted)[kThree])
{
    f32x4 s[kThree][2];
#pragma unroll
    for (int t = 0; t < kThree; ++t) s[t][0] = s[t][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const int k_lane_off = n * 512;
    auto read_k = [&](int i) {                          // i = 2 * ks + tb
        return *LDS_AT(bf16x8, lds_base, kbase + (i & 1) * 8192 + k_lane_off + (((4 * (i >> 1) + g) ^ n) << 4));
    };
    bf16x8 kf[2] = {read_k(0), read_k(1)};
#pragma unroll
    for (int i = 0; i < 16; ++i) {                      // key fragments two ahead of their products
        const bf16x8 k_now = kf[i & 1];
        if (i + 2 < 16) kf[i & 1] = read_k(i + 2);
#pragma unroll
        for (int t = 0; t < kThree; ++t) mfma_bf16_into_vgprs(s[t][i & 1], k_now, q[t].f[i >> 1]);
    }
    // 16 wait states between an 8-pass MFMA and a read of its result by another unit of the SIMD; every score
    // passes through this statement, so nothing reads one before it
    asm volatile("s_nop 7\n\ts_nop 7" : "+v"(s[0][0]), "+v"(s[0][1]), "+v"(s[1][0]), "+v"(s[1][1]), "+v"(s[2][0]), "+v"(s[2][1]));

    // (the scores are masked in place, and only in a unit that reaches past a token's end: no second copy of them)
    float m_ref[kThree];
    bool moved = false;
#pragma unroll
    for (int t = 0; t < kThree; ++t) {
        if (unit_t0 + kUnitTokens > t1[t]) {           // (a real branch: the empty statement keeps it from becoming 8 selects per unit)
            asm volatile("");
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int tok = unit_t0 + 16 * (j >> 2) + 4 * g + (j & 3);
                if (tok >= t1[t]) s[t][j >> 2][j & 3] = -INFINITY;
            }
        }
        float m_raw = -INFINITY;
#pragma unroll
        for (int j = 0; j < 8; ++j) m_raw = fmaxf(m_raw, s[t][j >> 2][j & 3]);
        const float m_seen = head_max(fmaxf(st[t].m, m_raw * scale_log2e));
        m_ref[t] = st[t].m == -INFINITY ? m_seen : st[t].m;       // set once, by the head's first unit with a token
        m_wanted[t] = m_seen;
        moved = moved || m_seen > m_ref[t] + kFixedReferenceLag;
    }
    if (__any(moved)) return false;
    bf16x8 pf[kThree];
#pragma unroll
    for (int t = 0; t < kThree; ++t) {
        const float m_safe = m_ref[t] == -INFINITY ? 0.f : m_ref[t];
        st[t].m = m_ref[t];
        float psum = 0.f;
#pragma unroll
        for (int j = 0; j < 8; j += 2) {
            // normalise by the sum of the rounded weights actually multiplied into V
            const float p0 = fast_exp2(__builtin_fmaf(s[t][j >> 2][j & 3], scale_log2e, -m_safe));
            const float p1 = fast_exp2(__builtin_fmaf(s[t][j >> 2][(j & 3) + 1], scale_log2e, -m_safe));
            typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
            const bf16x2 pb = {(__bf16)p0, (__bf16)p1};
            pf[t][j] = pb[0];
            pf[t][j + 1] = pb[1];
            const uint32_t bits = __builtin_bit_cast(uint32_t, pb);
            psum += __uint_as_float(bits << 16) + __uint_as_float(bits & 0xFFFF0000u);
        }
        st[t].l += psum;
    }
    const int v_row = 4 * g + (n >> 2);
    const int v_lane_off = v_row * 512 + ((n & 3) << 3);
    union VFrag { bf16x8 v; s16x4 h[2]; };
    auto read_v = [&](VFrag& f, int db) {
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
            f.h[tb] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_AT(s16x4, lds_base, vbase + tb * 8192 + v_lane_off + ((db ^ v_row) << 5)));
    };
    constexpr int kAhead = 3;
    VFrag f[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) read_v(f[i], i);
#pragma unroll
    for (int db = 0; db < 16; ++db) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < kThree; ++t) st[t].acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[db % kAhead].v, pf[t], st[t].acc[db], 0, 0, 0);
        if (db + kAhead < 16) read_v(f[db % kAhead], db + kAhead);
    }
    __builtin_amdgcn_sched_barrier(0);
    return true;
}

// ---- Three query tokens per sequence in ONE pass over a bf16 cache (Section 5.2: the new tokens of a
// multi-token step share the cache read, which multiplies the arithmetic per byte by their number).
// A workgroup is four waves, one per SIMD, wave = head group: a wave holds all kThree query tokens of its 16 heads
// (3 x 32 registers of query fragments, 3 x 64 accumulator registers: only one wave fits a SIMD's register
// file) and works through both units of every tile; key and value fragments read from LDS are shared by the kThree
// tokens (process_unit_three).  Same tiles, same two-slot ring and same schedule as decode_bf16_kernel; each wave
// brings 16 rows of a tile.  Query token j attends to the first len - (q_len - 1 - j) cached tokens.  Batches of
// at most 512 sequences (every wave works the schedule out by itself).
constexpr int kShortMultiFlag = kBf16LdsBytes;
constexpr int kShortMultiLdsBytes = kShortMultiFlag + 16;
template <bool PAGED>
__global__ __launch_bounds__(kMultiThreads) void short_bf16_multi_kernel(AttnArgs a)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const lds_ptr_t lds_base = (lds_ptr_t)smem;
    const uint32_t lds_addr0 = (uint32_t)(uintptr_t)lds_base;

    const int lane = threadIdx.x & 63;
    const int wq = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15;
    const int g = lane >> 4;

    auto issue_tile = [&](const Segment& sg, int tile, int slot, int page) {
        const int tile_t0 = sg.t0 + tile * kTile;
        const int64_t row0 = tile_row0<PAGED>(a, sg.b, tile_t0, page);
        const unsigned char* k_tile = (const unsigned char*)a.k + row0 * 512;
        const unsigned char* v_tile = (const unsigned char*)a.v + row0 * 512;
        int lane_now = lane;                                          // (the lane's offsets are formed here, per tile, not
        asm volatile("" : "+v"(lane_now));                            // ahead of the tile loop and kept in scarce registers)
        const int p16 = lane_now & 31;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int row = 16 * wq + 2 * u + (lane_now >> 5);        // row of the tile this lane fills
            int in_tile = row;
            if (tile_t0 + row > sg.t1 - 1) in_tile = sg.t1 - 1 - tile_t0;
            const int key = row & 15;
            const int ck = p16 ^ key;
            const int cv = ((((p16 >> 1) ^ key) << 1) | (p16 & 1));
            const int first_row = 16 * wq + 2 * u;                     // wave-uniform
            const uint32_t dst = lds_addr0 + slot * kSlotBytes + (first_row >> 5) * kUnitBytes + (first_row & 31) * 512;
            load_to_lds_16B(k_tile, (uint32_t)(in_tile * 512 + ck * 16), dst);
            load_to_lds_16B(v_tile, (uint32_t)(in_tile * 512 + cv * 16), dst + kUnitVOffset);
        }
    };
    QFrags q[kThree];
    auto load_q = [&](const Segment& sg) {
        int lane_now = lane;                                          // (addresses formed here, once per segment)
        asm volatile("" : "+v"(lane_now));
#pragma unroll
        for (int t = 0; t < kThree; ++t) load_q_fragments(q[t].f, a.q, a.q_len * sg.b + a.q0 + t, 16 * wq + (lane_now & 15), lane_now >> 4);
    };

    // A word of LDS behind the schedule's tables: set by a wave whose unit was refused (a score more than
    // 2^kFixedReferenceLag above its head's reference exponent), seen by all waves after the next barrier.
    stage_lengths(a, lds_base, kBf16SchedOffset);
    await_lengths<0>(a, false);
    Schedule sched = schedule_begin<kMultiThreads>(a, lds_base, kBf16SchedOffset, kMultiSwitch);
    Segment r;
    bool first_segment = true;
    while (schedule_next<kMultiThreads>(a, sched, r)) {
        if (!first_segment) __syncthreads();          // every wave is done with the previous segment's tiles
        first_segment = false;
        // Every segment leaves a partial result, also one that covers its whole sequence: partials are stored
        // straight from the accumulation registers, while a final result would have to pass all of them through
        // ordinary registers to be normalised.  The merge kernel normalises (AttnArgs::n_here >= 3).
        r.final_result = false;
        load_q(r);
        schedule_record(a, sched, r);
        int t1_mine[kThree];
        float m_floor[kThree];                            // reference exponents handed to the next attempt (-inf: none)
#pragma unroll
        for (int t = 0; t < kThree; ++t) {
            const int end_mine = r.len - (a.q_len - 1 - a.q0 - t);
            t1_mine[t] = r.t1 < end_mine ? r.t1 : end_mine;
            m_floor[t] = -INFINITY;
        }
        WaveState st[kThree];
        // One attempt streams the segment with fixed reference exponents.  If a unit is refused, its wave notes the
        // exponents it needs, raises the flag and stops computing; at the next barrier all waves see the flag and
        // the segment is streamed again from its first tile (every attempt ends with a higher reference for some
        // head, and a reference never exceeds the head's largest score: the attempts end).  Plausible attention
        // scores never get here; correctness does not depend on that.
        for (bool again = true; again;) {
            again = false;
            if (threadIdx.x == 0) *LDS_AT(int, lds_base, kShortMultiFlag) = 0;
#pragma unroll
            for (int t = 0; t < kThree; ++t) {
                init_state(st[t]);
                st[t].m = m_floor[t];
            }
            issue_tile(r, 0, 0, lookup_page<PAGED>(a, r.b, r.t0));
            int page_next = r.n_tiles > 1 ? lookup_page<PAGED>(a, r.b, r.t0 + kTile) : 0;
            bool refused = false;
            for (int it = 0; it < r.n_tiles; ++it) {
                const int slot = it & 1;
                wait_vmem_all();
                __syncthreads();                       // tile it has landed; the flag store of attempt start / of a refusal is visible
                if (*LDS_AT(int, lds_base, kShortMultiFlag) != 0) { again = true; break; }
                if (it + 1 < r.n_tiles) {
                    issue_tile(r, it + 1, slot ^ 1, page_next);
                    if (it + 2 < r.n_tiles) page_next = lookup_page<PAGED>(a, r.b, r.t0 + (it + 2) * kTile);
                }
                if (refused) continue;
#pragma unroll 1
                for (int u = 0; u < 2; ++u) {
                    const int unit = slot * kSlotBytes + u * kUnitBytes;
                    float m_wanted[kThree];
                    if (!process_unit_three(st, q, lds_base, unit, unit + kUnitVOffset, r.t0 + it * kTile + u * kUnitTokens,
                                                t1_mine, a.scale_log2e, n, g, m_wanted)) {
#pragma unroll
                        for (int t = 0; t < kThree; ++t) m_floor[t] = fmaxf(m_floor[t], m_wanted[t]);
                        if (lane == 0) *LDS_AT(int, lds_base, kShortMultiFlag) = 1;
                        refused = true;
                        break;
                    }
                }
            }
            if (!again) {
                // the last tile's refusal (if any) has not met a barrier yet
                __syncthreads();
                again = *LDS_AT(int, lds_base, kShortMultiFlag) != 0;
            }
            if (again) {
                wait_vmem_all();                       // a tile may still be on its way into the ring
                __syncthreads();                       // every wave has read the flag and left the tile loop
            }
        }
        int lane_now = lane;                          // (the result's addresses are formed here, once per segment)
        asm volatile("" : "+v"(lane_now));
#pragma unroll
        for (int t = 0; t < kThree; ++t) {
            finish_segment_two(st[t], a, r, t, wq, lane_now);
            __builtin_amdgcn_sched_barrier(0);        // one query token's accumulators at a time through ordinary registers
        }
    }
}

}  // namespace mfa
