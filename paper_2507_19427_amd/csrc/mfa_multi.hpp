// Decode attention over a bf16 cache for three and four query tokens per sequence in one pass over the cache.
//
// Workgroup: 4 waves, one per SIMD; wave = query token (three tokens: the fourth wave only brings tiles), and a wave works on
// its 64 heads as two blocks of 32 columns, 32 tokens (a unit) at a time:
//   scores  S^T[token, head] = K . Q^T    32x32x16 matrix instructions, A = key rows, B = query
//   output  O^T[d, head] += V^T . P^T     A = V^T, 32 dims x 16 tokens (transposing LDS reads), B = weights
// (lane = 32*h + n; a lane holds rows 8*(i/4) + 4*h + i%4, i = 0..15, of column n of a result).  The 16 scores of a lane are, in
// register order, the weights it has to supply to the second product; the value rows are read in the token order
// this implies.
//
// What bounds it: 64 matrix instructions of 32 cycles per unit and wave, about what memory takes to bring the unit, so everything
// else has to run beside them.  A wave is alone on its SIMD (256 accumulators, 128 registers of query), so the overlap is
// written out: the scores of unit s + 1 are taken beside the softmax of the second block of unit s, the weighted sum of unit s
// beside the softmax of the first block of unit s + 1.
// 64 x 4096 tokens, four query tokens, one product after the other (16 heads of all tokens per wave): 113.4 us a call, kernel 99.8; now
// 92.9 .. 99 by device, kernel 77 .. 82.  Of the kernel, without its matrix instructions, softmax and loads 32 remain (start, operand reads, 67 MB of
// partial results written); the merge that reads those takes 14.  Three units in flight instead of two: 1 % slower on average.
//
// The reference exponent of a column is set by its first unit and then stays: weights may grow to 2^kFixedReferenceLag relative to
// it, harmless in bf16 and fp32.  The true maximum is tracked beside it; if it ends up further ahead than that, the
// workgroup streams the segment once more with the maxima it has seen as references.  A first unit of nothing but -inf leaves
// the reference at -inf: any finite score after it is ahead of that, so such a segment takes the same way.
#pragma once
#include "mfa_lowbit.hpp"

namespace mfa {

constexpr int kMultiThreads = 256;
constexpr int kMultiDepth = 2;                        // units in flight (32 KB each)
constexpr int kMultiSlots = kMultiDepth + 1;          // ... beside the one in use; keys are used one unit ahead of values
constexpr int kMultiTensorUnit = kUnitTokens * 512;
constexpr int kMultiVBase = kMultiSlots * kMultiTensorUnit;
constexpr int kMultiFlag = 2 * kMultiVBase;
constexpr int kMultiSchedBase = kMultiFlag + 16;
constexpr int kMultiLdsBytes = kMultiSchedBase + kSchedLdsBytes;
constexpr int kMultiOps = 8;                          // direct loads of a wave per unit: four of keys, four of values
static_assert(kMultiLdsBytes <= 160 * 1024, "LDS of a compute unit");

struct MultiState {
    LowbitState half[2];      // of the columns 32*cb + n: element i of acc[db] is d = 32*db + 8*(i/4) + 4*h + i%4
};

__device__ __forceinline__ void mfma_bf16_scores_first(f32x16& d, const bf16x8& a, const bf16x8& b)
{
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_bf16_scores(f32x16& d, const bf16x8& a, const bf16x8& b)
{
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_bf16_output(f32x16& d, const bf16x8& a, const bf16x8& b)
{
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(a), "v"(b));
}

// LDS image of a unit: rows of 512 bytes; K: 16-byte piece c of row r at c ^ (r & 15); V: 32-byte group c of row r at
// c ^ 2*(r & 3) (a transposing read takes two groups of four rows per half wave: 256 bytes, every bank once).
struct MultiKeys {
    int lane_off;             // row n, piece h
    lds_ptr_t lds;
    int base;
    bf16x8 f[3];
    __device__ __forceinline__ void read(int i) { f[i % 3] = *LDS_AT(bf16x8, lds, base ^ ((i & 15) << 5)); }     // k step i % 16
    __device__ __forceinline__ void begin(int unit) { base = unit + lane_off; read(0); read(1); }
};
struct MultiValues {
    int lane_off;             // row 4*h + l16/4, group `side`
    lds_ptr_t lds;
    int base;
    union Frag { bf16x8 v; s16x4 p[2]; } f[3];
    __device__ __forceinline__ void read(int i)           // 32-dim block i / 2, tokens 16*(i & 1) ..
    {
#pragma unroll
        for (int m = 0; m < 2; ++m)
            f[i % 3].p[m] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_AT(s16x4, lds, (base ^ ((i >> 1) << 6)) + (16 * (i & 1) + 8 * m) * 512));
    }
    __device__ __forceinline__ void begin(int unit) { base = unit + lane_off; read(0); read(1); }
};

// Scores of one block of 32 columns -> weights.  step(k), k = 0..7, works on values 2k and 2k + 1; the normaliser sums the rounded
// weights.  MASKED: tokens at or past the end get the weight 0.
template <bool MASKED>
struct MultiSoftmax {
    f32x16& s;
    u32x4 (&w)[2];
    LowbitState& st;
    float c, m_safe;
    int tok_left;             // tokens left from the unit's first on, - 4*h
    __device__ __forceinline__ float masked(float x, int i) const { return MASKED && 8 * (i >> 2) + (i & 3) >= tok_left ? -INFINITY : x; }
    template <int K> __device__ __forceinline__ void step(Slot<K>)
    {
        const float x0 = masked(s[2 * K], 2 * K), x1 = masked(s[2 * K + 1], 2 * K + 1);
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        const bf16x2 pb = {(__bf16)fast_exp2(__builtin_fmaf(x0, c, -m_safe)), (__bf16)fast_exp2(__builtin_fmaf(x1, c, -m_safe))};
        int bits = __builtin_bit_cast(int, pb);
        pin(bits);
        st.s_max = fmaxf(fmaxf(st.s_max, x0), x1);    // (between the pinned weights and their first reader, which takes a wait state right behind them)
        pin(st.s_max);
        st.l += __uint_as_float((uint32_t)bits << 16);
        st.l += __uint_as_float((uint32_t)bits & 0xFFFF0000u);
        pin(st.l);
        w[K >> 2][K & 3] = (uint32_t)bits;
    }
    __device__ __forceinline__ void all()
    {
        for_slots([&](auto k) { step(k); }, std::make_integer_sequence<int, 8>{});
    }
};

template <bool PAGED, int NT>
__global__ __launch_bounds__(kMultiThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void decode_bf16_multi_kernel(AttnArgs a)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const lds_ptr_t lds = (lds_ptr_t)smem;
    const uint32_t lds_addr0 = (uint32_t)(uintptr_t)lds;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tok = wave;                             // query token
    const bool computes = NT == 4 || wave < NT;
    const int n = lane & 31, h = lane >> 5;

    // Direct loads: load u of a wave fills rows 8*u + 2*wave and the next of a unit; the permutation of the key pieces of odd u differs from that of
    // even u in bit 3 of the piece.
    const int row_mine = 2 * wave + h;                // (+ 8*u)
    const uint32_t k_src = (uint32_t)((n ^ row_mine) << 4), v_src = (uint32_t)((n ^ ((row_mine & 3) << 2)) << 4);
    const uint32_t lds_wave = lds_addr0 + 2 * wave * 512;

    struct Span { int b, t0, t1, n_units; };
    auto origin = [&](const Span& g, int unit) {
        unit = unit < g.n_units ? unit : g.n_units - 1;
        unit = __builtin_amdgcn_readfirstlane(unit);                    // keeps the page lookup a scalar load
        const int tile_t0 = g.t0 + (unit >> 1) * kTile;
        return tile_row0<PAGED>(a, g.b, tile_t0, lookup_page<PAGED>(a, g.b, tile_t0)) + (unit & 1) * kUnitTokens;
    };
    const uint32_t k_off[2] = {(uint32_t)(row_mine * 512) + k_src, (uint32_t)((row_mine + 8) * 512) + (k_src ^ 128)};
    const uint32_t v_off = (uint32_t)(row_mine * 512) + v_src;
    // Load i of the eight of an iteration (keys, then values), whole units only
    auto load_piece = [&](auto i, int64_t row_k, int64_t row_v, uint32_t k_dst, uint32_t v_dst) {
        constexpr int u = i.value & 3;
        if constexpr (i.value < 4)
            load_to_lds_16B_at<8 * u * 512>((const unsigned char*)a.k + row_k * 512 + (u >> 1) * 8192, k_off[u & 1], k_dst);
        else
            load_to_lds_16B_at<8 * u * 512>((const unsigned char*)a.v + row_v * 512 + u * 4096, v_off, v_dst);
    };
    // Keys or values of any unit; rows past the end re-read the last valid token
    auto load_unit = [&](bool value, const Span& g, int unit, int64_t row0, int slot) {
        unit = unit < g.n_units ? unit : g.n_units - 1;
        const int last = g.t1 - 1 - (g.t0 + unit * kUnitTokens);
        const unsigned char* base = (const unsigned char*)(value ? a.v : a.k) + row0 * 512;
        const uint32_t dst = lds_wave + (value ? kMultiVBase : 0) + slot * kMultiTensorUnit;
        int lane_now = lane;
        asm volatile("" : "+v"(lane_now));
#pragma unroll 1
        for (int u = 0; u < 4; ++u) {
            const int row = 8 * u + 2 * wave + (lane_now >> 5), piece = lane_now & 31;
            const int in_unit = row < last ? row : last;
            load_to_lds_16B(base, (uint32_t)(in_unit * 512 + ((value ? piece ^ ((row & 3) << 2) : piece ^ (row & 15)) << 4)), dst + 8 * u * 512);
        }
    };

    stage_lengths(a, lds, kMultiSchedBase);
    await_lengths<0>(a, false);
    Schedule sched = schedule_begin<kMultiThreads>(a, lds, kMultiSchedBase, kMultiSwitch);
    Segment r;
    while (schedule_next<kMultiThreads>(a, sched, r)) {
        // Every segment leaves a partial result, also one that covers its whole sequence; the merge kernel normalises
        // (AttnArgs::n_here >= 3).
        r.final_result = false;
        const Span span = {r.b, r.t0, r.t1, (r.t1 - r.t0 + kUnitTokens - 1) / kUnitTokens};
        const int n_units = span.n_units;
        const int n_whole = (r.t1 - r.t0) / kUnitTokens;
        const int end_mine = r.len - (a.q_len - 1 - a.q0 - tok);
        const int t1_mine = r.t1 < end_mine ? r.t1 : end_mine;
        // units without a masked token for any wave (tokens of the last units end before r.t1 for the earlier query tokens)
        const int t1_all = r.len - (a.q_len - 1 - a.q0) < r.t1 ? r.len - (a.q_len - 1 - a.q0) : r.t1;
        const int n_full = t1_all > r.t0 ? (t1_all - r.t0) / kUnitTokens : 0;
        auto tok_left = [&](int unit) { return t1_mine - (r.t0 + unit * kUnitTokens) - 4 * h; };
        auto k_of = [&](int slot) { return slot * kMultiTensorUnit; };
        auto v_of = [&](int slot) { return kMultiVBase + slot * kMultiTensorUnit; };

        bf16x8 q[2][16];
        {
            int lane_now = lane;                                       // (addresses formed here, once per segment)
            asm volatile("" : "+v"(lane_now));
            const int token = computes ? tok : 0;
            const bf16x8* src = (const bf16x8*)((const uint16_t*)a.q + (((size_t)r.b * a.q_len + a.q0 + token) * kHeads + (lane_now & 31)) * kHeadDim) + (lane_now >> 5);
#pragma unroll
            for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                for (int ks = 0; ks < 16; ++ks) q[cb][ks] = src[cb * 32 * (kHeadDim / 8) + 2 * ks];
        }
        MultiState st;
        st.half[0].m = st.half[1].m = -INFINITY;
        bool retried = false;
        for (bool again = true; again;) {
            if (threadIdx.x == 0) *LDS_AT(int, lds, kMultiFlag) = 0;
#pragma unroll 1
            for (int d = 0; d < kMultiDepth; ++d) {                     // (past the span's end: its last unit again)
                const int64_t o = origin(span, d);
                load_unit(false, span, d, o, d);
                load_unit(true, span, d, o, d);
            }
            if (!retried) schedule_record(a, sched, r);
            wait_vmem_but<0>();
            __syncthreads();
#pragma unroll
            for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                for (int ks = 0; ks < 16; ++ks) asm volatile("" : "+v"(q[cb][ks]));   // (landed: no wait of the compiler's inside the loops below)
            int64_t o[2] = {0, 0};                                     // of units s + kMultiDepth (values) and s + 1 + kMultiDepth (keys)
            if (kMultiDepth < n_units) {
                o[0] = origin(span, kMultiDepth);
                load_unit(false, span, kMultiDepth, o[0], kMultiDepth);
            }
            if (kMultiDepth + 1 < n_units) o[1] = origin(span, kMultiDepth + 1);

#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
#pragma unroll
                for (int i = 0; i < 8; ++i) st.half[cb].acc[i] = (f32x16)(0.f);
                output_ready(st.half[cb].acc);
                st.half[cb].s_max = -INFINITY;
                st.half[cb].l = 0.f;
            }
            const float c = a.scale_log2e;
            float m_safe[2];
            f32x16 sc[2];
            u32x4 w[2][2];                                             // weights of unit s: [column block][16-token step]
            MultiKeys keys{n * 512 + ((h ^ (n & 15)) << 4), lds};
            const int l16 = lane & 15, side = (lane >> 4) & 1;
            MultiValues values{(4 * h + (l16 >> 2)) * 512 + ((side ^ (2 * ((l16 >> 2) & 3))) << 5) + 8 * (l16 & 3), lds};
            // Scores of a unit: both column blocks in turn, the key operands read for each
            auto scores = [&](auto&& beside) {
                for_slots([&](auto k) {
                    constexpr int cb = k.value >> 4, ks = k.value & 15;
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (ks == 0) mfma_bf16_scores_first(sc[cb], keys.f[k.value % 3], q[cb][ks]);
                    else                   mfma_bf16_scores(sc[cb], keys.f[k.value % 3], q[cb][ks]);
                    if constexpr (k.value + 2 < 32) keys.read(k.value + 2);
                    beside(k);
                }, std::make_integer_sequence<int, 32>{});
                __builtin_amdgcn_sched_barrier(0);
            };
            auto weighted_sum = [&](auto&& beside) {
                for_slots([&](auto k) {
                    constexpr int f = k.value >> 1, cb = k.value & 1;
                    __builtin_amdgcn_sched_barrier(0);
                    mfma_bf16_output(st.half[cb].acc[f >> 1], values.f[f % 3].v, __builtin_bit_cast(bf16x8, w[cb][f & 1]));
                    if constexpr (cb == 0 && f + 2 < 16) values.read(f + 2);
                    beside(k);
                }, std::make_integer_sequence<int, 32>{});
                __builtin_amdgcn_sched_barrier(0);
            };
            // Vector-written weights are complete before a matrix instruction reads them (two wait states)
            auto weights_ready = [&]() { asm volatile("s_nop 1" : "+v"(w[0][0]), "+v"(w[0][1]), "+v"(w[1][0]), "+v"(w[1][1])); };

            int s = 0;
            int slot = 0, slot_prev = kMultiSlots - 1, slot_next = 1;   // of units s, s - 1 (= s + kMultiDepth) and s + 1
            if (computes) {
                keys.begin(k_of(0));
                scores([](auto) {});
                scores_ready(sc);
                const int left = tok_left(0);
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) {
                    float m = -INFINITY;
#pragma unroll
                    for (int i = 0; i < 16; ++i) m = fmaxf(m, 8 * (i >> 2) + (i & 3) >= left ? -INFINITY : sc[cb][i]);
                    if (st.half[cb].m == -INFINITY) st.half[cb].m = half_max(m) * c;      // (c > 0)
                    m_safe[cb] = st.half[cb].m == -INFINITY ? 0.f : st.half[cb].m;
                }
                MultiSoftmax<true>{sc[0], w[0], st.half[0], c, m_safe[0], left}.all();
            }
            auto advance = [&]() {
                o[0] = o[1];
                if (s + 2 + kMultiDepth < n_units) o[1] = origin(span, s + 2 + kMultiDepth);
                slot_prev = slot;
                slot = slot_next;
                slot_next = slot_next + 1 == kMultiSlots ? 0 : slot_next + 1;
                ++s;
            };
            // One iteration: scores of unit s + 1 beside the softmax of the second column block of unit s, then the weighted sum of unit s beside the
            // softmax of the first block of unit s + 1.  STEADY: requests keys s + 1 + kMultiDepth and values s + kMultiDepth, and no
            // token of units s and s + 1 is masked.
            auto iterate = [&](auto steady) {
                constexpr bool STEADY = decltype(steady)::value;
                const uint32_t k_dst = lds_wave + slot * kMultiTensorUnit, v_dst = lds_wave + kMultiVBase + slot_prev * kMultiTensorUnit;
                if (!computes) {
                    if constexpr (STEADY)
                        for_slots([&](auto i) { load_piece(i, o[1], o[0], k_dst, v_dst); }, std::make_integer_sequence<int, 8>{});
                    advance();
                    return;
                }
                keys.begin(k_of(slot_next));
                {
                    MultiSoftmax<!STEADY> f{sc[1], w[1], st.half[1], c, m_safe[1], STEADY ? 0 : tok_left(s)};
                    scores([&](auto k) {
                        if constexpr (k.value < 16 && (k.value & 1) == 0) f.step(Slot<k.value / 2>{});
                        if constexpr (STEADY && k.value >= 17 && k.value < 25) load_piece(Slot<k.value - 17>{}, o[1], o[0], k_dst, v_dst);
                        if constexpr (k.value == 29) values.begin(v_of(slot));
                    });
                }
                weights_ready();
                {
                    u32x4 w_next[2];
                    MultiSoftmax<!STEADY> f{sc[0], w_next, st.half[0], c, m_safe[0], STEADY ? 0 : tok_left(s + 1)};
                    weighted_sum([&](auto k) {
                        if constexpr (k.value == 2) scores_pass(sc);
                        if constexpr (k.value >= 3 && k.value < 27 && k.value % 3 == 0) f.step(Slot<k.value / 3 - 1>{});
                    });
                    w[0][0] = w_next[0];
                    w[0][1] = w_next[1];
                }
                advance();
            };
            // Iterations that request a whole group of whole units: every group in flight is complete, so a counted wait leaves
            // exactly the kMultiDepth - 1 youngest.
            while (s + 1 + kMultiDepth < n_whole && s + 1 < n_full) {
                wait_vmem_but<(kMultiDepth - 1) * kMultiOps>();
                __syncthreads();
                iterate(std::true_type{});
            }
            // The last iterations: whatever is left to request, everything awaited.
            while (s + 1 < n_units) {
                wait_vmem_but<0>();
                __syncthreads();
                if (s + 1 + kMultiDepth < n_units) load_unit(false, span, s + 1 + kMultiDepth, o[1], slot);
                if (s + kMultiDepth < n_units) load_unit(true, span, s + kMultiDepth, o[0], slot_prev);
                iterate(std::false_type{});
            }
            wait_vmem_but<0>();
            __syncthreads();
            bool outrun = false;
            float m_true[2];
            if (computes) {
                values.begin(v_of(slot));
                MultiSoftmax<true>{sc[1], w[1], st.half[1], c, m_safe[1], tok_left(s)}.all();
                weights_ready();
                weighted_sum([](auto) {});
#pragma unroll
                for (int cb = 0; cb < 2; ++cb) {
                    m_true[cb] = half_max(st.half[cb].s_max) * c;
                    outrun = outrun || m_true[cb] > st.half[cb].m + kFixedReferenceLag;
                }
                outrun = outrun && !retried;
                if (outrun) *LDS_AT(int, lds, kMultiFlag) = 1;
            }
            __syncthreads();                          // every wave is done reading the tile memory
            again = !retried && *LDS_AT(int, lds, kMultiFlag) != 0;
            if (again) {
                if (computes) {
#pragma unroll
                    for (int cb = 0; cb < 2; ++cb)
                        if (m_true[cb] > st.half[cb].m + kFixedReferenceLag) st.half[cb].m = m_true[cb];
                }
                retried = true;
                __syncthreads();                      // the flag has been read
            }
        }
        if (computes) {
            int lane_now = lane;                      // (the result's addresses are formed here, once per segment)
            asm volatile("" : "+v"(lane_now));
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) {
                output_ready(st.half[cb].acc);
                st.half[cb].l = half_sum(st.half[cb].l);
                finish_lowbit_two(st.half[cb], a, r, tok, cb, lane_now);
            }
        }
        __syncthreads();                              // the flag has been read; the tile memory is the next segment's
    }
}

}  // namespace mfa
