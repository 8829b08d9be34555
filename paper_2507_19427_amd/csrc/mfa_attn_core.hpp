// Device-side building blocks of the decode attention kernels (gfx950).  Common to all of them: waits, direct loads, the schedule,
// page lookup.  The kernels of four waves have shapes, matrix layouts and softmax rules of their own: mfa_lowbit.hpp
// (decode_lowbit_kernel), mfa_multi.hpp (decode_bf16_multi_kernel), mfa_multi_short.hpp (short_bf16_multi_kernel, on this file's unit image).
//
// Workgroup shape of decode_bf16_kernel (mfa_attn.hip) and short_lowbit_kernel (mfa_lowbit_short.hpp): 8 waves; wave = 4*grp + wq.
// wq selects 16 of the 64 query heads, grp which 32-token unit of every 64-token tile the wave processes (with two query
// tokens: which token).  The two waves that share a SIMD (same wq, different grp) keep independent online-softmax
// states, which finish_segment() merges through LDS, so one wave's MFMA work can overlap the other's softmax.
//
// LDS image of one 32-token unit (what process_unit reads), bf16:
//   K rows 0..31 then V rows 0..31, 512 B per row (256 bf16).
//   K row r stores its 16-byte chunk c at position c ^ (r & 15);
//   V row r stores its 32-byte chunk c at position c ^ (r & 15).
// With these swizzles the 16-row x 16-byte MFMA operand reads of K and the 16-row x 32-byte
// transposing reads of V each touch every LDS bank exactly once.
//
// MFMA shapes (v_mfma_f32_16x16x32_bf16; lane = 16*g + n):
//   scores   S^T[token, head] = K[token, :] . Q[head, :]^T     A = K rows, B = Q
//            lane holds S^T[token 4g+i, head n], i = 0..3, for each 16-token block
//   output   O^T[d, head] += V^T[d, token] . P^T[token, head]  A = V^T, B = P
//            lane holds O^T[d = 16*db + 4g + i, head n]
// The score block a lane ends up with is exactly the B-operand slice it must supply for the
// second product (8 tokens of its own head), so attention weights never move between lanes and
// the per-head statistics live in the lanes of that head.
#pragma once
#include <type_traits>
#include <utility>

#include "mfa_internal.hpp"

namespace mfa {

typedef __attribute__((address_space(3))) unsigned char* lds_ptr_t;
#define LDS_AT(T, base, byte_off) ((__attribute__((address_space(3))) T*)((base) + (byte_off)))

constexpr int kUnitTokens = 32;
constexpr int kUnitBytes = 32768;        // K 32x512 B then V 32x512 B
constexpr int kUnitVOffset = 16384;
constexpr int kAttnThreads = 512;

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// s_waitcnt that constrains only the vector-memory counter: vmcnt(0).
__device__ __forceinline__ void wait_vmem_all() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// ... leaving the N youngest operations in flight (gfx950: vmcnt is bits 3:0 and 15:14 of the immediate)
template <int N> __device__ __forceinline__ void wait_vmem_but()
{
    static_assert(N >= 0 && N < 64, "vmcnt has six bits");
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// Direct global->LDS load: 16 bytes per lane land at lds_addr + 16*lane (lds_addr is wave-uniform
// and travels in M0).  The global address is a wave-uniform base (scalar registers) plus a 32-bit
// byte offset per lane: no 64-bit vector arithmetic per load.  Issued as inline assembly so that
// the compiler does not make later LDS reads of *other* buffers wait for it; completion is
// awaited explicitly (wait_vmem_all() or a counted s_waitcnt) followed by a workgroup barrier.
// M0 is not otherwise live in these kernels.  The s_nop covers the wait state required between
// writing M0 and an LDS-direct load.  Everything brought in this way (cache rows, weight rows) is read
// once: the non-temporal hint keeps it from displacing reusable lines on its way through the caches,
// which alone is worth 11 to 14 % on the bf16 attention workloads.
__device__ __forceinline__ void load_to_lds_16B(const void* sbase, uint32_t voff, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt"
                 :: "v"(voff), "s"(sbase), "s"(lds_addr) : "memory");
}

// The same without the non-temporal hint, for rows that other workgroups read too.
__device__ __forceinline__ void load_to_lds_16B_keep(const void* sbase, uint32_t voff, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(voff), "s"(sbase), "s"(lds_addr) : "memory");
}

// The same with the LDS address as a base plus a compile-time offset.
template <int OFFSET>
__device__ __forceinline__ void load_to_lds_16B_at(const void* sbase, uint32_t voff, uint32_t lds_base)
{
    asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt"
                 :: "v"(voff), "s"(sbase), "s"(lds_base), "n"(OFFSET) : "memory", "scc");
}

// The same with the whole address in a pair of vector registers (for a base the compiler keeps there).
__device__ __forceinline__ void load_to_lds_16B_vaddr(const void* vaddr, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt"
                 :: "v"(vaddr), "s"(lds_addr) : "memory");
}
// Four bytes per lane: lane l's word lands at lds_addr + 4*l.
__device__ __forceinline__ void load_to_lds_4B(const void* sbase, uint32_t voff, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
                 :: "v"(voff), "s"(sbase), "s"(lds_addr) : "memory");
}

// max over the four lanes {n, n+16, n+32, n+48} that hold one head, without touching LDS:
// v_permlane32_swap exchanges the upper half of the first operand with the lower half of the
// second, v_permlane16_swap exchanges odd 16-lane rows of the first with even rows of the second.
__device__ __forceinline__ float head_max(float x)
{
    const unsigned u = __float_as_uint(x);
    const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const unsigned v = __float_as_uint(x);
    const auto b = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float head_sum(float x)
{
    const unsigned u = __float_as_uint(x);
    const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const unsigned v = __float_as_uint(x);
    const auto b = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Running state of one wave: 16 heads x 256 output dims, spread as described above.
struct WaveState {
    f32x4 acc[16];
    float m;     // reference exponent of the weights, log2 domain: within 8 below this head's running maximum (equal in the 4 lanes of a head)
    float l;     // this lane's share of the sum of weights
};

__device__ __forceinline__ void init_state(WaveState& st)
{
#pragma unroll
    for (int i = 0; i < 16; ++i) st.acc[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    st.m = -INFINITY;
    st.l = 0.f;
}

// Query fragments of this lane: B operand of the score product, d = 32*ks + 8*g + j.
__device__ __forceinline__ void load_q_fragments(bf16x8 (&qf)[8], const void* q, int b, int head, int g)
{
    const bf16x8* qp = (const bf16x8*)((const uint16_t*)q + ((size_t)b * kHeads + head) * kHeadDim + 8 * g);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qf[ks] = qp[ks * 4];
}

typedef int i32x8 __attribute__((ext_vector_type(8)));
// Query operands of one wave (its 16 heads): a lane holds head n, d = 32*ks + 8*g + j.
struct QFrags { bf16x8 f[8]; };

// One 32-token unit: scores, online softmax, weighted sum.
//   kbase      LDS byte offset of the unit's keys:   32 rows of 512 B, 16-byte chunk c of row r stored at c ^ (r & 15)
//   vbase      LDS byte offset of the unit's values: 32 rows of 512 B, 32-byte chunk c of row r stored at c ^ (r & 15)
//   unit_t0    index (within the sequence) of the unit's first token; tokens >= t1 are masked
//
// Raw scores of a unit (2 blocks of 16 tokens), before any scale: q . k for this lane's head and its 8 tokens.
struct RawScores { f32x4 s[2]; };
__device__ __forceinline__ RawScores qk_unit(const QFrags& q, lds_ptr_t lds_base, int kbase, int n, int g)
{
    f32x4 s[2] = {(f32x4){0.f, 0.f, 0.f, 0.f}, (f32x4){0.f, 0.f, 0.f, 0.f}};
    const int k_lane_off = n * 512;                     // K: row n of a 16-token block, swizzle key n
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
            const int off = kbase + tb * 8192 + k_lane_off + (((4 * ks + g) ^ n) << 4);
            const bf16x8 kf = *LDS_AT(bf16x8, lds_base, off);
            s[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, q.f[ks], s[tb], 0, 0, 0);
        }
    }
    RawScores r;
    r.s[0] = s[0];
    r.s[1] = s[1];
    return r;
}
// Online softmax of a unit from its raw scores, and the rescale of what has been accumulated so far.
// Returns the unit's attention weights as the B operand of the weighted sum (8 tokens of this lane's head).
__device__ __forceinline__ bf16x8 softmax_unit(WaveState& st, const RawScores& raw, int unit_t0, int t1, float scale_log2e, int g)
{
    const f32x4 s[2] = {raw.s[0], raw.s[1]};
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
    for (int j = 0; j < 8; j += 2) {
        // normalise by the sum of the rounded weights actually multiplied into V
        const float p0 = fast_exp2(__builtin_fmaf(sv[j], scale_log2e, -m_safe));
        const float p1 = fast_exp2(__builtin_fmaf(sv[j + 1], scale_log2e, -m_safe));
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        const bf16x2 pb = {(__bf16)p0, (__bf16)p1};
        pf[j] = pb[0];
        pf[j + 1] = pb[1];
        const uint32_t bits = __builtin_bit_cast(uint32_t, pb);
        psum += __uint_as_float(bits << 16) + __uint_as_float(bits & 0xFFFF0000u);
    }
    st.l = st.l * alpha + psum;

    if (__any(alpha != 1.0f)) {
#pragma unroll
        for (int db = 0; db < 16; ++db) st.acc[db] *= alpha;
    }
    return pf;
}

// Second half of a unit: O^T += V^T P^T over the unit's 32 tokens.
__device__ __forceinline__ void pv_unit(WaveState& st, lds_ptr_t lds_base, int vbase, const bf16x8& pf, int n, int g)
{
    const int v_row = 4 * g + (n >> 2);                 // V: row within a 16-token block (= swizzle key)
    const int v_lane_off = v_row * 512 + ((n & 3) << 3);   // (n & 3: which 8 bytes of the 32-byte chunk this lane supplies)
    union VFrag { bf16x8 v; s16x4 h[2]; };
    auto read_v = [&](VFrag& f, int db) {
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
            f.h[tb] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_AT(s16x4, lds_base, vbase + tb * 8192 + v_lane_off + ((db ^ v_row) << 5)));
    };
    // The operands of kAhead output blocks are on their way while one block is multiplied: an LDS read takes
    // several times as long as the MFMA it feeds, and a wave has only one other wave on its SIMD to hide it.
    constexpr int kAhead = 2;
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

__device__ __forceinline__ void process_unit(WaveState& st, const QFrags& q, lds_ptr_t lds_base, int kbase, int vbase, int unit_t0,
                                             int t1, float scale_log2e, int n, int g)
{
    const RawScores raw = qk_unit(q, lds_base, kbase, n, g);
    const bf16x8 pf = softmax_unit(st, raw, unit_t0, t1, scale_log2e, g);
    pv_unit(st, lds_base, vbase, pf, n, g);
}

// How far (log2) the weights of the kernels with a fixed reference exponent may grow before a segment is streamed again.
constexpr float kFixedReferenceLag = 40.0f;

// After the last tile the two waves that share 16 heads (grp 0 and 1: the two token halves of
// every tile) exchange halves of their accumulators through 64 KB of LDS at xbase (a tile buffer
// that is dead by then; the caller guarantees that no direct load into it is in flight) and a
// spare KB behind the tile memory: grp 0 finishes output blocks 0..7,
// grp 1 blocks 8..15, so all eight waves merge and store in parallel.  One split: the final
// result goes to `out`.  Several splits: the unnormalised partial goes to the workspace in
// lane order (float4 index (wq*16 + db)*64 + lane, fully coalesced), with (m, l) per head.
template <int KEEP, int SEND>
__device__ __forceinline__ void finish_half(WaveState& st, lds_ptr_t lds_base, int xbase, const AttnArgs& a, int b, int slot,
                                            bool final_result, int wq, int grp, int lane)
{
    const int n = lane & 15, g = lane >> 4;
    const int head = 16 * wq + n;
    const int mine = (wq * 2 + grp) * 8;              // my 8 KB exchange slots (1 KB each), from xbase on
    const int theirs = (wq * 2 + (grp ^ 1)) * 8;
    constexpr int kMlOff = 2 * 2 * kUnitBytes;        // (m, l) per head and wave: the spare KB behind the tile memory
#pragma unroll
    for (int i = 0; i < 8; ++i) *LDS_AT(f32x4, lds_base, xbase + (mine + i) * 1024 + lane * 16) = st.acc[SEND + i];
    if (g == 0) {                                     // m and (after head_sum) l are equal in the four lanes of a head
        *LDS_AT(float, lds_base, kMlOff + ((wq * 2 + grp) * 2 + 0) * 64 + n * 4) = st.m;
        *LDS_AT(float, lds_base, kMlOff + ((wq * 2 + grp) * 2 + 1) * 64 + n * 4) = st.l;
    }
    __syncthreads();
    const float m_o = *LDS_AT(float, lds_base, kMlOff + ((wq * 2 + (grp ^ 1)) * 2 + 0) * 64 + n * 4);
    const float l_o = *LDS_AT(float, lds_base, kMlOff + ((wq * 2 + (grp ^ 1)) * 2 + 1) * 64 + n * 4);
    const float m = fmaxf(st.m, m_o);                 // -inf if every score of the segment is: a partial without weight
    const float m_safe = m == -INFINITY ? 0.f : m;
    const float w_s = fast_exp2(st.m - m_safe);
    const float w_o = fast_exp2(m_o - m_safe);
    const float l = st.l * w_s + l_o * w_o;
    const float inv = 1.0f / l;
    float* o = a.out + ((size_t)b * kHeads + head) * kHeadDim + 4 * g;
    f32x4* part = (f32x4*)a.ws_acc + (size_t)slot * (kHeads * kHeadDim / 4) + (size_t)wq * 16 * 64 + lane;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const f32x4 other = *LDS_AT(f32x4, lds_base, xbase + (theirs + i) * 1024 + lane * 16);
        const f32x4 r = st.acc[KEEP + i] * w_s + other * w_o;
        if (final_result) *(f32x4*)(o + 16 * (KEEP + i)) = r * inv;
        else part[(KEEP + i) * 64] = r;
    }
    if (!final_result && grp == 0 && g == 0)
        *(float2*)(a.ws_ml + ((size_t)slot * kHeads + head) * 2) = make_float2(m, l);
}

// One piece of work: tokens [t0, t1) of sequence b (n_tiles tiles of 64, the last one possibly
// ragged).  Its result is the sequence's final output (final_result) or a partial in `slot`.
struct Segment {
    int b, t0, t1, n_tiles, slot;
    int len;              // the sequence's (clamped) length
    bool final_result;
    int seq_end;          // balanced schedule: the tiles up to the end of its sequence if it holds the sequence's first, else 0
};

// Every field of a segment is the same in all threads; saying so keeps the branches on them scalar.
__device__ __forceinline__ void make_uniform(Segment& r)
{
    r.b = __builtin_amdgcn_readfirstlane(r.b);
    r.t0 = __builtin_amdgcn_readfirstlane(r.t0);
    r.t1 = __builtin_amdgcn_readfirstlane(r.t1);
    r.n_tiles = __builtin_amdgcn_readfirstlane(r.n_tiles);
    r.slot = __builtin_amdgcn_readfirstlane(r.slot);
    r.len = __builtin_amdgcn_readfirstlane(r.len);
    r.final_result = __builtin_amdgcn_readfirstlane((int)r.final_result) != 0;
    r.seq_end = __builtin_amdgcn_readfirstlane(r.seq_end);
}

// xbase: LDS byte offset of the 64 KB the exchange may use (tile memory nobody reads any more).
__device__ __forceinline__ void finish_segment(WaveState& st, lds_ptr_t lds_base, int xbase, const AttnArgs& a, const Segment& r,
                                               int wq, int grp, int lane)
{
    st.l = head_sum(st.l);
    __syncthreads();                                  // every wave is done reading the tile buffers
    if (grp == 0) finish_half<0, 8>(st, lds_base, xbase, a, r.b, r.slot, r.final_result, wq, grp, lane);
    else          finish_half<8, 0>(st, lds_base, xbase, a, r.b, r.slot, r.final_result, wq, grp, lane);
}

// Several query tokens per sequence (a wave then holds all 256 output dims of its 16 heads for a query
// token, and has seen all tokens of the segment): no exchange, each wave stores its 16 rows.  The partial
// of a (segment, query token) sits at slot * n_here + query token in the same lane-order layout.  A query token
// that saw no cached token in this segment leaves m = -inf, l = 0 and a zero accumulator; as a final
// result that is the zero row.
__device__ __forceinline__ void finish_segment_two(WaveState& st, const AttnArgs& a, const Segment& r, int qtok, int wq, int lane)
{
    const int n = lane & 15, g = lane >> 4;
    const int head = 16 * wq + n;
    const float l = head_sum(st.l);
    const size_t row = (size_t)r.b * a.q_len + a.q0 + qtok;
    if (r.final_result) {
        const float inv = l > 0.f ? 1.0f / l : 0.f;
        float* o = a.out + (row * kHeads + head) * kHeadDim + 4 * g;
#pragma unroll
        for (int db = 0; db < 16; ++db) *(f32x4*)(o + 16 * db) = st.acc[db] * inv;
    } else {
        const size_t slot = (size_t)r.slot * a.n_here + qtok;
        f32x4* part = (f32x4*)a.ws_acc + slot * (kHeads * kHeadDim / 4) + (size_t)wq * 16 * 64 + lane;
#pragma unroll
        for (int db = 0; db < 16; ++db) part[db * 64] = st.acc[db];
        if (g == 0) *(float2*)(a.ws_ml + (slot * kHeads + head) * 2) = make_float2(st.m, l);
    }
}

// Page id of the tile that starts at token tile_t0 (paged cache only).  Looked up one tile ahead
// of its use so that the table read is never on the critical path of issuing a tile's loads.
template <bool PAGED>
__device__ __forceinline__ int lookup_page(const AttnArgs& a, int b, int tile_t0)
{
    // read through the constant address space: the table is not written while the kernel runs, and a
    // uniform index then makes this a scalar load, which the vector-memory waits do not have to cover
    typedef const __attribute__((address_space(4))) int32_t* const_table_t;
    if (!PAGED) return 0;
    const int page = ((const_table_t)a.block_table)[(size_t)b * a.max_blocks_per_seq + tile_t0 / kPage];
    return page < 0 ? 0 : (page >= a.n_pages ? a.n_pages - 1 : page);      // a bad id reads a wrong page, never outside the pool
}

template <bool PAGED>
__device__ __forceinline__ int64_t tile_row0(const AttnArgs& a, int b, int tile_t0, int page)
{
    return PAGED ? (int64_t)page * kPage : (int64_t)b * a.seq_stride_tokens + tile_t0;
}

__device__ __forceinline__ int clamped_len(const AttnArgs& a, int b)
{
    // (constant address space: not written while the kernel runs, and a uniform index makes it a scalar load)
    const int L = ((const __attribute__((address_space(4))) int32_t*)a.seq_lens)[b];
    return L < 0 ? 0 : (L > a.max_seq_len_hint ? a.max_seq_len_hint : L);
}

// ---- Which segments a workgroup works off.
//
// Fixed splits (n_wgs == 0): workgroup = (sequence, split), one segment of chunk_tokens tokens;
// the partial slot is the workgroup index; the first split of an empty sequence writes the zeros.
//
// Balanced (n_wgs > 0): with T_b = ceil(L_b / 64) tiles per sequence (and, where sequences begin in mid-range, the pad that
// stands for the cost of a switch ahead of them: batches of up to 512 sequences) and P the exclusive prefix
// sums of T, workgroup w takes the tile range [w*N/G, (w+1)*N/G) of the N = P[B] tiles laid end to
// end (G = min(n_wgs, N), so that no workgroup below G is idle) and cuts it at sequence boundaries.  The workgroups touching sequence b are
// consecutive, first(b)..last(b) with wg_of(t) = ((t+1)*G - 1) / N; the segment of workgroup w on
// sequence b uses partial slot w + b, which is unique because (w, b) grows in at least one
// coordinate from one segment to the next, and the slots of one sequence are consecutive.  The
// workgroup holding a sequence's first tile records (first slot, number of partials) for the
// merge; a sequence held by one workgroup is written finally and needs no merge.  Sequences
// without tokens are zero-filled by the merge kernel.
//
// LDS of the schedule, from a kernel-given offset `base` on: the staged lengths of batches of up to 512 sequences, eight
// wave totals and the result of the search of larger ones.
constexpr int kSchedTotals = 2048;
constexpr int kSchedFound = kSchedTotals + 8 * 4;
constexpr int kSchedLdsBytes = kSchedFound + 16;

constexpr int kSlotBytes = 2 * kUnitBytes;            // one 64-token tile: two unit images
// LDS of the bf16 kernels (and, from kBf16SchedOffset on, of short_lowbit_kernel): two tile slots, a KB for the per-head (m, l) exchanged at the end of a segment, and the
// schedule
constexpr int kBf16SchedOffset = 2 * kSlotBytes + 1024;
constexpr int kBf16LdsBytes = kBf16SchedOffset + kSchedLdsBytes;

// What starting on another sequence costs a workgroup, in tiles' worth of time (end of a segment, its result, and the start of the next
// with nothing in flight; decode_bf16_kernel has the next tile on its way already).  The schedule lays that many tiles ahead of every sequence's
// own, so that a range which holds a boundary holds fewer tiles: without them the few workgroups with two segments decide the time.  us per
// call without / with, lengths drawn from 1 .. the longest: 8 bit 40 x 9000 42.3 / 31.7, 100 x 5000 52.8 / 43.7, 60 x 12000 60.3 / 50.5,
// 23 x 20011 44.4 / 39.5; 4 bit 40 x 9000 38.6 / 28.6; 8 bit, two tokens, 60 x 6000 59.6 / 49.5; bf16, three tokens 16 x 4096 46.1 / 37.3, four
// 30 x 3000 53.7 / 41.9; bf16, one token, three draws each: 100 x 3000 45.3 .. 49.4 / 41.1 .. 45.7, 33 x 12000 45.6 .. 53.4 / 43.3 .. 50.9, two tokens 40 x 6000
// 48.4 .. 51.0 / 42.0 .. 45.0, but 128 x 1024..8192 within what two runs of one side differ by (121.7, 114.4, 112.8 / 120.4, 115.0, 111.3): its 38 tiles per
// workgroup leave little to balance.  Half or one and a half times as many: within 3 %.  Batches of more than 512 sequences have no pad.
constexpr int kBf16Switch = 2;
constexpr int kShortLowbitSwitch = 6;
constexpr int kLowbitSwitch = 8;
constexpr int kMultiSwitch = 3;
struct Schedule {
    int pad;            // tiles laid ahead of every sequence's own (what a switch costs), or 0
    int lo, hi;         // balanced: my tile range (lo moves on as segments are handed out); fixed: hi > lo while my one segment is still to do
    int n_tiles_all;    // N
    int n_wgs;          // G: workgroups that have a range (min of the grid size and N)
    int my_lo;          // start of my range
    int b, seq0, len;   // the sequence that lo may fall into, the tiles before it, and its (clamped) length
};

// floor(a / d) for 32-bit operands without the long emulated integer division (some hundred scalar
// instructions ahead of every workgroup's first load): double-precision reciprocal, then one step of
// correction in integers (the estimate is off by at most one).
__device__ __forceinline__ unsigned div_floor_u32(unsigned a, unsigned d)
{
    unsigned q = (unsigned)((double)a * __builtin_amdgcn_rcp((double)d));
    const unsigned long long prod = (unsigned long long)q * d;
    if (prod > a) --q;
    else if (prod + d <= a) ++q;
    return q;
}
// floor(x * N / G), in 32 bits when the products fit.  The common cases are no division: fewer tiles than workgroups (G = N), and
// a workgroup per compute unit (G = 256).
__device__ __forceinline__ int scaled_floor(int x, int N, int G)
{
    if (G == N) return x;
    const bool small = N < (1 << 20) && x <= (1 << 11);
    if (small && (G & (G - 1)) == 0) return (int)(((unsigned)x * (unsigned)N) >> __builtin_ctz(G));
    if (small) return (int)div_floor_u32((unsigned)x * (unsigned)N, (unsigned)G);
    return (int)((unsigned long long)x * (unsigned long long)N / (unsigned long long)G);
}
// ((t + 1) * G - 1) / N: at most G <= 4096, so a double-precision estimate is off by at most one whatever the size of the product.
__device__ __forceinline__ int wg_of_tile(int t, int G, int N)
{
    if (G == N) return t;
    asm volatile("" : "+s"(N));                       // (formed where it is used, once per sequence, not ahead of the segment loop)
    const unsigned long long a = ((unsigned long long)t + 1ull) * (unsigned)G - 1ull;
    unsigned q = (unsigned)((double)a * __builtin_amdgcn_rcp((double)N));
    const unsigned long long prod = (unsigned long long)q * (unsigned)N;
    if (prod > a) --q;
    else if (prod + (unsigned)N <= a) ++q;
    return (int)q;
}

// Inclusive prefix sum over the 64 lanes of a wave with data-parallel-primitive moves: shifts by
// 1, 2, 4, 8 inside each row of 16 lanes (lanes without a source add 0), then lane 15 of rows 0 and
// 2 is added to rows 1 and 3, then lane 31 to rows 2 and 3.
__device__ __forceinline__ int wave_inclusive_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);    // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);    // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);    // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);    // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);    // row_bcast:15 into rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);    // row_bcast:31 into rows 2, 3
    return v;
}

// Which range of the balanced schedule a workgroup takes.  Workgroups are handed to the device's eight
// compute dies in turn (workgroup i runs on die i % 8, each with its own L2), while the pieces of one
// sequence are consecutive ranges: numbering the ranges die by die puts neighbouring ranges, which read
// neighbouring memory and write neighbouring partial results, on one die (measured on the benchmark
// workload: 0.6 us per call).  Nothing but speed depends on where a workgroup really runs.
__device__ __forceinline__ int range_index()
{
    const int g = (int)gridDim.x, i = (int)blockIdx.x;
    return (g & 7) == 0 ? (i & 7) * (g >> 3) + (i >> 3) : i;
}

// Sequences of one length: are all ranges alike, a part of one sequence or the same number of whole ones?  (Then a switch costs all of them the same.)
__device__ __forceinline__ bool boundaries_on_edges(int B, int n_wgs) { return (B & (B - 1)) == 0 && (n_wgs & (n_wgs - 1)) == 0; }

// All threads of the workgroup call this; the values returned are the same in every thread.
//
// Batches of up to 512 sequences: every wave scans the whole batch by itself (64 lengths at a time), so the way
// to a workgroup's first segment crosses no barrier.  Larger batches: one cooperative scan, a run of consecutive
// sequences per thread.  Only the first sequence of a range is searched for; from there the lengths are read on as the segments
// are handed out.
//
// All of this runs once per workgroup, ahead of its first load of cache rows, and comes cold from the instruction cache (about 100
// cycles per 64 bytes): what it costs is its length in instructions.  Hence loops that are not unrolled, no division in the common
// cases, and the merge's record written later (schedule_record).  From the lengths' arrival to the first segment, 128 sequences: 2.1 us
// unrolled over eight groups of 64 with the lengths in registers and the record in between, 1.4 us now.
constexpr int kWaveScanChunks = 8;
// The lengths of such a batch reach the waves through LDS: every wave copies seq_lens[0 .. B) there with direct
// loads (all waves write the same bytes to the same place, so a wave that has waited for its own loads has the
// lengths without a barrier).  Direct loads are counted like every vector-memory operation but wait for nothing
// themselves, so a kernel can ask for the lengths, then for its first tile, and work the schedule out as soon as
// the lengths -- the older loads -- are there: stage_lengths(), further loads, await_lengths(.., loads issued
// since).
static_assert(kWaveScanChunks * 256 <= kSchedTotals, "staged lengths");
__device__ __forceinline__ bool lengths_are_staged(const AttnArgs& a) { return a.n_wgs != 0 && a.B <= kWaveScanChunks * 64; }
__device__ __forceinline__ void stage_lengths(const AttnArgs& a, lds_ptr_t lds_base, int base)
{
    if (!lengths_are_staged(a)) return;
    const int lane = threadIdx.x & 63;
    uint32_t dst = (uint32_t)(uintptr_t)lds_base + base;
#pragma unroll 1
    for (int c0 = 0; c0 < a.B; c0 += 64, dst += 256) {
        const int i = c0 + lane < a.B ? c0 + lane : a.B - 1;              // lanes past the batch repeat its last entry
        load_to_lds_4B(a.seq_lens, (uint32_t)i * 4u, dst);
    }
}
// LATER: vector-memory operations this wave has issued since stage_lengths when `later` (a tile asked for ahead)
template <int LATER>
__device__ __forceinline__ void await_lengths(const AttnArgs& a, bool later)
{
    if (!lengths_are_staged(a)) return;
    // the staged lengths have landed once only the loads issued after them are outstanding
    if (later) wait_vmem_but<LATER>();
    else       wait_vmem_but<0>();
}
template <int THREADS>
__device__ __forceinline__ Schedule schedule_begin(const AttnArgs& a, lds_ptr_t lds_base, int base, int switch_tiles)
{
    Schedule s;
    s.b = s.seq0 = s.len = s.n_tiles_all = s.n_wgs = s.lo = s.my_lo = s.pad = 0;
    s.hi = 1;
    if (a.n_wgs == 0) return s;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;

    if (a.B <= kWaveScanChunks * 64) {
        // lanes of the group of 64 sequences from c0 on: length, its tiles, and sums within the group up to and including the lane's
        int len, x, incl, incl_seqs;
        unsigned long long with_tiles;
        auto scan = [&](int c0) {
            const int i = c0 + lane;
            const int L = *LDS_AT(int, lds_base, base + i * 4);
            len = i >= a.B || L < 0 ? 0 : (L > a.max_seq_len_hint ? a.max_seq_len_hint : L);
            x = (len + kTile - 1) / kTile;
            incl = wave_inclusive_scan(x);
            with_tiles = __ballot(x != 0);
            incl_seqs = __builtin_amdgcn_mbcnt_hi((unsigned)(with_tiles >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)with_tiles, 0)) + (x != 0);
        };
        int c0 = 0, before = 0, before_seqs = 0, N = 0, n_seqs = 0;       // ahead of the group, and up to its end
        int x_first = 0;
        bool equal = true;
#pragma unroll 1
        for (;; c0 += 64) {
            scan(c0);
            if (c0 == 0) x_first = __builtin_amdgcn_readfirstlane(x);
            equal &= !__ballot(x != x_first && c0 + lane < a.B);
            before = N;
            before_seqs = n_seqs;
            N += __builtin_amdgcn_readlane(incl, 63);
            n_seqs += __builtin_popcountll(with_tiles);
            if (c0 + 64 >= a.B) break;
        }
        const int w = range_index();
        if (N > a.n_wgs && !(equal && boundaries_on_edges(a.B, a.n_wgs))) s.pad = switch_tiles;   // (up to a tile per workgroup nobody switches)
        N += s.pad * n_seqs;
        before += s.pad * before_seqs;
        const int G = a.n_wgs < N ? a.n_wgs : N;      // with fewer tiles than workgroups the last ones idle
        s.n_tiles_all = N;
        s.n_wgs = G;
        if (w >= G) { s.lo = s.hi = 0; return s; }
        s.lo = s.my_lo = __builtin_amdgcn_readfirstlane(scaled_floor(w, N, G));
        s.hi = __builtin_amdgcn_readfirstlane(scaled_floor(w + 1, N, G));
        // the one sequence with P[b] <= lo < P[b + 1], from the last group (still in registers) back
#pragma unroll 1
        while (before > s.lo) {
            c0 -= 64;
            scan(c0);
            before -= __builtin_amdgcn_readlane(incl, 63) + s.pad * __builtin_popcountll(with_tiles);
        }
        incl += s.pad * incl_seqs;
        const int src = __builtin_amdgcn_readfirstlane((int)__builtin_ctzll(__ballot(before + incl > s.lo)));
        s.b = c0 + src;
        s.len = __builtin_amdgcn_readlane(len, src);
        s.seq0 = before + __builtin_amdgcn_readlane(incl, src) - __builtin_amdgcn_readlane(x, src) - s.pad;
        return s;
    }

    // thread t scans sequences run*t .. run*t + run - 1
    const int run = (a.B + THREADS - 1) / THREADS;
    const int first = run * (int)threadIdx.x;
    int mine = 0;
    for (int i = first; i < first + run && i < a.B; ++i) mine += (clamped_len(a, i) + kTile - 1) / kTile;
    const int incl = wave_inclusive_scan(mine);
    if (lane == 63) *LDS_AT(int, lds_base, base + kSchedTotals + wave * 4) = incl;
    __syncthreads();
    int before = incl - mine, N = 0;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) {
        const int tw = *LDS_AT(int, lds_base, base + kSchedTotals + w * 4);
        N += tw;
        if (w < wave) before += tw;
    }
    const int G = a.n_wgs < N ? a.n_wgs : N;
    s.n_tiles_all = __builtin_amdgcn_readfirstlane(N);
    s.n_wgs = __builtin_amdgcn_readfirstlane(G);
    if (range_index() >= G) { s.lo = s.hi = 0; return s; }
    s.lo = s.my_lo = __builtin_amdgcn_readfirstlane(scaled_floor(range_index(), N, G));
    s.hi = __builtin_amdgcn_readfirstlane(scaled_floor(range_index() + 1, N, G));
    if (before <= s.lo && s.lo < before + mine)                       // exactly one thread
        for (int i = first, at = before; i < first + run && i < a.B; ++i) {
            const int len = clamped_len(a, i);
            const int x = (len + kTile - 1) / kTile;
            if (at <= s.lo && s.lo < at + x) {
                *LDS_AT(int, lds_base, base + kSchedFound) = i;
                *LDS_AT(int, lds_base, base + kSchedFound + 4) = at;
                *LDS_AT(int, lds_base, base + kSchedFound + 8) = len;
            }
            at += x;
        }
    __syncthreads();
    s.b = __builtin_amdgcn_readfirstlane(*LDS_AT(int, lds_base, base + kSchedFound));   // the one sequence with P[b] <= lo < P[b + 1]
    s.seq0 = __builtin_amdgcn_readfirstlane(*LDS_AT(int, lds_base, base + kSchedFound + 4));
    s.len = __builtin_amdgcn_readfirstlane(*LDS_AT(int, lds_base, base + kSchedFound + 8));
    return s;
}

// Where this workgroup's first tile lies if every sequence has the length of the hint: computed from the
// launch arguments alone (no device memory is read), with the same arithmetic as the schedule.  A load of rows from t0 up
// to the hint stays inside memory the caller has vouched for (rows below max_seq_len_hint of a sequence below B;
// paged: a table entry below ceil(hint / 64), clamped into the pool like every other).
struct FirstTileGuess { int b, t0; bool valid; };
__device__ __forceinline__ FirstTileGuess guess_first_tile(const AttnArgs& a, int switch_tiles)
{
    FirstTileGuess gs;
    gs.b = gs.t0 = 0;
    gs.valid = false;
    if (!lengths_are_staged(a)) return gs;            // (the guess rides on the staged lengths' head start)
    int T = (a.max_seq_len_hint + kTile - 1) / kTile;
    const int pad = a.B * T > a.n_wgs && !boundaries_on_edges(a.B, a.n_wgs) ? switch_tiles : 0;
    T += pad;
    const int N = a.B * T;
    const int G = a.n_wgs < N ? a.n_wgs : N;
    const int w = range_index();
    if (w >= G) return gs;
    const int lo = scaled_floor(w, N, G);
    gs.b = (int)div_floor_u32((unsigned)lo, (unsigned)T);
    const int tile = lo - gs.b * T - pad;
    gs.t0 = tile > 0 ? tile * kTile : 0;
    gs.b = __builtin_amdgcn_readfirstlane(gs.b);
    gs.t0 = __builtin_amdgcn_readfirstlane(gs.t0);
    gs.valid = gs.b < a.B && gs.t0 + kTile <= a.max_seq_len_hint;     // whole tiles only
    return gs;
}

// The holder of a sequence's first tile tells the merge which partial results there are.  Not needed before the segment's end: called
// once its loads are on their way.
__device__ __forceinline__ void schedule_record(const AttnArgs& a, const Schedule& s, const Segment& r)
{
    if (r.seq_end == 0) return;
    const int first = range_index();
    const int last = r.final_result ? first : wg_of_tile(r.seq_end - 1, s.n_wgs, s.n_tiles_all);
    if (threadIdx.x == 0) {
        a.ws_seg[2 * r.b] = first + r.b;
        a.ws_seg[2 * r.b + 1] = last - first + 1;
    }
}

// The next segment of this workgroup, or false when it has none left.  A false return for the very
// first request of a fixed-split workgroup on an empty sequence has written the zero result.
template <int THREADS>
__device__ __forceinline__ bool schedule_next(const AttnArgs& a, Schedule& s, Segment& r)
{
    if (s.lo >= s.hi) return false;
    if (a.n_wgs == 0) {
        s.hi = 0;
        const int item = blockIdx.x;
        r.b = item / a.n_splits;
        const int split = item - r.b * a.n_splits;
        const int L = clamped_len(a, r.b);
        r.t0 = split * a.chunk_tokens;
        r.t1 = (r.t0 + a.chunk_tokens < L) ? r.t0 + a.chunk_tokens : L;
        r.n_tiles = (r.t1 - r.t0 + kTile - 1) / kTile;
        r.len = L;
        r.slot = item;
        r.final_result = a.n_splits == 1;
        r.seq_end = 0;
        if (r.t0 >= r.t1) {
            if (split == 0) {
                float4* o = (float4*)(a.out + (size_t)r.b * kHeads * kHeadDim);
                for (int i = threadIdx.x; i < kHeads * kHeadDim / 4; i += THREADS) o[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
            return false;
        }
        make_uniform(r);
        return true;
    }
    int b = s.b, L = s.len;
    while (L == 0) {                                                  // sequences without tiles (one with tiles follows: lo < hi)
        const int lane = threadIdx.x & 63;
        const int ahead = b + 1 + lane < a.B ? clamped_len(a, b + 1 + lane) : 0;
        const unsigned long long hit = __ballot(ahead != 0);
        const int src = hit ? __builtin_ctzll(hit) : 63;
        b = __builtin_amdgcn_readfirstlane(b + 1 + src);
        L = __builtin_amdgcn_readlane(ahead, __builtin_amdgcn_readfirstlane(src));
    }
    const int seq0 = s.seq0 + s.pad, seq1 = seq0 + (L + kTile - 1) / kTile;
    const int end = s.hi < seq1 ? s.hi : seq1;
    if (s.lo < seq0) s.lo = seq0;
    if (s.lo >= end) { s.lo = s.hi; return false; }                  // the range ends in what is laid ahead of the sequence
    r.b = b;
    r.t0 = (s.lo - seq0) * kTile;
    r.t1 = (end - seq0) * kTile < L ? (end - seq0) * kTile : L;
    r.n_tiles = end - s.lo;
    r.len = L;
    r.final_result = seq0 >= s.my_lo && seq1 <= s.hi;                // the whole sequence lies in my range
    r.slot = range_index() + b;
    r.seq_end = s.lo == seq0 ? seq1 : 0;
    s.lo = end;
    s.seq0 = seq1;
    s.b = b + 1;
    // (asked for now, used when the next segment is: through the constant address space, a scalar load)
    if (end < s.hi) s.len = clamped_len(a, b + 1);
    make_uniform(r);
    return true;
}

}  // namespace mfa
