// Decode-step MFA attention for gfx950: 64 query heads of dimension 256 over one
// shared key head and one shared value head (paper, Section 2), one query token
// per sequence (or a pair, Section 5.2), independent sequences (Section 7.1).
//
// Work decomposition.  A workgroup works off segments: pieces
// [t0, t1) of one sequence's tokens, streamed once from HBM (mfa_attn_core.hpp:
// which segments a workgroup gets, how the waves share a tile, the MFMA operand
// layouts).  A segment that covers its whole sequence writes the final output;
// otherwise it leaves an unnormalised partial (acc, m, l) in the workspace that
// merge_splits_kernel reduces in order of position.
//
// bf16 cache: tiles of 64 tokens (= one cache page) are brought in with 16-byte
// global->LDS direct loads into a two-slot ring (64 KB per slot: two 32-token
// unit images).  The XOR swizzle of the unit image is applied on the global side
// of the direct load because its LDS side is fixed to base + 16*lane.
//
// 8-bit and 4-bit caches (e4m3 / e2m1 codes, one fp32 scale per token per
// tensor): mfa_lowbit.hpp and, for little work per workgroup, mfa_lowbit_short.hpp.
// Short contexts of any cache type: mfa_brief.hpp, one launch and nothing to merge.
// The key scale multiplies the score column of its token, the value scale rides
// on the attention weight of its token.
#include <hip/hip_ext.h>

#include "mfa_brief.hpp"
#include "mfa_kernel_choice.hpp"
#include "mfa_lowbit_short.hpp"
#include "mfa_merge_place.hpp"
#include "mfa_multi_short.hpp"

namespace mfa {

constexpr int kLoadsPerTileAndWave = 8;               // direct loads a wave of decode_bf16_kernel issues per tile (4 rows pairs x K, V)
// QL = query tokens per sequence.  1: wave = 4*(token half of the tile) + head group.  2: wave =
// 4*(query token of the pair q0, q0 + 1) + head group, and every wave works through both halves of each
// tile; query token j of q_len attends to the first len - (q_len - 1 - j) cached tokens (the new tokens are
// the last q_len of the cache).  More than two query tokens are worked off pair by pair, one launch each.
template <bool PAGED, int QL>
__global__ __launch_bounds__(kAttnThreads) void decode_bf16_kernel(AttnArgs a)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const lds_ptr_t lds_base = (lds_ptr_t)smem;
    const uint32_t lds_addr0 = (uint32_t)(uintptr_t)lds_base;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wq = wave & 3;
    const int grp = wave >> 2;
    const int n = lane & 15;
    const int g = lane >> 4;

    // Wave w brings rows [8w, 8w+8) of a tile's K and V: all in unit w/4.  Rows at or past the segment's
    // end re-read its last valid token, so nothing outside the sequence is touched and every LDS row
    // holds finite data (the weights of those rows are masked to zero).
    // (guessed: the tile named by guess_first_tile, whose position comes out of vector arithmetic; its
    // addresses stay in vector registers)
    auto issue_tile = [&](const Segment& sg, int tile, int slot, int page, bool guessed = false) {
        const int tile_t0 = sg.t0 + tile * kTile;
        const int64_t row0 = tile_row0<PAGED>(a, sg.b, tile_t0, page);
        const unsigned char* k_tile = (const unsigned char*)a.k + row0 * 512;   // wave-uniform: scalar registers
        const unsigned char* v_tile = (const unsigned char*)a.v + row0 * 512;
        const int p16 = lane & 31;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int row = 8 * wave + 2 * u + (lane >> 5);          // row of the tile this lane fills
            int in_tile = row;
            if (tile_t0 + row > sg.t1 - 1) in_tile = sg.t1 - 1 - tile_t0;
            const int key = row & 15;
            const int ck = p16 ^ key;
            const int cv = ((((p16 >> 1) ^ key) << 1) | (p16 & 1));
            const int first_row = 8 * wave + 2 * u;                   // wave-uniform
            const uint32_t dst = lds_addr0 + slot * kSlotBytes + (first_row >> 5) * kUnitBytes + (first_row & 31) * 512;
            if (guessed) {
                load_to_lds_16B_vaddr(k_tile + (uint32_t)(in_tile * 512 + ck * 16), dst);
                load_to_lds_16B_vaddr(v_tile + (uint32_t)(in_tile * 512 + cv * 16), dst + kUnitVOffset);
            } else {
                load_to_lds_16B(k_tile, (uint32_t)(in_tile * 512 + ck * 16), dst);
                load_to_lds_16B(v_tile, (uint32_t)(in_tile * 512 + cv * 16), dst + kUnitVOffset);
            }
        }
    };
    auto load_q = [&](QFrags& q, const Segment& sg) {
        load_q_fragments(q.f, a.q, QL == 2 ? a.q_len * sg.b + a.q0 + grp : sg.b, 16 * wq + n, g);
    };

    // The workgroup's segments are worked off as one stream of tiles: while the last tile of a segment is
    // multiplied, the first tile of the next one is already on its way into the other slot,
    // and the end-of-segment exchange uses the slot of the tile just finished.
    //
    // The very first tile is asked for before the schedule is known: the lengths are requested first
    // (stage_lengths), then the tile that would be this workgroup's first if every sequence had the length of
    // the hint -- its place follows from the launch arguments alone -- and the schedule is worked out while
    // those 64 KB are on their way (the lengths, requested earlier, arrive earlier).  When the schedule
    // disagrees (ragged lengths), the right tile goes into the other slot and the guessed one is never looked
    // at; the guess only ever names whole tiles below the hint, i.e. memory the caller has vouched for.
    stage_lengths(a, lds_base, kBf16SchedOffset);
    const FirstTileGuess guess = guess_first_tile(a, kBf16Switch);
    if (guess.valid) {
        Segment gs;
        gs.b = guess.b; gs.t0 = guess.t0; gs.t1 = guess.t0 + kTile;
        issue_tile(gs, 0, 0, lookup_page<PAGED>(a, guess.b, guess.t0), true);   // kLoadsPerTileAndWave loads
    }
    await_lengths<kLoadsPerTileAndWave>(a, guess.valid);
    Schedule sched = schedule_begin<kAttnThreads>(a, lds_base, kBf16SchedOffset, kBf16Switch);
    Segment r, r_next;
    if (!schedule_next<kAttnThreads>(a, sched, r)) {
        wait_vmem_all();                              // nothing may still be writing into this workgroup's LDS when it ends
        return;
    }
    QFrags q;
    load_q(q, r);
    int slot0 = 0;                                    // slot of the segment's first tile
    if (!(guess.valid && r.b == guess.b && r.t0 == guess.t0 && r.t0 + kTile <= r.t1)) {
        slot0 = guess.valid ? 1 : 0;
        issue_tile(r, 0, slot0, lookup_page<PAGED>(a, r.b, r.t0));
    }
    for (bool more = true; more;) {
        schedule_record(a, sched, r);
        const int end_mine = r.len - (a.q_len - 1 - a.q0 - grp);      // QL == 2: grp = query token of the pair
        const int t1_mine = QL == 2 ? (r.t1 < end_mine ? r.t1 : end_mine) : r.t1;
        WaveState st;
        init_state(st);
        int page_next = r.n_tiles > 1 ? lookup_page<PAGED>(a, r.b, r.t0 + kTile) : 0;
        more = false;
        for (int it = 0; it < r.n_tiles; ++it) {
            const int slot = (slot0 + it) & 1;
            wait_vmem_all();
            __syncthreads();
            if (it + 1 < r.n_tiles) {
                issue_tile(r, it + 1, slot ^ 1, page_next);
                if (it + 2 < r.n_tiles) page_next = lookup_page<PAGED>(a, r.b, r.t0 + (it + 2) * kTile);
            } else {
                more = schedule_next<kAttnThreads>(a, sched, r_next);
                if (more) issue_tile(r_next, 0, slot ^ 1, lookup_page<PAGED>(a, r_next.b, r_next.t0));
            }
            if (QL == 2) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int unit = slot * kSlotBytes + u * kUnitBytes;
                    process_unit(st, q, lds_base, unit, unit + kUnitVOffset, r.t0 + it * kTile + u * kUnitTokens,
                                 t1_mine, a.scale_log2e, n, g);
                }
            } else {
                const int unit = slot * kSlotBytes + grp * kUnitBytes;
                process_unit(st, q, lds_base, unit, unit + kUnitVOffset, r.t0 + it * kTile + grp * kUnitTokens,
                             t1_mine, a.scale_log2e, n, g);
            }
        }
        const int last_slot = (slot0 + r.n_tiles - 1) & 1;
        if (more) load_q(q, r_next);                  // ordinary loads (kept out of the tile loop, where the compiler's
                                                      // waits for them would also wait for the tile in flight)
        if (QL == 2) finish_segment_two(st, a, r, grp, wq, lane);
        else         finish_segment(st, lds_base, last_slot * kSlotBytes, a, r, wq, grp, lane);
        if (more) {
            r = r_next;
            slot0 = last_slot ^ 1;
        }
    }
}

// Merge the partial results of one sequence (fixed splits: slots b*n_splits ...; balanced schedule:
// the slots recorded by the workgroup that held the sequence's first tile):
//   out = sum_s 2^(m_s - m*) acc_s / sum_s 2^(m_s - m*) l_s,  m* = max_s m_s,
// summed in split order (m* is reached batch by batch, rescaling what has been summed).  One thread per float4 of the partial's lane-order layout; splits are
// taken four at a time so that their loads are independent and in flight together.
//
// How many waves share a row's partial results, and whether the blocks of a die take the rows of that die: mfa_merge_place.hpp, with both sides measured.
int merge_waves(const AttnArgs& a)
{
    if (a.n_wgs == 0 && a.chunk_tokens == kUnitTokens) return merge_waves_of_runs(a.n_splits);           // (brief_cut_runs)
    return merge_waves(a.B, a.n_here, a.q_len, a.n_wgs > 0 ? a.n_wgs / a.B : a.n_splits);
}
bool merge_by_die(const AttnArgs& a, int waves) { return merge_by_die(a.B, a.n_here, a.q_len, a.n_wgs, waves); }

// With many short sequences nearly every block only finds that a workgroup has written its row's result, and what counts is the way there:
// the rule is a template argument, the division by 1 .. 4 a shift or a multiplication, length and record one round trip.  us of the kernel
// at 4000 / 512 sequences of one tile: 44.7 / 6.6 without these, 27.6 / 4.8 now.
//
// WAVES > 1: a block takes 64 float4 of a row, each of its waves a run of consecutive partial results, and the
// waves' sums are added in order through LDS.
template <bool BY_DIE, int WAVES>                                     // (BY_DIE: only under the balanced schedule)
__global__ __launch_bounds__(WAVES == 1 ? 256 : 64 * WAVES) void merge_splits_kernel(AttnArgs a)
{
    constexpr int kThreads = WAVES == 1 ? 256 : 64;                   // positions of a block
    constexpr int kBlocksPerRow = kHeads * kHeadDim / 4 / kThreads;
    const int n_here = a.n_here;                                      // query tokens of this launch, 1 .. 4
    static_assert(kMaxQueryTokens == 4, "the division by n_here");
    const bool balanced = BY_DIE || a.n_wgs > 0;
    const int thread = WAVES == 1 ? threadIdx.x : threadIdx.x & 63;
    int row, p;                                                       // sequence * n_here + query token of the launch; position in the partial's lane-order layout
    if (BY_DIE) {
        row = merge_row(blockIdx.x, a.B * n_here, kBlocksPerRow);
        if (row < 0) return;
        p = (int)((blockIdx.x >> 3) % kBlocksPerRow) * kThreads + thread;
    } else {
        row = (int)(blockIdx.x / kBlocksPerRow);
        p = (int)(blockIdx.x % kBlocksPerRow) * kThreads + thread;
    }
    const int b = n_here == 3 ? (int)((unsigned)row / 3u) : row >> (n_here >> 1);
    const int qtok = row - b * n_here;
    const int lane = p & 63;
    const int db = (p >> 6) & 15;
    const int wq = p >> 10;
    const int h = 16 * wq + (lane & 15);
    const int d = 16 * db + 4 * (lane >> 4);
    // (the length and the sequence's slot record are asked for together: one round trip, not two; the record of
    // a sequence without tokens holds whatever the workspace held and is not used)
    int L = a.seq_lens[b];
    const int2 rec = balanced ? ((const int2*)a.ws_seg)[b] : make_int2(0, 0);      // first slot, number of partials
    L = L < 0 ? 0 : (L > a.max_seq_len_hint ? a.max_seq_len_hint : L);
    float4* const o = (float4*)(a.out + (((size_t)b * a.q_len + a.q0 + qtok) * kHeads + h) * kHeadDim + d);
    const int L_mine = L - (a.q_len - 1 - a.q0 - qtok);               // tokens this query token attends to
    int n_valid;
    size_t item0;
    if (balanced) {
        if (L == 0) { *o = make_float4(0.f, 0.f, 0.f, 0.f); return; }
        item0 = (size_t)rec.x;
        n_valid = rec.y;
        if (n_valid == 1 && n_here < 3) return;                       // one workgroup held it all and wrote the result
                                                                      // (the one-pass kernel for 3 / 4 tokens never does)
    } else {
        if (L == 0) return;                                           // zeros were written by the first split
        n_valid = (L + a.chunk_tokens - 1) / a.chunk_tokens;
        if (n_valid > a.n_splits) n_valid = a.n_splits;               // (brief_attn_kernel's runs: they have several units each)
        item0 = (size_t)b * a.n_splits;
    }
    if (L_mine <= 0) { *o = make_float4(0.f, 0.f, 0.f, 0.f); return; }   // (only with several query tokens and L < q_len)
    const size_t slot0 = item0 * n_here + qtok;                       // partial of (item, query token) at item*n_here + qtok
    const size_t slot_step = (size_t)n_here;
    const float2* ml_base = (const float2*)a.ws_ml + slot0 * kHeads + h;
    const float4* acc_base = (const float4*)a.ws_acc + slot0 * (kHeads * kHeadDim / 4) + p;

    // One pass with a running reference exponent: a batch's (m, l) pairs and accumulator pieces are loaded
    // together, so the weights do not wait for a first round trip that only fetches the maxima.
    constexpr int kBatch = WAVES == 1 ? 4 : 8;
    float m = -INFINITY;
    float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
    float l = 0.f;
    auto add = [&](const float2* ml, const float4* v, int n) {        // pieces 0 .. n - 1 of a batch (the others repeat the last)
        float m_new = m;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) m_new = fmaxf(m_new, ml[u].x);
        const float m_safe = m_new == -INFINITY ? 0.f : m_new;       // pieces without tokens have m = -inf
        const float keep = fast_exp2(m - m_safe);                    // 0 while nothing has been summed
        sum.x *= keep; sum.y *= keep; sum.z *= keep; sum.w *= keep;
        l *= keep;
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const float w = u < n ? fast_exp2(ml[u].x - m_safe) : 0.f;
            sum.x += w * v[u].x; sum.y += w * v[u].y; sum.z += w * v[u].z; sum.w += w * v[u].w;
            l += w * ml[u].y;
        }
        m = m_new;
    };
    const int wave = WAVES == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int first = n_valid * wave / WAVES, end = n_valid * (wave + 1) / WAVES;
    for (int s0 = first; s0 < end; s0 += kBatch) {
        float2 ml[kBatch];
        float4 v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int s = s0 + u < end ? s0 + u : end - 1;
            ml[u] = ml_base[(size_t)s * slot_step * kHeads];
            v[u] = acc_base[(size_t)s * slot_step * (kHeads * kHeadDim / 4)];
        }
        add(ml, v, end - s0);
    }
    // A last piece that is infinite has become NaN where it was repeated (0 times infinity): then piece by piece.  (Out of the way, since what counts here is how much code a
    // block has to fetch: a mask on every piece took 0.1 .. 0.3 us a call, whole batches apart from others up to 0.7.)
    if (__builtin_expect(__builtin_fmaf(sum.x, 0.f, __builtin_fmaf(sum.y, 0.f, __builtin_fmaf(sum.z, 0.f, sum.w * 0.f))) != 0.f, 0)) {
        const float m_safe = m == -INFINITY ? 0.f : m;
        float4 plain = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 1
        for (int s = first; s < end; ++s) {
            const float w = fast_exp2(ml_base[(size_t)s * slot_step * kHeads].x - m_safe);
            const float4 v = acc_base[(size_t)s * slot_step * (kHeads * kHeadDim / 4)];
            plain.x += w * v.x; plain.y += w * v.y; plain.z += w * v.z; plain.w += w * v.w;
        }
        auto fix = [](float& x, float y) { if (!(x * 0.f == 0.f)) x = y; };
        fix(sum.x, plain.x); fix(sum.y, plain.y); fix(sum.z, plain.z); fix(sum.w, plain.w);
    }
    if constexpr (WAVES > 1) {
        __shared__ float4 part[WAVES][64];
        __shared__ float2 part_ml[WAVES][64];
        part[wave][thread] = sum;
        part_ml[wave][thread] = make_float2(m, l);
        __syncthreads();
        if (wave != 0) return;
        m = -INFINITY;
        sum = make_float4(0.f, 0.f, 0.f, 0.f);
        l = 0.f;
        float2 ml[kBatch];
        float4 v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            ml[u] = u < WAVES ? part_ml[u % WAVES][thread] : make_float2(-INFINITY, 0.f);
            v[u] = u < WAVES ? part[u % WAVES][thread] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
        add(ml, v, WAVES);
    }
    const float inv = 1.0f / l;
    *o = make_float4(sum.x * inv, sum.y * inv, sum.z * inv, sum.w * inv);
}

// Copy the logical rows of every sequence out of a paged pool (test aid).
__global__ __launch_bounds__(256) void gather_paged_kernel(const uint32_t* pool, int32_t row_words,
                                                           const int32_t* block_table, int32_t max_blocks_per_seq,
                                                           int32_t n_pages, const int32_t* seq_lens, int32_t hint, uint32_t* dst,
                                                           int64_t dst_seq_stride_tokens)
{
    const int b = blockIdx.y;
    const int blk = blockIdx.x;
    int L = seq_lens[b];
    L = L < 0 ? 0 : (L > hint ? hint : L);
    const int tok0 = blk * kPage;
    if (tok0 >= L) return;
    const int n_tok = (L - tok0 < kPage) ? L - tok0 : kPage;
    int page = block_table[(size_t)b * max_blocks_per_seq + blk];
    page = page < 0 ? 0 : (page >= n_pages ? n_pages - 1 : page);
    const uint32_t* src = pool + (size_t)page * kPage * row_words;
    uint32_t* d = dst + ((size_t)b * dst_seq_stride_tokens + tok0) * row_words;
    for (int i = threadIdx.x; i < n_tok * row_words; i += 256) d[i] = src[i];
}

// Measurement aid: read two buffers once with plain 16-byte loads and do nothing else.  What
// this reaches is the practical ceiling for any kernel that must stream the same bytes.
__global__ __launch_bounds__(256) void stream_read_kernel(const uint4* __restrict__ a, const uint4* __restrict__ b,
                                                          size_t n16_per_block, uint32_t* sink)
{
    const uint4* pa = a + (size_t)blockIdx.x * n16_per_block;
    const uint4* pb = b + (size_t)blockIdx.x * n16_per_block;
    uint32_t acc = 0;
    for (size_t i = threadIdx.x; i < n16_per_block; i += 512) {
        // non-temporal like the attention kernels' own streaming loads (measured: the faster of the two policies)
        const u32x4 x0 = __builtin_nontemporal_load((const u32x4*)pa + i), x1 = __builtin_nontemporal_load((const u32x4*)pa + i + 256);
        const u32x4 y0 = __builtin_nontemporal_load((const u32x4*)pb + i), y1 = __builtin_nontemporal_load((const u32x4*)pb + i + 256);
        const u32x4 z = x0 ^ x1 ^ y0 ^ y1;
        acc ^= z[0] ^ z[1] ^ z[2] ^ z[3];
    }
    if (acc == 0x9e3779b9u) sink[0] = acc;     // keeps the loads alive; practically never true
}

hipError_t launch_stream_read(const void* a, const void* b, size_t bytes_each, void* sink, hipStream_t stream,
                              hipEvent_t ev_before, hipEvent_t ev_after)
{
    constexpr unsigned kBlocks = 2048;
    if (!(ev_before && ev_after)) ev_before = ev_after = nullptr;
    hipExtLaunchKernelGGL(stream_read_kernel, dim3(kBlocks), dim3(256), 0, stream, ev_before, ev_after, 0,
                          (const uint4*)a, (const uint4*)b, bytes_each / kBlocks / 16, (uint32_t*)sink);
    return hipGetLastError();
}

SplitPlan plan_splits(int32_t B, int32_t max_seq_len_hint, int32_t target_items)
{
    const int32_t max_tiles = (max_seq_len_hint + kTile - 1) / kTile;
    int32_t want = (target_items + B - 1) / B;
    if (want < 1) want = 1;
    if (want > max_tiles) want = max_tiles;
    const int32_t chunk_tiles = (max_tiles + want - 1) / want;
    SplitPlan p;
    p.chunk_tokens = chunk_tiles * kTile;
    p.n_splits = (max_tiles + chunk_tiles - 1) / chunk_tiles;
    return p;
}

int32_t balanced_workgroups(int32_t B, int32_t max_seq_len_hint, int32_t target_items)
{
    if (B > kMaxBalancedBatch) return 0;
    const int64_t max_tiles = (int64_t)B * ((max_seq_len_hint + kTile - 1) / kTile);
    return (int32_t)(max_tiles < target_items ? max_tiles : target_items);
}

namespace {

struct AttnKernel { const void* fn; unsigned threads, lds_bytes; };

template <int QL, int BITS>
AttnKernel lowbit_kernel(bool paged, bool short_work)
{
    if (short_work) return {paged ? (const void*)short_lowbit_kernel<true, QL, BITS> : (const void*)short_lowbit_kernel<false, QL, BITS>, kAttnThreads, kBf16LdsBytes};
    return {paged ? (const void*)decode_lowbit_kernel<true, QL, BITS> : (const void*)decode_lowbit_kernel<false, QL, BITS>, kLowbitThreads, LowbitShape<QL, BITS>::kLdsBytes};
}
template <int QL>
AttnKernel attn_kernel(mfa_kv_dtype kv_dtype, bool paged, bool short_work)
{
    if (kv_dtype == MFA_KV_BF16) return {paged ? (const void*)decode_bf16_kernel<true, QL> : (const void*)decode_bf16_kernel<false, QL>, kAttnThreads, kBf16LdsBytes};
    return kv_dtype == MFA_KV_FP4_E2M1 ? lowbit_kernel<QL, 4>(paged, short_work) : lowbit_kernel<QL, 8>(paged, short_work);
}
AttnKernel multi_kernel(int q_len, bool paged, bool short_work)
{
    if (short_work) return {paged ? (const void*)short_bf16_multi_kernel<true> : (const void*)short_bf16_multi_kernel<false>, kMultiThreads, kShortMultiLdsBytes};
    if (q_len == 3) return {paged ? (const void*)decode_bf16_multi_kernel<true, 3> : (const void*)decode_bf16_multi_kernel<false, 3>, kMultiThreads, kMultiLdsBytes};
    return {paged ? (const void*)decode_bf16_multi_kernel<true, 4> : (const void*)decode_bf16_multi_kernel<false, 4>, kMultiThreads, kMultiLdsBytes};
}

template <int BITS, int NH, int DS, bool CUT = false>
AttnKernel brief_form(bool paged)
{
    using S = BriefShape<BITS, NH, DS>;
    return {paged ? (const void*)brief_attn_kernel<true, BITS, NH, DS, CUT> : (const void*)brief_attn_kernel<false, BITS, NH, DS, CUT>, S::kThreads, S::kLdsBytes};
}
template <int BITS>
AttnKernel brief_kernel(bool paged, int parts, bool cut)
{
    static_assert(BriefShape<BITS, 1, 1>::kParts == kBriefCutParts, "workgroups per run");
    if (cut) return brief_form<BITS, 1, 1, true>(paged);
    return parts == 16 ? brief_form<BITS, 1, 4>(paged) : parts == 8 ? brief_form<BITS, 1, 2>(paged) : parts == 4 ? brief_form<BITS, 1, 1>(paged) : brief_form<BITS, 2, 1>(paged);
}
AttnKernel brief_kernel(mfa_kv_dtype kv_dtype, bool paged, int parts, bool cut)
{
    return kv_dtype == MFA_KV_BF16 ? brief_kernel<16>(paged, parts, cut) : kv_dtype == MFA_KV_FP8_E4M3 ? brief_kernel<8>(paged, parts, cut) : brief_kernel<4>(paged, parts, cut);
}
int cache_bits(mfa_kv_dtype kv_dtype) { return kv_dtype == MFA_KV_BF16 ? 16 : kv_dtype == MFA_KV_FP8_E4M3 ? 8 : 4; }
// Workgroups per row of brief_attn_kernel, 0 where another kernel takes the call (mfa_kernel_choice.hpp)
int brief_cut(const AttnArgs& a, mfa_kv_dtype kv_dtype)
{
    if (!a.may_be_brief) return 0;
    return brief_parts(cache_bits(kv_dtype), a.q_len, (int64_t)a.B * a.q_len, a.max_seq_len_hint);
}

// ... and else into how many runs it cuts a row, 0 likewise
int brief_cut_runs(const AttnArgs& a, mfa_kv_dtype kv_dtype)
{
    if (!a.may_be_brief) return 0;
    return brief_runs(cache_bits(kv_dtype), a.q_len, (int64_t)a.B * a.q_len, a.max_seq_len_hint);
}

// 64-token tiles per workgroup at the length of the hint (the host knows no other).
int64_t tiles_per_sequence(const AttnArgs& a) { return (a.max_seq_len_hint + kTile - 1) / kTile; }
int64_t tiles_per_workgroup(const AttnArgs& a) { return a.n_wgs > 0 ? a.B * tiles_per_sequence(a) / a.n_wgs : a.chunk_tokens / kTile; }
// Three query tokens over a bf16 cache: short_bf16_multi_kernel below 4 tiles per workgroup.  us per call, short / decode, 20 and 128 sequences of the
// length of the hint and drawn from 1 .. hint:
//   1 tile  30.4/31.7 31.5/32.6  33.3/34.8 34.2/34.8     3 tiles  40.3/38.2 36.1/36.2  42.3/41.2 43.7/42.8     5 tiles  49.1/44.0 39.5/39.0  50.7/46.9 49.0/45.3
// Four tokens always take decode_bf16_multi_kernel; a like kernel of 16 heads per wave took, against it:
//   1 tile  37.7/37.4  37.8/37.6     2 tiles  43.3/42.2  48.9/48.6     4 tiles  54.1/49.1  56.1/54.0     16 tiles  122.7/97.3  90.0/77.8
bool short_multi_work(const AttnArgs& a) { return a.q_len == 3 && tiles_per_workgroup(a) < 4; }

// Which of its two kernels a low-bit cache takes (mfa_kernel_choice.hpp)
bool short_lowbit_work(const AttnArgs& a, mfa_kv_dtype kv_dtype)
{
    return takes_short_lowbit_kernel(kv_dtype == MFA_KV_FP4_E2M1, a.q_len == 1, tiles_per_workgroup(a), tiles_per_sequence(a));
}
}  // namespace

hipError_t prepare_decode_attn_kernels()
{
    for (const int parts : {2, 4, 8, 16, 0})          // (0: runs)
        for (int form = 0; form < 6; ++form) {
            const AttnKernel k = brief_kernel(form < 2 ? MFA_KV_BF16 : form < 4 ? MFA_KV_FP8_E4M3 : MFA_KV_FP4_E2M1, (form & 1) != 0, parts, parts == 0);
            const hipError_t e = hipFuncSetAttribute(k.fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.lds_bytes);
            if (e != hipSuccess) return e;
        }
    for (int form = 0; form < 6; ++form) {            // three and four tokens, three tokens for little work; paged or not
        const AttnKernel k = multi_kernel(form / 2 == 1 ? 4 : 3, (form & 1) != 0, form / 2 == 2);
        const hipError_t e = hipFuncSetAttribute(k.fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.lds_bytes);
        if (e != hipSuccess) return e;
    }
    for (int dt = 0; dt < 3; ++dt)
        for (int form = 0; form < 8; ++form) {
            const mfa_kv_dtype kvd = dt == 0 ? MFA_KV_BF16 : (dt == 1 ? MFA_KV_FP8_E4M3 : MFA_KV_FP4_E2M1);
            const bool paged = (form & 1) != 0, short_work = (form & 2) != 0;
            const AttnKernel k = (form & 4) ? attn_kernel<2>(kvd, paged, short_work) : attn_kernel<1>(kvd, paged, short_work);
            const hipError_t e = hipFuncSetAttribute(k.fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.lds_bytes);
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

hipError_t launch_decode_attn(const AttnArgs& a, mfa_kv_dtype kv_dtype, hipStream_t stream,
                              hipEvent_t ev_before, hipEvent_t ev_after)
{
    const dim3 grid((unsigned)(a.n_wgs > 0 ? a.n_wgs : a.B * a.n_splits));
    if (kv_dtype != MFA_KV_BF16 && kv_dtype != MFA_KV_FP8_E4M3 && kv_dtype != MFA_KV_FP4_E2M1) return hipErrorNotSupported;
    if (a.q_len < 1 || a.q_len > kMaxQueryTokens) return hipErrorNotSupported;
    if (a.q_len != 1 && a.n_wgs == 0) return hipErrorNotSupported;     // several query tokens: balanced schedule only
    // The two events, when given, are attached to the streaming kernel's own dispatch: they take the
    // times at which that kernel starts and ends on the device, with no launch gap inside the interval.
    // (With more than two query tokens: the first pair's.)
    if (!(ev_before && ev_after)) ev_before = ev_after = nullptr;
    auto launch_merge = [&](const AttnArgs& args) {
        const int rows = args.B * args.n_here;
        const int waves = merge_waves(args);
        const bool by_die = merge_by_die(args, waves);
        const int per_row = waves == 1 ? kMergeBlocksPerRow : kHeads * kHeadDim / 4 / 64;
        const void* fn = waves == 8 ? (by_die ? (const void*)merge_splits_kernel<true, 8> : (const void*)merge_splits_kernel<false, 8>)
                       : waves == 4 ? (by_die ? (const void*)merge_splits_kernel<true, 4> : (const void*)merge_splits_kernel<false, 4>)
                                     : (by_die ? (const void*)merge_splits_kernel<true, 1> : (const void*)merge_splits_kernel<false, 1>);
        AttnArgs copy = args;
        void* params[] = {&copy};
        const hipError_t e = hipLaunchKernel(fn, dim3(by_die ? merge_blocks_by_die(rows, per_row) : (unsigned)(per_row * rows)), dim3(waves == 1 ? 256 : 64 * waves), params, 0, stream);
        return e != hipSuccess ? e : hipGetLastError();
    };
    if (const int parts = brief_cut(a, kv_dtype)) {
        AttnArgs args = a;
        void* params[] = {&args};
        const AttnKernel k = brief_kernel(kv_dtype, a.block_table != nullptr, parts, false);
        const unsigned rows = (unsigned)(a.B * a.q_len);
        const hipError_t e = hipExtLaunchKernel(k.fn, dim3(8u * (unsigned)parts * ((rows + 7) / 8)), dim3(k.threads), params, k.lds_bytes, stream, ev_before, ev_after, 0);
        return e != hipSuccess ? e : hipGetLastError();
    }
    if (const int runs = brief_cut_runs(a, kv_dtype)) {
        AttnArgs args = a;
        args.n_wgs = 0;                                                 // (partial results: at most kMostBriefRuns slots, fewer than any workspace with the default work distribution has)
        args.n_splits = runs;
        args.chunk_tokens = kUnitTokens;                                // (units are dealt out: as many runs have some as the length has units)
        args.n_here = a.q_len;
        void* params[] = {&args};
        const AttnKernel k = brief_kernel(kv_dtype, a.block_table != nullptr, 0, true);
        const unsigned items = (unsigned)(a.B * a.q_len * runs);
        hipError_t e = hipExtLaunchKernel(k.fn, dim3(8u * kBriefCutParts * ((items + 7) / 8)), dim3(k.threads), params, k.lds_bytes, stream, ev_before, ev_after, 0);
        if (e == hipSuccess) e = hipGetLastError();
        return e != hipSuccess ? e : launch_merge(args);
    }
    // Three and four query tokens over a bf16 cache, batches the per-wave schedule covers: one pass over the cache
    // by the kernel that keeps all of a sequence's query tokens in one wave.
    if (a.q_len >= 3 && kv_dtype == MFA_KV_BF16 && a.B <= kWaveScanChunks * 64) {
        AttnArgs args = a;
        args.q0 = 0;
        args.n_here = a.q_len;
        void* params[] = {&args};
        const AttnKernel k = multi_kernel(a.q_len, a.block_table != nullptr, short_multi_work(a));
        hipError_t e = hipExtLaunchKernel(k.fn, grid, dim3(k.threads), params, k.lds_bytes, stream, ev_before, ev_after, 0);
        if (e != hipSuccess) return e;
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_merge(args);
    }
    const bool short_work = kv_dtype != MFA_KV_BF16 && short_lowbit_work(a, kv_dtype);
    const AttnKernel kernel = a.q_len >= 2 ? attn_kernel<2>(kv_dtype, a.block_table != nullptr, short_work) : attn_kernel<1>(kv_dtype, a.block_table != nullptr, short_work);
    const int n_here = a.q_len == 1 ? 1 : 2;
    // Otherwise query tokens are worked off in pairs (q0, q0 + 1), one pass over the cache each; an odd count ends
    // with the pair (q_len - 2, q_len - 1), which computes token q_len - 2 a second time with the same result.
    // The passes share the partial-result workspace: they are ordered by the stream.
    for (int q0 = 0; q0 < a.q_len; q0 += 2) {
        AttnArgs args = a;
        args.q0 = q0 + n_here <= a.q_len ? q0 : a.q_len - n_here;
        args.n_here = n_here;
        void* params[] = {&args};
        hipError_t e = hipExtLaunchKernel(kernel.fn, grid, dim3(kernel.threads), params, kernel.lds_bytes, stream, q0 == 0 ? ev_before : nullptr,
                                          q0 == 0 ? ev_after : nullptr, 0);
        if (e != hipSuccess) return e;
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        if (a.n_wgs > 0 || a.n_splits > 1) {
            e = launch_merge(args);
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

hipError_t launch_gather_paged(const void* pool, int32_t row_bytes, const int32_t* block_table,
                               int32_t max_blocks_per_seq, int32_t n_pages, const int32_t* seq_lens, int32_t max_seq_len_hint,
                               int32_t B, void* dst, int64_t dst_seq_stride_tokens, hipStream_t stream)
{
    const int blocks = (max_seq_len_hint + kPage - 1) / kPage;
    hipLaunchKernelGGL(gather_paged_kernel, dim3((unsigned)blocks, (unsigned)B), dim3(256), 0, stream,
                       (const uint32_t*)pool, row_bytes / 4, block_table, max_blocks_per_seq, n_pages, seq_lens,
                       max_seq_len_hint, (uint32_t*)dst, dst_seq_stride_tokens);
    return hipGetLastError();
}

}  // namespace mfa
