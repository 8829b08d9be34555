// Low-rank query path of MFA (paper, Section 2): c = x.W_qa, RMS normalisation over the
// rank axis, q = c_hat.W_qb.  Three launches on the caller's stream:
//   1. split-K bf16 MFMA GEMM, fp32 partial sums of c into the workspace;
//   2. reduce the partials, normalise, apply the gain, round to bf16;
//   3. bf16 MFMA GEMM writing q in bf16.
// The key/value projection and the output projection of the same layer are built from the same products.
//
// With at most a few hundred rows of x a product is bound by streaming the weights once: a workgroup owns a strip of
// output columns and all (up to 128) rows of x, and what decides its speed is how the two streams, W from HBM and x from L2,
// share a compute unit's way to memory (measured on MI355X, W of 67 MB, 256 workgroups):
//   * A compute unit is served best with 16 .. 32 KB of W in flight: a stream alone takes 12.9 us with 16, 13.2 with 32, 14.7 with
//     64 and 15.3 with 128 KB (a matrix of 235 MB: 36.4 us with 32, 38.9 with 64).  More only waits longer.
//   * Loads of one wave come back in order.  x asked for behind W waits as long as W does: 256 KB of W and 512 KB of x per compute
//     unit take 22 us when the same waves load both, the sum of either alone, and 15.0 when different waves do.
//   * Rows of 512 bytes of W side by side stream faster than rows of 256 or 128 (235 MB: 34.8 / 36.4 / 37 us).
//   * x is fast only as whole 128-byte lines per load instruction (row-major fragments of 64 bytes: 26 against 60 .. 80 GB/s).
// gemm_loader_kernel follows from that, for any number of rows.
#include "mfa_attn_core.hpp"

namespace mfa {

namespace {

constexpr int kStripN = 64;                  // columns of a strip
constexpr int kMaxSplits = 32;               // k splits of a product, at most
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// How a product finds x:
//   kRows   bf16, row-major [M, K]
//   kTiled  bf16 in the order a wave loads it: element (m, k) at ((k/32)*rows_pad + (m & ~15))*32 + ((k%32)/8)*128 + (m%16)*8 + k%8, so that
//           16 rows x 32 k are one KB in lane order
//   kFloat  fp32, row-major [M, K], rounded to bf16 on the way
//   kFarRows  as kRows, for rows so long that those of a wave are more than kReach apart
enum class XKind { kRows, kTiled, kFloat, kFarRows };
constexpr bool bf16_rows(XKind k) { return k == XKind::kRows || k == XKind::kFarRows; }
__device__ __forceinline__ size_t tiled_index(int m, int k, int rows_pad)
{
    return ((size_t)(k >> 5) * rows_pad + (m & ~15)) * 32 + ((k & 31) >> 3) * 128 + (m & 15) * 8 + (k & 7);
}

// Buffer resource for `base`: loads through it at offsets below kReach read memory, all others (kOutside) and, with !valid, every
// load return zeros without touching it.
constexpr uint32_t kReach = 0x7FFFFFFFu, kOutside = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_at(const unsigned char* base, bool valid)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(base), 0, valid ? (int)kReach : 0, 0x00020000);
}

// Row-major x reaches the lanes by way of a small image of the wave's own in LDS: it is loaded in whole 128-byte lines, written row
// by row and read back as fragments.  bf16, 64 k of a row = 128 bytes: 16-byte chunk c of row r at c ^ ((r >> 1) & 7).  From fp32, 32 k of a
// row = 64 bytes of bf16: chunk c of row r at c ^ ((r >> 2) & 3).  Either way 16 rows x one chunk touch every bank once.
__device__ __forceinline__ int image64_at(int row, int chunk) { return row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4); }
__device__ __forceinline__ int image32_at(int row, int chunk) { return row * 64 + ((chunk ^ ((row >> 2) & 3)) << 4); }

// ---- The product.  Four waves only load W, with direct loads into a ring of stages in LDS (128 B rows, XOR-swizzled on the global side so
// that the transposing reads are conflict-free), each keeping a fixed number of loads in flight: as the oldest lands, the next is asked for.
// Eight waves multiply: A = W^T (16 columns x 32 k) from the LDS transposing read, one unit ahead of its MFMAs, B = x^T (32 k x 16 rows) from
// global memory two stages ahead, v_mfma_f32_16x16x32_bf16 giving C^T[column, row].  One barrier per stage, which waits for
// LDS reads but for nobody's global loads.  The eight waves are 4 row groups x 2: halves of a stage's k steps (the two sums are added
// through LDS) or, where the sums of both would not fit the registers, the halves of the columns.
// OUT_BF16 = false: fp32 partial sums to out[(kz*rows_pad + m)*N + n];  true: bf16 result to out[m*N + n] (requires gridDim.z == 1).
// MB = 1 or 2: 16-row blocks per wave; a workgroup covers 64 * MB rows of x.
// NS = 1 or 4: 64-column strips per workgroup.  NS = 4 (the output projection) reads rows of 512 bytes and x once per 256 columns.
// us per product at 4 / 64 / 128 rows, a kernel whose eight waves loaded 64 KB stages of W, loaded x and multiplied in turn -> this one:
//   7168 -> 512     5.2 / 6.8 / 10.2  ->  4.2 / 5.6 / 7.7        7168 -> 2048   9.5 / 12.4 / 17.3  ->  7.7 / 9.3 / 12.4
//   2048 -> 16384  16.1 / 18.3 / 22.6 -> 13.3 / 15.4 / 18.0     16384 -> 7168  42.8 / 43.9 / 59.9  -> 38.7 / 42.6 / 47.5 (up to 64 rows from fp32)
// In flight: 16 KB with NS = 1 (32: 14.5 / 16.3 / 19.1 for the third), 32 KB with NS = 4 (64: 39.2 / 43.4 / 48.6, 16: 43.7 at 64 rows).  Two loading
// waves instead of four: 16.6 / 16.8 / 18.9 for the third; eight: the same within 1 %.  x three stages ahead: 1 .. 2 % slower.
constexpr int kLoaders = 4;
constexpr int kMultipliers = 8;
constexpr int kLoaderThreads = (kMultipliers + kLoaders) * 64;

template <XKind X_KIND, int MB, int NS>
struct LoaderShape {
    static constexpr bool kSplitK = NS == 1 || MB == 1;
    static constexpr int kStageBytes = NS == 4 && MB == 1 ? 32768 : 16384;
    static constexpr int kStageRows = kStageBytes / (128 * NS);
    static constexpr int kSubBytes = kStageBytes / NS;                  // one strip's part of a stage
    static constexpr int kMySteps = kStageRows / 32 / (kSplitK ? 2 : 1);   // k steps of a multiplying wave per stage
    static constexpr int kMyStrips = kSplitK ? NS : NS / 2;
    static constexpr int kLoads = kStageBytes / 1024 / kLoaders;       // direct loads of a loading wave per stage
    static constexpr int kAhead = (NS == 1 ? 16384 : 32768) / kStageBytes;   // stages in flight
    static constexpr int kSlots = kAhead + 2;                          // (one being multiplied, one complete)
    static constexpr int kImageBytes = bf16_rows(X_KIND) ? MB * 2048 : X_KIND == XKind::kFloat ? MB * 1024 : 0;
    static constexpr int kImageBase = kSlots * kStageBytes;
    static constexpr int kCols = kStripN * NS;
    static constexpr int kRows = 64 * MB;
    static constexpr int kTileStride = kCols * 4 + 16;                  // rows of the result tile 16 bytes apart modulo the banks
    static constexpr int kRingBytes = kImageBase + kMultipliers * kImageBytes;
    static constexpr int kLdsBytes = kRingBytes > kRows * kTileStride ? kRingBytes : kRows * kTileStride;
    static_assert(kLdsBytes <= 160 * 1024, "LDS of a compute unit");
    static_assert(NS == 1 || NS == 4, "one strip, k steps shared out; or four, columns shared out");
    static_assert(!bf16_rows(X_KIND) || kMySteps == 2, "an image of row-major bf16 holds 64 k");
    static_assert(X_KIND != XKind::kFloat || kMySteps == 1, "an image of row-major fp32 holds 32 k");
};

// Swizzle key of a W row in LDS: its 32-byte chunk c is stored at position c ^ key.  A transposing
// read touches rows 8g + 4t + i (g = 0..3, i = 0..3) at one chunk each.  Rows are 128 bytes, so rows
// of equal parity share their banks; with key = 2*(g & 1) + i/2 the four rows of equal parity read
// by each half of the wave (g = 0, 1 or g = 2, 3) take the four chunk positions once each.
__device__ __forceinline__ int w_key(int row) { return (((row >> 3) & 1) << 1) | ((row >> 1) & 1); }

// Workgroup barrier that leaves this wave's global loads in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <bool OUT_BF16, XKind X_KIND, int MB, int NS>
__global__ __launch_bounds__(kLoaderThreads) void gemm_loader_kernel(const void* __restrict__ X, const uint16_t* __restrict__ W,
                                                                     void* __restrict__ out, int M, int K, int N, int k_per_split, int rows_pad)
{
    using S = LoaderShape<X_KIND, MB, NS>;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const lds_ptr_t lds_base = (lds_ptr_t)smem;
    const uint32_t lds_addr0 = (uint32_t)(uintptr_t)lds_base;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;

    // Groups of strips (the output projection): the workgroups are numbered die by die (workgroup i runs on die i % 8; nothing but speed
    // depends on it): a die's workgroups then share one or two slices of x, and its lines of W lie side by side.
    int group = blockIdx.x, kz = blockIdx.z;
    if (NS > 1) {
        const int n_groups = gridDim.x, n_wgs = n_groups * gridDim.z, id = blockIdx.x + n_groups * blockIdx.z, die = id & 7, rest = n_wgs & 7;
        const int place = die * (n_wgs >> 3) + (die < rest ? die : rest) + (id >> 3);
        kz = __builtin_amdgcn_readfirstlane(place / n_groups);
        group = place - kz * n_groups;
    }
    const int n0 = group * S::kCols;
    const int m0 = blockIdx.y * S::kRows;
    const int k_begin = kz * k_per_split;
    const int k_end = k_begin + k_per_split < K ? k_begin + k_per_split : K;
    const int n_stages = (k_end - k_begin + S::kStageRows - 1) / S::kStageRows;
    // Workgroups walk the stages of their k range starting at different points and wrapping round: at any moment
    // those that share an L2 then ask it for different parts of x instead of all for the same lines.
    const int phase = (int)((unsigned)(NS > 1 ? group : group >> 3) % (unsigned)n_stages);   // (without a k split, workgroups 8 apart share an L2)
    auto stage_k0 = [&](int it) { const int s = it + phase; return k_begin + (s < n_stages ? s : s - n_stages) * S::kStageRows; };

    f32x4 acc[MB][4 * S::kMyStrips];
    const int mp = wave & 3, half = (wave >> 2) & 1;
    const int kh = S::kSplitK ? half : 0, nh = S::kSplitK ? 0 : half;
    const int my_row0 = 16 * MB * mp;
    if (wave >= kMultipliers) {
        const int lw = wave - kMultipliers;
        constexpr int L = S::kLoads, A = S::kAhead;
        // load i of a stage: 8 rows of one strip.  (A half stage at the end of the k range: its first rows again, never multiplied.)
        auto request = [&](int it, int slot, int i) {
            const int k0 = stage_k0(it);
            const unsigned char* w_stage = (const unsigned char*)W + ((size_t)k0 * N + n0) * 2;   // wave-uniform
            const int l = L * lw + i;
            constexpr int kGroups = S::kStageRows / 8;
            const int strip = l / kGroups, first_row = 8 * (l % kGroups);
            const int in_stage = first_row + (lane >> 3);
            const int row = k0 + first_row < k_end ? in_stage : lane >> 3;
            const int p8 = lane & 7;                                   // 16-byte position in the 128-byte row
            const int c16 = (((p8 >> 1) ^ w_key(in_stage)) << 1) | (p8 & 1);
            load_to_lds_16B(w_stage, (uint32_t)row * (uint32_t)N * 2u + (uint32_t)(strip * 128 + c16 * 16),
                            lds_addr0 + slot * S::kStageBytes + strip * S::kSubBytes + first_row * 128);
        };
        int slot = 0;
        for (; slot < A && slot < n_stages; ++slot)
#pragma unroll
            for (int i = 0; i < L; ++i) request(slot, slot, i);
        for (int it = 0; it < n_stages; ++it) {
            // stage `it` is complete when no more than the A - 1 stages behind it are in flight.  The slot that stage it + A goes to was
            // multiplied before the last barrier but one.
            if (it + A < n_stages) {
#pragma unroll
                for (int i = 0; i < L; ++i) { wait_vmem_but<A * L - 1>(); request(it + A, slot, i); }
            } else if (A == 2 && it + 1 < n_stages) wait_vmem_but<L>();
            else wait_vmem_but<0>();
            slot = slot + 1 == S::kSlots ? 0 : slot + 1;
            lds_barrier();
        }
        static_assert(A <= 2, "waits at the end of the k range");
    } else {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < 4 * S::kMyStrips; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
        // Loads of x per stage: row-major in groups of 8 rows x 128 bytes, else one per 16-row block and k step.  Every element is
        // loaded by one wave, or by two where they share its k steps (!kSplitK).  Rows past M, and stages past the last, read nothing.
        constexpr int kXLoads = X_KIND == XKind::kTiled ? MB * S::kMySteps : 2 * MB;
        struct XRegs { u32x4 v[kXLoads]; };
        uint32_t x_off[kXLoads];
#pragma unroll
        for (int i = 0; i < kXLoads; ++i) {
            if (X_KIND == XKind::kTiled) x_off[i] = m0 + my_row0 + 16 * (i % MB) < M ? (uint32_t)(16 * lane + 1024 * (i % MB)) : kOutside;
            else                         x_off[i] = m0 + my_row0 + 8 * i + (lane >> 3) < M ? (uint32_t)(lane >> 3) * (uint32_t)K * (X_KIND == XKind::kFloat ? 4 : 2) + (lane & 7) * 16 : kOutside;
        }
        constexpr int kBytes = X_KIND == XKind::kFloat ? 4 : 2;
        const size_t x_step = X_KIND == XKind::kTiled ? (size_t)rows_pad * 64 : (size_t)32 * kBytes;     // bytes from a k step to the next
        const unsigned char* const x0 = (const unsigned char*)X + (X_KIND == XKind::kTiled ? (size_t)(m0 + my_row0) * 64 : (size_t)(m0 + my_row0) * K * kBytes);
        auto request_x = [&](XRegs& b, int it) {
            const int k0 = stage_k0(it < n_stages ? it : 0) + 32 * kh * S::kMySteps;
            const unsigned char* const x_stage = x0 + (size_t)(unsigned)(k0 >> 5) * x_step;
            const bool valid = it < n_stages && k0 < k_end;
            const __amdgpu_buffer_rsrc_t xr = buffer_at(x_stage, valid);
#pragma unroll
            for (int i = 0; i < kXLoads; ++i) {
                // (far rows: a resource per group of eight, at 0.05 .. 0.2 us a call)
                if (X_KIND == XKind::kFarRows) b.v[i] = __builtin_amdgcn_raw_buffer_load_b128(buffer_at(x_stage + (size_t)(8 * i) * K * kBytes, valid), x_off[i], 0, 0);
                else                           b.v[i] = __builtin_amdgcn_raw_buffer_load_b128(xr, x_off[i], X_KIND == XKind::kTiled ? (i / MB) * rows_pad * 64 : 8 * i * K * kBytes, 0);
            }
        };
        const int a_lane_off = (8 * g + (n >> 2)) * 128 + ((n & 3) << 3);         // row 8g + i, 8 bytes per lane
        const int a_key = ((g & 1) << 1) | ((n >> 3) & 1);                        // w_key of rows 8g + 4t + i
        // A operands of one k step and strip: for each 16-column block the two transposing reads that make W^T
        union AFrag { bf16x8 v; s16x4 h[2]; };
        auto read_a = [&](AFrag (&f)[4], int base, int ks) {
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    f[nb].h[t] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_AT(s16x4, lds_base, base + (32 * ks + 4 * t) * 128 + a_lane_off + ((nb ^ a_key) << 5)));
        };
        const int image = S::kImageBase + wave * S::kImageBytes;
        auto multiply = [&](const XRegs& b, int it, int slot) {
            if (m0 + my_row0 >= M || stage_k0(it) + 32 * kh * S::kMySteps >= k_end) return;   // no rows; half a stage at the end of the k range
            bf16x8 xf[MB * S::kMySteps];                                          // [own k step][row block]
            if constexpr (X_KIND == XKind::kTiled) {
#pragma unroll
                for (int i = 0; i < kXLoads; ++i) xf[i] = __builtin_bit_cast(bf16x8, b.v[i]);
            } else {
#pragma unroll
                for (int i = 0; i < kXLoads; ++i) {
                    const int r = 8 * i + (lane >> 3);
                    if constexpr (bf16_rows(X_KIND)) *LDS_AT(u32x4, lds_base, image + image64_at(r, lane & 7)) = b.v[i];
                    else {
                        const f32x4 f = __builtin_bit_cast(f32x4, b.v[i]);
                        bf16x4 h;
#pragma unroll
                        for (int c = 0; c < 4; ++c) h[c] = (__bf16)f[c];
                        *LDS_AT(bf16x4, lds_base, image + image32_at(r, (lane & 7) >> 1) + (lane & 1) * 8) = h;
                    }
                }
#pragma unroll
                for (int j = 0; j < S::kMySteps; ++j)
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb)
                        xf[j * MB + mb] = *LDS_AT(bf16x8, lds_base, image + (bf16_rows(X_KIND) ? image64_at(16 * mb + n, 4 * j + g) : image32_at(16 * mb + n, g)));
            }
            // units (own k step, strip): the operands of the next one are read from LDS while the current one is multiplied
            constexpr int T = S::kMyStrips, kUnits = S::kMySteps * T;
            const int base = slot * S::kStageBytes + nh * T * S::kSubBytes;
            AFrag f[2][4];
            read_a(f[0], base, kh * S::kMySteps);
#pragma unroll
            for (int u = 0; u < kUnits; ++u) {
                if (u + 1 < kUnits) read_a(f[(u + 1) & 1], base + ((u + 1) % T) * S::kSubBytes, kh * S::kMySteps + (u + 1) / T);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb)
                        acc[mb][(u % T) * 4 + nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[u & 1][nb].v, xf[(u / T) * MB + mb], acc[mb][(u % T) * 4 + nb], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        constexpr int kXAhead = 2;
        XRegs x[kXAhead];
#pragma unroll
        for (int d = 0; d < kXAhead; ++d) request_x(x[d], d);
        int slot = 0;
        for (int it = 0; it < n_stages; it += kXAhead)
#pragma unroll
            for (int d = 0; d < kXAhead; ++d) {
                if (it + d < n_stages) {
                    lds_barrier();
                    multiply(x[d], it + d, slot);
                }
                slot = slot + 1 == S::kSlots ? 0 : slot + 1;
                __builtin_amdgcn_sched_barrier(0);
                request_x(x[d], it + d + kXAhead);
                __builtin_amdgcn_sched_barrier(0);
            }
    }

    // The result tile meets in LDS (the ring is dead, no direct load is in flight), always as (kh 0 part) + (kh 1 part), and is
    // stored row by row: whole 128-byte lines.
    __syncthreads();
    const int own = (my_row0 + n) * S::kTileStride + 16 * g + nh * S::kMyStrips * kStripN * 4;
    if (wave < kMultipliers && (!S::kSplitK || kh == 1)) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int j = 0; j < 4 * S::kMyStrips; ++j) *LDS_AT(f32x4, lds_base, own + 16 * mb * S::kTileStride + 64 * j) = acc[mb][j];
    }
    __syncthreads();
    if (S::kSplitK) {
        if (wave < kMultipliers && kh == 0) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int j = 0; j < 4 * S::kMyStrips; ++j) {
                    const int at = own + 16 * mb * S::kTileStride + 64 * j;
                    *LDS_AT(f32x4, lds_base, at) = acc[mb][j] + *LDS_AT(f32x4, lds_base, at);
                }
        }
        __syncthreads();
    }
    constexpr int kPiece = OUT_BF16 ? 8 : 4;                            // columns a thread stores at a time: 16 bytes
    constexpr int kLanesPerRow = S::kCols / kPiece, kPieces = S::kRows * kLanesPerRow;
#pragma unroll
    for (int i = 0; i < (kPieces + kLoaderThreads - 1) / kLoaderThreads; ++i) {
        const int piece = i * kLoaderThreads + threadIdx.x, row = piece / kLanesPerRow, col = piece % kLanesPerRow * kPiece;
        if (piece >= kPieces || m0 + row >= M) break;
        const f32x4 lo = *LDS_AT(f32x4, lds_base, row * S::kTileStride + col * 4);
        if constexpr (OUT_BF16) {
            const f32x4 hi = *LDS_AT(f32x4, lds_base, row * S::kTileStride + col * 4 + 16);
            bf16x8 o;
#pragma unroll
            for (int c = 0; c < 4; ++c) { o[c] = (__bf16)lo[c]; o[4 + c] = (__bf16)hi[c]; }
            *(bf16x8*)((__bf16*)out + (size_t)(m0 + row) * N + n0 + col) = o;
        } else {
            *(f32x4*)((float*)out + ((size_t)kz * rows_pad + m0 + row) * N + n0 + col) = lo;
        }
    }
}

// One workgroup per row of x: c = sum of the split-K partials (in split order),
// c_hat = c / sqrt(mean(c^2) + eps) * gain.  A thread owns float4 pieces of the row; the partials
// of a piece are loaded eight splits at a time so that the loads are in flight together: eight splits and a rank
// of 2048 are one round trip.
constexpr int kNormThreads = 512;
__global__ __launch_bounds__(kNormThreads) void rmsnorm_reduce_kernel(const float* __restrict__ ws_c, const float* __restrict__ gain,
                                                             __bf16* __restrict__ chat, int r, int split_k, int rows_pad,
                                                             float eps)
{
    __shared__ float red[kNormThreads / 64];
    extern __shared__ float crow[];           // the reduced row's columns from 4 * kNormThreads on, kept between the two passes
    const int m = blockIdx.x;
    const int tid = threadIdx.x;
    const size_t split_stride = (size_t)rows_pad * r;
    // A thread's first four columns stay in registers, with their gain, which is asked for here and not when it is needed.
    auto sum_splits = [&](int j) {
        const float* p = ws_c + (size_t)m * r + j;
        f32x4 c = {0.f, 0.f, 0.f, 0.f};
        for (int z0 = 0; z0 < split_k; z0 += 8) {
            f32x4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int z = z0 + u < split_k ? z0 + u : split_k - 1;
                v[u] = *(const f32x4*)(p + (size_t)z * split_stride);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (z0 + u < split_k) c += v[u];
        }
        return c;
    };
    auto square = [](const f32x4& c) { return c[0] * c[0] + c[1] * c[1] + c[2] * c[2] + c[3] * c[3]; };
    const int j0 = 4 * tid;
    f32x4 c0 = {0.f, 0.f, 0.f, 0.f}, g0 = {1.f, 1.f, 1.f, 1.f};
    if (j0 < r) {
        if (gain) g0 = *(const f32x4*)(gain + j0);
        c0 = sum_splits(j0);
    }
    float ss = square(c0);
    for (int j = j0 + 4 * kNormThreads; j < r; j += 4 * kNormThreads) {
        const f32x4 c = sum_splits(j);
        *(f32x4*)(crow + j - 4 * kNormThreads) = c;
        ss += square(c);
    }
    for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    float total = 0.f;
#pragma unroll
    for (int i = 0; i < kNormThreads / 64; ++i) total += red[i];
    const float inv = 1.0f / sqrtf(total / (float)r + eps);
    for (int j = j0; j < r; j += 4 * kNormThreads) {
        const f32x4 c = j == j0 ? c0 : *(const f32x4*)(crow + j - 4 * kNormThreads);
        const f32x4 g = j == j0 || !gain ? g0 : *(const f32x4*)(gain + j);
        bf16x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = (__bf16)(c[i] * inv * g[i]);
        *(bf16x4*)(chat + tiled_index(m, j, rows_pad)) = o;
    }
}

// ---- the new token's cache record (Section 6: the cache holds one key row and one value row per
// token, 8 bits per element in the deployed system).
// One workgroup per sequence, thread t owns key element t or value element t - 256; all splits' loads are in flight together (with the
// place of the row looked up behind them: 28 splits, 64 sequences, 8 bit: 4.8 us, in groups of eight splits ahead of it, 4.4 now).  The fp32 rows are the
// sum of the projection's split-K partials in split order.  bf16 cache: round to nearest even.
// fp8 cache: per token and tensor scale = max(max|x|, 1e-12) / 448 and code = e4m3(x / scale), the
// quotient clamped to +-448; all in single precision with correctly rounded divisions, so that the
// codes are a function of the fp32 row alone.  The row written is seq_lens[b] (the tokens already
// cached); a row outside the cache or the block table is not written.
// 4-bit cache (BITS = 4): the same with e2m1's largest magnitude 6 in place of 448; the codes of
// elements 2i and 2i + 1 share byte i, the even one in the low four bits.
template <int BITS, bool PAGED>
__global__ __launch_bounds__(kKvWidth) void kv_record_kernel(const float* __restrict__ parts, int split_k, int rows_pad, KvAppendArgs a)
{
    __shared__ float red[kKvWidth / 64];
    const int b = blockIdx.x;
    const bool value = threadIdx.x >= kHeadDim;          // the same in all lanes of a wave
    const int t = threadIdx.x & (kHeadDim - 1);
    const float* const row0 = parts + (size_t)b * kKvWidth + threadIdx.x;
    const size_t split_stride = (size_t)rows_pad * kKvWidth;
    float p[kMaxSplits];
#pragma unroll
    for (int u = 0; u < kMaxSplits; ++u) {
        if (u % 8 == 0 && u >= split_k) break;           // (the groups of eight there are; all four: append of 2 rows of 64 k 6.5 us, 5.5 so, 64 rows of 7168 k 10.6, 9.9)
        p[u] = row0[(size_t)(u < split_k ? u : split_k - 1) * split_stride];
    }
    const int pos = a.seq_lens[b];
    int64_t row;
    if (PAGED) {
        const int blk = pos / kPage;
        if (pos < 0 || blk >= a.max_blocks_per_seq) return;
        const int page = a.block_table[(size_t)b * a.max_blocks_per_seq + blk];
        if (page < 0 || page >= a.n_pages) return;                  // never write outside the pools
        row = (int64_t)page * kPage + pos % kPage;
    } else {
        if (pos < 0 || pos >= a.seq_stride_tokens) return;
        row = (int64_t)b * a.seq_stride_tokens + pos;
    }
    float x = -0.f;                                     // -0 + x = x for every x, the sign of a zero included
#pragma unroll
    for (int u = 0; u < kMaxSplits; ++u)
        if (u < split_k) x += p[u];
    void* const cache = value ? a.v : a.k;
    if (BITS == 16) {
        ((__bf16*)cache)[row * kHeadDim + t] = (__bf16)x;
        return;
    }
    float top = fabsf(x);
    for (int off = 32; off > 0; off >>= 1) top = fmaxf(top, __shfl_xor(top, off));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = top;
    __syncthreads();
    const int w = value ? kHeadDim / 64 : 0;
    top = fmaxf(fmaxf(red[w], red[w + 1]), fmaxf(red[w + 2], red[w + 3]));
    constexpr float kTop = BITS == 8 ? 448.0f : 6.0f;
    const float scale = fmaxf(top, 1e-12f) / kTop;
    const float y = fminf(fmaxf(x / scale, -kTop), kTop);
    if (BITS == 8) {
        ((uint8_t*)cache)[row * kHeadDim + t] = (uint8_t)(__builtin_amdgcn_cvt_pk_fp8_f32(y, 0.f, 0, false) & 0xFF);
    } else {
        // the odd neighbour's quotient comes over by a lane shuffle; the even thread converts and stores the pair
        const float y1 = __shfl_down(y, 1);
        if ((t & 1) == 0) ((uint8_t*)cache)[row * (kHeadDim / 2) + (t >> 1)] = (uint8_t)(__builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, y, y1, 1.0f, 0) & 0xFF);
    }
    if (t == 0) (value ? a.v_scale : a.k_scale)[row] = scale;
}
static_assert(kHeadDim == 256, "kv_record_kernel reduces over four waves");

// fp32 [M, K] -> bf16 in the tiled order, for output projections of more than 64 rows (up to 64 the product converts by itself).  A wave takes
// 16 rows of one k step: reads whole 128-byte lines, writes one contiguous KB.
__global__ __launch_bounds__(256) void to_bf16_tiled_kernel(const float* __restrict__ src, __bf16* __restrict__ dst, int M, int K,
                                                            int rows_pad)
{
    const int lane = threadIdx.x & 63;
    const int ks = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int m = blockIdx.y * 16 + (lane >> 2);
    if (ks >= K / 32 || m >= M) return;
    const int k = 8 * (lane & 3);
    const f32x4* s = (const f32x4*)(src + (size_t)m * K + 32 * ks + k);
    const f32x4 lo = s[0], hi = s[1];
    bf16x8 o;
#pragma unroll
    for (int j = 0; j < 4; ++j) { o[j] = (__bf16)lo[j]; o[4 + j] = (__bf16)hi[j]; }
    *(bf16x8*)(dst + tiled_index(m, 32 * ks + k, rows_pad)) = o;
}

// y[m][n] = bf16(sum over splits, in split order, of the fp32 partials); eight splits' loads in flight together.
__global__ __launch_bounds__(256) void reduce_partials_bf16_kernel(const float* __restrict__ parts, __bf16* __restrict__ y, int N,
                                                                   int split_k, int rows_pad)
{
    const int m = blockIdx.y;
    const int n = (blockIdx.x * 256 + threadIdx.x) * 4;
    if (n >= N) return;
    const float* p = parts + (size_t)m * N + n;
    const size_t split_stride = (size_t)rows_pad * N;
    f32x4 c = {0.f, 0.f, 0.f, 0.f};
    for (int z0 = 0; z0 < split_k; z0 += 8) {
        f32x4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int z = z0 + u < split_k ? z0 + u : split_k - 1;
            v[u] = *(const f32x4*)(p + (size_t)z * split_stride);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (z0 + u < split_k) c += v[u];
    }
    union { __bf16 h[4]; uint2 u; } o;
#pragma unroll
    for (int j = 0; j < 4; ++j) o.h[j] = (__bf16)c[j];
    *(uint2*)(y + (size_t)m * N + n) = o.u;
}

}  // namespace

namespace {

// The kernel of one streaming product and what it covers.
struct GemmForm { const void* fn; unsigned threads, lds_bytes; int rows, cols; bool row_major_bf16; };

template <bool OUT_BF16, XKind X_KIND, int MB, int NS>
GemmForm loader_form()
{
    using S = LoaderShape<X_KIND, MB, NS>;
    return {(const void*)gemm_loader_kernel<OUT_BF16, X_KIND, MB, NS>, kLoaderThreads, S::kLdsBytes, S::kRows, S::kCols, bf16_rows(X_KIND)};
}
// Products over single strips: up to 64 rows, or tiles of 128.
template <bool OUT_BF16, XKind X_KIND>
GemmForm strip_form(int M)
{
    return M <= 64 ? loader_form<OUT_BF16, X_KIND, 1, 1>() : loader_form<OUT_BF16, X_KIND, 2, 1>();
}
// Products whose x is row-major bf16.  A wave's rows are reached by offsets into one resource, or, from 34.6 million k on, where 32 rows leave its reach, by a
// resource per eight rows.
constexpr bool within_reach(int rows, int K) { return (int64_t)(rows - 1) * K * 2 + 128 <= (int64_t)kReach; }
GemmForm rows_form(int M, int K) { return within_reach(32, K) ? strip_form<false, XKind::kRows>(M) : strip_form<false, XKind::kFarRows>(M); }
// The output projection over groups of four strips: up to 64 rows straight from the fp32 activations (64 rows: 42.6 us where the product over a
// converted copy takes 41.5, and the launch that converts 4 or 5), with more rows, where x is as large as a workgroup's share of W, from
// the converted copy (128 rows: 55.0 and 47.5 + 5).
bool converts_itself(int M, int strips_per_wg) { return strips_per_wg == 4 && M <= 64; }
GemmForm out_form(int M, int strips_per_wg)
{
    if (strips_per_wg == 4) return M <= 64 ? loader_form<false, XKind::kFloat, 1, 4>() : loader_form<false, XKind::kTiled, 2, 4>();
    return M <= 64 ? loader_form<false, XKind::kTiled, 1, 1>() : loader_form<false, XKind::kTiled, 2, 1>();
}

hipError_t launch_gemm(const GemmForm& f, const void* X, const void* W, void* out, int M, int K, int N, int k_per_split, int split_k,
                       int rows_pad, hipStream_t stream)
{
    const uint16_t* wp = (const uint16_t*)W;
    // Where not even eight rows are within reach, from 153 million k on, a launch per row (fp32 partial sums).
    const int rows = f.row_major_bf16 && !within_reach(8, K) ? 1 : M;
    for (int m = 0; m < M; m += rows) {
        const void* x_here = f.row_major_bf16 ? (const uint16_t*)X + (size_t)m * K : X;
        void* out_here = f.row_major_bf16 ? (float*)out + (size_t)m * N : out;
        int rows_here = rows;
        void* params[] = {&x_here, &wp, &out_here, &rows_here, &K, &N, &k_per_split, &rows_pad};
        const hipError_t e = hipLaunchKernel(f.fn, dim3(N / f.cols, (rows + f.rows - 1) / f.rows, split_k), dim3(f.threads), params, f.lds_bytes, stream);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

QProjPlan plan_linear(int32_t K, int32_t N, int32_t strips_per_wg)
{
    const int32_t strips = N / (kStripN * strips_per_wg);
    int32_t want = 256 / (strips > 0 ? strips : 1);
    if (want < 1) want = 1;
    if (want > kMaxSplits) want = kMaxSplits;
    const int32_t units = K / 64;                // a split is whole 64 k: what a wave takes at a time (every K here is a multiple of 64)
    const int32_t per = (units + want - 1) / want;
    QProjPlan p;
    p.k_per_split = per * 64;
    p.split_k = (units + per - 1) / per;
    p.strips_per_wg = strips_per_wg;
    return p;
}

// Output projection: groups of four strips (x once per 256 columns, W in rows of 512 bytes) pay for the fourfold k split, with more than 128 rows
// as well, and single strips do where the columns do not divide.  us per call, a plan of four strips up to 64 rows, pairs up to 128 and single ones beyond
// (on the kernel whose waves loaded and multiplied in turn) -> this one:  7168 columns, 256 / 512 / 1024 rows 163.7 / 322.0 / 576.3 -> 127.5 / 214.8 / 409.1;
// 1152 columns (pairs, now single strips), 4 / 64 / 128 / 256 rows 17.5 / 22.0 / 25.7 / 46.1 -> 14.6 / 20.6 / 25.3 / 39.3;
// 2176 columns 21.8 / 27.2 / 32.4 / 64.2 -> 20.3 / 27.4 / 32.1 / 53.2.
QProjPlan plan_out_proj(int32_t K, int32_t N)
{
    return plan_linear(K, N, N % (4 * kStripN) == 0 ? 4 : 1);
}

hipError_t prepare_query_proj_kernels()
{
    for (const int rows : {64, 128}) {
        const GemmForm forms[] = {strip_form<false, XKind::kRows>(rows), strip_form<false, XKind::kFarRows>(rows), strip_form<true, XKind::kTiled>(rows), out_form(rows, 1), out_form(rows, 4)};
        for (const GemmForm& f : forms) {
            const hipError_t e = hipFuncSetAttribute(f.fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)f.lds_bytes);
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

namespace {
size_t norm_lds_bytes(int q_rank) { return q_rank > 4 * kNormThreads ? (q_rank - 4 * kNormThreads) * sizeof(float) : 0; }
}  // namespace

hipError_t launch_query_proj(const QProjArgs& a, hipStream_t stream)
{
    const int m_blocks = (a.B + kQProjRows - 1) / kQProjRows;
    const int rows_pad = m_blocks * kQProjRows;
    hipError_t e = launch_gemm(rows_form(a.B, a.d_model), a.x, a.w_qa, a.ws_c, a.B, a.d_model, a.q_rank, a.k_per_split, a.split_k,
                               rows_pad, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(rmsnorm_reduce_kernel, dim3(a.B), dim3(kNormThreads), norm_lds_bytes(a.q_rank), stream,
                       (const float*)a.ws_c, a.gain, (__bf16*)a.ws_chat, a.q_rank, a.split_k, rows_pad, a.eps);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_gemm(strip_form<true, XKind::kTiled>(a.B), a.ws_chat, a.w_qb, a.q_out, a.B, a.q_rank, a.n_out, a.q_rank, 1, rows_pad, stream);
}

namespace {

template <int BITS>
hipError_t launch_record_bits(const KvAppendArgs& a, const float* parts, int split_k, int rows_pad, hipStream_t stream)
{
    if (a.block_table) hipLaunchKernelGGL((kv_record_kernel<BITS, true>), dim3(a.B), dim3(kKvWidth), 0, stream, parts, split_k, rows_pad, a);
    else               hipLaunchKernelGGL((kv_record_kernel<BITS, false>), dim3(a.B), dim3(kKvWidth), 0, stream, parts, split_k, rows_pad, a);
    return hipGetLastError();
}

hipError_t launch_record(const KvAppendArgs& a, mfa_kv_dtype kv_dtype, const float* parts, int split_k, int rows_pad, hipStream_t stream)
{
    if (kv_dtype == MFA_KV_FP8_E4M3) return launch_record_bits<8>(a, parts, split_k, rows_pad, stream);
    if (kv_dtype == MFA_KV_FP4_E2M1) return launch_record_bits<4>(a, parts, split_k, rows_pad, stream);
    return launch_record_bits<16>(a, parts, split_k, rows_pad, stream);
}

}  // namespace

hipError_t launch_kv_record(const KvAppendArgs& a, const float* kv, mfa_kv_dtype kv_dtype, hipStream_t stream)
{
    return launch_record(a, kv_dtype, kv, 1, a.B, stream);
}

hipError_t launch_kv_append(const KvAppendArgs& a, mfa_kv_dtype kv_dtype, hipStream_t stream)
{
    const int m_blocks = (a.B + kQProjRows - 1) / kQProjRows;
    const int rows_pad = m_blocks * kQProjRows;
    const hipError_t e = launch_gemm(rows_form(a.B, a.d_model), a.x, a.w_kv, a.ws_c, a.B, a.d_model, kKvWidth, a.plan.k_per_split,
                                     a.plan.split_k, rows_pad, stream);
    if (e != hipSuccess) return e;
    return launch_record(a, kv_dtype, a.ws_c, a.plan.split_k, rows_pad, stream);
}

hipError_t launch_out_proj(const OutProjArgs& a, hipStream_t stream)
{
    const int m_blocks = (a.B + kQProjRows - 1) / kQProjRows;
    const int rows_pad = m_blocks * kQProjRows;
    const bool fused = converts_itself(a.B, a.plan.strips_per_wg);
    hipError_t e = hipSuccess;
    if (!fused) {
        hipLaunchKernelGGL(to_bf16_tiled_kernel, dim3((a.n_in / 32 + 3) / 4, (a.B + 15) / 16), dim3(256), 0, stream, a.attn, (__bf16*)a.ws_act,
                           a.B, a.n_in, rows_pad);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    e = launch_gemm(out_form(a.B, a.plan.strips_per_wg), fused ? (const void*)a.attn : a.ws_act, a.w_o, a.ws_c, a.B, a.n_in, a.d_model,
                    a.plan.k_per_split, a.plan.split_k, rows_pad, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(reduce_partials_bf16_kernel, dim3((a.d_model / 4 + 255) / 256, a.B), dim3(256), 0, stream, (const float*)a.ws_c,
                       (__bf16*)a.y, a.d_model, a.plan.split_k, rows_pad);
    return hipGetLastError();
}

}  // namespace mfa
