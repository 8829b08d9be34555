// Decode attention over the 8-bit and 4-bit caches (e4m3 / e2m1 codes, one fp32 scale per token and tensor) for
// gfx950.  Codes stay codes from HBM to the matrix cores: keys meet the query and values meet the weights on
// v_mfma_scale_f32_32x32x64_f8f6f4, with the bf16 query and the fp32 weights split into two e4m3 terms each.
//
// Workgroup: 4 waves, one per SIMD (a wave needs more than 256 of its 512 registers).  A wave works on 32 columns, a
// column being a (query token, head) pair, and 64 tokens at a time:
//   one query token:   64 columns; wave = 2*tp + cg takes columns 32*cg.. and the tiles of parity tp
//   two query tokens: 128 columns; wave = 2*token + (half of the heads) takes every tile
// MFMA shapes (lane = 32*h + n; a lane holds rows 8*(i/4) + 4*h + i%4, i = 0..15, of column n of D):
//   scores  S^T[token, column] = K . Q^T    A = 32 key rows x 64 dims, B = query; two blocks of 32 tokens
//   output  O^T[d, column] += V^T . P^T     A = V^T, 32 dims x 64 tokens (transposing LDS reads), B = weights
// The 32 scores a lane ends up with (16 per token block) are, in register order, the 32 bytes it has to supply as
// the B operand of the second product, so weights never move between lanes; the value rows are read from LDS in the
// token order this implies (LowbitLanes::va).
//
// Operand element order (measured with one-hot operands).  Byte 16*hi + lo of lane half h of an 8-bit operand is
// k = 32*hi + 16*h + lo, element j of lane half h of a 4-bit operand is k = 32*h + j.  Two 8-bit operands therefore match
// byte for byte; where a 4-bit operand meets an 8-bit one the rows or dims are chosen to match.
//
// What bounds it.  8 bit, one token: memory (6.9 TB/s in the steady stream).  4 bit, and two query tokens: the matrix pipe, 2 x 16
// instructions of 64 cycles per wave and stage, and what does not hide behind it.  About 9 us per launch go to the first segment's
// start and the end (8 bit, 128 x 8192 tokens, us from the first workgroup's start: first segment known 2.05, everything requested 4.0, query converted
// 6.2, first tile done 8.4, last product 80.7, result stored 82.6), which is why launches with little work have a kernel of
// their own.  Alternatives measured at 128 x 8192 tokens, 8 bit / 4 bit / 8 bit two tokens: values expanded to bf16 (the other
// kernel) 114 / 95 / 175 us, this one 102 / 79 / 154 and, with fewer wait states and the scales folded, 100 / 75 / 148;
// eight waves of 16 columns on these instructions 108 / 85 / 162.
// Error against 64 bits at 8192 tokens: 6.3e-4 of a row's largest element (bf16 weights: 1.7e-3).
//
// The accumulators are not rescaled (LowbitState): a segment in which a score outruns its first tile's by 2^40 is streamed twice, where the
// other kernel moves its reference on.  128 x 8192 tokens, one token per sequence 400 times its score late in a segment, other
// kernel / this one, 8 bit / 4 bit / 8 bit two tokens: 117/179, 100/135, 185/258 us; without such scores 121/108, 104/83, 188/162 on the same device.
#pragma once
#include "mfa_attn_core.hpp"

namespace mfa {

typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kLowbitThreads = 256;

// LDS of a workgroup.  A stage is the tiles the workgroup works on at a time (two for one query token, a tile per wave
// pair; one for two).  Keys are used one iteration ahead of the values of the same tile: iteration s reads the keys of
// stage s + 1 and the values of stage s, and requests keys s + 1 + kDepth and values s + kDepth.  kDepth stages are in
// flight: 32 KB of keys and values per compute unit, 64 KB where one stage is as large (8 bit, one token).  64 KB everywhere,
// against this, in us: 4 bit 60 x 12000 ragged 42.6 / 41.8, 100 x 5000 ragged 37.8 / 37.1, two tokens 40 x 7000 ragged 36.7 / 35.5;
// 8 bit, two tokens 60 x 6000 ragged 45.3 / 44.6; equal lengths 0.3 .. 1 % slower.
template <int QL, int BITS>
struct LowbitShape {
    static constexpr int kTiles = QL == 1 ? 2 : 1;
    static constexpr int kRowBytes = BITS == 8 ? 256 : 128;              // one cached row of K or V
    static constexpr int kTileBytes = kTile * kRowBytes;
    static constexpr int kStageBytes = kTiles * kTileBytes;               // of K or of V
    static constexpr int kDepth = kStageBytes >= 16384 ? 1 : 16384 / kStageBytes;
    static constexpr int kSlots = kDepth + 1;                             // (a stage in use beside those in flight)
    static constexpr int kVBase = kSlots * kStageBytes;
    static constexpr int kScaleStage = kTiles * kTile * 4;                // fp32 scales of one tensor of a stage (they come with the keys)
    static constexpr int kKScaleBase = kVBase + kSlots * kStageBytes;
    static constexpr int kVScaleBase = kKScaleBase + kSlots * kScaleStage;
    static constexpr int kKcBase = kVScaleBase + kSlots * kScaleStage;    // key scales of the tile a wave is at, times the softmax scale: 256 bytes per wave
    static constexpr int kFlag = kKcBase + 4 * kTile * 4;                 // restart flag
    static constexpr int kSchedBase = kFlag + 16;
    // Four areas of 32 query rows (16 KB; only used before the first tile): the slots no stage of the prologue lands in, then memory
    // of their own.
    static constexpr int kQOwn = (kSchedBase + kSchedLdsBytes + 1023) / 1024 * 1024;
    static constexpr int kQInSlots = kStageBytes / 16384;                 // waves per free slot (2, 1 or none)
    static constexpr int query_area(int i)
    {
        if (i < kQInSlots) return kDepth * kStageBytes + i * 16384;
        if (i < 2 * kQInSlots) return kVBase + kDepth * kStageBytes + (i - kQInSlots) * 16384;
        return kQOwn + (i - 2 * kQInSlots) * 16384;
    }
    static constexpr int kLdsBytes = kQOwn + (kQInSlots < 2 ? (4 - 2 * kQInSlots) * 16384 : 0);
    static constexpr int kLoadsPerTile = kTileBytes / (4 * 1024);         // 1 KB direct loads of a wave per tile of K or V
    static constexpr int kOps = 2 * kTiles * kLoadsPerTile + 1;           // vector-memory operations of a wave per stage
    static_assert(kLdsBytes <= 160 * 1024, "LDS of a compute unit");
    static_assert(QL == 2 || 4 * 16384 + 4 * 256 <= kKcBase, "the exchange at a segment's end fits the tiles and their scales");
};

// The query of one column, split into two e4m3 terms: q * 2^e = hi + lo with e chosen per head so that the largest |q|
// of the head lands in [128, 256): hi is the nearest e4m3 value and lo the remainder, which e4m3 holds exactly (the 8
// significant bits of bf16 are 4 + 4) down to 2^-9, i.e. to 2^-17 of the head's largest element.
struct SplitQuery { i32x8 hi[4]; i32x8 lo[4]; int scale; };              // [64-dim chunk]; scale: 2^-e as the matrix instruction's scale operand takes it

// max over the two lanes {n, n + 32} that hold one column
__device__ __forceinline__ float half_max(float x)
{
    const unsigned u = __float_as_uint(x);
    const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
__device__ __forceinline__ float half_sum(float x)
{
    const unsigned u = __float_as_uint(x);
    const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}

// The query rows go to LDS with direct loads (piece p, 16 bytes, of row r at p ^ r), are converted there, and the operands
// are read back.  Loops that are not unrolled: code that runs once per segment comes cold from
// the instruction cache, about 100 cycles per 64 bytes; unrolled, the conversion took 7000 cycles, most of it fetching.
// With one query token the two waves of the same heads share the work: each brings half of the rows and converts half of the
// dims, from one 16 KB area to another; with two every wave has rows of its own and converts them in place.
template <int QL> constexpr int kQueryOps = QL == 1 ? 8 : 16;         // direct loads (two rows each) of a wave
__device__ __forceinline__ void request_query(const void* qptr, size_t row0, uint32_t lds_dst, int first, int count, int lane)
{
    const unsigned char* src = (const unsigned char*)qptr + row0 * kHeadDim * 2;
#pragma unroll 1
    for (int u = first; u < first + count; ++u) {
        const int row = 2 * u + (lane >> 5);
        load_to_lds_16B_keep(src, (uint32_t)(row * 512 + (((lane & 31) ^ row) << 4)), lds_dst + u * 1024);
    }
}
// The four pieces of chunk c (64 dims) that a lane holds.  Dims of bytes 16*hi + lo of a lane are 64c + 32h + 16hi + lo against e4m3
// keys read in plain order, 64c + 32hi + 16h + lo against e2m1 keys.
template <int BITS>
__device__ __forceinline__ int query_piece(int base, int c, int i, int lane)
{
    const int n = lane & 31, h = lane >> 5;
    return base + n * 512 + (((8 * c + (BITS == 8 ? 4 * h + i : 4 * (i >> 1) + 2 * h + (i & 1))) ^ n) << 4);
}
template <int QL, int BITS>
__device__ __forceinline__ void split_query(SplitQuery& q, lds_ptr_t lds, int in, int out, int grp, int lane)
{
    if (QL == 1) __syncthreads();                                      // both waves' rows are there

    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    typedef short s16x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    u16x2 top = {0, 0};                                                // largest magnitude, as bit patterns
#pragma unroll 2
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const u32x4 x = *LDS_AT(u32x4, lds, query_piece<BITS>(in, c, i, lane));
#pragma unroll
            for (int w = 0; w < 4; ++w) top = __builtin_elementwise_max(top, __builtin_bit_cast(u16x2, x[w] & 0x7FFF7FFFu));
        }
    const float amax = half_max(__uint_as_float((uint32_t)(top[0] > top[1] ? top[0] : top[1]) << 16));
    int e = (int)((__float_as_uint(amax) >> 23) & 0xFFu);          // biased exponent of the largest element
    e = e < 24 ? 24 : e;                                           // (all-zero or vanishing heads: any scale will do)
    q.scale = e - 7;
    const float inv_scale = __uint_as_float((uint32_t)(e - 7) << 23);   // 2^-e: amax / inv_scale in [128, 256)
#pragma unroll 1
    for (int c = QL == 1 ? 2 * grp : 0; c < (QL == 1 ? 2 * grp + 2 : 4); ++c) {
        u32x4 hi4[2], lo4[2];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const u32x4 x = *LDS_AT(u32x4, lds, query_piece<BITS>(in, c, i, lane));
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                const uint32_t u0 = x[2 * w], u1 = x[2 * w + 1];
                s16x2 hi = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16((s16x2){0, 0}, __builtin_bit_cast(bf16x2, u0), inv_scale, false);
                hi = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(hi, __builtin_bit_cast(bf16x2, u1), inv_scale, true);
                const int hi_bits = __builtin_bit_cast(int, hi);
                const f32x2 b01 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(hi_bits, inv_scale, false);
                const f32x2 b23 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(hi_bits, inv_scale, true);
                s16x2 lo = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32((s16x2){0, 0}, __uint_as_float(u0 << 16) - b01[0],
                                                                    __uint_as_float(u0 & 0xFFFF0000u) - b01[1], inv_scale, false);
                lo = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(lo, __uint_as_float(u1 << 16) - b23[0],
                                                              __uint_as_float(u1 & 0xFFFF0000u) - b23[1], inv_scale, true);
                hi4[i >> 1][2 * (i & 1) + w] = (uint32_t)hi_bits;
                lo4[i >> 1][2 * (i & 1) + w] = __builtin_bit_cast(uint32_t, lo);
            }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            *LDS_AT(u32x4, lds, query_piece<BITS>(out, c, i, lane)) = hi4[i];
            *LDS_AT(u32x4, lds, query_piece<BITS>(out, c, 2 + i, lane)) = lo4[i];
        }
    }
    if (QL == 1) __syncthreads();
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        union { i32x8 v; u32x4 h[2]; } hi, lo;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            hi.h[i] = *LDS_AT(u32x4, lds, query_piece<BITS>(out, c, i, lane));
            lo.h[i] = *LDS_AT(u32x4, lds, query_piece<BITS>(out, c, 2 + i, lane));
        }
        q.hi[c] = hi.v;
        q.lo[c] = lo.v;
    }
}

// A lane's LDS offsets inside a tile image (see the layouts at LowbitTile below).
template <int BITS>
struct LowbitLanes {
    int ka;        // first key operand piece; the others differ from it in address bits 4 .. 7 only (the images are aligned)
    int va;        // first transposing read of the value operand of the first 32-dim block
};
// LDS image of a tile: 64 rows, 16-byte pieces permuted within a row so that operand reads touch every bank once.
//   K, 8 bit: piece c of row r at c ^ (r & 15)             (an operand read: 16 rows x one piece per 256 bytes of banks)
//   K, 4 bit: piece c of row r at c ^ ((r >> 1) & 7)       (rows are 128 bytes: two rows span the banks)
//   V, 8 bit: 32-byte group c of row r at c ^ ((r & 3) | 4*((r >> 3) & 1))
//   V, 4 bit: piece c of row r at c ^ (((r >> 3) & 3) | 4*((r >> 1) & 1))
// A transposing read gives a group of 16 lanes 16 columns (bytes or nibbles) of the 8 (16) rows that its lanes name.
// The rows a lane's operand bytes stand for follow from the score layout: byte 16*b + i is token 32b + 8*(i/4) + 4h + i%4.
//   8 bit, read m of 4: rows 16m + 4h + {0..3, 8..11}
//   4 bit, read m of 2: rows 32h + 4m + {0..3, 8..11, 16..19, 24..27}
template <int BITS>
__device__ __forceinline__ LowbitLanes<BITS> lowbit_lanes(int lane)
{
    LowbitLanes<BITS> a;
    const int n = lane & 31, h = lane >> 5, l16 = lane & 15, side = (lane >> 4) & 1;
    if constexpr (BITS == 8) {
        a.ka = n * 256 + (((2 * h) ^ (n & 15)) << 4);                  // (+ piece 4*c + i: flips bits 6, 7 and bit 4)
        const int r8 = l16 >> 1;                                       // row named by this lane, of the 8
        const int row = 4 * h + (r8 & 3) + 8 * (r8 >> 2);
        a.va = row * 256 + (r8 << 5) + 16 * side + 8 * (l16 & 1);      // (+ block i: bits 5 .. 7)
    } else {
        a.ka = n * 128 + ((h ^ ((n >> 1) & 7)) << 4);                  // (+ piece 2*c: bits 5, 6)
        const int row = 32 * h + 8 * (l16 >> 2) + (l16 & 3);
        const int key = (l16 >> 2) | (((l16 >> 1) & 1) << 2);
        a.va = row * 128 + (key << 4) + 8 * side;                      // (+ block i: bits 4 .. 6)
    }
    return a;
}

// Running state of one wave: 32 columns x 256 output dims.
//
// The reference exponent of a column's weights is set by its first tile and then stays: weights may grow to
// 2^kFixedReferenceLag relative to it, which costs nothing (the weights enter the product with a power-of-two scale per tile, and
// sums are fp32), and the accumulators never pass through vector registers to be rescaled.  The true maximum is
// tracked beside it; if it ends up further ahead than that, the workgroup streams the segment once more with the
// maxima it has seen as references (decode_lowbit_kernel).  So it does if a weight times its value scale has passed kLargeWeight, from
// where on sums could leave fp32, and a lower reference is to blame: 2^24 tokens times the largest code, 448, stay finite
// below 2^95.
constexpr float kLargeWeight = 1.2089258e24f;        // 2^80
// The true maximum is tracked from the reference on (an exponent is one fused multiply-add), so a reference far below the scores that count would
// hide them in its own rounding: a first tile below kLowestReference leaves none (-inf: exponents from 0 on), and the restart
// takes the maximum as it is.  Below kLowestScore a score is no more than -inf (differences between such scores are rounding).
constexpr float kLowestReference = -16777216.0f;     // -2^24: rounded to at most 1
constexpr float kLowestScore = -1.2676506e30f;       // -2^100
struct LowbitState {
    f32x16 acc[8];       // [32-dim block]; element i: d = 32*db + 8*(i/4) + 4*h + i%4
    float m;             // reference exponent, log2 domain (-inf: the column has no token here)
    float s_max;         // this lane's largest score so far, log2 domain, from the reference on (from 0 on while that is -inf); decode_bf16_multi_kernel: the raw score
    float w_top;         // this lane's largest weight times value scale so far (magnitude)
    float l;             // this lane's share of the sum of weights
};

struct SplitWeights { i32x8 hi, lo; int e_hi, e_lo; };                 // value = hi * 2^(e_hi - 127) + lo * 2^(e_lo - 127)

// The matrix instructions are written out: the accumulators are only ever touched by them, so they live in the accumulation
// half of the register file (as "a" operands), and everything else -- query terms, scores, operands -- has the other half;
// left to the compiler, scores and accumulators are copied between the halves every tile.  The hazard between a
// matrix instruction and a vector instruction that reads its result is therefore covered by hand: 24 wait states
// (scores_ready, output_ready), or two more matrix instructions issued in between (the pipe takes one every 16 passes).  The
// build checks the machine code for it (asm_check.py: check_matrix_hazards).
template <int BITS> struct KeyOperand { typedef i32x8 type; };
template <> struct KeyOperand<4> { typedef u32x4 type; };
template <int BITS> using OperandA = typename KeyOperand<BITS>::type;                     // 32 bytes (8 bit) or 16 bytes per lane
// (the scale operand of A is the unit scale, E8M0 127; the query's is its head's 2^-e, so that all columns' scores come in one unit)
template <int BITS>
__device__ __forceinline__ void mfma_scores_first(f32x16& d, const OperandA<BITS>& a, const i32x8& b, int one, int b_scale)
{
    if constexpr (BITS == 8)
        asm volatile("v_mfma_scale_f32_32x32x64_f8f6f4 %0, %1, %2, 0, %3, %4 op_sel_hi:[0,0,0]" : "=&v"(d) : "v"(a), "v"(b), "v"(one), "v"(b_scale));
    else
        asm volatile("v_mfma_scale_f32_32x32x64_f8f6f4 %0, %1, %2, 0, %3, %4 op_sel_hi:[0,0,0] cbsz:4" : "=&v"(d) : "v"(a), "v"(b), "v"(one), "v"(b_scale));
}
template <int BITS>
__device__ __forceinline__ void mfma_scores(f32x16& d, const OperandA<BITS>& a, const i32x8& b, int one, int b_scale)
{
    if constexpr (BITS == 8)
        asm volatile("v_mfma_scale_f32_32x32x64_f8f6f4 %0, %1, %2, %0, %3, %4 op_sel_hi:[0,0,0]" : "+v"(d) : "v"(a), "v"(b), "v"(one), "v"(b_scale));
    else
        asm volatile("v_mfma_scale_f32_32x32x64_f8f6f4 %0, %1, %2, %0, %3, %4 op_sel_hi:[0,0,0] cbsz:4" : "+v"(d) : "v"(a), "v"(b), "v"(one), "v"(b_scale));
}
template <int BITS>
__device__ __forceinline__ void mfma_output(f32x16& d, const OperandA<BITS>& a, const i32x8& b, int one, int b_scale)
{
    if constexpr (BITS == 8)
        asm volatile("v_mfma_scale_f32_32x32x64_f8f6f4 %0, %1, %2, %0, %3, %4 op_sel_hi:[0,0,0]" : "+a"(d) : "v"(a), "v"(b), "v"(one), "v"(b_scale));
    else
        asm volatile("v_mfma_scale_f32_32x32x64_f8f6f4 %0, %1, %2, %0, %3, %4 op_sel_hi:[0,0,0] cbsz:4" : "+a"(d) : "v"(a), "v"(b), "v"(one), "v"(b_scale));
}
__device__ __forceinline__ void scores_pass(f32x16 (&s)[2]) { asm volatile("" : "+v"(s[0]), "+v"(s[1])); }      // nothing reads a score before this
__device__ __forceinline__ void scores_ready(f32x16 (&s)[2]) { asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" : "+v"(s[0]), "+v"(s[1])); }
__device__ __forceinline__ void output_ready(f32x16 (&acc)[8])
{
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" : "+a"(acc[0]), "+a"(acc[1]), "+a"(acc[2]), "+a"(acc[3]), "+a"(acc[4]), "+a"(acc[5]), "+a"(acc[6]), "+a"(acc[7]));
}
// Vector-written operands of a matrix instruction are complete (two wait states).
__device__ __forceinline__ void operands_ready(SplitWeights& w) { asm volatile("s_nop 1" : "+v"(w.hi), "+v"(w.lo), "+v"(w.e_hi), "+v"(w.e_lo)); }

// The two products of a tile, 16 matrix instructions (of 64 cycles) each.  `beside(k)` is called after instruction k with
// k a compile-time constant: independent work placed there runs in the shadow of the matrix pipe (a wave is alone on
// its SIMD, so nothing else would; and a wave issues one instruction every 4 cycles, so a slot holds about 15).
// The scheduling fences keep it where it was put.  Operands are read from LDS two fragments (four instructions) ahead; begin()
// reads the first two.
template <int K> using Slot = std::integral_constant<int, K>;
template <class F, int... K>
__device__ __forceinline__ void for_slots(F&& f, std::integer_sequence<int, K...>) { (f(Slot<K>{}), ...); }

template <int BITS>
struct KeyReader {
    const LowbitLanes<BITS>& ln;
    lds_ptr_t lds;
    int first;
    OperandA<BITS> f[3];
    __device__ __forceinline__ void read(int i)                        // fragment i: chunk i / 2, token block i & 1
    {
        const int c = i >> 1, b = i & 1;
        if constexpr (BITS == 8) {
            union { i32x8 v; u32x4 h[2]; } x;
            x.h[0] = *LDS_AT(u32x4, lds, (first ^ (c << 6)) + b * 32 * 256);
            x.h[1] = *LDS_AT(u32x4, lds, (first ^ (c << 6) ^ 16) + b * 32 * 256);
            f[i % 3] = x.v;
        } else {
            f[i % 3] = *LDS_AT(u32x4, lds, (first ^ (c << 5)) + b * 32 * 128);
        }
    }
    __device__ __forceinline__ void begin(int base) { first = base + ln.ka; read(0); read(1); }
};
template <int BITS>
struct ValueReader {
    const LowbitLanes<BITS>& ln;
    lds_ptr_t lds;
    int first;
    OperandA<BITS> f[3];
    __device__ __forceinline__ void read(int db)                       // 32-dim block db
    {
        union { OperandA<BITS> v; i32x2 p[BITS == 8 ? 4 : 2]; } x;
        if constexpr (BITS == 8) {
#pragma unroll
            for (int m = 0; m < 4; ++m) x.p[m] = __builtin_amdgcn_ds_read_tr8_b64_v2i32(LDS_AT(i32x2, lds, (first ^ (db << 5)) + m * 16 * 256));
        } else {
#pragma unroll
            for (int m = 0; m < 2; ++m) x.p[m] = __builtin_amdgcn_ds_read_tr4_b64_v2i32(LDS_AT(i32x2, lds, (first ^ (db << 4)) + m * 4 * 128));
        }
        f[db % 3] = x.v;
    }
    __device__ __forceinline__ void begin(int base) { first = base + ln.va; read(0); read(1); }
};

template <int BITS, class F>
__device__ __forceinline__ void qk_tile(f32x16 (&s)[2], const SplitQuery& q, KeyReader<BITS>& keys, F&& beside)
{
    const int one = 0x7F;
    for_slots([&](auto k) {
        constexpr int f = k.value >> 1;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr ((k.value & 1) == 0) {
            if constexpr (f < 2) mfma_scores_first<BITS>(s[f & 1], keys.f[f % 3], q.lo[f >> 1], one, q.scale);
            else                 mfma_scores<BITS>(s[f & 1], keys.f[f % 3], q.lo[f >> 1], one, q.scale);
            if constexpr (f + 2 < 8) keys.read(f + 2);
        } else {
            mfma_scores<BITS>(s[f & 1], keys.f[f % 3], q.hi[f >> 1], one, q.scale);
        }
        beside(k);
    }, std::make_integer_sequence<int, 16>{});
    __builtin_amdgcn_sched_barrier(0);
}

template <int BITS, class F>
__device__ __forceinline__ void pv_tile(f32x16 (&acc)[8], const SplitWeights& w, ValueReader<BITS>& values, F&& beside)
{
    const int one = 0x7F;
    for_slots([&](auto k) {
        constexpr int db = k.value >> 1;
        __builtin_amdgcn_sched_barrier(0);
        if constexpr ((k.value & 1) == 0) {
            mfma_output<BITS>(acc[db], values.f[db % 3], w.lo, one, w.e_lo);
            if constexpr (db + 2 < 8) values.read(db + 2);
        } else {
            mfma_output<BITS>(acc[db], values.f[db % 3], w.hi, one, w.e_hi);
        }
        beside(k);
    }, std::make_integer_sequence<int, 16>{});
    __builtin_amdgcn_sched_barrier(0);
}

// Keeps a value where the program text has it, relative to the matrix instructions (both are volatile).
__device__ __forceinline__ void pin(float& x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void pin(int& x) { asm volatile("" : "+v"(x)); }

// Scores of a tile -> weights times value scales (fp32).  step(k), k = 0 .. 15, works on values 2k and 2k + 1 (value
// 16*b + i is element i of token block b).  MASKED: tokens tok0 + .. at or past t1 get the weight 0.
template <bool MASKED>
struct ScoresToWeights {
    f32x16 (&s)[2];
    float (&out)[32];
    LowbitState& st;
    float m_safe;            // reference exponent, 0 for a column without tokens
    lds_ptr_t lds;
    int ks_off, vs_off;      // LDS offsets of the tile's scales (the keys' times the softmax scale), this lane's half (+ 16*h) included
    int tok_left;            // t1 - tok0 - 4*h
    f32x4 ksc[3], vsc[3];    // of tokens 8i + 4h .. (values 4i ..) at [i % 3]: read two groups ahead
    float w_max, psum[2];

    __device__ __forceinline__ void read(int i)
    {
        ksc[i % 3] = *LDS_AT(f32x4, lds, ks_off + i * 32);
        vsc[i % 3] = *LDS_AT(f32x4, lds, vs_off + i * 32);
    }
    __device__ __forceinline__ void begin()
    {
        read(0);
        read(1);
        w_max = psum[0] = psum[1] = 0.f;
    }
    __device__ __forceinline__ float masked(float x, int v) const { return MASKED && 8 * (v >> 2) + (v & 3) >= tok_left ? -INFINITY : x; }
    __device__ __forceinline__ void weigh(float x0, float x1, int v)      // scores from the reference on
    {
        const float p0 = fast_exp2(x0);
        const float p1 = fast_exp2(x1);
        float y0 = p0 * vsc[(v >> 2) % 3][v & 3];
        float y1 = p1 * vsc[(v >> 2) % 3][(v & 3) + 1];
        pin(y0);
        pin(y1);
        // (the sums stand between the pinned weights and their first reader: the compiler puts a wait state where an instruction reads what the
        // one before it, an assembly block, has written)
        psum[0] += p0;
        psum[1] += p1;
        pin(psum[0]);
        pin(psum[1]);
        w_max = fmaxf(fmaxf(w_max, fabsf(y0)), fabsf(y1));
        out[v] = y0;
        out[v + 1] = y1;
        pin(w_max);
    }
    template <int K> __device__ __forceinline__ void step(Slot<K>)
    {
        constexpr int v = 2 * K;
        if constexpr ((K & 1) == 0 && K / 2 + 2 < 8) read(K / 2 + 2);
        const float x0 = masked(__builtin_fmaf(s[v >> 4][v & 15], ksc[(v >> 2) % 3][v & 3], -m_safe), v);
        const float x1 = masked(__builtin_fmaf(s[v >> 4][(v & 15) + 1], ksc[(v >> 2) % 3][(v & 3) + 1], -m_safe), v + 1);
        st.s_max = fmaxf(fmaxf(st.s_max, x0), x1);
        pin(st.s_max);
        weigh(x0, x1, v);
    }
    __device__ __forceinline__ void sum_up()
    {
        st.l += psum[0] + psum[1];
        st.w_top = fmaxf(st.w_top, w_max);
    }
    // The segment's first tile, in one go: sets the reference.  (Tokens past the end have a key scale of 1 here.)  The exponents are formed as in
    // step(), one fused multiply-add from score and scale: a product rounded ahead of the subtraction would set tokens of this tile apart from
    // equal ones of the next by the rounding of a large score.
    __device__ __forceinline__ void first()
    {
        w_max = psum[0] = psum[1] = 0.f;
        if (tok_left < kTile) {                       // (a real branch, and no comparison made ahead of it)
            asm volatile("" : "+v"(tok_left));
#pragma unroll
            for (int v = 0; v < 32; ++v) s[v >> 4][v & 15] = masked(s[v >> 4][v & 15], v);
        }
        f32x4 k4[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            k4[i] = *LDS_AT(f32x4, lds, ks_off + i * 32);
#pragma unroll
            for (int j = 0; j < 4; ++j) st.s_max = fmaxf(st.s_max, s[i >> 2][4 * (i & 3) + j] * k4[i][j]);
        }
        if (st.m == -INFINITY) {
            const float top = half_max(st.s_max);
            st.m = top < kLowestReference ? -INFINITY : top;
        }
        m_safe = st.m == -INFINITY ? 0.f : st.m;
        st.s_max -= m_safe;
#pragma unroll
        for (int v = 0; v < 32; v += 2) {
            if ((v & 3) == 0) vsc[(v >> 2) % 3] = *LDS_AT(f32x4, lds, vs_off + (v >> 2) * 32);
            weigh(__builtin_fmaf(s[v >> 4][v & 15], k4[v >> 2][v & 3], -m_safe), __builtin_fmaf(s[v >> 4][(v & 15) + 1], k4[v >> 2][(v & 3) + 1], -m_safe), v);
        }
        sum_up();
    }
};

// ... -> two e4m3 terms with one power-of-two scale per column and tile (the scale operand of the matrix instruction
// undoes it): w = hi * 2^k + lo * 2^(k-5), k such that the largest |w| of the tile's 64 tokens lies in [128, 256) * 2^k.
// hi keeps 4 significant bits, the remainder (at most half a step of hi) 4 more and its sign: at least the 8 bits of a bf16
// weight down to 2^-13 of the tile's largest (where hi becomes subnormal), below that an error of at most 2^-22 of the
// largest (half a subnormal step of lo).  A bf16 weight would keep its 8 bits there too; it shows only in dims where the heavy
// tokens' codes are 0 (test_light_tokens_beside_a_heavy_one).  scale() picks k, steps i = 0 .. 7 convert the 32 values.
struct WeightsToOperands {
    float (&p)[32];
    SplitWeights& w;
    float s_hi, s_lo;

    __device__ __forceinline__ void scale(float w_max)
    {
        int e = (int)((__float_as_uint(half_max(w_max)) >> 23) & 0xFFu);
        e = e < 13 ? 13 : e;
        w.e_hi = e - 7;
        w.e_lo = e - 12;
        s_hi = __uint_as_float((uint32_t)(e - 7) << 23);
        s_lo = __uint_as_float((uint32_t)(e - 12) << 23);
    }
    // Two steps take eight values: the even one their first terms and what those stand for, the odd one the remainders.  Eight, so that
    // each conversion has two others between the half-register write of its operand and itself (four at a time take wait states
    // there; with those ahead of the first readers of pinned values, 4 bit, 128 x 8192 tokens: 80.1 us, without 78.1).  (One block: left to the compiler, every conversion comes with a cleared
    // destination and a wait state of its own.)
    f32x2 t[4];
    template <int I> __device__ __forceinline__ void step(Slot<I>)
    {
        constexpr int i = 8 * (I / 2);
        if constexpr ((I & 1) == 0) {
            int hi0, hi1;
            asm volatile("v_cvt_scalef32_pk_fp8_f32 %0, %6, %7, %14\n\t"
                         "v_cvt_scalef32_pk_fp8_f32 %0, %8, %9, %14 op_sel:[0,0,0,1]\n\t"
                         "v_cvt_scalef32_pk_fp8_f32 %1, %10, %11, %14\n\t"
                         "v_cvt_scalef32_pk_fp8_f32 %1, %12, %13, %14 op_sel:[0,0,0,1]\n\t"
                         "v_cvt_scalef32_pk_f32_fp8 %2, %0, %14\n\t"
                         "v_cvt_scalef32_pk_f32_fp8 %3, %0, %14 op_sel:[1,0,0]\n\t"
                         "v_cvt_scalef32_pk_f32_fp8 %4, %1, %14\n\t"
                         "v_cvt_scalef32_pk_f32_fp8 %5, %1, %14 op_sel:[1,0,0]"
                         : "=&v"(hi0), "=&v"(hi1), "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3])
                         : "v"(p[i]), "v"(p[i + 1]), "v"(p[i + 2]), "v"(p[i + 3]), "v"(p[i + 4]), "v"(p[i + 5]), "v"(p[i + 6]), "v"(p[i + 7]), "v"(s_hi));
            w.hi[I] = hi0;
            w.hi[I + 1] = hi1;
        } else {
            int lo0, lo1;
            const float r0 = p[i] - t[0][0], r1 = p[i + 1] - t[0][1], r2 = p[i + 2] - t[1][0], r3 = p[i + 3] - t[1][1];
            const float r4 = p[i + 4] - t[2][0], r5 = p[i + 5] - t[2][1], r6 = p[i + 6] - t[3][0], r7 = p[i + 7] - t[3][1];
            asm volatile("v_cvt_scalef32_pk_fp8_f32 %0, %2, %3, %10\n\t"
                         "v_cvt_scalef32_pk_fp8_f32 %0, %4, %5, %10 op_sel:[0,0,0,1]\n\t"
                         "v_cvt_scalef32_pk_fp8_f32 %1, %6, %7, %10\n\t"
                         "v_cvt_scalef32_pk_fp8_f32 %1, %8, %9, %10 op_sel:[0,0,0,1]"
                         : "=&v"(lo0), "=&v"(lo1) : "v"(r0), "v"(r1), "v"(r2), "v"(r3), "v"(r4), "v"(r5), "v"(r6), "v"(r7), "v"(s_lo));
            w.lo[I - 1] = lo0;
            w.lo[I] = lo1;
        }
    }
};

// End of a segment, one query token: the two waves that share 32 columns (tp = 0, 1: the even and the odd tiles) exchange
// halves of their accumulators through 64 KB of dead tile memory (and 1 KB behind it: tiles or their scales, dead as
// well); tp 0 finishes dims 0..127, tp 1 the rest.
// Partials keep the lane-order layout of the other kernels (float4 index (head/16*16 + d/16)*64 + d/4%4*16 + head%16).
__device__ __forceinline__ size_t partial_index(int head, int dq)           // dq = d / 4
{
    return (size_t)((head >> 4) * 16 + (dq >> 2)) * 64 + (dq & 3) * 16 + (head & 15);
}
__device__ __forceinline__ f32x4 quad(const f32x16& x, int i) { return (f32x4){x[4 * i], x[4 * i + 1], x[4 * i + 2], x[4 * i + 3]}; }
template <int KEEP, int SEND>
__device__ __forceinline__ void finish_lowbit_half(LowbitState& st, lds_ptr_t lds, const AttnArgs& a, const Segment& r, int cg, int tp, int lane)
{
    constexpr int kMl = 4 * 16384;
    const int n = lane & 31, h = lane >> 5, head = 32 * cg + n;
    const int mine = (cg * 2 + tp), theirs = (cg * 2 + (tp ^ 1));
#pragma unroll
    for (int i = 0; i < 16; ++i) *LDS_AT(f32x4, lds, mine * 16384 + i * 1024 + lane * 16) = quad(st.acc[SEND + (i >> 2)], i & 3);
    if (h == 0) {
        *LDS_AT(float, lds, kMl + mine * 256 + n * 4) = st.m;
        *LDS_AT(float, lds, kMl + mine * 256 + 128 + n * 4) = st.l;
    }
    __syncthreads();
    const float m_o = *LDS_AT(float, lds, kMl + theirs * 256 + n * 4);
    const float l_o = *LDS_AT(float, lds, kMl + theirs * 256 + 128 + n * 4);
    const float m = fmaxf(st.m, m_o);                 // -inf if every score of the segment is: a partial without weight
    const float m_safe = m == -INFINITY ? 0.f : m;
    float w_s = fast_exp2(st.m - m_safe);
    float w_o = fast_exp2(m_o - m_safe);
    const float l = st.l * w_s + l_o * w_o;
    f32x4* dst;
    if (r.final_result) {                             // dims 4*dq.. of the row, dq = 8*(block) + 2*(quad) + h: 2 float4 apart per quad
        const float inv = 1.0f / l;
        w_s *= inv;
        w_o *= inv;
        dst = (f32x4*)(a.out + ((size_t)r.b * kHeads + head) * kHeadDim) + h;
    } else {
        dst = (f32x4*)a.ws_acc + (size_t)r.slot * (kHeads * kHeadDim / 4) + partial_index(head, h);
        if (tp == 0 && h == 0) *(float2*)(a.ws_ml + ((size_t)r.slot * kHeads + head) * 2) = make_float2(m, l);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const f32x4 other = *LDS_AT(f32x4, lds, theirs * 16384 + i * 1024 + lane * 16);
        const f32x4 res = quad(st.acc[KEEP + (i >> 2)], i & 3) * w_s + other * w_o;
        const int dq = 8 * (KEEP + (i >> 2)) + 2 * (i & 3);              // (+ h: even, so partial_index(head, dq + h) = partial_index(head, h) + ..)
        dst[r.final_result ? dq : (dq >> 2) * 64 + (dq & 3) * 16] = res;
    }
}

// Two query tokens: a wave holds all dims of its columns and has seen all tokens of the segment.  A token that saw no
// cached token leaves m = -inf, l = 0 and a zero accumulator; as a final result that is the zero row.
__device__ __forceinline__ void finish_lowbit_two(LowbitState& st, const AttnArgs& a, const Segment& r, int qtok, int hh, int lane)
{
    const int n = lane & 31, h = lane >> 5, head = 32 * hh + n;
    float scale = 1.0f;
    f32x4* dst;
    if (r.final_result) {
        scale = st.l > 0.f ? 1.0f / st.l : 0.f;
        dst = (f32x4*)(a.out + (((size_t)r.b * a.q_len + a.q0 + qtok) * kHeads + head) * kHeadDim) + h;
    } else {
        const size_t slot = (size_t)r.slot * a.n_here + qtok;
        dst = (f32x4*)a.ws_acc + slot * (kHeads * kHeadDim / 4) + partial_index(head, h);
        if (h == 0) *(float2*)(a.ws_ml + (slot * kHeads + head) * 2) = make_float2(st.m, st.l);
    }
#pragma unroll
    for (int i = 0; i < 32; ++i) {
        const int dq = 8 * (i >> 2) + 2 * (i & 3);
        dst[r.final_result ? dq : (dq >> 2) * 64 + (dq & 3) * 16] = quad(st.acc[i >> 2], i & 3) * scale;
    }
}

template <bool PAGED, int QL, int BITS>
__global__ __launch_bounds__(kLowbitThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void decode_lowbit_kernel(AttnArgs a)
{
    using S = LowbitShape<QL, BITS>;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const lds_ptr_t lds = (lds_ptr_t)smem;
    const uint32_t lds_addr0 = (uint32_t)(uintptr_t)lds;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int hh = wave & 1;                          // which 32 heads
    const int grp = wave >> 1;                        // one query token: tile parity; two: query token of the pair
    const int h = lane >> 5;
    const LowbitLanes<BITS> ln = lowbit_lanes<BITS>(lane);

    // Direct loads: load u of a wave fills rows kRowStep*u + kRowsPerLoad*wave + (lane's row) of a tile; the rows of one
    // lane differ by a multiple of 16 (8 bit) or 32 (4 bit), so its permutation of the pieces is the same in all of them.
    constexpr int kRowsPerLoad = 1024 / S::kRowBytes;
    constexpr int kLanesPerRow = S::kRowBytes / 16;
    constexpr int kRowStep = 4 * kRowsPerLoad;
    auto first_row = [&](int l) { return kRowsPerLoad * wave + l / kLanesPerRow; };
    auto source = [&](bool value, int l) {                            // byte offset in the row of the piece that lane l brings
        const int row = first_row(l), piece = l % kLanesPerRow;
        if (BITS == 8) return 16 * (value ? piece ^ (2 * ((row & 3) | (4 * ((row >> 3) & 1)))) : piece ^ (row & 15));
        return 16 * (value ? piece ^ (((row >> 3) & 3) | (4 * ((row >> 1) & 1))) : piece ^ ((row >> 1) & 7));
    };
    const uint32_t lds_wave = lds_addr0 + kRowsPerLoad * wave * S::kRowBytes;
    uint32_t k_off[S::kLoadsPerTile], v_off[S::kLoadsPerTile];        // of a whole tile
#pragma unroll
    for (int u = 0; u < S::kLoadsPerTile; ++u) {
        k_off[u] = (uint32_t)((first_row(lane) + kRowStep * u) * S::kRowBytes + source(false, lane));
        v_off[u] = (uint32_t)((first_row(lane) + kRowStep * u) * S::kRowBytes + source(true, lane));
    }
    auto k_dst_of = [&](int slot) { return lds_wave + slot * S::kStageBytes; };
    auto v_dst_of = [&](int slot) { return lds_wave + S::kVBase + slot * S::kStageBytes; };

    // Tiles [t0, t1) of sequence b.  Tiles past the end of a span (the second of an odd last stage) repeat its last tile: their
    // tokens are masked.  Rows at or past t1 re-read the last valid token.
    struct Span { int b, t0, t1, n_tiles; };
    struct StageOrigin { int64_t row[S::kTiles]; };
    auto origin = [&](const Span& g, int stage) {
        StageOrigin o;
#pragma unroll
        for (int j = 0; j < S::kTiles; ++j) {
            int tile = S::kTiles * stage + j;
            tile = tile < g.n_tiles ? tile : g.n_tiles - 1;
            tile = __builtin_amdgcn_readfirstlane(tile);                // keeps the page lookup a scalar load
            const int tile_t0 = g.t0 + tile * kTile;
            o.row[j] = tile_row0<PAGED>(a, g.b, tile_t0, lookup_page<PAGED>(a, g.b, tile_t0));
        }
        return o;
    };
    // An even wave brings key scales, an odd one value scales, of tile scale_tile of the stage.
    const int scale_tile = S::kTiles == 2 ? wave >> 1 : 0;
    const float* const scale_src = (wave & 1) ? a.v_scale : a.k_scale;
    const uint32_t scale_dst = lds_addr0 + ((wave & 1) ? S::kVScaleBase : S::kKScaleBase) + scale_tile * kTile * 4;
    auto load_scales = [&](const StageOrigin& o, int slot, uint32_t off) {
        load_to_lds_4B(scale_src + (S::kTiles == 2 && scale_tile ? o.row[S::kTiles - 1] : o.row[0]), off, scale_dst + slot * S::kScaleStage);
    };
    // Piece i of the 2 * kTiles * kLoadsPerTile of an iteration (keys, then values), whole tiles only
    auto load_piece = [&](auto i, const StageOrigin& ok, const StageOrigin& ov, uint32_t k_dst, uint32_t v_dst) {
        constexpr bool value = i.value >= S::kTiles * S::kLoadsPerTile;
        constexpr int j = (i.value / S::kLoadsPerTile) % S::kTiles, u = i.value % S::kLoadsPerTile;
        load_to_lds_16B_at<j * S::kTileBytes + kRowStep * u * S::kRowBytes>((const unsigned char*)(value ? a.v : a.k) + (value ? ov : ok).row[j] * S::kRowBytes,
                                                                            value ? v_off[u] : k_off[u], value ? v_dst : k_dst);
    };
    // Keys (with the scales of both tensors) or values of any stage (not unrolled: see request_query)
    auto load_stage = [&](bool value, const Span& g, int stage, const StageOrigin& o, int slot) {
        int lane_now = lane;                                            // (offsets formed here, not kept in registers)
        asm volatile("" : "+v"(lane_now));
        const unsigned char* base = (const unsigned char*)(value ? a.v : a.k);
        const uint32_t dst = value ? v_dst_of(slot) : k_dst_of(slot);
        const int src = source(value, lane_now);
#pragma unroll
        for (int j = 0; j < S::kTiles; ++j) {
            int tile = S::kTiles * stage + j;
            tile = tile < g.n_tiles ? tile : g.n_tiles - 1;
            const int last = g.t1 - 1 - (g.t0 + tile * kTile);          // last valid row of the tile (>= 0)
#pragma unroll 1
            for (int u = 0; u < S::kLoadsPerTile; ++u) {
                const int row = first_row(lane_now) + kRowStep * u;
                const int in_tile = row < last ? row : last;
                load_to_lds_16B(base + o.row[j] * S::kRowBytes, (uint32_t)(in_tile * S::kRowBytes + src), dst + j * S::kTileBytes + kRowStep * u * S::kRowBytes);
            }
            if (!value && j == scale_tile) load_scales(o, slot, (uint32_t)(4 * (lane_now < last ? lane_now : last)));
        }
    };
    auto query_row = [&](int b) { return ((size_t)(QL == 2 ? a.q_len * b + a.q0 + grp : b)) * kHeads + 32 * hh; };
    // (one query token: from area hh to area 2 + hh; two: area `wave`)
    const int q_in = QL == 1 ? (hh ? S::query_area(1) : S::query_area(0)) : wave == 0 ? S::query_area(0) : wave == 1 ? S::query_area(1) : wave == 2 ? S::query_area(2) : S::query_area(3);
    const int q_out = QL == 1 ? (hh ? S::query_area(3) : S::query_area(2)) : q_in;
    // Everything a segment starts with: the query, then keys and values of the first kDepth stages
    auto request_start = [&](const Span& g) {
        int lane_now = lane;
        asm volatile("" : "+v"(lane_now));
        request_query(a.q, query_row(g.b), lds_addr0 + q_in, QL == 1 ? 8 * grp : 0, kQueryOps<QL>, lane_now);
#pragma unroll 1
        for (int d = 0; d < S::kDepth; ++d) {
            const StageOrigin o = origin(g, d);                         // (past the span's end: its last tile again)
            load_stage(false, g, d, o, d);
            load_stage(true, g, d, o, d);
        }
    };

    // (A first segment asked for ahead of the schedule, where it would be if every sequence had the length of the hint,
    // changes nothing when they do -- 56.1 against 56.3 us, 64 x 8192 tokens at 8 bits -- and costs 1 .. 2.5 us
    // when they do not: the wrong 96 KB per workgroup come first.)
    stage_lengths(a, lds, S::kSchedBase);
    await_lengths<0>(a, false);
    Schedule sched = schedule_begin<kLowbitThreads>(a, lds, S::kSchedBase, kLowbitSwitch);
    Segment r;
    while (schedule_next<kLowbitThreads>(a, sched, r)) {
        const Span span = {r.b, r.t0, r.t1, r.n_tiles};
        const int n_stages = (r.n_tiles + S::kTiles - 1) / S::kTiles;
        const int n_whole = (r.t1 - r.t0) / (S::kTiles * kTile);      // stages without a row past the end: n_stages or one less
        const int end_mine = r.len - (a.q_len - 1 - a.q0 - grp);      // QL == 2: grp = query token of the pair
        const int t1_mine = QL == 2 ? (r.t1 < end_mine ? r.t1 : end_mine) : r.t1;
        const int my_tile = QL == 1 ? grp : 0;                         // this wave's tile of a stage
        auto tok_left = [&](int stage) { return t1_mine - (r.t0 + (S::kTiles * stage + my_tile) * kTile) - 4 * h; };
        auto k_of = [&](int slot) { return slot * S::kStageBytes + my_tile * S::kTileBytes; };
        auto v_of = [&](int slot) { return S::kVBase + slot * S::kStageBytes + my_tile * S::kTileBytes; };
        // Key scales of this wave's tile, times softmax scale * log2(e) (the query's 2^-e is in the scores already): a token's for every lane, so
        // that a score becomes an exponent in one fused multiply-add.  Written and read by the wave itself: LDS keeps the order.
        auto take_key_scale = [&](int slot) { return *LDS_AT(float, lds, S::kKScaleBase + slot * S::kScaleStage + my_tile * kTile * 4 + lane * 4); };
        auto put_key_scale = [&](float ks) { *LDS_AT(float, lds, S::kKcBase + wave * kTile * 4 + lane * 4) = ks * a.scale_log2e; };
        const int kc = S::kKcBase + wave * kTile * 4 + 16 * h;
        auto vs_of = [&](int slot) { return S::kVScaleBase + slot * S::kScaleStage + my_tile * kTile * 4 + 16 * h; };

        LowbitState st;
        st.m = -INFINITY;
        SplitQuery q;
        bool retried = false;
        for (bool again = true; again;) {
        // Prologue: the start of the segment (the query is converted while its tiles are on their way), then the keys of one stage more.
        if (threadIdx.x == 0) *LDS_AT(int, lds, S::kFlag) = 0;
        request_start(span);
        if (!retried) schedule_record(a, sched, r);
        wait_vmem_but<S::kDepth * S::kOps>();
        {
            int lane_now = lane;
            asm volatile("" : "+v"(lane_now));
            split_query<QL, BITS>(q, lds, q_in, q_out, grp, lane_now);
        }
        wait_vmem_but<0>();
        __syncthreads();
        StageOrigin o[2];                                              // of stages s + kDepth (values) and s + 1 + kDepth (keys)
        if (S::kDepth < n_stages) {
            o[0] = origin(span, S::kDepth);
            load_stage(false, span, S::kDepth, o[0], S::kDepth);
        }
        if (S::kDepth + 1 < n_stages) o[1] = origin(span, S::kDepth + 1);

#pragma unroll
        for (int i = 0; i < 8; ++i) st.acc[i] = (f32x16)(0.f);
        output_ready(st.acc);
        st.s_max = -INFINITY;
        st.w_top = 0.f;
        st.l = 0.f;
        float wt[32];                                                  // weights (times value scales) of stage s's tile
        float w_max, m_safe;
        KeyReader<BITS> keys{ln, lds};
        keys.begin(k_of(0));
        {
            f32x16 sc[2];
            put_key_scale(lane < tok_left(0) + 4 * h ? take_key_scale(0) : 1.f);
            qk_tile<BITS>(sc, q, keys, [](auto) {});
            scores_ready(sc);
            ScoresToWeights<true> f{sc, wt, st, 0.f, lds, kc, vs_of(0), tok_left(0)};
            f.first();
            w_max = f.w_max;
            m_safe = f.m_safe;
        }
        int s = 0;
        int slot = 0, slot_prev = S::kSlots - 1, slot_next = 1 % S::kSlots;   // of stages s, s - 1 (= s + kDepth) and s + 1
        auto advance = [&]() {
            o[0] = o[1];
            if (s + 2 + S::kDepth < n_stages) o[1] = origin(span, s + 2 + S::kDepth);
            slot_prev = slot;
            slot = slot_next;
            slot_next = slot_next + 1 == S::kSlots ? 0 : slot_next + 1;
            ++s;
        };
        // One iteration: scores of stage s + 1 beside the conversion of stage s's weights, then the weighted sum of stage s beside the
        // softmax of stage s + 1.  STEADY: requests keys s + 1 + kDepth and values s + kDepth, and stage s + 1 has whole tiles
        // only.
        auto iterate = [&](auto steady) {
            constexpr bool STEADY = decltype(steady)::value;
            constexpr int kLoads = 2 * S::kTiles * S::kLoadsPerTile, kPerSlot = 2, kLoadSlots = STEADY ? kLoads / kPerSlot : 0;
            constexpr int kConvert = STEADY ? 7 : 2;                   // first slot of the conversion
            constexpr int kKeyScale = 4;
            keys.begin(k_of(slot_next));
            f32x16 sc[2];
            SplitWeights w;
            WeightsToOperands f2{wt, w};
            ValueReader<BITS> values{ln, lds};
            ScoresToWeights<!STEADY> f1{sc, wt, st, m_safe, lds, kc, vs_of(slot_next), STEADY ? 0 : tok_left(s + 1)};
            float key_scale;
            const uint32_t k_dst = k_dst_of(slot), v_dst = v_dst_of(slot_prev);      // keys s + 1 + kDepth take the slot of keys s
            qk_tile<BITS>(sc, q, keys, [&](auto k) {
                if constexpr (k.value < kLoadSlots)
                    for_slots([&](auto i) { load_piece(Slot<k.value * kPerSlot + i.value>{}, o[1], o[0], k_dst, v_dst); }, std::make_integer_sequence<int, kPerSlot>{});
                if constexpr (STEADY && k.value == kLoadSlots) load_scales(o[1], slot, (uint32_t)(4 * lane));
                if constexpr (k.value == 0) f2.scale(w_max);
                if constexpr (k.value >= kConvert && k.value < kConvert + 8) f2.step(Slot<k.value - kConvert>{});
                if constexpr (k.value == kKeyScale) key_scale = take_key_scale(slot_next);
                if constexpr (k.value == kKeyScale + 2) put_key_scale(key_scale);
                if constexpr (k.value == 14) values.begin(v_of(slot));
                if constexpr (k.value == 15) f1.begin();
            });
            operands_ready(w);
            pv_tile<BITS>(st.acc, w, values, [&](auto k) {
                if constexpr (k.value == 0) scores_pass(sc);
                if constexpr (k.value >= 1) f1.step(Slot<k.value - 1>{});
                if constexpr (k.value == 15) f1.step(Slot<15>{});
            });
            f1.sum_up();
            w_max = f1.w_max;
            advance();
        };
        // Iterations that request a whole group of whole tiles: every group in flight is complete, so a counted wait leaves
        // exactly the kDepth - 1 youngest.
        while (s + 1 + S::kDepth < n_whole) {
            wait_vmem_but<(S::kDepth - 1) * S::kOps>();
            __syncthreads();
            iterate(std::true_type{});
        }
        // The last iterations: whatever is left to request, everything awaited.
        while (s + 1 < n_stages) {
            wait_vmem_but<0>();
            __syncthreads();
            if (s + 1 + S::kDepth < n_stages) load_stage(false, span, s + 1 + S::kDepth, o[1], slot);
            if (s + S::kDepth < n_stages) load_stage(true, span, s + S::kDepth, o[0], slot_prev);
            iterate(std::false_type{});
        }
        {
            wait_vmem_but<0>();
            __syncthreads();
            SplitWeights w;
            WeightsToOperands f2{wt, w};
            ValueReader<BITS> values{ln, lds};
            values.begin(v_of(slot));
            f2.scale(w_max);
            for_slots([&](auto k) { f2.step(k); }, std::make_integer_sequence<int, 8>{});
            operands_ready(w);
            pv_tile<BITS>(st.acc, w, values, [](auto) {});
        }
        // A column whose largest score has outrun its reference too far: the workgroup streams the segment once more, the
        // maxima as references.  (A reference of -inf, left by a first tile of nothing but -inf, is outrun by any finite score;
        // a column without tokens has s_max = -inf too and keeps it.)
        const float top = half_max(st.s_max) + m_safe;
        const float m_true = top < kLowestScore ? -INFINITY : top;
        const bool outrun = !retried && (m_true > st.m + kFixedReferenceLag || (m_true > st.m && half_max(st.w_top) > kLargeWeight));
        if (outrun) *LDS_AT(int, lds, S::kFlag) = 1;
        __syncthreads();                              // every wave is done reading the tile memory
        again = !retried && *LDS_AT(int, lds, S::kFlag) != 0;
        if (again) {
            if (outrun) st.m = m_true;
            retried = true;
            __syncthreads();                          // the flag has been read
        }
        }
        output_ready(st.acc);
        st.l = half_sum(st.l);
        int lane_now = lane;                          // (the result's addresses are formed here, once per segment)
        asm volatile("" : "+v"(lane_now));
        if (QL == 2) {
            finish_lowbit_two(st, a, r, grp, hh, lane_now);
        } else {
            if (grp == 0) finish_lowbit_half<0, 4>(st, lds, a, r, hh, 0, lane_now);
            else          finish_lowbit_half<4, 0>(st, lds, a, r, hh, 1, lane_now);
        }
        __syncthreads();                              // the exchange area is the tile memory of the next segment
    }
}

}  // namespace mfa
