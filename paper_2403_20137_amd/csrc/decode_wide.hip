// Split pass of decode attention for many (virtual) query heads per kv-head on the matrix cores: 16-bit I/O, 4- and
// 8-bit mantissas, every block size, contiguous and paged caches (Sec. III run-time flow; several query tokens per
// sequence bring n_q_tokens * G virtual heads).
//
// With G rows a cached element takes 2 G multiply-adds, so from some G on the pass is bound by arithmetic, not by
// memory, and the arithmetic has to go into full matrix-core tiles:
//   * A workgroup decodes a tile of cached rows once, to bf16 in LDS (a code times its block's power of two is
//     exact there), and its four wavefronts, 32 virtual heads each, multiply with it (decode_split_wide).  With 64 heads or
//     fewer two wavefronts take the same heads and share the tokens of the tile out, and with 32 or fewer every
//     wavefront decodes and multiplies its own tokens (decode_split_few).
//   * Both products are formed transposed, v_mfma_f32_32x32x16_bf16 with S^T = K Q^T and O^T = V^T P^T: a lane then
//     holds scores, running maximum, sum and outputs of ONE head, the softmax needs one exchange with the other half
//     of the wavefront, and the registers that hold S^T are, converted, the second operand of the value product -- the
//     order of the tokens in its reduction is free, and V^T is laid out in LDS in the order S^T leaves them in.
//   * The query is not rounded: a bf16 query (or one cast to BFP) is one bf16 operand, an fp16 query is two (8 + 3
//     bits).  softmax_scale * log2(e) multiplies the score in fp32.  Probabilities above 32 heads are three bf16 limbs, all of
//     their 24 bits; up to 32 two (16 bits), as in the other passes for 16-bit I/O.  (Not two binary16 limbs, which take two thirds
//     of the matrix and a third of the limb instructions, 67 us for the 77 below: they have an absolute step, 2^-36 of the largest
//     probability, and where the heaviest token's values are zero the output is the sum of the light ones alone.)
// Bound by: vector ALUs and matrix cores (decode_split_wide, per wavefront, 64 tokens and 32 heads: 64 MFMAs of 32 cycles and
// some 530 vector instructions of 4 cycles, 32 exponentials of 8 among them).  256 virtual heads (64 query tokens, groups of
// 4) over 4 x 8192 tokens x 8 kv-heads: 77 us a call, fp16 I/O 86 (80 and 125 with one half of LDS, decoding and products one after
// the other; 1490 in the general pass).
// Up to 32 heads: vector ALUs 70 % busy (490 instructions per 32 tokens); 20 heads over 8 x 12000 tokens x 8 kv-heads: 40 us a
// call, against 66 us in two launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>
#include <utility>

#include "decode_args.h"
#include "decode_dev.h"
#include "decode_spans.h"
#include "kvbfp_internal.h"
#include "quantize_dev.h"

namespace {

using kvbfp::DecodeArgs;
using namespace kvbfp::dev;

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kThreads = 256;
constexpr int kRows = 32;                      // virtual heads per wavefront
constexpr uint32_t kKeyUp = 2;                 // decode_split_few: added to the keys' exponent bytes
// The sums are relative to a reference that a score may exceed by kSlack before they are rescaled (a branch and 64 products nearly
// every tile otherwise), so a sum of weighted values may be 2^kSlack above what it is with the largest score as the reference.  Values
// with bytes up to kOrdinary bear that with room to spare (those up to 218 would: below 2^92 each, times 2^kSlack, times the
// 2^31 tokens a sequence can have at most, is below 2^128).  From the first larger byte on a wavefront's reference is its largest score,
// and what wavefronts and workgroups hand on is relative to that in any case.
constexpr float kSlack = 4.f;
constexpr int kOrdinary = 200;

// packs the upper halves of two fp32 patterns: (lo, hi) -> one register of two bf16
__device__ __forceinline__ uint32_t pack_hi(uint32_t lo, uint32_t hi) { return __builtin_amdgcn_perm(hi, lo, 0x07060302u); }
__device__ __forceinline__ uint32_t pack_lo(uint32_t lo, uint32_t hi) { return __builtin_amdgcn_perm(hi, lo, 0x05040100u); }
__device__ __forceinline__ uint32_t bits(bf16x2 v) { return __builtin_bit_cast(uint32_t, v); }

// Eight 4-bit codes -> bf16 pairs (c0,c2), (c4,c6), (c1,c3), (c5,c7), scaled by 2^(E - 136) per unit (value * 2^-7):
// the nibble s|mmm widened to the byte s0000mmm is the FP8-E4M3 subnormal (-1)^s m 2^-9.
__device__ __forceinline__ void unpack8_p4(uint32_t w, float scale, uint32_t (&p)[4]) {
    uint32_t lo, hi;
    spread4(w, lo, hi);
    p[0] = bits(__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, scale, false));
    p[1] = bits(__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, scale, true));
    p[2] = bits(__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, scale, false));
    p[3] = bits(__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, scale, true));
}
// Four 8-bit codes -> fp32, scaled by 2^(E - 136) per unit (value * 2^-3).  The byte s mmmm lll is the sum of the FP8
// numbers s000mmmm (at eight times the scale) and s0000lll; the sum has at most 7 significant bits, so its upper
// half is the bf16 number.
// `field`: the exponent byte at bit 23 (nothing else of the scale operand counts).
__device__ __forceinline__ void unpack4_p8(uint32_t w, uint32_t field, float (&x)[4]) {
    const float s_lo = __uint_as_float(field), s_hi = __uint_as_float(field + (3u << 23));
    uint32_t hi, lo;
    spread8(w, hi, lo);
    const f32x2 h01 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(hi, s_hi, false), h23 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(hi, s_hi, true);
    const f32x2 l01 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(lo, s_lo, false), l23 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(lo, s_lo, true);
    x[0] = h01[0] + l01[0]; x[1] = h01[1] + l01[1];
    x[2] = h23[0] + l23[0]; x[3] = h23[1] + l23[1];
}

// Exponent bytes at the ends of their range.  The conversions take the byte as their scale operand, which fits all but the
// largest ones, and leave value * 2^-kShift in bf16, which holds all but the smallest blocks exactly.  A 16-token stage with
// one of the smallest is converted at kUp powers of two more, which its scores and probabilities make up for; a block whose byte
// is then too large for the operand is converted at kDown fewer and its bf16 numbers are raised where they lie (bf16 itself
// holds them: code 127 at byte 255 + kUp is below 2^128).  So every byte is exact beside every other.
template <int P>
struct ExpRange {
    static constexpr uint32_t kTop = P == 4 ? 254u : 251u;         // largest byte whose scale operand (8-bit: + 3) is finite
    static constexpr uint32_t kUp = 2u, kDown = 8u;
    __device__ static bool tiny(uint32_t E) { return E - 1u < 2u; }
    __device__ static bool high(uint32_t E, uint32_t up) { return E + up > kTop; }
    __device__ static uint32_t operand(uint32_t E, uint32_t up) { return high(E, up) ? E + up - kDown : E + up; }
};
// a pair of bf16 numbers times 2^kDown (normal numbers and zeros)
__device__ __forceinline__ uint32_t raise_pair(uint32_t w, bool lo, bool hi) {
    return w + (lo && (w & 0x7FFFu) ? 8u << 7 : 0u) + (hi && (w & 0x7FFF0000u) ? 8u << 23 : 0u);
}

__device__ __forceinline__ float other_half(float v) { return __shfl_xor(v, 32); }
__device__ __forceinline__ float both_halves_max(float v) {
    const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(x[0]), __uint_as_float(x[1]));
}

// The query operand: lane (head l32, half), MFMA m: the 8 channels of group `group(m, half)`, in key slot order, QL bf16
// limbs.  ROWS heads of the workgroup (`used` of them there) are requested ahead of everything else (loads return in
// order), pass through LDS in cache channel order, and every wavefront takes the 32 from `row0` on.
template <int ROWS>
struct QueryRows {
    static constexpr int kPieces = ROWS * 16 / kThreads;               // 16 pieces of 16 bytes per head
    u32x4 w[kPieces];
    int perm;
    __device__ __forceinline__ void request(const DecodeArgs& a, int b, int kvh, int s_first, int used) {
        const int tid = threadIdx.x;
        perm = a.perm_k ? (a.perm_k[kvh * kD + (tid & (kD - 1))] & (kD - 1)) : (tid & (kD - 1));   // masked: device data the host cannot check
        const bool vec = ((uintptr_t)a.q & 15u) == 0;
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            const int row = (tid >> 4) + i * (kThreads / 16);
            const uint16_t* src = (const uint16_t*)a.q + kvbfp::query_row(a, b, kvh, s_first + min(row, used - 1)) * kD + (tid & 15) * 8;
            if (vec) {
                w[i] = *(const u32x4*)src;
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) w[i][k] = (uint32_t)src[2 * k] | ((uint32_t)src[2 * k + 1] << 16);
            }
        }
    }
    // smem: ROWS * 256 bytes, inv_s: kD ints.  Called by the whole workgroup; ends with a barrier.  Returns what the scores
    // of this lane's head are to be multiplied with on top of score_mul.
    template <int P, int QL, class Group>
    __device__ __forceinline__ float build(const DecodeArgs& a, int dt, int used, int row0, uint8_t* smem, int* inv_s, float query_mul,
                                          Group&& group, bf16x8 (&q_op)[QL][8]) {
        const int tid = threadIdx.x, l32 = tid & 31, half = (tid >> 5) & 1;
        // cache position of every channel; position c goes to slot order inside its group of 8
        if (tid < kD) inv_s[perm] = P == 8 ? tid : ((tid & ~7) | ((tid & 1) ? 4 + ((tid & 7) >> 1) : ((tid & 7) >> 1)));
        lds_only_barrier();
        int at[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) at[k] = inv_s[(tid & 15) * 8 + k] & (kD - 1);
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            const int row = (tid >> 4) + i * (kThreads / 16);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const uint32_t h = row < used ? (w[i][k >> 1] >> (16 * (k & 1))) & 0xFFFFu : 0u;
                *(uint16_t*)(smem + row * 256 + (((at[k] >> 3) ^ (row & 15)) * 16) + (at[k] & 7) * 2) = (uint16_t)h;
            }
        }
        lds_only_barrier();
        const int row = row0 + l32;
        u32x4 raw[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) raw[m] = *(const u32x4*)(smem + row * 256 + ((group(m, half) ^ (row & 15)) * 16));
        lds_only_barrier();                             // the queries give way to the cached rows
        if (QL == 1 && dt == KVBFP_BF16 && a.q_mant_bits == 0 && query_mul == 1.0f) {      // the operand as it is
#pragma unroll
            for (int m = 0; m < 8; ++m) q_op[0][m] = __builtin_bit_cast(bf16x8, raw[m]);
            return 1.f;
        }
        auto value = [&](int m, int k) {
            const uint32_t h = (raw[m][k >> 1] >> (16 * (k & 1))) & 0xFFFFu;
            return dt == KVBFP_F16 ? (float)__builtin_bit_cast(_Float16, (unsigned short)h) : __uint_as_float(h << 16);
        };
        int cast_e[8];                                  // power of two of a mantissa step, if the query is cast to BFP
        if (a.q_mant_bits) {                            // like a cached row
            // a group of 8 channels lies in one block; the maximum of a block is that of its groups, here or in the other half
            float top[8], other[8];
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                top[m] = 0.f;
#pragma unroll
                for (int k = 0; k < 8; ++k) top[m] = fmaxf(top[m], fabsf(value(m, k)));
                other[m] = other_half(top[m]);
            }
            const int sh = a.log2_block - 3;            // groups per block, log2
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                float t = 0.f;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    t = (group(j, half) >> sh) == (group(m, half) >> sh) ? fmaxf(t, top[j]) : t;
                    t = (group(j, half ^ 1) >> sh) == (group(m, half) >> sh) ? fmaxf(t, other[j]) : t;
                }
                const uint32_t amax = __float_as_uint(t);
                const uint32_t bumped = (amax + (1u << (24 - a.q_mant_bits))) >> 23;
                cast_e[m] = (amax == 0 ? 0 : (int)max(bumped, 1u)) - 127 - (a.q_mant_bits - 2);
            }
        }
        // A small power of two is folded in as far as the head's largest element stays above 2^-8, the rest of it multiplies
        // the scores: below 2^-126 bf16 loses bits.  (No sum of 128 products then reaches the end of the fp32 range.)
        float lift = 1.f;
        if (fabsf(query_mul) < 1.f && query_mul != 0.f) {
            float top = 0.f;
#pragma unroll
            for (int m = 0; m < 8; ++m)
#pragma unroll
                for (int k = 0; k < 8; ++k) top = fmaxf(top, fabsf(value(m, k)));
            int e = 0;
            (void)frexpf(fmaxf(top, other_half(top)) * fabsf(query_mul), &e);
            lift = ldexpf(1.f, min(max(-8 - e, 0), -ilogbf(query_mul)));
        }
        query_mul *= lift;
#pragma unroll
        for (int m = 0; m < 8; ++m) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                float v = value(m, k);
                if (a.q_mant_bits) v = ldexpf(rintf(ldexpf(v, -cast_e[m])), cast_e[m]);
                v *= query_mul;                         // a power of two and the sign of the scale: exact
                const uint32_t top_bits = __float_as_uint(v) & 0xFFFF0000u;
                q_op[0][m][k] = __builtin_bit_cast(__bf16, (unsigned short)(top_bits >> 16));
                if (QL == 2) q_op[QL - 1][m][k] = (__bf16)(v - __uint_as_float(top_bits));
            }
            __builtin_amdgcn_sched_barrier(0);          // one group of 8 at a time: the rows in flight hold the registers
        }
        return 1.f / lift;
    }
};

// kvbfp_append_decode_attention: the current token's rows (position pos), cast and stored by one wavefront before it requests
// its first tile; returns when they are stored.  Lanes 0-7 take the key row, lanes 8-15 the value row; the others run along
// with zeros (the block maximum is a cross-lane reduction).
template <int P>
__device__ __forceinline__ void append_row(const DecodeArgs& a, int dt, int b, int kvh, int lane, int64_t pos) {
    const int sub = lane & 7, which = (lane >> 3) & 1;
    const bool live = lane < 16;
    const int32_t* pr = which ? a.perm_v : a.perm_k;
    const uint16_t* src = (const uint16_t*)(which ? a.v_new : a.k_new) + (int64_t)b * a.new_stride_b + (int64_t)kvh * a.new_stride_h;
    float x[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int c = (pr && live) ? (pr[kvh * kD + sub * 16 + i] & (kD - 1)) : sub * 16 + i;
        x[i] = live ? load_as_float(src, dt, c) : 0.f;
    }
    uint8_t* const mant = const_cast<uint8_t*>(which ? a.v_mant : a.k_mant);
    uint8_t* const exps = const_cast<uint8_t*>(which ? a.v_exp : a.k_exp);
    const int64_t row = kvbfp::cache_row(a, b, kvh, pos);
    if (a.log2_block == 4) kvbfp::cast::encode_store<P, 16>(x, sub, live, mant, exps, row);
    else if (a.log2_block == 5) kvbfp::cast::encode_store<P, 32>(x, sub, live, mant, exps, row);
    else if (a.log2_block == 6) kvbfp::cast::encode_store<P, 64>(x, sub, live, mant, exps, row);
    else kvbfp::cast::encode_store<P, 128>(x, sub, live, mant, exps, row);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// Merges the 4 / RG wavefronts that hold the same heads over different tokens (wavefront w: heads 32 (w % RG) ..) and
// writes this split's partial result for `count` heads from head `h` on.  LDS: o_s, o_s2 [2][32][kD + 4] floats each, ml_s [4][32][3].
// The sums are relative to m_run, what is written to the largest score, m_top.
template <int RG>
__device__ __forceinline__ void merge_waves(const DecodeArgs& a, const kvbfp::spans::Span& span, int h, int count, float* o_s, float* o_s2, float* ml_s,
                                            int wave, int lane, const f32x16 (&o)[4], float m_run, float m_top, float l_run) {
    constexpr int kOStride = kD + 4;
    const int half = lane >> 5, l32 = lane & 31;
    auto row_of = [&](int w, int r) { return (w < 2 ? o_s : o_s2) + ((w & 1) * kRows + r) * kOStride; };
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *(f32x4*)(row_of(wave, l32) + 32 * ct + 8 * i + 4 * half) = f32x4{o[ct][4 * i], o[ct][4 * i + 1], o[ct][4 * i + 2], o[ct][4 * i + 3]};
    if (half == 0) {
        ml_s[(wave * kRows + l32) * 3] = m_run;
        ml_s[(wave * kRows + l32) * 3 + 1] = l_run;
        ml_s[(wave * kRows + l32) * 3 + 2] = m_top;
    }
    lds_only_barrier();
    // four channels per thread (a head's weights are worked out once for them): 64 heads over 300 tokens 21.4 us a call with
    // one, 15.0 with four; 32 heads over 4 x 3000 26.0 and 20.0
    for (int i = threadIdx.x; i < count * (kD / 4); i += kThreads) {
        const int g = i / (kD / 4), c = 4 * (i % (kD / 4));
        const int w0 = g / kRows, r = g % kRows;
        float m[4 / RG], M = -INFINITY;
#pragma unroll
        for (int t = 0; t < 4 / RG; ++t) {
            m[t] = ml_s[((w0 + t * RG) * kRows + r) * 3];
            M = fmaxf(M, ml_s[((w0 + t * RG) * kRows + r) * 3 + 2]);
        }
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        float lsum = 0.f;
#pragma unroll
        for (int t = 0; t < 4 / RG; ++t) {
            if (m[t] > -INFINITY) {
                const float f = exp2f(m[t] - M);
                const f32x4 x = *(const f32x4*)(row_of(w0 + t * RG, r) + c);
#pragma unroll
                for (int k = 0; k < 4; ++k) acc[k] = fmaf(f, x[k], acc[k]);
                lsum = fmaf(f, ml_s[((w0 + t * RG) * kRows + r) * 3 + 1], lsum);
            }
        }
        *(f32x4*)(a.part_o + span.row(h + g) * kD + c) = acc;
        if (c == 0) {
            float* ml = a.part_ml + span.row(h + g) * 2;
            ml[0] = M;
            ml[1] = lsum;
        }
    }
}

// P = mantissa bits; N16: blocks of 16 (a 16-byte chunk of 4-bit codes then spans two blocks).
// RG = groups of 32 heads per workgroup (2 or 4), 4 / RG wavefronts share the tokens of a tile; QL = bf16 limbs of the query.
// grid = (n_splits, H_kv * row_tiles, B), block = 256; a workgroup takes the heads of `groups` (<= RG) groups of 32,
// and every n_splits-th tile of TT tokens.
//
// The next tile is decoded into the other half of the LDS while this one is multiplied with, and the next probabilities are formed
// between the value products, so that the vector instructions of a wavefront fill the time of its own matrix instructions.
// Registers: with 8-bit mantissas, fp16 queries and more than 64 heads 4 of them are spilled.
template <int P, bool N16, int RG, int QL>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void decode_split_wide(DecodeArgs a, int dt, int row_tiles, int groups, float score_mul, float query_mul) {
    constexpr int kShift = P == 4 ? 7 : 3;             // decoded to bf16, values are value * 2^-kShift
    constexpr int TG = 4 / RG;                         // wavefronts that share the tokens of a tile
    constexpr int kLog2Tile = 6, TT = 1 << kLog2Tile;  // tokens per tile; every wavefront decodes 16 of them
    constexpr int CB = TT / 32 / TG;                   // blocks of 32 tokens per wavefront
    constexpr int kRowB = kD * P / 8;
    constexpr int kKeyChunks = P == 4 ? 1 : 2;         // 16-byte chunks of a key row per thread and pass
    constexpr int kValWords = P == 4 ? 1 : 2;          // dwords (8 channels) of a value row per thread
    // marks of a stage of 16 tokens: keys, values raised by kUp; a value byte above kOrdinary
    constexpr uint32_t kKeysUp = 1, kValuesUp = 2, kLarge = 4;
    constexpr int kKeyBytes = TT * 256, kValBytes = kD * TT * 2, kTileBytes = kKeyBytes + kValBytes;
    constexpr int kOStride = kD + 4;
    constexpr int kMerge = TG > 1 ? 2 * kRows * kOStride * 4 : 0;          // two wavefronts' outputs
    constexpr int kSmem = kTileBytes > kMerge ? kTileBytes : kMerge;
    static_assert(RG * kRows * 256 <= kSmem, "the raw queries of the set-up fit");
    __shared__ __align__(1024) uint8_t smem[kSmem];    // (two arrays: the compiler then knows that what it writes to one is not read from the other)
    __shared__ __align__(1024) uint8_t smem_odd[kSmem];
    __shared__ float ml_s[TG > 1 ? 4 * kRows * 3 : 1];
    __shared__ int perm_s[kD];
    __shared__ uint32_t marks_s[2];                    // of the tile in either half of the LDS: its four stages, one byte each

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int half = lane >> 5, l32 = lane & 31;
    kvbfp::spans::Span span;
    const int kvh = blockIdx.y / row_tiles, rt = blockIdx.y % row_tiles;
    const int s_first = rt * groups * kRows;                     // first virtual head of the workgroup
    const int s_count = min(groups * kRows, a.G - s_first);      // its heads
    if (!kvbfp::spans::take(a, kvbfp::spans::request_lengths(a, gridDim.z), kLog2Tile, span)) return;
    const int split = span.split, b = span.b;
    const int rg = wave % RG, tg = wave / RG;
    const int my_s = s_first + rg * kRows + l32;                 // this lane's head
    const bool active = rg * kRows < s_count;                    // wave-uniform
    const int h0 = kvh * a.G;
    const int64_t L = span.L;
    const int64_t t_first = (int64_t)split * TT;
    if (t_first >= L) {       // nothing cached in this split
        for (int i = tid; i < s_count * kD; i += kThreads)
            a.part_o[span.row(h0 + s_first + i / kD) * kD + i % kD] = 0.f;
        for (int i = tid; i < s_count; i += kThreads) {
            float* ml = a.part_ml + span.row(h0 + s_first + i) * 2;
            ml[0] = -INFINITY;
            ml[1] = 0.f;
        }
        return;
    }

    QueryRows<RG * kRows> query;
    query.request(a, b, kvh, s_first, s_count);

    // ---- packed rows of one tile, as loaded: this wavefront's 16 tokens
    const int log2_nb = 7 - a.log2_block;              // exponent bytes per row
    struct Raw {
        u32x4 k[kKeyChunks];
        uint32_t ke[2];
        uint32_t v[4][kValWords];
        uint32_t ve[4];
    };
    const int k_tok = lane >> 2, k_chunk = lane & 3;   // keys: token of the stage, 16-byte chunk (8-bit: and chunk + 4)
    const int v_quad = lane >> 4, v_word = lane & 15;  // values: tokens 4 v_quad .. + 3, channels 8 v_word .. + 7
    auto fetch = [&](const int64_t T0, Raw& r) {
        int64_t st = T0 + 16 * wave;               // first token of the stage, wave-uniform
        if (st >= L) st = (L - 1) & ~(int64_t)15;  // beyond the end: rows that are not used
        const int last = (int)min((int64_t)15, L - 1 - st);
        const int64_t row0 = kvbfp::cache_row(a, b, kvh, st);
        const uint8_t* __restrict__ km = a.k_mant + row0 * kRowB;
        const uint8_t* __restrict__ vm = a.v_mant + row0 * kRowB;
        const uint8_t* __restrict__ kx = a.k_exp + (row0 << log2_nb);
        const uint8_t* __restrict__ vx = a.v_exp + (row0 << log2_nb);
        // what follows from the lane is worked out here each time: held through the loop, it spills with two limbs of the query, and
        // the requests then wait for it (256 heads, fp16 I/O, 4 x 8192 tokens: 92 us a call)
        int l = lane;
        asm volatile("" : "+v"(l));
        const int chunk = l & 3, word = l & 15;
        const uint32_t ke_at0 = (uint32_t)((P == 4 ? 32 : 16) * chunk) >> a.log2_block;
        const uint32_t ke_at1 = (uint32_t)(64 + 16 * chunk) >> a.log2_block;        // (8 bits)
        const uint32_t ve_at = (uint32_t)(8 * word) >> a.log2_block;
        const uint32_t kr = (uint32_t)min(l >> 2, last);
#pragma unroll
        for (int i = 0; i < kKeyChunks; ++i)
            r.k[i] = __builtin_nontemporal_load((const u32x4*)(km + (kr * kRowB + chunk * 16 + i * 64)));
        if (P == 4 && N16) {
            r.ke[0] = *(const uint16_t*)(kx + ((kr << log2_nb) + ke_at0));
        } else {
            r.ke[0] = kx[(kr << log2_nb) + ke_at0];
            if (P == 8) r.ke[1] = kx[(kr << log2_nb) + ke_at1];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t vr = (uint32_t)min(4 * (l >> 4) + i, last);
            if constexpr (P == 4) {
                r.v[i][0] = __builtin_nontemporal_load((const uint32_t*)(vm + (vr * kRowB + word * 4)));
            } else {
                const u32x2 w = __builtin_nontemporal_load((const u32x2*)(vm + (vr * kRowB + word * 8)));
                r.v[i][0] = w[0];
                r.v[i][kValWords - 1] = w[1];
            }
            r.ve[i] = vx[(vr << log2_nb) + ve_at];
        }
    };
    auto key_byte = [&](const Raw& r, int i) -> uint32_t {       // of the blocks of this lane's key chunk(s)
        if constexpr (P == 4) return !N16 ? r.ke[0] : i ? r.ke[0] >> 8 : r.ke[0] & 0xFFu;
        else return r.ke[i];
    };
    // Where things lie in a tile's half of the LDS.  Keys: [TT tokens][16 groups of 8 channels], 16 bytes each, the group's place
    // exchanged with token % 16 so that the reads of 16 neighbouring tokens hit different banks.  Values, behind them: [128
    // channels][TT / 8 groups of 8 tokens], the four tokens of a quad side by side per channel; quads 0 and 2 of 16 tokens make the
    // first 16 bytes and 1 and 3 the second, the order in which S^T leaves them in the two halves of a wavefront; row and
    // place exchanged with the channel's bits, at(ch, place) = (ch ^ (ch >> 6 & 1)) * 128 + ((place ^ ch ^ (ch >> 3)) & 7) * 16, so
    // that neither the writes (equal bits 0-2) nor the reads (16 neighbouring channels) meet in a bank.  All of it is exclusive
    // ors of a lane's base with constants; the bases are made opaque tile by tile, which leaves the compiler the half of the
    // LDS and the block of channels as immediate offsets and no second set of addresses to hold in registers.
    const int tok = 16 * wave + k_tok;
    uint32_t key_put = tok * 256 + (((4 * (P == 4 ? k_chunk : 0) + 2 * (P == 4 ? 0 : k_chunk)) ^ (tok & 15)) * 16);      // group d (8 bits: 8 i + e): ^ 16 d
    uint32_t val_put = kKeyBytes + (8 * v_word + (v_word >> 3)) * 128 + (((2 * wave + (v_quad & 1)) ^ (v_word & 7)) * 16) + (v_quad >> 1) * 8;   // channel c of 8: ^ 144 c
    uint32_t key_get = (tg * CB * 32 + l32) * 256 + ((half ^ (l32 & 15)) * 16);                                         // products m: ^ 32 m, block of tokens: + 8192
    // step n, block of channels ct: ^ 32 (n ^ 2 (ct & 1)) ^ 128 (ct >> 1), + 4096 ct
    uint32_t val_get = kKeyBytes + l32 * 128 + (((4 * tg * (CB & 1) + half) ^ (l32 & 7) ^ (l32 >> 3)) * 16);
    // keys to bf16 in LDS, a quarter of what this lane holds of them
    auto decode_keys = [&](const Raw& r, uint8_t* const tile, auto quarter) {
        constexpr int d = decltype(quarter)::value;
        if constexpr (P == 4) {
            uint32_t q[4];
            unpack8_p4(r.k[0][d], __uint_as_float(key_byte(r, d >> 1) << 23), q);
            *(u32x4*)(tile + (key_put ^ (16 * d))) = u32x4{q[0], q[1], q[2], q[3]};
        } else {
            constexpr int i = (d >> 1) * (kKeyChunks - 1), e = d & 1;
            float x[4], y[4];
            unpack4_p8(r.k[i][2 * e], r.ke[i] << 23, x);
            unpack4_p8(r.k[i][2 * e + 1], r.ke[i] << 23, y);
            const u32x4 w = {pack_hi(__float_as_uint(x[0]), __float_as_uint(x[1])), pack_hi(__float_as_uint(x[2]), __float_as_uint(x[3])),
                             pack_hi(__float_as_uint(y[0]), __float_as_uint(y[1])), pack_hi(__float_as_uint(y[2]), __float_as_uint(y[3]))};
            *(u32x4*)(tile + (key_put ^ (16 * (8 * i + e)))) = w;
        }
    };
    auto put = [&](uint8_t* const tile, const int c, const uint32_t t01, const uint32_t t23) {      // values; c = channel % 8
        *(u32x2*)(tile + (val_put ^ (144 * c))) = u32x2{t01, t23};
    };
    auto put_pairs = [&](uint8_t* const tile, const uint32_t (&q)[4][4]) {                          // as unpack8_p4 leaves them
#pragma unroll
        for (int x = 0; x < 4; ++x) {              // pair x: channels (0,2), (4,6), (1,3), (5,7)
            const int c = x < 2 ? 4 * x : 4 * (x - 2) + 1;
            put(tile, c, pack_lo(q[0][x], q[1][x]), pack_lo(q[2][x], q[3][x]));
            put(tile, c + 2, pack_hi(q[0][x], q[1][x]), pack_hi(q[2][x], q[3][x]));
        }
    };

    // the current token (one row tile only): by the wavefront that decodes its row
    if (a.k_new != nullptr && (int)(((L - 1) / TT) % span.n) == split && (int)(((L - 1) >> 4) & 3) == wave)
        append_row<P>(a, dt, b, kvh, lane, L - 1);

    Raw raw;
    fetch(t_first, raw);

    bf16x8 q_op[QL][8];
    const float mul = score_mul * query.template build<P, QL>(a, dt, s_count, rg * kRows, smem, perm_s, query_mul, [](int m, int h) { return 2 * m + h; }, q_op);

    const int64_t lim = L - kvbfp::hidden_tokens(a, my_s);         // this head sees tokens below
    const int64_t all_see = L - (a.n_q_tokens - 1);                // every head does
    float m_run = -INFINITY, l_run = 0.f;
    f32x16 o[4];
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[ct][i] = 0.f;

    const int64_t step = (int64_t)span.n * TT;
    const int my_tok0 = tg * CB * 32;                              // first token of this wavefront inside a tile
    // S^T of 32 tokens x 32 heads; register i of a block: token 8 (i / 4) + 4 half + i % 4.  meanwhile(m), m = 0..7: vector
    // instructions for the time of the m-th products (the barriers keep the compiler from moving them behind the last).
    auto scores = [&](const uint8_t* const tile, f32x16 (&s)[CB], auto&& meanwhile) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int i = 0; i < 16; ++i) s[cb][i] = 0.f;
        bf16x8 ka[2][CB];
        auto read = [&](const int m) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) ka[m & 1][cb] = *(const bf16x8*)(tile + (key_get ^ (32 * m)) + 8192 * cb);
        };
        read(0);
        static_for<8>([&](auto at) {
            constexpr int m = decltype(at)::value;
            if (m < 7) read(m + 1);
#pragma unroll
            for (int l = 0; l < QL; ++l)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) s[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[m & 1][cb], q_op[l][m], s[cb], 0, 0, 0);
            meanwhile(at);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    auto hide = [&](const int64_t T0, f32x16 (&s)[CB]) {           // what a head must not see
        const int sees = (int)min((int64_t)TT, max((int64_t)0, lim - T0)) - my_tok0 - 4 * half;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int i = 0; i < 16; ++i) s[cb][i] = 32 * cb + 8 * (i >> 2) + (i & 3) < sees ? s[cb][i] : -INFINITY;
    };
    auto value_get = [&](const int n, const int ct) { return (val_get ^ (32 * (n ^ (2 * (ct & 1)))) ^ (128 * (ct >> 1))) + 4096 * ct; };
    auto largest = [&](const f32x16 (&s)[CB]) {                    // of this lane's head; -inf only if it sees none of the tile
        float tmax = s[0][0];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int i = 0; i < 16; ++i) tmax = fmaxf(tmax, s[cb][i]);
        return both_halves_max(tmax) * mul;
    };

    int64_t T0 = t_first;
    // A tile's exponent bytes, made operands of the conversions in place (see ExpRange), and what its stage is marked with.  Returns this
    // lane's blocks that were converted at kDown fewer: keys bits 0, 1, values 4 + token.
    auto mark = [&](Raw& r, const int at) -> uint32_t {
        using R = ExpRange<P>;
        const uint32_t ke[2] = {key_byte(r, 0), key_byte(r, 1)};
        const uint32_t v_top = max(max(r.ve[0], r.ve[1]), max(r.ve[2], r.ve[3])), top = max(v_top, max(ke[0], ke[1]));
        const uint32_t low = min(min(min(r.ve[0], r.ve[1]), min(r.ve[2], r.ve[3])), min(ke[0], ke[1]));
        uint32_t marks = 0, raise = 0;                 // marks: wave-uniform
        if (__builtin_amdgcn_ballot_w64(top > (uint32_t)kOrdinary || low <= 2u) != 0) {      // (also where a block is all zero)
            const uint32_t up_k = __builtin_amdgcn_ballot_w64(R::tiny(ke[0]) || R::tiny(ke[1])) != 0 ? R::kUp : 0;
            const uint32_t up_v = __builtin_amdgcn_ballot_w64(R::tiny(r.ve[0]) || R::tiny(r.ve[1]) || R::tiny(r.ve[2]) || R::tiny(r.ve[3])) != 0 ? R::kUp : 0;
            marks = (up_k ? kKeysUp : 0u) | (up_v ? kValuesUp : 0u) | (__builtin_amdgcn_ballot_w64(v_top > (uint32_t)kOrdinary) != 0 ? kLarge : 0u);
            raise = (R::high(ke[0], up_k) ? 1u : 0u) | (R::high(ke[1], up_k) ? 2u : 0u);
            if constexpr (P == 4) {
                r.ke[0] = N16 ? (R::operand(ke[0], up_k) | (R::operand(ke[1], up_k) << 8)) : R::operand(ke[0], up_k);
            } else {
                r.ke[0] = R::operand(ke[0], up_k);
                r.ke[1] = R::operand(ke[1], up_k);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                raise |= R::high(r.ve[i], up_v) ? 16u << i : 0u;
                r.ve[i] = R::operand(r.ve[i], up_v);
            }
        }
        if (lane == 0) ((uint8_t*)&marks_s[at])[wave] = (uint8_t)marks;
        return raise;
    };
    // A quarter of the keys (pieces 0-3) or values (4-7) to bf16 in LDS.  Values wait in q for the rest of their words: 4 bits,
    // pairs of channels by token, stored by finish(); 8 bits, channels of tokens 0 and 1 of a word, stored with those of tokens 2 and 3.
    struct Values {
        uint32_t q[4][P == 4 ? 4 : 1];
        u32x4 two;
    };
    auto decode = [&](const Raw& r, uint8_t* const tile, Values& v, auto part) {
        constexpr int piece = decltype(part)::value;
        if constexpr (piece < 4) {
            decode_keys(r, tile, part);
        } else if constexpr (P == 4) {
            unpack8_p4(r.v[piece - 4][0], __uint_as_float(r.ve[piece - 4] << 23), v.q[piece - 4]);
        } else {
            constexpr int w = (piece - 4) >> 1, h = (piece - 4) & 1;
            float x[4], y[4];
            unpack4_p8(r.v[2 * h][w], r.ve[2 * h] << 23, x);
            unpack4_p8(r.v[2 * h + 1][w], r.ve[2 * h + 1] << 23, y);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t two = pack_hi(__float_as_uint(x[c]), __float_as_uint(y[c]));
                if constexpr (h == 0) v.two[c] = two;
                else put(tile, 4 * w + c, v.two[c], two);
            }
        }
    };
    auto finish = [&](uint8_t* const tile, const Values& v, const uint32_t raise) {
        if constexpr (P == 4) put_pairs(tile, v.q);
        if (__builtin_amdgcn_ballot_w64(raise != 0) != 0) {        // what this lane wrote
#pragma unroll 1
            for (int g = 0; g < 4; ++g) {
                const bool up = (raise >> (g >> 1)) & 1u;
                u32x4* const at = (u32x4*)(tile + (key_put ^ (16 * (P == 4 ? g : 8 * (g >> 1) + (g & 1)))));
                const u32x4 w = *at;
                *at = u32x4{raise_pair(w[0], up, up), raise_pair(w[1], up, up), raise_pair(w[2], up, up), raise_pair(w[3], up, up)};
            }
#pragma unroll 1
            for (int c = 0; c < 8; ++c) {
                u32x2* const at = (u32x2*)(tile + (val_put ^ (144 * c)));
                const u32x2 w = *at;
                *at = u32x2{raise_pair(w[0], raise & 16u, raise & 32u), raise_pair(w[1], raise & 64u, raise & 128u)};
            }
        }
    };
    auto decode_all = [&](Raw& r, uint8_t* const tile, const int at) {
        const uint32_t raise = mark(r, at);
        Values v;
        static_for<8>([&](auto i) { decode(r, tile, v, i); });
        finish(tile, v, raise);
    };
    // sums relative to m_run; the largest score may exceed it by kSlack
    float m_top = -INFINITY;
    uint32_t seen = 0;                                             // marks of the tiles so far
    auto raise_reference = [&](const float tmax, const uint32_t marks) {
        m_top = fmaxf(m_top, tmax);
        seen |= marks;
        if (__builtin_amdgcn_ballot_w64(m_top > m_run + ((seen & (0x01010101u * kLarge)) ? 0.f : kSlack)) != 0) {
            const float alpha = exp2_raw(m_run - (m_top == -INFINITY ? 0.f : m_top));
            l_run *= alpha;
            m_run = m_top;
#pragma unroll
            for (int ct = 0; ct < 4; ++ct) o[ct] *= alpha;
        }
    };
    // O^T += V^T P^T, 16 tokens a step.  A probability is three bf16 limbs, all of its 24 bits at every size (a token whose values
    // are zero takes any weight, and what is left is the sum of the others).
    auto products = [&](const uint8_t* const tile, f32x16 (&s)[CB], const uint32_t marks) {
        const float m_p = (m_run == -INFINITY ? 0.f : m_run) - (float)kShift;      // probabilities carry 2^kShift
        u32x4 limb[2][3];
        bf16x8 va[4];
        float psum = 0.f;
        // of step n: values of a stage that was raised by kUp take probabilities that are lower by as much
        auto up_of = [&](const int n) { return (marks >> (8 * (my_tok0 / 16 + n))) & kValuesUp; };
        float part, m_n;
        // two of the eight probabilities of step n
        auto limbs = [&](const int n, const int j) {
            if (j == 0) {
                part = 0.f;
                m_n = m_p + (up_of(n) ? (float)ExpRange<P>::kUp : 0.f);
            }
            float x = exp2_raw(fmaf(s[n >> 1][8 * (n & 1) + 2 * j], mul, -m_n));
            float y = exp2_raw(fmaf(s[n >> 1][8 * (n & 1) + 2 * j + 1], mul, -m_n));
            part += x;
            part += y;
#pragma unroll
            for (int l = 0; l < 3; ++l) {
                limb[n & 1][l][j] = pack_hi(__float_as_uint(x), __float_as_uint(y));
                x -= __uint_as_float(__float_as_uint(x) & 0xFFFF0000u);
                y -= __uint_as_float(__float_as_uint(y) & 0xFFFF0000u);
            }
            if (j == 3) psum = fmaf(part, up_of(n) ? (float)(1 << ExpRange<P>::kUp) : 1.f, psum);
        };
        auto read = [&](const int n, const int ct) { va[ct] = *(const bf16x8*)(tile + value_get(n, ct)); };
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) read(0, ct);
#pragma unroll
        for (int j = 0; j < 4; ++j) limbs(0, j);
#pragma unroll
        for (int n = 0; n < 2 * CB; ++n) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {          // three products of a pair of blocks of channels, and vector instructions of the next step for their time
#pragma unroll
                for (int k = 3 * (j & 1); k < 3 * (j & 1) + 3; ++k) {
                    const int ct = (j & 2) + (k & 1);
                    o[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[ct], __builtin_bit_cast(bf16x8, limb[n & 1][k >> 1]), o[ct], 0, 0, 0);
                }
                if (n + 1 < 2 * CB) {
                    if (j & 1) {
                        read(n + 1, j & 2);
                        read(n + 1, (j & 2) + 1);
                    }
                    limbs(n + 1, j);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        l_run += psum;
    };

    decode_all(raw, smem, 0);
    if (T0 + step < L) fetch(T0 + step, raw);
    // One tile from half AT of the LDS, the next one decoded into the other.  False: there is none.
    auto tile_of = [&](auto AT) -> bool {
        constexpr int at = decltype(AT)::value;
        uint8_t* const tile = at ? smem_odd : smem;
        uint8_t* const next = at ? smem : smem_odd;
        asm volatile("" : "+v"(key_put), "+v"(val_put), "+v"(key_get), "+v"(val_get));
        lds_only_barrier();
        if (T0 >= L) return false;
        if (active) {
            const uint32_t marks = __builtin_amdgcn_readfirstlane(marks_s[at]);
            f32x16 s[CB];
            Values v;
            const uint32_t raise = mark(raw, at ^ 1);
            scores(tile, s, [&](auto m) { decode(raw, next, v, m); });    // (behind the last tile: once more what it holds, for nobody)
            finish(next, v, raise);
            if (T0 + 2 * step < L) fetch(T0 + 2 * step, raw);
            if (marks & (0x01010101u * kKeysUp)) {                 // of the stage of 16 tokens a register's token lies in
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) s[cb][i] *= ((marks >> (8 * (my_tok0 / 16 + 2 * cb + (i >> 3)))) & kKeysUp) ? 0.25f : 1.f;
            }
            if (T0 + TT > all_see) hide(T0, s);
            raise_reference(largest(s), marks);
            products(tile, s, marks);
        } else if (T0 + step < L) {
            decode_all(raw, next, at ^ 1);
            if (T0 + 2 * step < L) fetch(T0 + 2 * step, raw);
        }
        T0 += step;
        return true;
    };
    while (tile_of(std::integral_constant<int, 0>{}) && tile_of(std::integral_constant<int, 1>{})) {}
    if constexpr (TG == 1) raise_reference(-INFINITY, kLarge);     // (the merge of wavefronts does it otherwise)
    l_run *= 1.0f / (float)(1 << kShift);
    l_run += other_half(l_run);

    // ---- partial result of this split: registers 4i .. 4i+3 of block ct are channels 32 ct + 8 i + 4 half ..
    if constexpr (TG == 1) {
        if (!active || my_s - s_first >= s_count) return;
        float* const po = a.part_o + span.row(h0 + my_s) * kD;
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *(f32x4*)(po + 32 * ct + 8 * i + 4 * half) = f32x4{o[ct][4 * i], o[ct][4 * i + 1], o[ct][4 * i + 2], o[ct][4 * i + 3]};
        if (half == 0) {
            float* ml = a.part_ml + span.row(h0 + my_s) * 2;
            ml[0] = m_run;
            ml[1] = l_run;
        }
    } else {       // merge the wavefronts that shared the tokens
        merge_waves<RG>(a, span, h0 + s_first, s_count, (float*)smem, (float*)smem_odd, ml_s, wave, lane, o, m_run, m_top, l_run);
    }
}

// Up to 32 heads: the cache is read once, so the pass is bound by memory, and what counts is how much of it is on its way.
// The four wavefronts take 32 tokens each of a tile of 128 and share nothing until the merge: keys go from memory to
// registers, where they are the first operand of S^T = K Q^T as they are decoded (a lane holds half of a token's row);
// values are transposed through 8 KB of LDS of the wavefront's own.  No barrier in the loop, and kDepth tiles per wavefront
// in flight (one for 8-bit mantissas, whose rows take twice the registers, and for fp16 queries, whose second limb takes 32:
// with two those variants spill, 8 bits 76 -> 68 us, 12 heads with fp16 I/O over 8 x 12000 tokens 46.1 -> 42.4 us).
template <int P, int N, int QL>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void decode_split_few(DecodeArgs a, int dt, float score_mul, float query_mul) {
    constexpr int kShift = P == 4 ? 7 : 3;             // of the values; keys are value * 2^-(kShift - kKeyUp)
    constexpr int kDepth = P == 8 || QL == 2 ? 1 : 2;
    constexpr int NB = kD / N;
    constexpr int kRowB = kD * P / 8;
    constexpr int kKeyChunks = kRowB / 32;             // 16-byte chunks of a key row per lane (every other one)
    constexpr int kValWords = P / 4;                   // dwords (8 channels) of a value row per lane
    constexpr int TT = 32;                             // tokens per wavefront and tile
    constexpr int kOStride = kD + 4;
    constexpr int kMerge = 4 * kRows * kOStride * 4 + 4 * kRows * 3 * 4;
    __shared__ __align__(16) uint8_t smem[kMerge];     // queries, then the transposed values (8 KB per wavefront), then the merge
    __shared__ int perm_s[kD];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int half = lane >> 5, l32 = lane & 31;
    kvbfp::spans::Span span;
    if (!kvbfp::spans::take(a, kvbfp::spans::request_lengths(a, gridDim.z), 7, span)) return;
    const int split = span.split, kvh = blockIdx.y, b = span.b;
    const int h0 = kvh * a.G;
    const int64_t L = span.L;
    if ((int64_t)split * 128 >= L) {       // nothing cached in this split
        for (int i = tid; i < a.G * kD; i += kThreads) a.part_o[span.row(h0 + i / kD) * kD + i % kD] = 0.f;
        if (tid < a.G) {
            float* ml = a.part_ml + span.row(h0 + tid) * 2;
            ml[0] = -INFINITY;
            ml[1] = 0.f;
        }
        return;
    }
    const int64_t t_first = (int64_t)split * 128 + wave * TT;
    const int64_t step = (int64_t)span.n * 128;
    QueryRows<kRows> query;
    query.request(a, b, kvh, 0, a.G);

    // Plane rows of the two 16-token stages of the tile at T (wave-uniform).  Paged: the page numbers are requested a tile
    // ahead by the lanes (an ordinary load, so that it queues with the rows and is not waited for by itself).
    const int64_t unit = ((int64_t)b * a.H_kv + kvh) * a.max_seq;
    int page_next = 0;
    auto request_pages = [&](const int64_t T) {
        if (a.block_table && T < L) {
            int64_t t = T + 16 * ((lane >> 4) & 1);
            if (t >= L) t = L - 1;
            page_next = a.block_table[(int64_t)b * a.table_stride + (t >> a.log2_page)];
        }
    };
    auto stage_row = [&](const int64_t T, const int st) -> int64_t {
        const int64_t t = T + 16 * st;
        if (!a.block_table) return unit + t;
        int page = __builtin_amdgcn_readlane(page_next, 16 * st);
        page = page < 0 ? 0 : (page >= a.n_pages ? a.n_pages - 1 : page);
        return (((int64_t)page * a.H_kv + kvh) << a.log2_page) + (t & (((int64_t)1 << a.log2_page) - 1));
    };
    // (exponents as loaded: keys, all bytes of the lane's row; values, the byte of this lane's channels per token)
    struct Raw {
        u32x4 k[kKeyChunks];
        uint32_t ke[N == 16 ? 2 : 1];
        uint32_t v[2][4][kValWords];
        uint32_t ve[2][4];
    };
    const int v_quad = lane >> 4, v_word = lane & 15;
    auto load_keys = [&](Raw& r, const uint8_t* km, const uint8_t* kx) {       // a lane's row
#pragma unroll
        for (int i = 0; i < kKeyChunks; ++i) r.k[i] = __builtin_nontemporal_load((const u32x4*)(km + 32 * i));
        if constexpr (N == 16) {
            const u32x2 e = *(const u32x2*)kx;
            r.ke[0] = e[0];
            r.ke[N == 16 ? 1 : 0] = e[1];
        } else if constexpr (N == 32) {
            r.ke[0] = *(const uint32_t*)kx;
        } else if constexpr (N == 64) {
            r.ke[0] = *(const uint16_t*)kx;
        } else {
            r.ke[0] = *kx;
        }
    };
    auto load_value = [&](Raw& r, const int st, const int i, const uint8_t* vm, const uint8_t* vx, const uint32_t vr) {
        if constexpr (P == 4) {
            r.v[st][i][0] = __builtin_nontemporal_load((const uint32_t*)(vm + (vr * kRowB + v_word * 4)));
        } else {
            const u32x2 w = __builtin_nontemporal_load((const u32x2*)(vm + (vr * kRowB + v_word * 8)));
            r.v[st][i][0] = w[0];
            r.v[st][i][kValWords - 1] = w[1];
        }
        r.ve[st][i] = vx[vr * NB + (8 * v_word) / N];
    };
    auto fetch = [&](const int64_t T, Raw& r) {        // T < L; requests the pages of the tile after it
        const int64_t row0 = stage_row(T, 0);
        const bool two = T + 16 < L;                   // wave-uniform
        const int64_t row1 = two ? stage_row(T, 1) : row0;
        request_pages(T + step);
        const int last0 = (int)min((int64_t)15, L - 1 - T), last1 = two ? (int)min((int64_t)15, L - 1 - (T + 16)) : last0;
        const int64_t kr = (l32 >= 16 ? row1 : row0) + min(l32 & 15, l32 >= 16 ? last1 : last0);
        load_keys(r, a.k_mant + kr * kRowB + half * 16, a.k_exp + kr * NB);
#pragma unroll
        for (int st = 0; st < 2; ++st) {
            const uint8_t* __restrict__ vm = a.v_mant + (st ? row1 : row0) * kRowB;
            const uint8_t* __restrict__ vx = a.v_exp + (st ? row1 : row0) * NB;
#pragma unroll
            for (int i = 0; i < 4; ++i) load_value(r, st, i, vm, vx, (uint32_t)min(4 * v_quad + i, st ? last1 : last0));
        }
    };
    // scale operands (only the exponent field counts) of the 16-byte key chunk i, of its blocks of 16, of a value row
    auto key_exp = [&](const Raw& r, const int i, const int sub) -> uint32_t {      // byte in the exponent field
        const int ch = (P == 4 ? 32 : 16) * 2 * i + 16 * sub;                      // first channel for half 0
        constexpr int kHalf = P == 4 ? 32 : 16;                                    // half 1: that many channels on
        if constexpr (N == 128) return r.ke[0] << 23;
        const int at0 = ch / N, at1 = (ch + kHalf) / N;                            // constants once unrolled
        const uint32_t w = r.ke[N == 16 ? at0 / 4 : 0];                            // (at1 never crosses the dword)
        const int sh = half ? 8 * (at1 & 3) : 8 * (at0 & 3);
        return __builtin_amdgcn_alignbit(w, w, (uint32_t)((sh + 32 - 23) & 31));
    };

    // the current token: by the wavefront whose tile holds it
    if (a.k_new != nullptr && (int)(((L - 1) >> 7) % span.n) == split && (int)(((L - 1) >> 5) & 3) == wave)
        append_row<P>(a, dt, b, kvh, lane, L - 1);

    Raw raw[kDepth];
    request_pages(t_first);
#pragma unroll
    for (int d = 0; d < kDepth; ++d)
        if (t_first + d * step < L) fetch(t_first + d * step, raw[d]);

    // MFMA m multiplies the 8 channels of key group group_of(m, half)
    auto group_of = [](int m, int h) { return P == 4 ? 8 * (m >> 2) + 4 * h + (m & 3) : 4 * (m >> 1) + 2 * h + (m & 1); };
    bf16x8 q_op[QL][8];
    const float mul = score_mul * query.template build<P, QL>(a, dt, a.G, 0, smem, perm_s, query_mul, group_of, q_op);

    // [128 channels][4 groups of 8 tokens], row and place exchanged with the channel's bits so that neither the writes (equal
    // bits 0-2) nor the reads (16 neighbouring channels) meet in a bank
    uint8_t* const v_lds = smem + wave * (kD * TT * 2);
    auto value_at = [](int ch, int place) { return (ch ^ ((ch >> 3) & 3)) * (TT * 2) + ((place ^ (((ch >> 2) ^ (ch >> 5)) & 3)) * 16); };
    const int64_t lim = L - kvbfp::hidden_tokens(a, l32);
    const int64_t all_see = L - (a.n_q_tokens - 1);
    float m_run = -INFINITY, l_run = 0.f;
    f32x16 o[4];
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[ct][i] = 0.f;

    float m_top = -INFINITY, slack = kSlack;                       // 4 bits: see kSlack
    auto raise_reference = [&] {
        if (__builtin_amdgcn_ballot_w64(m_top > m_run + slack) != 0) {
            const float alpha = exp2_raw(m_run - (m_top == -INFINITY ? 0.f : m_top));
            l_run *= alpha;
            m_run = m_top;
#pragma unroll
            for (int ct = 0; ct < 4; ++ct) o[ct] *= alpha;
        }
    };
    auto tile = [&](const int64_t T0, Raw& r) {
        uint32_t v_top = 0;
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int i = 0; i < 4; ++i) v_top = max(v_top, r.ve[st][i]);
        if (__builtin_amdgcn_ballot_w64(v_top > kOrdinary) != 0) slack = 0.f;
        // ---- values to LDS, the four tokens of a quad side by side per channel; quads 0 and 2 of a stage make its first 16
        // bytes, 1 and 3 the second (the order in which S^T leaves the tokens)
#pragma unroll
        for (int st = 0; st < 2; ++st) {
            const int place = 2 * st + (v_quad & 1);
            auto put = [&](const int c, const uint32_t t01, const uint32_t t23) {
                const int ch = 8 * v_word + c;
                *(u32x2*)(v_lds + value_at(ch, place) + (v_quad >> 1) * 8) = u32x2{t01, t23};
            };
            if constexpr (P == 4) {
                uint32_t q[4][4];
#pragma unroll
                for (int i = 0; i < 4; ++i) unpack8_p4(r.v[st][i][0], __uint_as_float(r.ve[st][i] << 23), q[i]);
#pragma unroll
                for (int x = 0; x < 4; ++x) {          // pair x: channels (0,2), (4,6), (1,3), (5,7)
                    const int c = x < 2 ? 4 * x : 4 * (x - 2) + 1;
                    put(c, pack_lo(q[0][x], q[1][x]), pack_lo(q[2][x], q[3][x]));
                    put(c + 2, pack_hi(q[0][x], q[1][x]), pack_hi(q[2][x], q[3][x]));
                }
            } else {
#pragma unroll
                for (int w = 0; w < kValWords; ++w) {
                    float x[4][4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) unpack4_p8(r.v[st][i][w], r.ve[st][i] << 23, x[i]);
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        put(4 * w + c, pack_hi(__float_as_uint(x[0][c]), __float_as_uint(x[1][c])), pack_hi(__float_as_uint(x[2][c]), __float_as_uint(x[3][c])));
                }
            }
        }
        // ---- S^T.  The keys' exponent bytes are raised by kKeyUp: bf16 then holds the smallest blocks too (bytes 1 and 2).
        // Where a byte of the tile has no room for that, all of them stay as they are and the scores make up for it
        // (the look at them costs 1 % of the instructions).
        constexpr uint32_t kRaise = kKeyUp * 0x01010101u;
        bool above = false;
#pragma unroll
        for (int i = 0; i < (N == 16 ? 2 : 1); ++i)
            above |= (((r.ke[i] & 0x7F7F7F7Fu) + (0x7Fu - (ExpRange<P>::kTop - kKeyUp - 128u)) * 0x01010101u) & r.ke[i] & 0x80808080u) != 0;
        const bool raised = __builtin_amdgcn_ballot_w64(above) == 0;
        if (raised) {
#pragma unroll
            for (int i = 0; i < (N == 16 ? 2 : 1); ++i) r.ke[i] += kRaise;
        }
        f32x16 s;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            u32x4 kw;
            if constexpr (P == 4) {
                uint32_t q[4];
                unpack8_p4(r.k[m >> 2][m & 3], __uint_as_float(key_exp(r, m >> 2, N == 16 ? (m & 3) >> 1 : 0)), q);
                kw = u32x4{q[0], q[1], q[2], q[3]};
            } else {
                float x[4], y[4];
                unpack4_p8(r.k[m >> 1][2 * (m & 1)], key_exp(r, m >> 1, 0), x);
                unpack4_p8(r.k[m >> 1][2 * (m & 1) + 1], key_exp(r, m >> 1, 0), y);
                kw = u32x4{pack_hi(__float_as_uint(x[0]), __float_as_uint(x[1])), pack_hi(__float_as_uint(x[2]), __float_as_uint(x[3])),
                           pack_hi(__float_as_uint(y[0]), __float_as_uint(y[1])), pack_hi(__float_as_uint(y[2]), __float_as_uint(y[3]))};
            }
            const bf16x8 ka = __builtin_bit_cast(bf16x8, kw);
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, q_op[0][m], s, 0, 0, 0);
            if (QL == 2) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, q_op[QL - 1][m], s, 0, 0, 0);
        }
        if (!raised) {
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] *= (float)(1 << kKeyUp);
        }
        // the rows are used up: the tile kDepth ahead is requested into the same registers
        if (T0 + kDepth * step < L) {
            fetch(T0 + kDepth * step, r);
        }
        if (T0 + TT > all_see) {                       // register i: token 8 (i / 4) + 4 half + i % 4
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = T0 + 8 * (i >> 2) + 4 * half + (i & 3) < lim ? s[i] : -INFINITY;
        }
        // ---- online softmax, base 2
        float tmax = s[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) tmax = fmaxf(tmax, s[i]);
        float alpha = 1.f;
        if constexpr (P == 4) {
            m_top = fmaxf(m_top, both_halves_max(tmax) * mul);         // -inf only if this head has seen no token
            raise_reference();
        } else {                                             // (bound by memory: the branch there costs as much as it saves)
            tmax = fmaxf(tmax, other_half(tmax)) * mul;
            const float m_new = fmaxf(m_run, tmax);
            alpha = exp2_raw(m_run - (m_new == -INFINITY ? 0.f : m_new));
            m_run = m_new;
        }
        const float m_p = (m_run == -INFINITY ? 0.f : m_run) - (float)kShift;     // probabilities carry 2^kShift
        uint32_t p_hi[8], p_lo[8];
        float psum = 0.f;
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
            const float p0 = exp2_raw(fmaf(s[i], mul, -m_p));
            const float p1 = exp2_raw(fmaf(s[i + 1], mul, -m_p));
            psum += p0;
            psum += p1;
            p_hi[i / 2] = pack_hi(__float_as_uint(p0), __float_as_uint(p1));
            bf16x2 lo;
            lo[0] = (__bf16)(p0 - __uint_as_float(__float_as_uint(p0) & 0xFFFF0000u));
            lo[1] = (__bf16)(p1 - __uint_as_float(__float_as_uint(p1) & 0xFFFF0000u));
            p_lo[i / 2] = bits(lo);
        }
        if constexpr (P == 4) {
            l_run += psum;
        } else {
            l_run = l_run * alpha + psum;
            if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
                for (int ct = 0; ct < 4; ++ct) o[ct] *= alpha;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");     // the values were written by other lanes of this wavefront
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // ---- O^T += V^T P^T
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const bf16x8 ph = __builtin_bit_cast(bf16x8, u32x4{p_hi[4 * kk], p_hi[4 * kk + 1], p_hi[4 * kk + 2], p_hi[4 * kk + 3]});
            const bf16x8 pl = __builtin_bit_cast(bf16x8, u32x4{p_lo[4 * kk], p_lo[4 * kk + 1], p_lo[4 * kk + 2], p_lo[4 * kk + 3]});
#pragma unroll
            for (int ct = 0; ct < 4; ct += 2) {        // (two blocks in turn: no product waits for the one before it)
                const bf16x8 v0 = *(const bf16x8*)(v_lds + value_at(32 * ct + l32, 2 * kk + half));
                const bf16x8 v1 = *(const bf16x8*)(v_lds + value_at(32 * ct + 32 + l32, 2 * kk + half));
                o[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v0, ph, o[ct], 0, 0, 0);
                o[ct + 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v1, ph, o[ct + 1], 0, 0, 0);
                o[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v0, pl, o[ct], 0, 0, 0);
                o[ct + 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v1, pl, o[ct + 1], 0, 0, 0);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");     // the next tile overwrites them
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    for (int64_t T0 = t_first; T0 < L; T0 += kDepth * step) {
#pragma unroll
        for (int d = 0; d < kDepth; ++d)
            if (T0 + d * step < L) tile(T0 + d * step, raw[d]);
    }
    if constexpr (P == 8) m_top = m_run;
    l_run = (l_run + other_half(l_run)) * (1.0f / (float)(1 << kShift));

    // ---- merge the four wavefronts
    lds_only_barrier();
    merge_waves<1>(a, span, h0, a.G, (float*)smem, (float*)smem + 2 * kRows * kOStride, (float*)smem + 4 * kRows * kOStride, wave, lane, o, m_run, m_top, l_run);
}

template <int P, bool N16, int RG>
void launch_ql(const DecodeArgs& a, int dt, dim3 grid, int row_tiles, int groups, float score_mul, float query_mul, hipStream_t s) {
    if (dt == KVBFP_F16 && a.q_mant_bits == 0)
        decode_split_wide<P, N16, RG, 2><<<grid, kThreads, 0, s>>>(a, dt, row_tiles, groups, score_mul, query_mul);
    else
        decode_split_wide<P, N16, RG, 1><<<grid, kThreads, 0, s>>>(a, dt, row_tiles, groups, score_mul, query_mul);
}
template <int P, int N>
void launch_few_n(const DecodeArgs& a, int dt, dim3 grid, float score_mul, float query_mul, hipStream_t s) {
    if (dt == KVBFP_F16 && a.q_mant_bits == 0) decode_split_few<P, N, 2><<<grid, kThreads, 0, s>>>(a, dt, score_mul, query_mul);
    else decode_split_few<P, N, 1><<<grid, kThreads, 0, s>>>(a, dt, score_mul, query_mul);
}
template <int P>
void launch_few(const DecodeArgs& a, int dt, int block, dim3 grid, float score_mul, float query_mul, hipStream_t s) {
    if (block == 16) launch_few_n<P, 16>(a, dt, grid, score_mul, query_mul, s);
    else if (block == 32) launch_few_n<P, 32>(a, dt, grid, score_mul, query_mul, s);
    else if (block == 64) launch_few_n<P, 64>(a, dt, grid, score_mul, query_mul, s);
    else launch_few_n<P, 128>(a, dt, grid, score_mul, query_mul, s);
}
template <int P, bool N16>
void launch_rg(const DecodeArgs& a, int dt, dim3 grid, int row_tiles, int groups, float score_mul, float query_mul, hipStream_t s) {
    if (groups == 2) launch_ql<P, N16, 2>(a, dt, grid, row_tiles, groups, score_mul, query_mul, s);
    else launch_ql<P, N16, 4>(a, dt, grid, row_tiles, groups, score_mul, query_mul, s);
}

}  // namespace

namespace kvbfp {

// Row tiles (workgroups that share the heads of a kv-head out) and groups of 32 heads in each, as even as they go.
WidePlan plan_wide(int G, int64_t units, int64_t max_len, int max_splits) {
    WidePlan w;
    const int groups = (G + kRows - 1) / kRows;
    w.row_tiles = (groups + 3) / 4;
    w.groups = (groups + w.row_tiles - 1) / w.row_tiles;
    // two workgroups fit a compute unit; as many splits as fill one round of them, not more than there are tiles.  (Down to
    // one, which leaves slots empty from 257 to 511 workgroups: 40 sequences x 4096 tokens, 5 query tokens x 4 heads, 320
    // workgroups, take 83 us a call in equal and 60 in log-uniform lengths, 122 and 70 in the passes that served them before.)
    const int tile = w.groups > 1 ? 64 : 128;
    const int64_t tiles = (max_len + tile - 1) / tile;
    int64_t n = 512 / (units * w.row_tiles);
    if (n > tiles) n = tiles;
    if (n > max_splits) n = max_splits;
    w.n_splits = n < 1 ? 1 : (int32_t)n;
    w.log2_tile = w.groups > 1 ? 6 : 7;
    return w;
}

hipError_t launch_decode_split_wide(const DecodeArgs& a, int mant_bits, int dtype, int block, int batch, const WidePlan& w, hipStream_t s) {
    if (dtype == KVBFP_F32) return hipErrorInvalidValue;
    const dim3 grid((unsigned)a.n_splits, (unsigned)(a.H_kv * w.row_tiles), (unsigned)batch);
    // softmax_scale * log2(e) = f * 2^e, f in [1, 2), multiplies the score, with the 2^kShift that the decoded keys lack;
    // only its sign and a power of two far from 1 (keys or queries far from 1 go with it) are folded into the query,
    // within the exponents that leave that factor finite
    int e = 0;
    const float f = std::frexp(std::fabs(a.scale_log2e), &e);
    const int at = std::abs(e - 1) <= 8 ? 0 : std::max(-119, std::min(119, e - 1));
    const bool few = w.row_tiles == 1 && w.groups == 1;
    const int shift = (mant_bits == 4 ? 7 : 3) - (few ? (int)kKeyUp : 0);
    const float score_mul = a.scale_log2e != 0.f ? std::ldexp(2.f * f, e - 1 - at + shift) : 1.f;
    const float query_mul = a.scale_log2e != 0.f ? std::copysign(std::ldexp(1.0f, at), a.scale_log2e) : 0.f;
    if (few) {
        if (mant_bits == 4) launch_few<4>(a, dtype, block, grid, score_mul, query_mul, s);
        else launch_few<8>(a, dtype, block, grid, score_mul, query_mul, s);
    } else if (mant_bits == 4 && block == 16) launch_rg<4, true>(a, dtype, grid, w.row_tiles, w.groups, score_mul, query_mul, s);
    else if (mant_bits == 4) launch_rg<4, false>(a, dtype, grid, w.row_tiles, w.groups, score_mul, query_mul, s);
    else launch_rg<8, false>(a, dtype, grid, w.row_tiles, w.groups, score_mul, query_mul, s);
    return hipGetLastError();
}

}  // namespace kvbfp
