// Split pass of decode attention for many (virtual) query heads per kv-head on the matrix cores: 16-bit I/O, 4- and
// 8-bit mantissas, every block size, contiguous and paged caches (Sec. III run-time flow; several query tokens per
// sequence bring n_q_tokens * G virtual heads).
//
// With G rows a cached element takes 2 G multiply-adds, so from some G on the pass is bound by arithmetic, not by
// memory, and the arithmetic has to go into full matrix-core tiles:
//   * A workgroup decodes a tile of cached rows once, to bf16 in LDS (a code times its block's power of two is
//     exact there), and its four wavefronts, 32 virtual heads each, multiply with it.  With 64 heads or fewer two
//     or all four wavefronts take the same heads and share the tokens of the tile out instead.
//   * Both products are formed transposed, v_mfma_f32_32x32x16_bf16 with S^T = K Q^T and O^T = V^T P^T: a lane then
//     holds scores, running maximum, sum and outputs of ONE head, the softmax needs one exchange with the other half
//     of the wavefront, and the registers that hold S^T are, converted, the second operand of the value product -- the
//     order of the tokens in its reduction is free, and V^T is laid out in LDS in the order S^T leaves them in.
//   * The query is not rounded: a bf16 query (or one cast to BFP) is one bf16 operand, an fp16 query is two (8 + 3
//     bits).  softmax_scale * log2(e) multiplies the score in fp32.  Probabilities are two bf16 limbs (16 bits), as in the other passes for 16-bit I/O.
// Bound by: 64 and more heads, the vector ALUs and the matrix cores about alike (per wavefront, 64 tokens and 32 heads:
// 48 MFMAs of 32 cycles, some 320 vector instructions of softmax and 110 of decoding, 4 cycles each).  256 virtual heads (64
// query tokens, groups of 4) over 4 x 8192 tokens x 8 kv-heads: 67 us against 1470 us in the general pass.  32 heads and
// fewer: waiting for the rows of the next tile (two workgroups per compute unit, one tile ahead).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "decode_args.h"
#include "decode_dev.h"
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

// packs the upper halves of two fp32 patterns: (lo, hi) -> one register of two bf16
__device__ __forceinline__ uint32_t pack_hi(uint32_t lo, uint32_t hi) { return __builtin_amdgcn_perm(hi, lo, 0x07060302u); }
__device__ __forceinline__ uint32_t pack_lo(uint32_t lo, uint32_t hi) { return __builtin_amdgcn_perm(hi, lo, 0x05040100u); }
__device__ __forceinline__ uint32_t bits(bf16x2 v) { return __builtin_bit_cast(uint32_t, v); }

// Eight 4-bit codes -> bf16 pairs (c0,c2), (c4,c6), (c1,c3), (c5,c7), scaled by 2^(E - 136) per unit (value * 2^-7):
// the nibble s|mmm widened to the byte s0000mmm is the FP8-E4M3 subnormal (-1)^s m 2^-9.
__device__ __forceinline__ void unpack8_p4(uint32_t w, float scale, uint32_t (&p)[4]) {
    const uint32_t lo = ((w << 4) & 0x80808080u) | (w & 0x07070707u);
    const uint32_t hi = (w & 0x80808080u) | ((w >> 4) & 0x07070707u);
    p[0] = bits(__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, scale, false));
    p[1] = bits(__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, scale, true));
    p[2] = bits(__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, scale, false));
    p[3] = bits(__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, scale, true));
}
// Four 8-bit codes -> fp32, scaled by 2^(E - 136) per unit (value * 2^-3).  The byte s mmmm lll is the sum of the FP8
// numbers s000mmmm (at eight times the scale) and s0000lll; the sum has at most 7 significant bits, so its upper
// half is the bf16 number.
__device__ __forceinline__ void unpack4_p8(uint32_t w, uint32_t E, float (&x)[4]) {
    const float s_lo = __uint_as_float(E << 23), s_hi = __uint_as_float((E + 3u) << 23);
    const uint32_t hi = ((w >> 3) & 0x0F0F0F0Fu) | (w & 0x80808080u), lo = w & 0x87878787u;
    const f32x2 h01 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(hi, s_hi, false), h23 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(hi, s_hi, true);
    const f32x2 l01 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(lo, s_lo, false), l23 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(lo, s_lo, true);
    x[0] = h01[0] + l01[0]; x[1] = h01[1] + l01[1];
    x[2] = h23[0] + l23[0]; x[3] = h23[1] + l23[1];
}

// channel of k-slot x of the 8-channel group `grp` of a key row in LDS
template <int P>
__device__ __forceinline__ int slot_channel(int grp, int x) {
    return 8 * grp + (P == 8 ? x : (x < 4 ? 2 * x : 2 * (x - 4) + 1));
}

// Exponent bytes at the ends of their range.  The conversions take the byte as their scale operand, which fits all but the
// largest ones, and leave value * 2^-kShift in bf16, which holds all but the smallest blocks exactly.  A 16-token stage
// with such a byte is converted at another power of two, and what its scores and probabilities are multiplied with makes
// up for it; the general pass, which has no such limits, is not needed for them.
enum ExpMode { kExpPlain = 0, kExpHigh = 1, kExpLow = 2 };
template <int P>
struct ExpRange {
    static constexpr uint32_t kTop = P == 4 ? 254u : 251u;         // largest byte whose scale operand (8-bit: + 3) is finite
    static constexpr uint32_t kDown = P == 4 ? 1u : 8u, kUp = 2u;  // taken off / added to the byte at the two ends
    __device__ static uint32_t operand(uint32_t E, int mode) {
        return mode == kExpPlain ? E : (mode == kExpHigh ? E - min(E, kDown) : E + kUp);
    }
    __device__ static float undo(uint32_t mode) { return mode == kExpPlain ? 1.f : (mode == kExpHigh ? (float)(1u << kDown) : 0.25f); }
};
// mode of the stage whose bytes the lanes of a wavefront hold (any number of calls or-ed together)
template <int P>
__device__ __forceinline__ int exp_mode(bool above_top, bool above_low, bool tiny) {
    if (__builtin_amdgcn_ballot_w64(above_top) != 0) return kExpHigh;
    return __builtin_amdgcn_ballot_w64(tiny) != 0 && __builtin_amdgcn_ballot_w64(above_low) == 0 ? kExpLow : kExpPlain;
}

__device__ __forceinline__ float other_half(float v) { return __shfl_xor(v, 32); }

// P = mantissa bits; N16: blocks of 16 (a 16-byte chunk of 4-bit codes then spans two blocks).
// RG = groups of 32 heads per workgroup, 4 / RG wavefronts share the tokens of a tile; QL = bf16 limbs of the query.
// grid = (n_splits, H_kv * row_tiles, B), block = 256; a workgroup takes the heads of `groups` (<= RG) groups of 32,
// and every n_splits-th tile of TT tokens.
template <int P, bool N16, int RG, int QL>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void decode_split_wide(DecodeArgs a, int dt, int row_tiles, int groups, float score_mul, float query_mul) {
    constexpr int kShift = P == 4 ? 7 : 3;             // decoded values are value * 2^-kShift
    constexpr int TG = 4 / RG;                         // wavefronts that share the tokens of a tile
    constexpr int TT = RG == 1 ? 128 : 64;             // tokens per tile
    constexpr int CB = TT / 32 / TG;                   // blocks of 32 tokens per wavefront
    constexpr int SP = TT / 64;                        // decode passes: a wavefront decodes 16 tokens of every 64
    constexpr int kRowB = kD * P / 8;
    constexpr int kKeyChunks = P == 4 ? 1 : 2;         // 16-byte chunks of a key row per thread and pass
    constexpr int kValWords = P == 4 ? 1 : 2;          // dwords (8 channels) of a value row per thread
    // keys: [TT tokens][16 groups of 8 channels], 16 bytes each, the group's place exchanged with token % 16 so that
    // the reads of 16 neighbouring tokens hit different banks; values: [128 channels][TT / 8 groups of 8 tokens], the
    // place exchanged with the channel's bits for both the writes (same bits 0-2, different bits 3-5) and the reads.
    constexpr int kKeyBytes = TT * 256, kValBytes = kD * TT * 2;
    constexpr int kOStride = kD + 4;
    constexpr int kMerge = TG > 1 ? 4 * kRows * kOStride * 4 + 4 * kRows * 2 * 4 : 0;
    constexpr int kQueryBytes = RG * kRows * 256;      // raw queries during the set-up
    constexpr int kSmemA = kKeyBytes + kValBytes > kMerge ? kKeyBytes + kValBytes : kMerge;
    constexpr int kSmem = kSmemA > kQueryBytes ? kSmemA : kQueryBytes;
    __shared__ __align__(16) uint8_t smem[kSmem];
    __shared__ int perm_s[kD];
    __shared__ uint32_t modes_s[SP];                   // ExpMode of the tile's 16-token stages, one byte each: keys | values << 4
    uint8_t* const k_lds = smem;
    uint8_t* const v_lds = smem + kKeyBytes;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int half = lane >> 5, l32 = lane & 31;
    const int split = blockIdx.x, kvh = blockIdx.y / row_tiles, rt = blockIdx.y % row_tiles, b = blockIdx.z;
    const int rg = wave % RG, tg = wave / RG;
    const int s_first = rt * groups * kRows;                     // first virtual head of the workgroup
    const int s_count = min(groups * kRows, a.G - s_first);      // its heads
    const int my_s = s_first + rg * kRows + l32;                 // this lane's head
    const bool active = rg * kRows < s_count;                    // wave-uniform
    const int64_t h0 = (int64_t)b * a.H_q + (int64_t)kvh * a.G;

    int64_t L64 = a.seq_len ? (int64_t)a.seq_len[b] : a.max_len;
    L64 = L64 < 0 ? 0 : (L64 > a.max_len ? a.max_len : L64);
    const int64_t L = L64;
    const int64_t t_first = (int64_t)split * TT;
    if (t_first >= L) {       // nothing cached in this split
        for (int i = tid; i < s_count * kD; i += kThreads)
            a.part_o[((h0 + s_first + i / kD) * a.n_splits + split) * kD + i % kD] = 0.f;
        for (int i = tid; i < s_count; i += kThreads) {
            float* ml = a.part_ml + ((h0 + s_first + i) * a.n_splits + split) * 2;
            ml[0] = -INFINITY;
            ml[1] = 0.f;
        }
        return;
    }

    // ---- packed rows of one tile, as loaded: this wavefront's 16 tokens of every 64
    const int log2_nb = 7 - a.log2_block;              // exponent bytes per row
    struct Raw {
        u32x4 k[SP][kKeyChunks];
        uint32_t ke[SP][2];
        uint32_t v[SP][4][kValWords];
        uint32_t ve[SP][4];
    };
    const int k_tok = lane >> 2, k_chunk = lane & 3;   // keys: token of the stage, 16-byte chunk (8-bit: and chunk + 4)
    const int v_quad = lane >> 4, v_word = lane & 15;  // values: tokens 4 v_quad .. + 3, channels 8 v_word .. + 7
    const uint32_t ke_at0 = P == 4 ? (uint32_t)((32 * k_chunk) >> a.log2_block) : (uint32_t)((16 * k_chunk) >> a.log2_block);
    const uint32_t ke_at1 = P == 4 ? ke_at0 + 1 : (uint32_t)((64 + 16 * k_chunk) >> a.log2_block);
    const uint32_t ve_at = (uint32_t)((8 * v_word) >> a.log2_block);
    auto fetch = [&](const int64_t T0, Raw& r) {
#pragma unroll
        for (int p = 0; p < SP; ++p) {
            int64_t st = T0 + 64 * p + 16 * wave;      // first token of the stage, wave-uniform
            if (st >= L) st = (L - 1) & ~(int64_t)15;  // beyond the end: rows that are not used
            const int last = (int)min((int64_t)15, L - 1 - st);
            const int64_t row0 = kvbfp::cache_row(a, b, kvh, st);
            const uint8_t* __restrict__ km = a.k_mant + row0 * kRowB;
            const uint8_t* __restrict__ vm = a.v_mant + row0 * kRowB;
            const uint8_t* __restrict__ kx = a.k_exp + (row0 << log2_nb);
            const uint8_t* __restrict__ vx = a.v_exp + (row0 << log2_nb);
            const uint32_t kr = (uint32_t)min(k_tok, last);
#pragma unroll
            for (int i = 0; i < kKeyChunks; ++i)
                r.k[p][i] = __builtin_nontemporal_load((const u32x4*)(km + (kr * kRowB + k_chunk * 16 + i * 64)));
            if (P == 4 && N16) {
                r.ke[p][0] = *(const uint16_t*)(kx + ((kr << log2_nb) + ke_at0));
            } else {
                r.ke[p][0] = kx[(kr << log2_nb) + ke_at0];
                if (P == 8) r.ke[p][1] = kx[(kr << log2_nb) + ke_at1];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t vr = (uint32_t)min(4 * v_quad + i, last);
                if constexpr (P == 4) {
                    r.v[p][i][0] = __builtin_nontemporal_load((const uint32_t*)(vm + (vr * kRowB + v_word * 4)));
                } else {
                    const u32x2 w = __builtin_nontemporal_load((const u32x2*)(vm + (vr * kRowB + v_word * 8)));
                    r.v[p][i][0] = w[0];
                    r.v[p][i][kValWords - 1] = w[1];
                }
                r.ve[p][i] = vx[(vr << log2_nb) + ve_at];
            }
        }
    };
    // decoded to bf16 in LDS
    auto decode = [&](Raw& r) {
#pragma unroll
        for (int p = 0; p < SP; ++p) {
            using R = ExpRange<P>;
            const uint32_t ke[2] = {P == 4 && N16 ? (r.ke[p][0] & 0xFFu) : r.ke[p][0], P == 4 ? (N16 ? r.ke[p][0] >> 8 : r.ke[p][0]) : r.ke[p][1]};
            const uint32_t top = max(max(max(r.ve[p][0], r.ve[p][1]), max(r.ve[p][2], r.ve[p][3])), max(ke[0], ke[1]));
            const uint32_t low = min(min(min(r.ve[p][0], r.ve[p][1]), min(r.ve[p][2], r.ve[p][3])), min(ke[0], ke[1]));
            int mode_k = kExpPlain, mode_v = kExpPlain;
            if (__builtin_amdgcn_ballot_w64(top > R::kTop || low <= 2u) != 0) {     // (also where a block is all zero)
                constexpr uint32_t kLowTop = R::kTop - R::kUp;
                auto tiny = [](uint32_t E) { return E - 1u < 2u; };
                const uint32_t kt = max(ke[0], ke[1]);
                mode_k = exp_mode<P>(kt > R::kTop, kt > kLowTop, tiny(ke[0]) || tiny(ke[1]));
                const uint32_t vt = max(max(r.ve[p][0], r.ve[p][1]), max(r.ve[p][2], r.ve[p][3]));
                mode_v = exp_mode<P>(vt > R::kTop, vt > kLowTop, tiny(r.ve[p][0]) || tiny(r.ve[p][1]) || tiny(r.ve[p][2]) || tiny(r.ve[p][3]));
                if constexpr (P == 4) {
                    r.ke[p][0] = N16 ? (R::operand(ke[0], mode_k) | (R::operand(ke[1], mode_k) << 8)) : R::operand(ke[0], mode_k);
                } else {
                    r.ke[p][0] = R::operand(ke[0], mode_k);
                    r.ke[p][1] = R::operand(ke[1], mode_k);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) r.ve[p][i] = R::operand(r.ve[p][i], mode_v);
            }
            if (lane == 0) ((uint8_t*)&modes_s[p])[wave] = (uint8_t)(mode_k | (mode_v << 4));
            const int tok = 64 * p + 16 * wave + k_tok;
            uint8_t* const krow = k_lds + tok * 256;
#pragma unroll
            for (int i = 0; i < kKeyChunks; ++i) {
                if constexpr (P == 4) {
                    const float s0 = __uint_as_float((N16 ? (r.ke[p][0] & 0xFFu) : r.ke[p][0]) << 23);
                    const float s1 = N16 ? __uint_as_float((r.ke[p][0] >> 8) << 23) : s0;
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        uint32_t q[4];
                        unpack8_p4(r.k[p][i][d], d < 2 ? s0 : s1, q);
                        *(u32x4*)(krow + (((4 * k_chunk + d) ^ (tok & 15)) * 16)) = u32x4{q[0], q[1], q[2], q[3]};
                    }
                } else {
#pragma unroll
                    for (int d = 0; d < 2; ++d) {
                        float x[4], y[4];
                        unpack4_p8(r.k[p][i][2 * d], r.ke[p][i], x);
                        unpack4_p8(r.k[p][i][2 * d + 1], r.ke[p][i], y);
                        const u32x4 w = {pack_hi(__float_as_uint(x[0]), __float_as_uint(x[1])), pack_hi(__float_as_uint(x[2]), __float_as_uint(x[3])),
                                         pack_hi(__float_as_uint(y[0]), __float_as_uint(y[1])), pack_hi(__float_as_uint(y[2]), __float_as_uint(y[3]))};
                        *(u32x4*)(krow + (((8 * i + 2 * k_chunk + d) ^ (tok & 15)) * 16)) = w;
                    }
                }
            }
            // values: the four tokens of each channel side by side.  In a group of 16 tokens the quads 0 and 2 make the
            // first 16 bytes and 1 and 3 the second: the order in which S^T leaves them in the two halves of a wavefront.
            const int place = 2 * (4 * p + wave) + (v_quad & 1);
            auto put = [&](const int c, const uint32_t t01, const uint32_t t23) {      // c = channel % 8
                const int ch = 8 * v_word + c;
                const int at = ch * (TT * 2) + ((place ^ ((v_word ^ c) & 7)) * 16) + (v_quad >> 1) * 8;
                *(u32x2*)(v_lds + at) = u32x2{t01, t23};
            };
            if constexpr (P == 4) {
                uint32_t q[4][4];
#pragma unroll
                for (int i = 0; i < 4; ++i) unpack8_p4(r.v[p][i][0], __uint_as_float(r.ve[p][i] << 23), q[i]);
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
                    for (int i = 0; i < 4; ++i) unpack4_p8(r.v[p][i][w], r.ve[p][i], x[i]);
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        put(4 * w + c, pack_hi(__float_as_uint(x[0][c]), __float_as_uint(x[1][c])), pack_hi(__float_as_uint(x[2][c]), __float_as_uint(x[3][c])));
                }
            }
        }
    };

    // ---- kvbfp_append_decode_attention (one row tile only): the current token, position L - 1, is cast and stored by
    // the one wavefront that decodes that row, before it requests the row's tile.  Lanes 0-7 take the key row, lanes
    // 8-15 the value row; the others run along with zeros (the block maximum is a cross-lane reduction).
    const bool appends = a.k_new != nullptr && (int)(((L - 1) / TT) % a.n_splits) == split && (int)(((L - 1) >> 4) & 3) == wave;
    const int64_t T_new = (L - 1) / TT * TT;             // the tile that holds it
    const int nr_sub = lane & 7, nr_which = (lane >> 3) & 1;
    int nr_c[16];
    float nr_x[16];
    auto new_row_perm = [&] {
        const int32_t* pr = nr_which ? a.perm_v : a.perm_k;
#pragma unroll
        for (int i = 0; i < 16; ++i) nr_c[i] = (pr && lane < 16) ? (pr[kvh * kD + nr_sub * 16 + i] & (kD - 1)) : nr_sub * 16 + i;
    };
    auto new_row_load = [&] {
        const uint16_t* src = (const uint16_t*)(nr_which ? a.v_new : a.k_new) + (int64_t)b * a.new_stride_b + (int64_t)kvh * a.new_stride_h;
#pragma unroll
        for (int i = 0; i < 16; ++i) nr_x[i] = lane < 16 ? load_as_float(src, dt, nr_c[i]) : 0.f;
    };
    auto new_row_store = [&] {
        uint8_t* const mant = const_cast<uint8_t*>(nr_which ? a.v_mant : a.k_mant);
        uint8_t* const exps = const_cast<uint8_t*>(nr_which ? a.v_exp : a.k_exp);
        const int64_t row = kvbfp::cache_row(a, b, kvh, L - 1);
        const bool live = lane < 16;
        if (a.log2_block == 4) kvbfp::cast::encode_store<P, 16>(nr_x, nr_sub, live, mant, exps, row);
        else if (a.log2_block == 5) kvbfp::cast::encode_store<P, 32>(nr_x, nr_sub, live, mant, exps, row);
        else if (a.log2_block == 6) kvbfp::cast::encode_store<P, 64>(nr_x, nr_sub, live, mant, exps, row);
        else kvbfp::cast::encode_store<P, 128>(nr_x, nr_sub, live, mant, exps, row);
    };
    auto stores_done = [&] { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
    if (appends) {
        new_row_perm();
        if (T_new == t_first) {
            new_row_load();
            new_row_store();
            stores_done();
        }
    }

    Raw raw;
    fetch(t_first, raw);
    if (appends && T_new != t_first) new_row_load();     // waited for after the set-up

    // ---- query operand: lane (head l32, half), MFMA m: channels of the groups 2m + half, in key slot order
    bf16x8 q_op[QL][8];
    {
        if (tid < kD) perm_s[tid] = a.perm_k ? (a.perm_k[kvh * kD + tid] & (kD - 1)) : tid;     // masked: device data the host cannot check
        const bool vec = ((uintptr_t)a.q & 15u) == 0;
        for (int i = tid; i < RG * kRows * 16; i += kThreads) {        // 16 pieces of 16 bytes per head
            const int row = i >> 4;
            u32x4 w = {0u, 0u, 0u, 0u};
            if (row < s_count) {
                const uint16_t* src = (const uint16_t*)a.q + kvbfp::query_row(a, b, kvh, s_first + row) * kD + (i & 15) * 8;
                if (vec) {
                    w = *(const u32x4*)src;
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k) w[k] = (uint32_t)src[2 * k] | ((uint32_t)src[2 * k + 1] << 16);
                }
            }
            *(u32x4*)(smem + row * 256 + (((i & 15) ^ (row & 15)) * 16)) = w;
        }
        lds_only_barrier();
        const int row = rg * kRows + l32;
        float x[8][8];
        float top[8];                                   // largest magnitude of channels 16m .. 16m + 15
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            top[m] = 0.f;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int c = perm_s[slot_channel<P>(2 * m + half, k)];
                const uint32_t h = *(const uint16_t*)(smem + row * 256 + (((c >> 3) ^ (row & 15)) * 16) + (c & 7) * 2);
                x[m][k] = dt == KVBFP_F16 ? (float)__builtin_bit_cast(_Float16, (unsigned short)h) : __uint_as_float(h << 16);
                top[m] = fmaxf(top[m], fabsf(x[m][k]));
            }
        }
        if (a.q_mant_bits) {                            // cast to BFP first, in cache channel order, like a cached row
#pragma unroll
            for (int m = 0; m < 8; ++m) top[m] = fmaxf(top[m], other_half(top[m]));
            if (a.log2_block >= 5) {
#pragma unroll
                for (int m = 0; m < 8; m += 2) top[m] = top[m + 1] = fmaxf(top[m], top[m + 1]);
            }
            if (a.log2_block >= 6) {
#pragma unroll
                for (int m = 0; m < 8; m += 4) top[m] = top[m + 1] = top[m + 2] = top[m + 3] = fmaxf(top[m], top[m + 2]);
            }
            if (a.log2_block >= 7) {
                const float t = fmaxf(top[0], top[4]);
#pragma unroll
                for (int m = 0; m < 8; ++m) top[m] = t;
            }
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                const uint32_t amax = __float_as_uint(top[m]);
                const uint32_t bumped = (amax + (1u << (24 - a.q_mant_bits))) >> 23;
                const int E = amax == 0 ? 0 : (int)max(bumped, 1u);
                const int e = E - 127 - (a.q_mant_bits - 2);
#pragma unroll
                for (int k = 0; k < 8; ++k) x[m][k] = ldexpf(rintf(ldexpf(x[m][k], -e)), e);
            }
        }
#pragma unroll
        for (int m = 0; m < 8; ++m) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float v = x[m][k] * query_mul;    // a power of two and the sign of the scale: exact
                const uint32_t top_bits = __float_as_uint(v) & 0xFFFF0000u;
                q_op[0][m][k] = __builtin_bit_cast(__bf16, (unsigned short)(top_bits >> 16));
                if (QL == 2) q_op[QL - 1][m][k] = (__bf16)(v - __uint_as_float(top_bits));
            }
        }
        lds_only_barrier();                             // the queries give way to the first tile
    }
    if (appends && T_new != t_first) new_row_store();

    const int64_t lim = L - kvbfp::hidden_tokens(a, my_s);         // this head sees tokens below
    const int64_t all_see = L - (a.n_q_tokens - 1);                // every head does
    float m_run = -INFINITY, l_run = 0.f;
    f32x16 o[4];
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[ct][i] = 0.f;

    const int64_t step = (int64_t)a.n_splits * TT;
    const int my_tok0 = tg * CB * 32;                              // first token of this wavefront inside a tile
    for (int64_t T0 = t_first; T0 < L; T0 += step) {
        decode(raw);
        if (appends && T0 + step == T_new) stores_done();
        if (T0 + step < L) fetch(T0 + step, raw);
        lds_only_barrier();
        if (active) {
            // ---- S^T: 32 tokens x 32 heads per block
            f32x16 s[CB];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
#pragma unroll
                for (int i = 0; i < 16; ++i) s[cb][i] = 0.f;
                const int tok = my_tok0 + 32 * cb + l32;
                const uint8_t* const krow = k_lds + tok * 256;
#pragma unroll
                for (int m = 0; m < 8; ++m) {
                    const bf16x8 ka = *(const bf16x8*)(krow + (((2 * m + half) ^ (tok & 15)) * 16));
                    s[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, q_op[0][m], s[cb], 0, 0, 0);
                    if (QL == 2) s[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka, q_op[QL - 1][m], s[cb], 0, 0, 0);
                }
            }
            // register i of a block: token 8 (i / 4) + 4 half + i % 4
            uint32_t modes[SP];
            uint32_t any_mode = 0;
#pragma unroll
            for (int p = 0; p < SP; ++p) any_mode |= modes[p] = __builtin_amdgcn_readfirstlane(modes_s[p]);
            auto mode_at = [&](int cb, int i) {            // of the stage of 16 tokens this register's token lies in
                const int st = my_tok0 / 16 + 2 * cb + (i >> 3);
                uint32_t w = modes[0];
                if constexpr (SP == 2) w = st >= 4 ? modes[SP - 1] : w;
                return w >> (8 * (st & 3));
            };
            if (any_mode != 0) {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) s[cb][i] *= ExpRange<P>::undo(mode_at(cb, i) & 0xFu);
            }
            if (T0 + TT > all_see) {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int64_t t = T0 + my_tok0 + 32 * cb + 8 * (i >> 2) + 4 * half + (i & 3);
                        s[cb][i] = t < lim ? s[cb][i] : -INFINITY;
                    }
            }
            // ---- online softmax, base 2
            float tmax = s[0][0];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int i = 0; i < 16; ++i) tmax = fmaxf(tmax, s[cb][i]);
            tmax = fmaxf(tmax, other_half(tmax)) * score_mul;      // -inf only if this head sees none of the tile
            const float m_new = fmaxf(m_run, tmax);
            const float m_ref = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = exp2_raw(m_run - m_ref);
            const float m_p = m_ref - (float)kShift;               // probabilities carry 2^kShift
            uint32_t p_hi[CB][8], p_lo[CB][8];
            float psum = 0.f;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int i = 0; i < 16; i += 2) {
                    const float p0 = exp2_raw(fmaf(s[cb][i], score_mul, -m_p));
                    const float p1 = exp2_raw(fmaf(s[cb][i + 1], score_mul, -m_p));
                    psum += p0;
                    psum += p1;
                    p_hi[cb][i / 2] = pack_hi(__float_as_uint(p0), __float_as_uint(p1));
                    bf16x2 lo;
                    lo[0] = (__bf16)(p0 - __uint_as_float(__float_as_uint(p0) & 0xFFFF0000u));
                    lo[1] = (__bf16)(p1 - __uint_as_float(__float_as_uint(p1) & 0xFFFF0000u));
                    p_lo[cb][i / 2] = bits(lo);
                }
            if (any_mode != 0) {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int i = 0; i < 16; i += 2) {
                        const float u = ExpRange<P>::undo((mode_at(cb, i) >> 4) & 0xFu);
                        auto scaled = [&](uint32_t w) {
                            return pack_hi(__float_as_uint(__uint_as_float(w << 16) * u), __float_as_uint(__uint_as_float(w & 0xFFFF0000u) * u));
                        };
                        p_hi[cb][i / 2] = scaled(p_hi[cb][i / 2]);
                        p_lo[cb][i / 2] = scaled(p_lo[cb][i / 2]);
                    }
            }
            l_run = l_run * alpha + psum;
            m_run = m_new;
            if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
                for (int ct = 0; ct < 4; ++ct) o[ct] *= alpha;
            }
            // ---- O^T += V^T P^T
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) {
                    const bf16x8 ph = __builtin_bit_cast(bf16x8, u32x4{p_hi[cb][4 * kk], p_hi[cb][4 * kk + 1], p_hi[cb][4 * kk + 2], p_hi[cb][4 * kk + 3]});
                    const bf16x8 pl = __builtin_bit_cast(bf16x8, u32x4{p_lo[cb][4 * kk], p_lo[cb][4 * kk + 1], p_lo[cb][4 * kk + 2], p_lo[cb][4 * kk + 3]});
                    const int place = 2 * (my_tok0 / 16 + 2 * cb + kk) + half;
#pragma unroll
                    for (int ct = 0; ct < 4; ++ct) {
                        const int ch = 32 * ct + l32;
                        const bf16x8 va = *(const bf16x8*)(v_lds + ch * (TT * 2) + ((place ^ ((ch ^ (ch >> 3)) & 7)) * 16));
                        o[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, ph, o[ct], 0, 0, 0);
                        o[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pl, o[ct], 0, 0, 0);
                    }
                }
        }
        lds_only_barrier();                                        // the next tile overwrites this one
    }
    l_run = (l_run + other_half(l_run)) * (1.0f / (float)(1 << kShift));

    // ---- partial result of this split: registers 4i .. 4i+3 of block ct are channels 32 ct + 8 i + 4 half ..
    if constexpr (TG == 1) {
        if (!active || my_s - s_first >= s_count) return;
        float* const po = a.part_o + ((h0 + my_s) * a.n_splits + split) * kD;
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *(f32x4*)(po + 32 * ct + 8 * i + 4 * half) = f32x4{o[ct][4 * i], o[ct][4 * i + 1], o[ct][4 * i + 2], o[ct][4 * i + 3]};
        if (half == 0) {
            float* ml = a.part_ml + ((h0 + my_s) * a.n_splits + split) * 2;
            ml[0] = m_run;
            ml[1] = l_run;
        }
    } else {       // merge the wavefronts that shared the tokens
        float* const o_s = (float*)smem;                           // [wave][head][kOStride]
        float* const ml_s = (float*)(smem + 4 * kRows * kOStride * 4);
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *(f32x4*)(o_s + (wave * kRows + l32) * kOStride + 32 * ct + 8 * i + 4 * half) = f32x4{o[ct][4 * i], o[ct][4 * i + 1], o[ct][4 * i + 2], o[ct][4 * i + 3]};
        if (half == 0) {
            ml_s[(wave * kRows + l32) * 2] = m_run;
            ml_s[(wave * kRows + l32) * 2 + 1] = l_run;
        }
        lds_only_barrier();
        for (int i = tid; i < s_count * kD; i += kThreads) {
            const int g = i / kD, c = i % kD;
            const int w0 = g / kRows, r = g % kRows;
            float M = -INFINITY;
#pragma unroll
            for (int t = 0; t < TG; ++t) M = fmaxf(M, ml_s[((w0 + t * RG) * kRows + r) * 2]);
            float acc = 0.f, lsum = 0.f;
#pragma unroll
            for (int t = 0; t < TG; ++t) {
                const float mw = ml_s[((w0 + t * RG) * kRows + r) * 2];
                if (mw > -INFINITY) {
                    const float f = exp2f(mw - M);
                    acc = fmaf(f, o_s[((w0 + t * RG) * kRows + r) * kOStride + c], acc);
                    lsum = fmaf(f, ml_s[((w0 + t * RG) * kRows + r) * 2 + 1], lsum);
                }
            }
            a.part_o[((h0 + s_first + g) * a.n_splits + split) * kD + c] = acc;
            if (c == 0) {
                float* ml = a.part_ml + ((h0 + s_first + g) * a.n_splits + split) * 2;
                ml[0] = M;
                ml[1] = lsum;
            }
        }
    }
}

template <int P, bool N16, int RG>
void launch_ql(const DecodeArgs& a, int dt, dim3 grid, int row_tiles, int groups, float score_mul, float query_mul, hipStream_t s) {
    if (dt == KVBFP_F16 && a.q_mant_bits == 0)
        decode_split_wide<P, N16, RG, 2><<<grid, kThreads, 0, s>>>(a, dt, row_tiles, groups, score_mul, query_mul);
    else
        decode_split_wide<P, N16, RG, 1><<<grid, kThreads, 0, s>>>(a, dt, row_tiles, groups, score_mul, query_mul);
}
template <int P, bool N16>
void launch_rg(const DecodeArgs& a, int dt, dim3 grid, int row_tiles, int groups, float score_mul, float query_mul, hipStream_t s) {
    if (groups == 1) launch_ql<P, N16, 1>(a, dt, grid, row_tiles, groups, score_mul, query_mul, s);
    else if (groups == 2) launch_ql<P, N16, 2>(a, dt, grid, row_tiles, groups, score_mul, query_mul, s);
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
    // two workgroups fit a compute unit; as many splits as fill one round of them, not more than there are tiles
    const int tile = w.groups > 1 ? 64 : 128;
    const int64_t tiles = (max_len + tile - 1) / tile;
    int64_t n = 512 / (units * w.row_tiles);
    if (n > tiles) n = tiles;
    if (n > max_splits) n = max_splits;
    w.n_splits = n < 1 ? 1 : (int32_t)n;
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
    const int shift = mant_bits == 4 ? 7 : 3;
    const float score_mul = a.scale_log2e != 0.f ? std::ldexp(2.f * f, e - 1 - at + shift) : 1.f;
    const float query_mul = a.scale_log2e != 0.f ? std::copysign(std::ldexp(1.0f, at), a.scale_log2e) : 0.f;
    if (mant_bits == 4 && block == 16) launch_rg<4, true>(a, dtype, grid, w.row_tiles, w.groups, score_mul, query_mul, s);
    else if (mant_bits == 4) launch_rg<4, false>(a, dtype, grid, w.row_tiles, w.groups, score_mul, query_mul, s);
    else launch_rg<8, false>(a, dtype, grid, w.row_tiles, w.groups, score_mul, query_mul, s);
    return hipGetLastError();
}

}  // namespace kvbfp
