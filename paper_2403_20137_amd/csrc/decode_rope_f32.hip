// Split pass of decode attention over keys cached BEFORE the rotary embedding, in fp32
// (Alg. 1 step 5; Sec. II-D; Sec. III run-time flow: rows are fetched, rotated in the reordered channel
// order, then multiplied with the reordered query).  8-bit mantissas, fp32 I/O and exponent planes of any alignment; what
// has 4 bits and 16-bit I/O takes decode_rope.hip.  Up to four query heads of a KV head per workgroup.
//
// The rotation is moved from the keys to the operands around them.  With q2[m] = -s'[m] q[i'[m]]
// (partner and sign vectors of the reordered pairs), the score of token t is
//     sum_m k'[m] ( q[m] cos(t Th[m]) + q2[m] sin(t Th[m]) ),
// and with t = t0 + tau (t0 = first token of a wavefront's 64-token tile, tau = 0..63)
//     = sum_m (k'[m] cos(tau Th[m])) A1[m] + (k'[m] sin(tau Th[m])) A2[m],
//     A1 = q cos(t0 Th) + q2 sin(t0 Th),   A2 = q2 cos(t0 Th) - q sin(t0 Th).
//   * A lane holds one token: its row of codes in registers, one channel at a time a number times cosine and sine, and
//     v_mfma_f32_4x4x1_16b_f32 adds the outer product with the four heads' A1 and A2 of that channel -- 16 blocks of four
//     tokens each, the block of A that holds the channel broadcast to all of them (16 channels share a register).  Lane l
//     then has the scores of token l, register h those of head h.  A matrix instruction takes the place of four fused
//     multiply-adds (it rounds like one) and of their operands' broadcast.
//   * cos/sin(tau Th[m]), tau < 64, never change: one fp32 table per workgroup in LDS, built in double precision.
//   * A1, A2 are rebuilt once per tile from the phasor of t0, which is stepped in double precision from tile to tile.
//   * A code is a binary16 integer, exactly, and the product with the table entry one v_fma_mix; the power of two of a block
//     multiplies the sum of 16 products (the integer-mantissa products plus one exponent addition per block of Sec. II-B).
// Values, softmax and the merge of the four wavefronts are those of the register-staged plain pass: probabilities are three
// bf16 limbs (24 bits), and a tile with an exponent byte that the values' conversion to bf16 does not hold exactly, or with a
// weight that the limbs do not hold, takes fp32 multiply-adds for its values.
// Bound by instruction issue: per wavefront and 64 tokens, 8 bits, some 1230 vector instructions of 4 cycles and 320 matrix instructions of
// about 9, which hardly overlap and are two thirds of the time (without half of the small matrix instructions a call took 8 us less,
// without the values 8, with the table's entries in registers nothing).  Calls with 8 kv-heads, 4 heads, one token a thread and all products
// on the vector ALUs before -> now: 8 bits, bf16, 8 x 16384 tokens 241 -> 86 us, fp32 7 x 59535 1301 -> 253, fp32 with 4 bits 4 x 8192
// 64 -> 25.9, 1 x 1000 tokens, 8 bits 23.5 -> 14.6.  Against 64 bits fp32 outputs are 0.93 (4 bits) and 0.85 times (8 bits) as far off as
// those were, 2.6 and 2.4e-7 of their norm in the mean of 60 calls of any shape.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>
#include <utility>

#include "decode_args.h"
#include "decode_dev.h"
#include "decode_spans.h"
#include "kvbfp_internal.h"

namespace {

using kvbfp::DecodeArgs;
using namespace kvbfp::dev;

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// The values' conversions make pairs of channels of a dword, P = 4: (0,2), (4,6), (1,3), (5,7), P = 8: (0,1), (2,3); where channel x is
template <int P>
__device__ constexpr int pair_of(int x) { return P == 4 ? (x & 1) * 2 + (x >> 2) : x >> 1; }
template <int P>
__device__ constexpr int half_of(int x) { return P == 4 ? (x >> 1) & 1 : x & 1; }

// P = mantissa bits, N = block.  grid = (n_splits, ceil(G / 4) * H_kv, B), block = 256: a workgroup serves four heads of a kv-head (the last
// ones maybe fewer), and all of a call are in one launch, since with few and short sequences a launch of four heads leaves most of the chip
// idle and takes as long as one of all.  8 kv-heads, launches one after the other -> one (all products on the vector ALUs, four heads a
// workgroup, before either): 1 x 1000 tokens, 8 heads, 8 bits 25.8 -> 14.7 us (24.3), 16 heads 48.2 -> 14.9 (24.6), 64 heads 185 -> 20.9
// (29.3), 8 x 16384 tokens, 8 heads 175 -> 154 (469), fp32 4 x 8192, 8 heads 47.4 -> 39.3 (117).  The groups of heads of a kv-head, which read the same rows, are H_kv * n_splits workgroups apart: on the same die where that is a multiple of 8.
template <int P, int N>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void decode_split_rope_f32(DecodeArgs a, int dt) {
    constexpr int NB = kD / N;
    constexpr int NH = 4;
    constexpr int PL = 3;                                       // bf16 limbs of a probability: all of its 24 bits
    constexpr int kRowB = kD * P / 8;
    constexpr int kChunks = kRowB / 16;                         // 16-byte pieces of a row
    constexpr int kWord = 32 / P;                               // codes in a dword
    constexpr int kValWords = P / 4;                            // dwords (8 channels) of a value row per lane
    constexpr int kExpWords = NB == 8 ? 2 : 1;                  // dwords of a row's exponent bytes
    // values are converted to value * 2^-kShift in bf16 with the exponent byte as the scale operand, exactly for bytes from 3 to kTop
    constexpr int kShift = P == 4 ? 7 : 3;
    constexpr uint32_t kTop = P == 4 ? 254u : 251u;
    // [128 channels][64 tau] pairs (cos, sin), tau exchanged with the bits of the channel (stores come from channels side by side, and
    // only four of them meet in a bank).  Before the table is built the same memory holds the queries, after the main loop
    // the per-wavefront outputs for the merge.
    __shared__ __align__(16) unsigned char tab_raw[kD * kSuper * 8];
    auto swizzle = [](int c) { return (c >> 1) & 15; };
    float (*raw)[kD] = reinterpret_cast<float (*)[kD]>(tab_raw);                 // [NH][kD], original channel order
    float (*q1_s)[kD] = raw + NH;                                                // scaled, cache order
    float (*q2_s)[kD] = q1_s + NH;
    // What lane (b, h) = 4 b + h takes for the operand registers r = 4 rh + x, channels 16 r + b: [q | q2][rh][lane][x]
    __shared__ __align__(16) float q_op_s[2][2][64][4];
    __shared__ float top_s[NH];
    // Per wavefront: the phasor of its tile's t0, [cos | sin][rh][b][x]; then the probabilities of the tile,
    // [limb][head][token] (or as fp32 numbers, [head][token])
    constexpr int kWaveBytes = PL * NH * kSuper * 2;
    static_assert(kWaveBytes >= 2 * 2 * 16 * 4 * 4 && kWaveBytes >= NH * kSuper * 4, "the phasor fits, and fp32 probabilities do");
    __shared__ __align__(16) unsigned char wave_s[kWaves][kWaveBytes];
    __shared__ __align__(16) uint32_t ve_s[kWaves][kExpWords][kSuper];           // exponent bytes of the tile's value rows
    __shared__ float ml_s[kWaves][NH][2];
    static_assert(sizeof(tab_raw) >= sizeof(float) * kWaves * NH * kD, "the merge buffer fits the table");
    float (*o_s)[NH][kD] = reinterpret_cast<float (*)[NH][kD]>(tab_raw);

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;    // scalar: tile bases stay in SGPRs
    const int j = lane & 15, kg = lane >> 4;
    int kvh = blockIdx.y, group = 0;
    if (a.G > NH) {
        group = kvh / a.H_kv;
        kvh -= group * a.H_kv;
    }
    const int g_base = NH * group, g_cnt = min(NH, a.G - g_base);
    // what the set-up reads ahead of everything else but the lengths, before those have arrived: the query as it lies in memory, the
    // vectors of this thread's channel (a load through the permutation would be one more round trip)
    const int len0 = kvbfp::spans::request_lengths(a, gridDim.z);
    const int my_c = tid & (kD - 1);
    uint32_t q_bits[NH * kD / 256];
    auto request_queries = [&](const int seq) {
#pragma unroll
        for (int k = 0; k < NH * kD / 256; ++k) {
            const int g = (tid + 256 * k) / kD;
            const int64_t idx = kvbfp::query_row(a, seq, kvh, g_base + min(g, g_cnt - 1)) * kD + my_c;
            q_bits[k] = dt == KVBFP_F32 ? ((const uint32_t*)a.q)[idx] : (uint32_t)((const uint16_t*)a.q)[idx];
        }
    };
    request_queries(blockIdx.z);
    const int perm_c = a.perm_k ? (a.perm_k[kvh * kD + my_c] & (kD - 1)) : my_c;       // masked: device data the host cannot check
    const int partner_c = a.rope_partner[kvh * kD + my_c] & (kD - 1);
    const float sign_c = a.rope_sign[kvh * kD + my_c];
    const double th0 = (double)a.rope_theta[kvh * kD + lane], th1 = (double)a.rope_theta[kvh * kD + 64 + lane];
    __builtin_amdgcn_sched_barrier(0);
    kvbfp::spans::Span span;
    if (!kvbfp::spans::take(a, len0, 8, span)) return;
    if (span.b != (int)blockIdx.z) request_queries(span.b);
    const int split = span.split, b = span.b;
    const int h0 = kvh * a.G + g_base;

    const int64_t L = span.L;
    const int64_t t_begin = (int64_t)split * 256;
    const int64_t t_end = L;

    if (t_begin >= t_end) {
        for (int i = tid; i < g_cnt * kD; i += 256) {
            if (a.direct) kvbfp::spans::write_output(a, dt, b, kvh, g_base + i / kD, i % kD, 0.f, 0.f);
            else a.part_o[span.row(h0 + i / kD) * kD + (i % kD)] = 0.f;
        }
        if (!a.direct && tid < g_cnt) {
            float* ml = a.part_ml + span.row(h0 + tid) * 2;
            ml[0] = -INFINITY;
            ml[1] = 0.f;
        }
        return;
    }

    const int64_t base = ((int64_t)b * a.H_kv + kvh) * a.max_seq + t_begin;
    const uint8_t* __restrict__ k_mant = a.k_mant + base * kRowB;
    const uint8_t* __restrict__ v_mant = a.v_mant + base * kRowB;
    const uint8_t* __restrict__ k_exp = a.k_exp + base * NB;
    const uint8_t* __restrict__ v_exp = a.v_exp + base * NB;
    const int n_tok = (int)(t_end - t_begin);
    const bool exp_words = (((uintptr_t)a.k_exp | (uintptr_t)a.v_exp) & (NB - 1)) == 0;      // a row's bytes can be read at once

    // The rows of one 64-token tile as a lane loads them: the key row of token `lane` with its exponent bytes (requested a tile
    // ahead, piece by piece as the pieces of this tile are used up), and 8 channels of 16 value rows (requested at the top of the
    // tile; rows 16u + 4kg + i, channels 8j ..).
    u32x4 kw[kChunks];
    uint32_t kex[kExpWords];
    auto load_exponents = [&](const uint8_t* p, uint32_t (&e)[kExpWords]) {
        if (exp_words) {
            if constexpr (NB == 8) {
                const u32x2 w = *(const u32x2*)p;
                e[0] = w[0];
                e[kExpWords - 1] = w[1];
            } else if constexpr (NB == 4) {
                e[0] = *(const uint32_t*)p;
            } else if constexpr (NB == 2) {
                e[0] = *(const uint16_t*)p;
            } else {
                e[0] = *p;
            }
        } else {
#pragma unroll
            for (int w = 0; w < kExpWords; ++w) {
                e[w] = 0;
#pragma unroll
                for (int i = 0; i < (NB < 4 ? NB : 4); ++i) e[w] |= (uint32_t)p[4 * w + i] << (8 * i);
            }
        }
    };
    const int T_step = span.n * kWaves * kSuper, T_first = wave * kSuper;
    // (row of this lane in the tile at T: rows past the last cached token re-read it; beyond the last tile every lane re-reads one row)
    auto key_row = [&](const int T) -> uint32_t { return (uint32_t)min(T + lane, n_tok - 1); };
    {
        const uint32_t r = key_row(T_first);
#pragma unroll
        for (int i = 0; i < kChunks; ++i) kw[i] = *(const u32x4*)(k_mant + (size_t)r * kRowB + 16 * i);
        load_exponents(k_exp + (size_t)r * NB, kex);
    }

    // ---------------- set-up (the first tile's keys are on their way: barriers that order LDS only)
#pragma unroll
    for (int k = 0; k < NH * kD / 256; ++k) {
        const int g = (tid + 256 * k) / kD;
        const float f = dt == KVBFP_F32 ? __uint_as_float(q_bits[k])
                        : dt == KVBFP_F16 ? (float)__builtin_bit_cast(_Float16, (unsigned short)q_bits[k]) : __uint_as_float(q_bits[k] << 16);
        raw[g][my_c] = g < g_cnt ? f : 0.f;
    }
    lds_only_barrier();
#pragma unroll
    for (int k = 0; k < NH * kD / 256; ++k) {
        const int g = (tid + 256 * k) / kD;
        q1_s[g][my_c] = raw[g][perm_c] * a.scale_log2e;
    }
    lds_only_barrier();
#pragma unroll
    for (int k = 0; k < NH * kD / 256; ++k) {
        const int g = (tid + 256 * k) / kD;
        q2_s[g][my_c] = -sign_c * q1_s[g][partner_c];
    }
    lds_only_barrier();
    {       // the largest |q|, |q2| of each head, by a wavefront
        const float2 x = *(const float2*)&q1_s[wave][2 * lane], y = *(const float2*)&q2_s[wave][2 * lane];
        float top = row_max(fmaxf(fmaxf(fabsf(x.x), fabsf(x.y)), fmaxf(fabsf(y.x), fabsf(y.y))));
        top = fmaxf(top, __shfl_xor(top, 16));
        top = fmaxf(top, __shfl_xor(top, 32));
        if (lane == 0) top_s[wave] = top;
    }
    lds_only_barrier();
    // Queries between 2^-60 and 2^60 (softmax_scale * log2(e) in them) are taken as they are; where a head's are not, every head's
    // are brought to [1, 2) and the powers of two go to the blocks' sums, so that nothing leaves the range of fp32 in between.
    int q_exp[NH];
    bool plain = true;
#pragma unroll
    for (int g = 0; g < NH; ++g) {
        const uint32_t e = (__float_as_uint(top_s[g]) >> 23) & 0xFFu;
        q_exp[g] = (int)min(e, 254u) - 127;
        plain = plain && (e == 0u ? top_s[g] == 0.f : e - 67u <= 120u);
    }
    plain = __builtin_amdgcn_readfirstlane(plain);
#pragma unroll
    for (int g = 0; g < NH; ++g) q_exp[g] = plain ? 0 : __builtin_amdgcn_readfirstlane(q_exp[g]);
#pragma unroll
    for (int k = 0; k < NH * kD / 256; ++k) {
        const int g = (tid + 256 * k) / kD;
        const int r = my_c >> 4, bl = my_c & 15;
        const int e = plain ? 0 : (int)min((__float_as_uint(top_s[g]) >> 23) & 0xFFu, 254u) - 127;
        q_op_s[0][r >> 2][4 * bl + g][r & 3] = ldexpf(q1_s[g][my_c], -e);
        q_op_s[1][r >> 2][4 * bl + g][r & 3] = ldexpf(q2_s[g][my_c], -e);
    }
    // Phasors of this lane's two channels, lane and lane + 64, at the wavefront's first t0, and of the step to its next.
    double pc[2], ps[2], step_c[2], step_s[2];
    phasor((double)(t_begin + T_first), th0, pc[0], ps[0]);
    phasor((double)(t_begin + T_first), th1, pc[1], ps[1]);
    step_c[0] = step_c[1] = step_s[0] = step_s[1] = 0.0;
    if (T_first + T_step < n_tok) {
        phasor((double)T_step, th0, step_c[0], step_s[0]);
        phasor((double)T_step, th1, step_c[1], step_s[1]);
    }
    lds_only_barrier();        // the queries give way to the table
    {
        // The table: thread (channel, half) takes 32 entries, each from the two before it: cos((n+1) x) = 2 cos x cos(n x) - cos((n-1) x),
        // and the sine alike (in double precision: what that loses for small angles is below 2^-40).
        const double th = (wave & 1) ? th1 : th0;
        const int half = tid >> 7;
        double c1, s1, c, s;
        phasor(1.0, th, c1, s1);
        phasor((double)(32 * half), th, c, s);
        double cb = c, sb = s;                                   // the one before
        turn(cb, sb, c1, -s1);
        const double twice = 2.0 * c1;
        f32x2* const row = (f32x2*)tab_raw + my_c * kSuper + 32 * half;
        const int sw = swizzle(my_c);
#pragma unroll 8
        for (int i = 0; i < 32; ++i) {
            row[i ^ sw] = f32x2{(float)c, (float)s};
            const double cn = fma(twice, c, -cb), sn = fma(twice, s, -sb);
            cb = c;
            sb = s;
            c = cn;
            s = sn;
        }
    }
    lds_only_barrier();

    const int a_head = j >> 2, a_par = (j >> 1) & 1, a_limb = j & 1;
    const uint32_t sel_even = a_par ? 0x01000c0cu : 0x0c0c0100u;
    const uint32_t sel_odd = a_par ? 0x03020c0cu : 0x0c0c0302u;
    // this lane's block of the value rows' exponent bytes: word of the row, and the rotation that brings the byte to the exponent field
    const int ve_word = NB == 8 ? j >> 3 : 0;
    const int ve_byte = ((8 * j) / N) & 3;
    const uint32_t ve_rot = (uint32_t)((8 * ve_byte + 32 - 23) & 31);

    float m_run = -INFINITY, l_run = 0.f;
    f32x4 o_acc[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) o_acc[m] = f32x4{0.f, 0.f, 0.f, 0.f};

    const f32x2* tab[16];                                        // by the swizzle
#pragma unroll
    for (int i = 0; i < 16; ++i) tab[i] = (const f32x2*)tab_raw + (lane ^ i);
    float* const ph = (float*)wave_s[wave];                      // [cos | sin][rh][b][x]
    uint16_t* const p_s = (uint16_t*)wave_s[wave];               // [limb][head][token]
    auto fence = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };

    for (int T0 = T_first; T0 < n_tok; T0 += T_step) {
        const int left = n_tok - T0;                             // cached tokens from T0 on (>= 1)
        // ---------------- value rows
        uint32_t vw[16][kValWords], vex[kExpWords];
        load_exponents(v_exp + (size_t)key_row(T0) * NB, vex);
        {
            const uint8_t* __restrict__ vp = v_mant + (size_t)T0 * kRowB;
            auto load = [&](const int i, const uint32_t at) {
                if constexpr (P == 4) {
                    vw[i][0] = __builtin_nontemporal_load((const uint32_t*)(vp + at));
                } else {
                    const u32x2 w = __builtin_nontemporal_load((const u32x2*)(vp + at));
                    vw[i][0] = w[0];
                    vw[i][kValWords - 1] = w[1];
                }
            };
            if (left >= kSuper) {                                // a complete tile: one offset per lane, the row as an immediate
                const uint32_t at = (uint32_t)(4 * kg * kRowB + j * P);
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int i = 0; i < 4; ++i) load(4 * u + i, at + (uint32_t)((16 * u + i) * kRowB));
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int i = 0; i < 4; ++i) load(4 * u + i, (uint32_t)(min(16 * u + 4 * kg + i, left - 1) * kRowB + j * P));
            }
        }
        // ---------------- the tile's query operands: lane (b, h), register r: channel 16 r + b of head h
        float A1[8], A2[8];
        fence();                                                 // (the probabilities of the tile before have been read)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            ph[((0 + i) * 16 + j) * 4 + kg] = (float)pc[i];      // channel lane + 64 i: r = 4 i + kg, b = j
            ph[((2 + i) * 16 + j) * 4 + kg] = (float)ps[i];
            turn(pc[i], ps[i], step_c[i], step_s[i]);
        }
        fence();
#pragma unroll
        for (int rh = 0; rh < 2; ++rh) {
            const f32x4 x = *(const f32x4*)q_op_s[0][rh][lane], y = *(const f32x4*)q_op_s[1][rh][lane];
            const f32x4 c = *(const f32x4*)&ph[((0 + rh) * 16 + (lane >> 2)) * 4], s = *(const f32x4*)&ph[((2 + rh) * 16 + (lane >> 2)) * 4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                A1[4 * rh + i] = fmaf(x[i], c[i], y[i] * s[i]);
                A2[4 * rh + i] = fmaf(y[i], c[i], -(x[i] * s[i]));
            }
        }

        // ---------------- scores: s[h] = head h, token `lane`
        float s[NH] = {0.f, 0.f, 0.f, 0.f};
        {
            const uint32_t next = key_row(T0 + T_step < n_tok ? T0 + T_step : n_tok);
            const uint8_t* __restrict__ const kp = k_mant + (size_t)next * kRowB;
            // 4 channels a step: while the matrix cores take the products of one step, the vector ALUs form those of the next and the
            // table entries of the one after it are read.  Every 16 channels the sums (of cosines and of sines, so that no matrix
            // instruction waits for the one before it) are multiplied by their block's power of two and added up.
            f32x2 t[2][4];
            float kc[2][4], ks[2][4];
            uint32_t lo, hi;                                     // P = 4: the dword's codes as FP8 bytes
            auto read = [&](auto G) {
                constexpr int g = decltype(G)::value;
#pragma unroll
                for (int x = 0; x < 4; ++x) t[g & 1][x] = tab[swizzle(4 * g + x)][(4 * g + x) * kSuper];
            };
            auto form = [&](auto G) {
                constexpr int g = decltype(G)::value;
                f16x2 k[2];                                      // P = 4: channels (0,2), (1,3); P = 8: (0,1), (2,3)
                if constexpr (P == 4) {
                    constexpr int d = g / 2;
                    if constexpr (g % 2 == 0) spread4(kw[d / 4][d % 4], lo, hi);
                    k[0] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(lo, 512.0f, g % 2 != 0);
                    k[1] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(hi, 512.0f, g % 2 != 0);
                } else {
                    spread8(kw[g / 4][g % 4], hi, lo);
                    k[0] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(hi, 4096.0f, false) + __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(lo, 512.0f, false);
                    k[1] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(hi, 4096.0f, true) + __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(lo, 512.0f, true);
                }
                if constexpr (4 * (g + 1) % (4 * kWord) == 0) kw[4 * g / (4 * kWord)] = *(const u32x4*)(kp + 16 * (4 * g / (4 * kWord)));
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const float v = P == 4 ? (float)k[x & 1][x >> 1] : (float)k[x >> 1][x & 1];
                    kc[g & 1][x] = fmaf(v, t[g & 1][x][0], 0.f);
                    ks[g & 1][x] = fmaf(v, t[g & 1][x][1], 0.f);
                }
            };
            f32x4 acc[2][2];
            auto finish = [&](auto Q) {                          // 16 channels; a code of byte E is worth 2^(E - 125 - P)
                constexpr int q = decltype(Q)::value, blk = 16 * q / N;
                const int e = (int)((kex[blk / 4] >> (8 * (blk & 3))) & 0xFFu) - (125 + P);
                if (plain) {
                    const float scale = ldexpf(1.0f, e);
#pragma unroll
                    for (int h = 0; h < NH; ++h) s[h] = fmaf(scale, acc[q & 1][0][h] + acc[q & 1][1][h], s[h]);
                } else {
#pragma unroll
                    for (int h = 0; h < NH; ++h) s[h] += ldexpf(acc[q & 1][0][h] + acc[q & 1][1][h], e + q_exp[h]);
                }
            };
            read(std::integral_constant<int, 0>{});
            read(std::integral_constant<int, 1>{});
            form(std::integral_constant<int, 0>{});
            __builtin_amdgcn_sched_barrier(0);
            static_for<kD / 4>([&](auto G) {
                constexpr int g = decltype(G)::value, q = g / 4;
                if constexpr (g % 4 == 0) acc[q & 1][0] = acc[q & 1][1] = f32x4{0.f, 0.f, 0.f, 0.f};
                if constexpr (g + 2 < kD / 4) read(std::integral_constant<int, (g + 2) % (kD / 4)>{});
                static_for<4>([&](auto X) {
                    constexpr int x = decltype(X)::value, c = 4 * g + x;
                    acc[q & 1][0] = __builtin_amdgcn_mfma_f32_4x4x1f32(A1[c / 16], kc[g & 1][x], acc[q & 1][0], 4, c % 16, 0);
                    acc[q & 1][1] = __builtin_amdgcn_mfma_f32_4x4x1f32(A2[c / 16], ks[g & 1][x], acc[q & 1][1], 4, c % 16, 0);
                });
                if constexpr (g + 1 < kD / 4) form(std::integral_constant<int, (g + 1) % (kD / 4)>{});
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x2, 2, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (g % 4 == 0 && q > 0) finish(std::integral_constant<int, q - 1 < 0 ? 0 : q - 1>{});
            });
            finish(std::integral_constant<int, 7>{});
            load_exponents(k_exp + (size_t)next * NB, kex);
        }
#pragma unroll
        for (int h = 0; h < NH; ++h) s[h] = lane < left ? s[h] : -INFINITY;
        {                                                        // now lane (j, kg): head kg, tokens 16u + j
            u32x4 w = {__float_as_uint(s[0]), __float_as_uint(s[1]), __float_as_uint(s[2]), __float_as_uint(s[3])};
            transpose_rows(w);
#pragma unroll
            for (int u = 0; u < 4; ++u) s[u] = __uint_as_float(w[u]);
        }

        // ---------------- online softmax
        bool light;                                              // the tile's probabilities are fp32 numbers (the same for a wavefront)
        {
            const float tmax = row_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
            const float m_new = fmaxf(m_run, tmax);
            const float m_ref = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = exp2f(m_run - m_ref);            // (keeps subnormal numbers)
            const float m_p = m_ref - (float)kShift;             // probabilities carry 2^kShift
            float psum = 0.f;
            fence();                                             // (the phasor has been read)
            // Below 2^-110 the third limb loses bits to bf16's smallest number, 2^-133, and below 2^-126 exp2_raw has none: a tile with
            // such a weight that fp32 still holds keeps them in fp32, which holds 24 bits down to 2^-126 and something down to 2^-149, and
            // takes fp32 multiply-adds for its values.  (A light token counts where its values are larger by as much.)
            constexpr float kLow = (float)kShift - 150.5f, kHigh = -109.5f;
            const float m_mid = m_p + 0.5f * (kLow + kHigh);
            const float off = fminf(fminf(fabsf(s[0] - m_mid), fabsf(s[1] - m_mid)), fminf(fabsf(s[2] - m_mid), fabsf(s[3] - m_mid)));
            const bool low = off < 0.5f * (kHigh - kLow);
            light = __builtin_amdgcn_ballot_w64(low) != 0;
            if (light) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float pw = exp2f(s[u] - m_ref);
                    ((float*)p_s)[kg * kSuper + 16 * u + j] = pw;
                    psum = fmaf(pw, (float)(1 << kShift), psum);
                }
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float pw = exp2_raw(s[u] - m_p);
                    float rest = pw;
#pragma unroll
                    for (int l = 0; l < PL; ++l) {
                        const __bf16 limb = (__bf16)rest;
                        rest -= (float)limb;
                        p_s[(l * NH + kg) * kSuper + 16 * u + j] = __builtin_bit_cast(unsigned short, limb);
                    }
                    psum += pw - rest;                           // what the limbs hold
                }
            }
            l_run = l_run * alpha + psum;
            m_run = m_new;
            if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
                for (int m = 0; m < 4; ++m) o_acc[m] *= alpha;
            }
        }
        // exponent bytes of this lane's value row: 1, 2 or above kTop?
        uint32_t out = 0;
#pragma unroll
        for (int w = 0; w < kExpWords; ++w) {
            const uint32_t low = vex[w] & 0x7F7F7F7Fu;
            const uint32_t small = ~(low + 0x7D7D7D7Du) & (low + 0x7F7F7F7Fu) & ~vex[w];
            const uint32_t large = (low + (0x7Fu - (kTop - 128u)) * 0x01010101u) & vex[w];
            out |= (small | large) & 0x80808080u;
            ve_s[wave][w][lane] = vex[w];
        }
        fence();

        // ---------------- values of the same 64 tokens
        if (!light && __builtin_amdgcn_ballot_w64(out != 0) == 0) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const u32x4 ve = *(const u32x4*)&ve_s[wave][ve_word][16 * u + 4 * kg];
                // bf16 pairs, one per MFMA: P = 4 channels (0,2), (4,6), (1,3), (5,7) of 8; P = 8 (0,1) .. (6,7), high and low pieces
                constexpr int kPieces = P == 4 ? 1 : 2;
                bf16x2 v[4][4][kPieces];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float scale = __uint_as_float(__builtin_amdgcn_alignbit(ve[i], ve[i], ve_rot));    // (nothing but the exponent field counts)
                    if constexpr (P == 4) {
                        uint32_t lo, hi;
                        spread4(vw[4 * u + i][0], lo, hi);
                        v[i][0][0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, scale, false);
                        v[i][1][0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, scale, true);
                        v[i][2][0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, scale, false);
                        v[i][3][0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, scale, true);
                    } else {
                        const float scale8 = __uint_as_float(__float_as_uint(scale) + (3u << 23));
#pragma unroll
                        for (int w = 0; w < kValWords; ++w) {
                            uint32_t lo, hi;
                            spread8(vw[4 * u + i][w], hi, lo);
                            v[i][2 * w][0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, scale8, false);
                            v[i][2 * w + 1][0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, scale8, true);
                            v[i][2 * w][kPieces - 1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, scale, false);
                            v[i][2 * w + 1][kPieces - 1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, scale, true);
                        }
                    }
                }
                // a third limb takes a second round with that limb in the rows of limb 0 and zeros in the others
#pragma unroll
                for (int round = 0; round < 2; ++round) {
                    uint2 pp = *(const uint2*)&p_s[((round == 0 ? a_limb : PL - 1) * NH + a_head) * kSuper + 16 * u + 4 * kg];
                    if (round == 1 && a_limb == 1) pp = make_uint2(0u, 0u);
                    const bf16x8 ap = __builtin_bit_cast(bf16x8, u32x4{__builtin_amdgcn_perm(pp.x, pp.x, sel_even), __builtin_amdgcn_perm(pp.x, pp.x, sel_odd),
                                                                       __builtin_amdgcn_perm(pp.y, pp.y, sel_even), __builtin_amdgcn_perm(pp.y, pp.y, sel_odd)});
#pragma unroll
                    for (int x = 0; x < kPieces; ++x)
#pragma unroll
                        for (int m = 0; m < 4; ++m)
                            o_acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ap, join(v[0][m][x], v[1][m][x], v[2][m][x], v[3][m][x]), o_acc[m], 0, 0, 0);
                }
            }
        } else {       // one by one: this lane's head kg, channels 8j ..
            const int count = min(left, kSuper);
#pragma unroll 1
            for (int t = 0; t < count; ++t) {
                float pw = 0.f;
                if (light) {
                    pw = ((const float*)p_s)[kg * kSuper + t];
                } else {
#pragma unroll
                    for (int l = 0; l < PL; ++l) pw += __uint_as_float((uint32_t)p_s[(l * NH + kg) * kSuper + t] << 16);
                    pw *= 1.0f / (float)(1 << kShift);
                }
                const uint32_t* const wp = (const uint32_t*)(v_mant + (size_t)(T0 + t) * kRowB + j * P);
                const float scale = ldexpf(1.0f, (int)((ve_s[wave][ve_word][t] >> (8 * ve_byte)) & 0xFFu) - (125 + P));
#pragma unroll
                for (int x = 0; x < 8; ++x) {                    // the accumulator of a channel is an even one's or an odd one's first row
                    const uint32_t code = (wp[x / kWord] >> (P * (x % kWord))) & ((1u << P) - 1u);
                    const float mag = (float)(code & ((1u << (P - 1)) - 1u));
                    const float value = ((code >> (P - 1)) ? -mag : mag) * scale;
                    // P = 4: pair 0 (0,2), 1 (4,6), 2 (1,3), 3 (5,7); P = 8: pair x / 2
                    const int m = pair_of<P>(x % kWord) + (P == 8 ? 2 * (x / kWord) : 0), row = 2 * half_of<P>(x % kWord);
                    o_acc[m][row] = fmaf(pw, value, o_acc[m][row]);
                }
            }
        }
    }

    // ---------------- per-wavefront result to LDS (nobody needs the table any more after the barrier)
    __syncthreads();
    {
        const float lsum = row_sum(l_run);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            // channels of pair m in a lane's 8
            const int even = P == 4 ? 4 * (m & 1) + (m >> 1) : 2 * m, odd = P == 4 ? even + 2 : even + 1;
            o_s[wave][kg][8 * j + even] = o_acc[m][0] + o_acc[m][1];
            o_s[wave][kg][8 * j + odd] = o_acc[m][2] + o_acc[m][3];
        }
        if (j == 0) {
            ml_s[wave][kg][0] = m_run;
            ml_s[wave][kg][1] = lsum * (1.0f / (float)(1 << kShift));
        }
    }
    __syncthreads();

    for (int i = tid; i < g_cnt * kD; i += 256) {
        const int g = i / kD, c = i % kD;
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) M = fmaxf(M, ml_s[w][g][0]);
        float acc = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const float mw = ml_s[w][g][0];
            if (mw > -INFINITY) acc = fmaf(exp2f(mw - M), o_s[w][g][c], acc);
        }
        if (a.direct) {
            float den = 0.f;
#pragma unroll
            for (int w = 0; w < kWaves; ++w)
                if (ml_s[w][g][0] > -INFINITY) den = fmaf(exp2f(ml_s[w][g][0] - M), ml_s[w][g][1], den);
            kvbfp::spans::write_output(a, dt, b, kvh, g_base + g, c, acc, den);
        } else {
            a.part_o[span.row(h0 + g) * kD + c] = acc;
        }
    }
    if (!a.direct && tid < g_cnt) {
        const int g = tid;
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) M = fmaxf(M, ml_s[w][g][0]);
        float lsum = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const float mw = ml_s[w][g][0];
            if (mw > -INFINITY) lsum = fmaf(exp2f(mw - M), ml_s[w][g][1], lsum);
        }
        float* ml = a.part_ml + span.row(h0 + g) * 2;
        ml[0] = M;
        ml[1] = lsum;
    }
}

template <int P>
hipError_t launch_rope(const DecodeArgs& a, int dt, int block, dim3 grid, hipStream_t s) {
    if (block == 16) decode_split_rope_f32<P, 16><<<grid, 256, 0, s>>>(a, dt);
    else if (block == 32) decode_split_rope_f32<P, 32><<<grid, 256, 0, s>>>(a, dt);
    else if (block == 64) decode_split_rope_f32<P, 64><<<grid, 256, 0, s>>>(a, dt);
    else if (block == 128) decode_split_rope_f32<P, 128><<<grid, 256, 0, s>>>(a, dt);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace

namespace kvbfp {

// Contiguous cache, all heads (a.g_base and a.g_cnt are not read).
hipError_t launch_decode_split_rope_f32(const DecodeArgs& a, int mant_bits, int dtype, int block, int batch, hipStream_t s) {
    if (a.block_table || !a.rope_theta || !a.rope_partner || !a.rope_sign) return hipErrorInvalidValue;
    const dim3 grid((unsigned)a.n_splits, (unsigned)((a.G + 3) / 4 * a.H_kv), (unsigned)batch);
    return mant_bits == 4 ? launch_rope<4>(a, dtype, block, grid, s) : launch_rope<8>(a, dtype, block, grid, s);
}

}  // namespace kvbfp
