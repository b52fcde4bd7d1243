// Fast split pass of decode attention for 4-bit mantissas on gfx950 (Sec. III run-time flow).
//
// Why matrix cores: with G query heads sharing one KV head, a cached element takes 2*G multiply-
// adds but arrives at 0.53 bytes.  At 8 TB/s the vector ALUs (64 lanes x 4 SIMDs x 256 CUs, one
// fp32 op per lane per clock without packed math) can spend about 2.5 instructions per element;
// unpacking a sign-magnitude nibble costs >= 1.25 of them, which leaves no room for even G = 1
// worth of dot2 instructions at full bandwidth, let alone G = 4.  The skinny products
// (G x 128) . (128 x T) and (G x T) . (T x 128) therefore go to the MFMA pipe, which is otherwise
// idle, and the vector ALUs only unpack.
//
// Unpacking without integer->float conversions: a code s|mmm widened to the byte s0000mmm is the
// OCP FP8-E4M3 subnormal (-1)^s * m * 2^-9, so v_cvt_scalef32_pk_bf16_fp8 turns two codes into
// two exact bf16 values and applies the block's power-of-two scale in the same instruction.
// Cost per 8 codes: 6 bit operations + 4 conversions.
//
// Score product  S = Q . K^T  (v_mfma_f32_16x16x32_bf16, A = query rows, B = keys):
//   lane (j = lane%16, kg = lane/16) loads the 16-byte chunk kg of the key row of token j
//   (32 channels, i.e. whole blocks) and feeds it to 4 MFMAs; A holds the query split into three
//   bf16 limbs (24 significant bits) in rows 4*head + limb, so the product keeps fp32 accuracy.
// Value product  O = P . V  (same instruction, A = probabilities, B = values):
//   the reduction index enumerates (token, channel parity): a converted register already holds
//   the two channels of one token, and the probabilities sit in rows (head, parity, limb) with
//   zeros in the other parity's slots, so no transposition of the 4-bit data is ever needed.
//   Lane (j, kg) loads dword j (8 channels) of the value rows of tokens 4kg..4kg+3.
// Each wavefront owns every fourth 64-token tile of its split and keeps its own online-softmax
// state; the four wavefronts of a workgroup merge once at the end.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>
#include <utility>

#include "decode_args.h"
#include "decode_dev.h"
#include "decode_spans.h"
#include "kvbfp_internal.h"
#include "quantize_dev.h"
#include "decode_lds.h"

namespace {

using kvbfp::DecodeArgs;

using namespace kvbfp::dev;

// A code m of a block with exponent byte E stands for m * 2^(E - 129).  Read as the FP8 subnormal
// m * 2^-9 and converted with the scale operand 2^(E - 127) -- the byte E itself in the exponent field,
// which is all the conversion looks at -- it becomes the bf16 value m * 2^(E - 136) = value * 2^-kShift,
// exact for every E >= 3 (bf16 keeps denormals down to 2^-133; blocks with E = 1, 2, magnitudes below
// 2^-124, lose low-order bits, an absolute error under 2^-126).  E = 255 (a block maximum within a
// factor 1.07 of the largest fp32 number) would read as an infinite scale and is not supported here.
constexpr int kShift = 7;

// N = block size, HG = groups of four query heads per KV head (G <= 4*HG).
// grid = (n_splits, H_kv, B), block = 256 (four wavefronts).
// PL = bf16 limbs of a probability: 2 (16 bits, enough for 16-bit outputs) or 3 (24 bits, fp32 outputs).
// PAGED: the planes are a pool of pages and every 16-token stage of a tile looks up its page (a separate instantiation: the
// contiguous case keeps its 32-bit offsets from one scalar base).
// THREE: three wavefronts per SIMD.  Otherwise two, whose registers hold the tiles in two instantiations without a branch around the
// requests.  Three do better over pages and with blocks of 128, whose exponents pass between lanes (12 x 8192 tokens over 16-token
// pages 41.8 us, 48.1 with two; blocks of 128 33.5 and 35.8); elsewhere plan_f32 (attention.hip) decides together with the splits.
template <int N, int HG, int PL, bool PAGED, bool SHARE, bool THREE = HG == 1 && (PAGED || N == 128)>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(THREE ? 3 : 2, 4)))
void decode_split_mfma_p4(DecodeArgs a, int dt) {
    constexpr int NB = kD / N;
    constexpr int NH = HG * 4;
    constexpr int kQStride = kD + 4;                            // (four heads side by side are read from different banks)
    __shared__ __align__(16) float q_s[NH][kQStride];           // scaled, permuted queries
    __shared__ __align__(16) uint16_t p_s[kWaves][HG][PL][4][kSuper];  // probabilities, bf16 limbs
    __shared__ float o_s[kWaves][NH][kD];                       // per-wavefront outputs for the merge
    __shared__ float ml_s[kWaves][NH][2];

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int j = lane & 15, kg = lane >> 4;
    const int len0 = SHARE ? kvbfp::spans::request_lengths(a, gridDim.z) : 0;
    kvbfp::spans::Span span;
    if (!kvbfp::spans::take<SHARE, true>(a, len0, 8, span)) return;
    const int split = span.split, kvh = blockIdx.y, b = span.b;
    const int h0 = kvh * a.G + a.g_base;      // first (virtual) head of this launch

    const int64_t L = span.L;
    // 256-token tiles are dealt out round-robin: split s takes tiles s, s + n, s + 2 n, ...;
    // "split-relative" tokens below count from t_begin
    const int64_t t_begin = (int64_t)split * 256;
    const int64_t t_end = L;

    if (t_begin >= t_end) {   // nothing cached in this split
        for (int i = tid; i < a.g_cnt * kD; i += 256) {
            if (!SHARE && a.direct == 1) kvbfp::spans::write_output(a, dt, b, kvh, a.g_base + i / kD, i % kD, 0.f, 0.f);
            else a.part_o[span.row(h0 + i / kD) * kD + (i % kD)] = 0.f;
        }
        if (tid < a.g_cnt) {
            float* ml = a.part_ml + span.row(h0 + tid) * 2;
            ml[0] = -INFINITY;
            ml[1] = 0.f;
        }
        return;
    }

    // Plane bases of this (batch, kv-head) are wave-uniform (scalar registers); everything inside
    // the split is addressed with 32-bit offsets from them.
    // (Paged cache: the bases are those of the pool and every 16-token stage of a tile looks up its page.)
    const int64_t base = PAGED ? 0 : ((int64_t)b * a.H_kv + kvh) * a.max_seq + t_begin;
    const uint8_t* __restrict__ k_mant = a.k_mant + base * 64;
    const uint8_t* __restrict__ v_mant = a.v_mant + base * 64;
    const uint8_t* __restrict__ k_exp = a.k_exp + base * NB;
    const uint8_t* __restrict__ v_exp = a.v_exp + base * NB;
    const int n_tok = (int)(t_end - t_begin);       // tokens from this split's first tile to the end of the sequence
    // several query tokens: head slot s sees tokens below lim[.] only (split-relative), and a tile counts
    // as full only if every head sees all of it
    const int n_vis = (int)(L - t_begin);
    const int n_full = min(n_tok, n_vis - (a.n_q_tokens - 1));
    int lim[HG];
#pragma unroll
    for (int hg = 0; hg < HG; ++hg) lim[hg] = n_vis - kvbfp::hidden_tokens(a, a.g_base + hg * 4 + kg);

    // exponent byte(s) of key chunk kg of a row
    const uint32_t ke_col = N == 16 ? 2u * kg : (N == 32 ? (uint32_t)kg : (N == 64 ? (uint32_t)(kg >> 1) : 0u));
    // The packed rows of one 64-token tile as this lane uses them: key chunk kg of rows 16u + j, value dword j of rows
    // 16u + 4kg + i, each with its exponent bytes.  The rows of the wavefront's next tile are requested as soon as these are
    // used up, keys before the softmax and values at the end of a tile, and those of the first tile before the set-up
    // (which waits for LDS only): a round trip to memory takes longer than the arithmetic of a tile.  4 x 8192 tokens, 8
    // kv-heads, blocks of 16, fp32 I/O: a call took 22.2 us with it, 32.6 with every tile's rows requested when they are needed (18.4 now,
    // with the query ahead of the rows, two tiles for every split and steady tiles); 10 x 8000 tokens, blocks of 32 35.3 against 55.1.
    struct Rows {
        u32x4 k[4];
        uint32_t ke[4], v[4][4], ve[4][N == 128 ? 1 : 4];      // (one exponent a row: that of row 16u + j, handed over where it is used)
    };
    auto fetch_keys = [&](const int T0, Rows& r) {
        kvbfp::StageBases sb{};
        if constexpr (PAGED) sb = kvbfp::stage_bases(a, b, kvh, t_begin + T0, t_end);
        const int left = n_tok - T0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const size_t base_u = PAGED ? (size_t)(sb.v[u] + t_begin + T0) : (size_t)T0;
            const uint8_t* __restrict__ kp = k_mant + base_u * 64;
            const uint8_t* __restrict__ kep = k_exp + base_u * NB;
            const uint32_t row = (uint32_t)min(16 * u + j, left - 1);        // rows past the last cached token re-read it
            r.k[u] = __builtin_nontemporal_load((const u32x4*)(kp + (row * 64u + (uint32_t)kg * 16u)));   // streamed once: keep it out of the caches' way
            if (N == 16) r.ke[u] = *(const uint16_t*)(kep + (row * NB + ke_col));
            else r.ke[u] = kep[row * NB + ke_col];
        }
    };
    auto fetch_values = [&](const int T0, Rows& r) {
        kvbfp::StageBases sb{};
        if constexpr (PAGED) sb = kvbfp::stage_bases(a, b, kvh, t_begin + T0, t_end);
        const int left = n_tok - T0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const size_t base_u = PAGED ? (size_t)(sb.v[u] + t_begin + T0) : (size_t)T0;
            const uint8_t* __restrict__ vp = v_mant + base_u * 64;
            const uint8_t* __restrict__ vep = v_exp + base_u * NB;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t row = (uint32_t)min(16 * u + 4 * kg + i, left - 1);
                r.v[u][i] = __builtin_nontemporal_load((const uint32_t*)(vp + (row * 64u + 4u * (uint32_t)j)));
                if constexpr (N != 128) r.ve[u][N == 128 ? 0 : i] = vep[row * NB + (uint32_t)((8 * j) / N)];
            }
            if constexpr (N == 128) r.ve[u][0] = vep[min(16 * u + j, left - 1)];
        }
    };
    const int T_first = wave * kSuper, T_step = span.n * kWaves * kSuper;     // this wavefront's tiles
    // The query as it lies in memory and its permutation ahead of the first tile's rows: loads return in order, and a load through
    // the permutation would be a round trip behind them.
    constexpr int kQPerThread = NH * kD / 256;
    uint32_t q_bits[kQPerThread];
#pragma unroll
    for (int k = 0; k < kQPerThread; ++k) {
        const int i = tid + 256 * k, g = i / kD;
        const int64_t idx = kvbfp::query_row(a, b, kvh, a.g_base + min(g, a.g_cnt - 1)) * kD + i % kD;   // clamped: rows beyond the count are zeroed below
        q_bits[k] = dt == KVBFP_F32 ? ((const uint32_t*)a.q)[idx] : (uint32_t)((const uint16_t*)a.q)[idx];
    }
    const int perm_c = a.perm_k ? (a.perm_k[kvh * kD + tid % kD] & (kD - 1)) : tid % kD;
    Rows rows;
    if (T_first < n_tok) {
        fetch_keys(T_first, rows);
        fetch_values(T_first, rows);
    }

    // q' = permuted query (optionally cast to BFP) * softmax_scale*log2(e) * 2^kShift; head slots beyond G are zero
    {
        const float two_k = (float)(1 << kShift);
        float* const raw = &o_s[0][0][0];           // [NH][kD], original channel order
#pragma unroll
        for (int k = 0; k < kQPerThread; ++k) {
            const int i = tid + 256 * k;
            const float f = dt == KVBFP_F32 ? __uint_as_float(q_bits[k]) : load_as_float(&q_bits[k], dt, 0);
            raw[i] = i / kD < a.g_cnt ? f : 0.f;
        }
        lds_only_barrier();
        float v[kQPerThread];
#pragma unroll
        for (int k = 0; k < kQPerThread; ++k) v[k] = raw[((tid + 256 * k) / kD) * kD + perm_c];
        if (a.q_mant_bits) {
            float* const cast = &o_s[1][0][0];      // [NH][kD], cache channel order
#pragma unroll
            for (int k = 0; k < kQPerThread; ++k) cast[tid + 256 * k] = v[k];
            lds_only_barrier();
            bfp_round_queries(cast, (uint32_t*)&o_s[2][0][0], NH, a.log2_block, a.q_mant_bits);
#pragma unroll
            for (int k = 0; k < kQPerThread; ++k) v[k] = cast[tid + 256 * k];
        }
#pragma unroll
        for (int k = 0; k < kQPerThread; ++k) q_s[(tid + 256 * k) / kD][tid % kD] = (v[k] * a.scale_log2e) * two_k;
        lds_only_barrier();
    }

    // A operands of the score product: row r = lane%16 = 4*head + limb, k-slot (kg, x) of MFMA d
    // is channel 32*kg + 8*d + slot_channel(x).
    bf16x8 aq[HG][4];
    {
        const int gi = j >> 2, limb = j & 3;
#pragma unroll
        for (int hg = 0; hg < HG; ++hg)
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const f32x4 q0 = *(const f32x4*)&q_s[hg * 4 + gi][32 * kg + 8 * d], q1 = *(const f32x4*)&q_s[hg * 4 + gi][32 * kg + 8 * d + 4];
#pragma unroll
                for (int x = 0; x < 8; ++x) {
                    const int c = slot_channel(x);
                    const float f = c < 4 ? q0[c & 3] : q1[c & 3];
                    const __bf16 l0 = (__bf16)f;
                    const float r1 = f - (float)l0;
                    const __bf16 l1 = (__bf16)r1;
                    const float r2 = r1 - (float)l1;
                    const __bf16 l2 = (__bf16)r2;
                    aq[hg][d][x] = limb == 0 ? l0 : (limb == 1 ? l1 : (limb == 2 ? l2 : (__bf16)0.0f));
                }
            }
    }

    // selectors that place a probability in the low (parity 0) or high (parity 1) half of an
    // A register of the value product; row r = j = 4*head + 2*parity + limb
    const int a_head = j >> 2, a_par = (j >> 1) & 1, a_limb = j & 1;
    const uint32_t sel_even = a_par ? 0x01000c0cu : 0x0c0c0100u;   // halfword 0 of the source
    const uint32_t sel_odd = a_par ? 0x03020c0cu : 0x0c0c0302u;    // halfword 1 of the source

    float m_run[HG], l_run[HG];
    f32x4 o_acc[HG][4];
#pragma unroll
    for (int hg = 0; hg < HG; ++hg) {
        m_run[hg] = -INFINITY;
        l_run[hg] = 0.f;
#pragma unroll
        for (int m = 0; m < 4; ++m) o_acc[hg][m] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    // One 64-token tile starting at token T0 of the split.  FULL: all 64 tokens are cached, no
    // clamping or masking; otherwise rows are clamped to the last cached token and masked.
    // Steady: the next tile is requested from all tiles but the last, which is the other instantiation whether it is full or not,
    // and so without a branch around the requests: with one the compiler cannot tell which of them are on their way, and waits
    // for a tile's values where it needs the keys.  The scheduling barriers keep the requests behind the last use of their
    // registers.  Blocks of 16, 8 kv-heads, 4 heads, with the branch and three wavefronts per SIMD (168 registers and spills) -> now:
    // 4 x 8192 tokens 20.7 -> 18.4 us, 32 x 8192 76.8 -> 62.6, 20 ragged sequences of up to 16384 36.1 -> 30.7.
    // Two groups of heads: with blocks of 16, 64 and 128 the second instantiation takes all 256 registers and spills up to 7, for no gain (4 x
    // 8192 tokens, 8 heads 23.6 us with it and 23.7, 1 x 32768 25.1 and 24.3, 8 x 16384 49.0 and 50.1, blocks of 128 8 x 8192 33.0 and 32.9); with
    // blocks of 32 it takes 255 and spills none, 1 % less in the mean of 370 calls (11 x 24162 tokens 93.9 -> 90.4 us, 2 x 32866 27.3 -> 26.2).
    constexpr bool kSteady = (HG == 1 || N == 32) && !PAGED && !THREE;
    auto tile = [&](const int T0, auto full_tag) {
        constexpr bool FULL = decltype(full_tag)::value;
        const int left = n_tok - T0;                 // cached tokens from T0 on (>= 1)

        // ---------------- scores of 64 tokens
        f32x4 s_acc[HG][4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const u32x4 raw = rows.k[u];
            const float sc0 = scale_operand(N == 16 ? (rows.ke[u] & 0xFFu) : rows.ke[u]);
            const float sc1 = N == 16 ? scale_operand(rows.ke[u] >> 8) : sc0;
#pragma unroll
            for (int hg = 0; hg < HG; ++hg) s_acc[hg][u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const Unpacked4 kk = unpack8_p4(raw[d], d < 2 ? sc0 : sc1);
                const bf16x8 bk = join(kk.p[0], kk.p[1], kk.p[2], kk.p[3]);
#pragma unroll
                for (int hg = 0; hg < HG; ++hg)
                    s_acc[hg][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aq[hg][d], bk, s_acc[hg][u], 0, 0, 0);
            }
        }
        const bool more = kSteady ? FULL : T0 + T_step < n_tok;       // wave-uniform
        if constexpr (kSteady) __builtin_amdgcn_sched_barrier(0);
        if (more) fetch_keys(T0 + T_step, rows);
        if constexpr (kSteady) __builtin_amdgcn_sched_barrier(0);

        // ---------------- online softmax; lane (j, kg) owns head kg of each group, tokens 16u + j
#pragma unroll
        for (int hg = 0; hg < HG; ++hg) {
            float s[4];
            float tmax = -INFINITY;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float v = s_acc[hg][u][0] + s_acc[hg][u][1] + s_acc[hg][u][2];   // the three limbs
                s[u] = (FULL || 16 * u + j < min(left, lim[hg] - T0)) ? v : -INFINITY;
                tmax = fmaxf(tmax, s[u]);
            }
            tmax = row_max(tmax);           // -inf only if this head sees none of the tile (several query tokens)
            const float m_new = fmaxf(m_run[hg], tmax);
            const float m_ref = m_new == -INFINITY ? 0.f : m_new;   // keeps the differences below well defined
            const float alpha = exp2_raw(m_run[hg] - m_ref);           // 0 on the first tile, 1 when the maximum stays
            const float m_p = m_ref - (float)kShift;                    // probabilities carry 2^kShift (values come as 2^-kShift)
            float psum = 0.f;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float pw = exp2_raw(s[u] - m_p);
                const __bf16 ph = (__bf16)pw;
                const float r1 = pw - (float)ph;
                const __bf16 pl = (__bf16)r1;
                p_s[wave][hg][0][kg][16 * u + j] = __builtin_bit_cast(unsigned short, ph);
                p_s[wave][hg][1][kg][16 * u + j] = __builtin_bit_cast(unsigned short, pl);
                if (PL == 3) {
                    const __bf16 p3 = (__bf16)(r1 - (float)pl);
                    p_s[wave][hg][PL - 1][kg][16 * u + j] = __builtin_bit_cast(unsigned short, p3);
                    psum += ((float)ph + (float)pl) + (float)p3;
                } else {
                    psum += (float)ph + (float)pl;
                }
            }
            l_run[hg] = l_run[hg] * alpha + psum;                   // per-lane partial; summed at the end
            m_run[hg] = m_new;
            // Rescale the running output only when some head's maximum moved (exact: alpha == 1
            // otherwise).  The accumulators sit in the MFMA result registers, so skipping saves the
            // round trip.  This lane's rows all belong to head kg.
            if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
                for (int m = 0; m < 4; ++m) o_acc[hg][m] *= alpha;
            }
        }

        // the probabilities just written are read back below by other lanes of this wavefront
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

        // ---------------- values of the same 64 tokens
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            Unpacked4 vv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t E = N == 128 ? (uint32_t)__shfl((int)rows.ve[u][0], 20 * kg + i) : rows.ve[u][N == 128 ? 0 : i];
                vv[i] = unpack8_p4(rows.v[u][i], scale_operand(E));
            }
#pragma unroll
            for (int hg = 0; hg < HG; ++hg) {
                // probabilities of tokens 16u + 4kg .. +3 for this lane's row (head, parity, limb); a third
                // limb takes a second round with that limb in the rows of limb 0 and zeros in the others
#pragma unroll
                for (int round = 0; round < (PL == 3 ? 2 : 1); ++round) {
                    uint2 pp = *(const uint2*)&p_s[wave][hg][round == 0 ? a_limb : PL - 1][a_head][16 * u + 4 * kg];
                    if (round == 1 && a_limb == 1) pp = make_uint2(0u, 0u);
                    uint32_t ar[4];
                    ar[0] = __builtin_amdgcn_perm(pp.x, pp.x, sel_even);
                    ar[1] = __builtin_amdgcn_perm(pp.x, pp.x, sel_odd);
                    ar[2] = __builtin_amdgcn_perm(pp.y, pp.y, sel_even);
                    ar[3] = __builtin_amdgcn_perm(pp.y, pp.y, sel_odd);
                    const bf16x8 ap = __builtin_bit_cast(bf16x8, u32x4{ar[0], ar[1], ar[2], ar[3]});
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        const bf16x8 bv = join(vv[0].p[m], vv[1].p[m], vv[2].p[m], vv[3].p[m]);
                        o_acc[hg][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ap, bv, o_acc[hg][m], 0, 0, 0);
                    }
                }
            }
        }
        if constexpr (kSteady) __builtin_amdgcn_sched_barrier(0);
        if (more) fetch_values(T0 + T_step, rows);
        if constexpr (kSteady) __builtin_amdgcn_sched_barrier(0);
        // the next tile overwrites the probability buffer
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };

    {
        int T0 = T_first;
        // (a tile with another one 256 tokens or more behind it is seen whole by every head: at most 63 tokens are hidden from one)
        for (; kSteady ? T0 + T_step < n_tok : T0 + kSuper <= n_full; T0 += T_step) tile(T0, std::true_type{});
        if (T0 < n_tok) tile(T0, std::false_type{});     // at most one ragged tile per wavefront
    }

    // ---------------- per-wavefront result to LDS: lane (j, kg) holds head kg, channels 8j..8j+7
#pragma unroll
    for (int hg = 0; hg < HG; ++hg) {
        const float lsum = row_sum(l_run[hg]);
        const int head = hg * 4 + kg;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            // rows (parity 0: hi, lo), (parity 1: hi, lo); MFMA m holds slots (m) -> channels below
            const int c_even = 8 * j + slot_channel(2 * m);       // parity 0 channel of pair m
            const int c_odd = 8 * j + slot_channel(2 * m + 1);    // parity 1 channel of pair m
            o_s[wave][head][c_even] = o_acc[hg][m][0] + o_acc[hg][m][1];
            o_s[wave][head][c_odd] = o_acc[hg][m][2] + o_acc[hg][m][3];
        }
        if (j == 0) {
            ml_s[wave][head][0] = m_run[hg];
            ml_s[wave][head][1] = lsum * (1.0f / (float)(1 << kShift));      // the probabilities carried 2^kShift
        }
    }
    __syncthreads();

    // ---------------- merge the four wavefronts, write this split's partial result
    for (int i = tid; i < a.g_cnt * kD; i += 256) {
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
        if (!SHARE && a.direct == 1) {
            float den = 0.f;
#pragma unroll
            for (int w = 0; w < kWaves; ++w)
                if (ml_s[w][g][0] > -INFINITY) den = fmaf(exp2f(ml_s[w][g][0] - M), ml_s[w][g][1], den);
            kvbfp::spans::write_output(a, dt, b, kvh, a.g_base + g, c, acc, den);
        } else {
            a.part_o[span.row(h0 + g) * kD + c] = acc;
        }
    }
    if ((SHARE || a.direct != 1) && tid < a.g_cnt) {
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


// The LDS-DMA pipeline (decode_lds.h) for 4-bit mantissas.
template <int N, int HG, bool PAGED, bool SHARE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu((N != 32 && HG == 2) ? 2 : 3, 4)))
void decode_split_lds_p4(DecodeArgs a, int dt) {
    kvbfp::lds::decode_split_lds_body<4, N, HG, PAGED, SHARE>(a, dt);
}

// The same with eight wavefronts, for calls whose workgroups take a sequence each (attention.hip has when and the figures).
template <int N, int HG, bool PAGED>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 4)))
void decode_split_lds_p4_w8(DecodeArgs a, int dt) {
    kvbfp::lds::decode_split_lds_body<4, N, HG, PAGED, false, false, 8>(a, dt);
}

// 16-bit I/O: the LDS pipeline, every block size.  fp32 I/O: the register-staged pass with three probability
// limbs and the three-limb bf16 query (the FP8 query limbs of the LDS pipeline carry 16 bits, too few for the
// 1e-5 bar).
template <int HG, bool PAGED, bool SHARE>
hipError_t launch_reg(const DecodeArgs& a, int dt, int block, bool three, dim3 grid, hipStream_t s) {
    if constexpr (HG == 1 && !PAGED) {
        if (three && block != 128) {
            if (block == 16) decode_split_mfma_p4<16, 1, 3, false, SHARE, true><<<grid, 256, 0, s>>>(a, dt);
            else if (block == 32) decode_split_mfma_p4<32, 1, 3, false, SHARE, true><<<grid, 256, 0, s>>>(a, dt);
            else if (block == 64) decode_split_mfma_p4<64, 1, 3, false, SHARE, true><<<grid, 256, 0, s>>>(a, dt);
            else return hipErrorInvalidValue;
            return hipGetLastError();
        }
    }
    if (block == 16) decode_split_mfma_p4<16, HG, 3, PAGED, SHARE><<<grid, 256, 0, s>>>(a, dt);
    else if (block == 32) decode_split_mfma_p4<32, HG, 3, PAGED, SHARE><<<grid, 256, 0, s>>>(a, dt);
    else if (block == 64) decode_split_mfma_p4<64, HG, 3, PAGED, SHARE><<<grid, 256, 0, s>>>(a, dt);
    else if (block == 128) decode_split_mfma_p4<128, HG, 3, PAGED, SHARE><<<grid, 256, 0, s>>>(a, dt);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

template <int HG, bool PAGED, bool SHARE>
hipError_t launch_lds(const DecodeArgs& a, int dt, int block, dim3 grid, hipStream_t s) {
    if (block == 16) decode_split_lds_p4<16, HG, PAGED, SHARE><<<grid, 256, 0, s>>>(a, dt);
    else if (block == 32) decode_split_lds_p4<32, HG, PAGED, SHARE><<<grid, 256, 0, s>>>(a, dt);
    else if (block == 64) decode_split_lds_p4<64, HG, PAGED, SHARE><<<grid, 256, 0, s>>>(a, dt);
    else if (block == 128) decode_split_lds_p4<128, HG, PAGED, SHARE><<<grid, 256, 0, s>>>(a, dt);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

template <int HG, bool PAGED>
hipError_t launch_lds_w8(const DecodeArgs& a, int dt, int block, dim3 grid, hipStream_t s) {
    if (block == 16) decode_split_lds_p4_w8<16, HG, PAGED><<<grid, 512, 0, s>>>(a, dt);
    else if (block == 32) decode_split_lds_p4_w8<32, HG, PAGED><<<grid, 512, 0, s>>>(a, dt);
    else if (block == 64) decode_split_lds_p4_w8<64, HG, PAGED><<<grid, 512, 0, s>>>(a, dt);
    else if (block == 128) decode_split_lds_p4_w8<128, HG, PAGED><<<grid, 512, 0, s>>>(a, dt);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

template <int HG, bool PAGED>
hipError_t launch_n(const DecodeArgs& a, int dt, int block, int waves, bool three, dim3 grid, hipStream_t s) {
    if (waves == 8) return launch_lds_w8<HG, PAGED>(a, dt, block, grid, s);
    if (dt == KVBFP_F32) return a.share_above ? launch_reg<HG, PAGED, true>(a, dt, block, three, grid, s) : launch_reg<HG, PAGED, false>(a, dt, block, three, grid, s);
    return a.share_above ? launch_lds<HG, PAGED, true>(a, dt, block, grid, s) : launch_lds<HG, PAGED, false>(a, dt, block, grid, s);
}

}  // namespace

namespace kvbfp {

hipError_t launch_decode_split_mfma(const DecodeArgs& a, int dtype, int block, int batch, int waves, bool three, hipStream_t s) {
    if (waves == 8 && (dtype == KVBFP_F32 || a.share_above)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)a.n_splits, (unsigned)a.H_kv, (unsigned)batch);
    if (a.block_table) return a.g_cnt <= 4 ? launch_n<1, true>(a, dtype, block, waves, three, grid, s) : launch_n<2, true>(a, dtype, block, waves, three, grid, s);
    return a.g_cnt <= 4 ? launch_n<1, false>(a, dtype, block, waves, three, grid, s) : launch_n<2, false>(a, dtype, block, waves, three, grid, s);
}

}  // namespace kvbfp
