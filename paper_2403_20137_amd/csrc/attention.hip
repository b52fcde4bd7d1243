// Decode attention over the packed BFP cache for gfx950 (Sec. III run-time flow: cached keys are
// read back in block format and multiplied with the permuted query; the rest is ordinary softmax
// attention; values are handled the same way).
//
// Split-K over the sequence: pass 1 gives every (batch, kv-head, split) its own workgroup, which
// streams its token range once, keeps an online softmax (running maximum m, normaliser l,
// unnormalised output o) for the query heads that share the KV head, and writes (m, l, o) to the
// workspace; pass 2 merges the splits with the usual log-sum-exp weights, normalises, restores the
// original channel order of the values and rounds once to the output type.
//
// All softmax arithmetic is done in base 2: the query is pre-multiplied by softmax_scale*log2(e),
// so exp(x) becomes the native 2^x.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <mutex>

#include "decode_args.h"
#include "decode_dev.h"
#include "decode_spans.h"
#include "kvbfp_internal.h"

using kvbfp::DecodeArgs;

namespace {

constexpr int kD = 128;
constexpr int kTile = kvbfp::kTokenTile;   // tokens per tile = threads per workgroup
constexpr int kHeadsPerWg = 4;             // query heads handled by one workgroup of the generic kernel


__device__ __forceinline__ float load_as_float(const void* p, int dt, int64_t i) {
    if (dt == KVBFP_F32) return ((const float*)p)[i];
    const uint32_t h = ((const uint16_t*)p)[i];
    if (dt == KVBFP_F16) return (float)__builtin_bit_cast(_Float16, (unsigned short)h);
    return __uint_as_float(h << 16);
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Signed integer value of a sign-magnitude code as a float.
template <int P>
__device__ __forceinline__ float code_value(uint32_t c) {
    const float m = (float)(c & ((1u << (P - 1)) - 1u));
    return (c >> (P - 1)) ? -m : m;
}

// Generic split pass: fp32 FMAs everywhere, any block size, any group size (query heads are processed
// four per workgroup; larger groups re-read the cache).  The fallback for what the matrix-core passes
// do not take: more than 32 (virtual) heads per kv-head with fp32 I/O, planes that are not 16-byte aligned.
// grid = (n_splits, H_kv * ceil(G/4), B), block = 256.
template <int P>
__global__ __launch_bounds__(kTile) void decode_split_generic(DecodeArgs a, int dt) {
    constexpr int kRowBytes = kD * P / 8;
    constexpr int kRowVec = kRowBytes / 16;
    __shared__ float qs[kHeadsPerWg][kD];
    __shared__ float sc[kHeadsPerWg][kTile];
    __shared__ float alpha_s[kHeadsPerWg];
    __shared__ float ored[4][kHeadsPerWg][kD];

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int split = blockIdx.x;
    const int gg_count = (a.G + kHeadsPerWg - 1) / kHeadsPerWg;
    const int kvh = blockIdx.y / gg_count;
    const int g0 = (blockIdx.y % gg_count) * kHeadsPerWg;
    const int n_act = min(kHeadsPerWg, a.G - g0);
    const int b = blockIdx.z;
    const int h0 = kvh * a.G + g0;   // first query head of this workgroup

    int64_t L = a.seq_len ? (int64_t)a.seq_len[b] : a.max_len;
    L = L < 0 ? 0 : (L > a.max_len ? a.max_len : L);
    // 256-token tiles are dealt out round-robin: split s takes tiles s, s + n_splits, s + 2 n_splits, ...
    const int64_t t_begin = (int64_t)split * kTile;
    const int64_t t_end = L;
    const int64_t tile_step = (int64_t)a.n_splits * kTile;
    const int nb = kD >> a.log2_block;

    if (t_begin >= t_end) {   // nothing cached in this split
        for (int i = tid; i < n_act * kD; i += kTile) {
            const int g = i / kD, j = i % kD;
            a.part_o[(((int64_t)b * a.H_q + h0 + g) * a.n_splits + split) * kD + j] = 0.f;
        }
        if (tid < n_act) {
            float* ml = a.part_ml + (((int64_t)b * a.H_q + h0 + tid) * a.n_splits + split) * 2;
            ml[0] = -INFINITY;
            ml[1] = 0.f;
        }
        return;
    }

    // q' = permuted query (optionally cast to BFP) times softmax_scale*log2(e); unused head slots are zero
    for (int i = tid; i < kHeadsPerWg * kD; i += kTile) {
        const int g = i / kD, j = i % kD;
        float v = 0.f;
        if (g < n_act) {
            const int c = a.perm_k ? (a.perm_k[kvh * kD + j] & (kD - 1)) : j;   // masked: device data the host cannot check
            v = load_as_float(a.q, dt, kvbfp::query_row(a, b, kvh, g0 + g) * kD + c);
        }
        qs[g][j] = a.q_mant_bits ? v : v * a.scale_log2e;
    }
    __syncthreads();
    if (a.q_mant_bits) {
        kvbfp::dev::bfp_round_queries(&qs[0][0], (uint32_t*)&sc[0][0], kHeadsPerWg, a.log2_block, a.q_mant_bits);
        for (int i = tid; i < kHeadsPerWg * kD; i += kTile) (&qs[0][0])[i] *= a.scale_log2e;
        __syncthreads();
    }

    float m_run = -INFINITY, l_run = 0.f;          // wave g owns head g0+g (uniform per wave)
    float o[kHeadsPerWg][2];
#pragma unroll
    for (int g = 0; g < kHeadsPerWg; ++g) o[g][0] = o[g][1] = 0.f;
    const int cp = lane;                            // V phase: channels 2cp, 2cp+1

    for (int64_t tile0 = t_begin; tile0 < t_end; tile0 += tile_step) {
        // rows of the planes are addressed as base + token; a paged cache with pages of 64 tokens or more has one
        // base per 64 tokens, the share of a wavefront in both phases below; with smaller pages every token looks
        // up its own row
        const int64_t tw = tile0 + wave * 64;
        const bool per_token = a.block_table != nullptr && a.log2_page < 6;
        const int64_t base = (tw < t_end && !per_token) ? kvbfp::cache_row(a, b, kvh, tw) - tw : 0;
        // ---- scores: one cached token per thread
        const int64_t t = tile0 + tid;
        float s[kHeadsPerWg];
#pragma unroll
        for (int g = 0; g < kHeadsPerWg; ++g) s[g] = -INFINITY;
        if (t < t_end) {
            uint4 raw[kRowVec];
            const int64_t krow = per_token ? kvbfp::cache_row(a, b, kvh, t) : base + t;
            const uint4* rp = (const uint4*)(a.k_mant + krow * kRowBytes);
#pragma unroll
            for (int i = 0; i < kRowVec; ++i) raw[i] = rp[i];
            const uint8_t* ep = a.k_exp + krow * nb;
#pragma unroll
            for (int g = 0; g < kHeadsPerWg; ++g) s[g] = 0.f;
#pragma unroll
            for (int c = 0; c < kD / 16; ++c) {      // 16 channels at a time (never straddles a block)
                const int E = ep[(c * 16) >> a.log2_block];
                const float scale = ldexpf(1.0f, E - 127 - (P - 2));
                float v[16];
                if (P == 4) {
                    const uint4 r = raw[c / 2];
                    const uint32_t w0 = (c & 1) ? r.z : r.x, w1 = (c & 1) ? r.w : r.y;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        v[i] = code_value<4>((w0 >> (4 * i)) & 0xFu);
                        v[8 + i] = code_value<4>((w1 >> (4 * i)) & 0xFu);
                    }
                } else {
                    const uint4 r = raw[c];
                    const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
                    for (int i = 0; i < 16; ++i) v[i] = code_value<8>((w[i / 4] >> (8 * (i % 4))) & 0xFFu);
                }
#pragma unroll
                for (int g = 0; g < kHeadsPerWg; ++g) {
                    float acc = 0.f;
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc = fmaf(qs[g][c * 16 + i], v[i], acc);
                    s[g] = fmaf(scale, acc, s[g]);
                }
            }
        }
#pragma unroll
        for (int g = 0; g < kHeadsPerWg; ++g)        // several query tokens: head slot g0+g does not see the last few tokens
            sc[g][tid] = t < L - kvbfp::hidden_tokens(a, g0 + g) ? s[g] : -INFINITY;
        __syncthreads();

        // ---- online softmax: wave g updates head g
        {
            const int g = wave;
            float sv[kTile / 64];
            float tmax = -INFINITY;
#pragma unroll
            for (int k = 0; k < kTile / 64; ++k) {
                sv[k] = sc[g][lane + 64 * k];
                tmax = fmaxf(tmax, sv[k]);
            }
            tmax = wave_max(tmax);                  // -inf only if this head sees none of the tile (several query tokens)
            const float m_new = fmaxf(m_run, tmax);
            const float m_ref = m_new == -INFINITY ? 0.f : m_new;
            float tsum = 0.f;
#pragma unroll
            for (int k = 0; k < kTile / 64; ++k) {
                const float pw = exp2f(sv[k] - m_ref);   // 2^-inf = 0 for padding
                sc[g][lane + 64 * k] = pw;
                tsum += pw;
            }
            tsum = wave_sum(tsum);
            const float al = exp2f(m_run - m_ref);       // 0 on the first tile
            l_run = l_run * al + tsum;
            m_run = m_new;
            if (lane == 0) alpha_s[g] = al;
        }
        __syncthreads();

        // ---- values: wave w takes tokens [64w, 64w+64) of the tile, lane = channel pair
#pragma unroll
        for (int g = 0; g < kHeadsPerWg; ++g) {
            const float al = alpha_s[g];
            o[g][0] *= al;
            o[g][1] *= al;
        }
        const int64_t tw0 = tile0 + wave * 64;
        const int cnt = (int)max((int64_t)0, min((int64_t)64, t_end - tw0));
        auto add_value_row = [&](const int k, const int64_t vrow) {
            const int E = a.v_exp[vrow * nb + ((2 * cp) >> a.log2_block)];
            const float scale = ldexpf(1.0f, E - 127 - (P - 2));
            float v0, v1;
            if (P == 4) {
                const uint32_t byte = a.v_mant[vrow * kRowBytes + cp];
                v0 = code_value<4>(byte & 0xFu) * scale;
                v1 = code_value<4>(byte >> 4) * scale;
            } else {
                const uint32_t two = ((const uint16_t*)(a.v_mant + vrow * kRowBytes))[cp];
                v0 = code_value<8>(two & 0xFFu) * scale;
                v1 = code_value<8>(two >> 8) * scale;
            }
#pragma unroll
            for (int g = 0; g < kHeadsPerWg; ++g) {
                const float pw = sc[g][wave * 64 + k];
                o[g][0] = fmaf(pw, v0, o[g][0]);
                o[g][1] = fmaf(pw, v1, o[g][1]);
            }
        };
        if (per_token) {      // its own loop: the look-up stays out of the common one
            for (int k = 0; k < cnt; ++k) add_value_row(k, kvbfp::cache_row(a, b, kvh, tw0 + k));
        } else {
            for (int k = 0; k < cnt; ++k) add_value_row(k, base + tw0 + k);
        }
        __syncthreads();   // sc and alpha_s are rewritten by the next tile
    }

    // ---- merge the four token slices and write the partial result of this split
#pragma unroll
    for (int g = 0; g < kHeadsPerWg; ++g) {
        ored[wave][g][2 * cp] = o[g][0];
        ored[wave][g][2 * cp + 1] = o[g][1];
    }
    __syncthreads();
    for (int i = tid; i < n_act * kD; i += kTile) {
        const int g = i / kD, j = i % kD;
        const float v = ored[0][g][j] + ored[1][g][j] + ored[2][g][j] + ored[3][g][j];
        a.part_o[(((int64_t)b * a.H_q + h0 + g) * a.n_splits + split) * kD + j] = v;
    }
    if (lane == 0 && wave < n_act) {
        float* ml = a.part_ml + (((int64_t)b * a.H_q + h0 + wave) * a.n_splits + split) * 2;
        ml[0] = m_run;
        ml[1] = l_run;
    }
}

__device__ __forceinline__ uint16_t narrow_bf16(float v) {
    uint32_t u = __float_as_uint(v);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// Pass 2: merge the splits of one (batch, query head).  block = 512 threads: kChan channels times 512 / kChan
// slices of the splits; grid = (H_q, B, 128 / kChan).  A round trip to memory costs far more than anything computed
// here, so every thread first puts kCombineBatch partial-output loads in flight (enough for all splits in one go
// up to kCombineBatch * slices of them), then the (m, l) pairs go through LDS, and the slices are added through LDS
// at the end.  Few (batch, head) pairs with many splits -- one long sequence -- take the 32-channel form: four
// times the workgroups, a quarter of the bytes through each compute unit.
constexpr int kCombineThreads = 512;
template <int kCombineBatch, int kChan, bool SHARED>
__global__ __launch_bounds__(kCombineThreads) void decode_combine(DecodeArgs a, int dt) {
    constexpr int kSlices = kCombineThreads / kChan;
    constexpr int kMaxLds = 1024;
    __shared__ float m_s[kMaxLds];
    __shared__ float l_s[kMaxLds];
    __shared__ float red[kSlices][2][kChan];
    __shared__ float red_m[kSlices];
    const int jl = threadIdx.x % kChan, sl = threadIdx.x / kChan;
    const int j = blockIdx.z * kChan + jl;      // channel (cache order)
    const int h = blockIdx.x, b = blockIdx.y;
    int at = -1, count = 0;
    if (SHARED) {
        at = a.places[2 * b];
        count = a.places[2 * b + 1];
    }
    kvbfp::spans::Parts parts = kvbfp::spans::parts_of(a, b, h);

    // where this channel goes in the output row: requested with the partial outputs, not after the sums (a load here
    // costs nothing, at the end it is one more round trip to memory)
    const int kvh = h / a.G;
    const int c_raw = a.perm_v ? a.perm_v[kvh * kD + j] : j;
    float v[kCombineBatch];                     // first batch of this thread's partial outputs: splits sl + kSlices k
    auto first_batch = [&] {
#pragma unroll
        for (int k = 0; k < kCombineBatch; ++k) {
            const int i = sl + k * kSlices;
            v[k] = i < parts.n ? a.part_o[(parts.first + i * parts.step) * kD + j] : 0.f;
        }
    };
    first_batch();
    if (SHARED && at >= 0) {                    // (requested where they are if nothing was shared out, without waiting for the table)
        parts = kvbfp::spans::shared_parts(a, at, count, h);
        first_batch();
    }
    const float* const ml = a.part_ml + parts.first * 2;
    const float* const po = a.part_o + parts.first * kD;
    const int n = parts.n;
    const bool staged = n <= kMaxLds;           // otherwise (m, l) are read from global memory each time
    if (staged) {
        for (int i = threadIdx.x; i < n; i += kCombineThreads) {
            const float2 t = *(const float2*)(ml + 2 * i * parts.step);
            m_s[i] = t.x;
            l_s[i] = t.y;
        }
        __syncthreads();
    }
    auto m_of = [&](int i) { return staged ? m_s[i] : ml[2 * i * parts.step]; };
    auto l_of = [&](int i) { return staged ? l_s[i] : ml[2 * i * parts.step + 1]; };
    // Each slice works relative to the maximum of its own splits (a short, unrolled scan instead of
    // one long serial loop over all of them); the slices are brought to the common maximum at the end.
    float mk[kCombineBatch];
    float Ms = -INFINITY;
#pragma unroll
    for (int k = 0; k < kCombineBatch; ++k) {
        const int i = sl + k * kSlices;
        mk[k] = i < n ? m_of(i) : -INFINITY;
        Ms = fmaxf(Ms, mk[k]);
    }
    for (int i = sl + kCombineBatch * kSlices; i < n; i += kSlices) Ms = fmaxf(Ms, m_of(i));
    float num = 0.f, den = 0.f;
    if (Ms > -INFINITY) {                       // empty splits carry m = -inf -> weight 0
#pragma unroll
        for (int k = 0; k < kCombineBatch; ++k) {
            const int i = sl + k * kSlices;
            if (i < n) {
                const float w = exp2f(mk[k] - Ms);
                num = fmaf(w, v[k], num);
                den = fmaf(w, l_of(i), den);
            }
        }
        for (int i = sl + kCombineBatch * kSlices; i < n; i += kSlices) {
            const float w = exp2f(m_of(i) - Ms);
            num = fmaf(w, po[i * parts.step * kD + j], num);
            den = fmaf(w, l_of(i), den);
        }
    }
    red[sl][0][jl] = num;
    red[sl][1][jl] = den;
    if (jl == 0) red_m[sl] = Ms;
    __syncthreads();
    if (sl != 0) return;
    float M = -INFINITY;
#pragma unroll
    for (int k = 0; k < kSlices; ++k) M = fmaxf(M, red_m[k]);
    num = 0.f;
    den = 0.f;
    if (M > -INFINITY) {
#pragma unroll
        for (int k = 0; k < kSlices; ++k) {
            const float w = exp2f(red_m[k] - M);        // 0 for a slice without cached tokens
            num = fmaf(w, red[k][0][jl], num);
            den = fmaf(w, red[k][1][jl], den);
        }
    }
    const float r = den > 0.f ? num / den : 0.f;
    const int c = c_raw & (kD - 1);             // masked: the store stays inside the row
    const int64_t oi = kvbfp::query_row(a, b, kvh, h % a.G) * kD + c;
    if (dt == KVBFP_F32) ((float*)a.out)[oi] = r;
    else if (dt == KVBFP_F16) ((uint16_t*)a.out)[oi] = __builtin_bit_cast(unsigned short, (_Float16)r);
    else ((uint16_t*)a.out)[oi] = narrow_bf16(r);
}

// The same for up to 32 splits with a wavefront per (batch, query head), two channels per lane: no barrier, every
// partial output of the head in flight at once, four heads per workgroup.  With 32 virtual heads or more per kv-head the
// partial outputs are tens of megabytes and this is a streaming pass: bound by memory there (8192 heads, 8 splits, 34 MB:
// 20.6 us with a 512-thread workgroup per head, 8.2 us with this one), by the launch and one round trip otherwise (4.6 us).
constexpr int kRowSplits = 32;
template <bool SHARED>
__global__ __launch_bounds__(256) void decode_combine_rows(DecodeArgs a, int dt, int batch) {
    __shared__ float out_s[4][kD];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int bh = blockIdx.x * 4 + wave;       // b * H_q + h
    if (bh >= batch * a.H_q) return;
    const int b = bh / a.H_q, h = bh % a.H_q;
    const int kvh = h / a.G;
    const int n = a.n_splits;                   // <= kRowSplits
    int at = -1, count_all = 0;                 // (requested with the rows: where nothing was shared out it costs no time)
    if (SHARED) {
        at = a.places[2 * b];
        count_all = a.places[2 * b + 1];
    }
    const float2 ml = lane < n ? ((const float2*)a.part_ml)[(int64_t)bh * n + lane] : make_float2(-INFINITY, 0.f);
    const float2* const po = (const float2*)(a.part_o + (int64_t)bh * n * kD) + lane;
    float2 v[kRowSplits];
#pragma unroll
    for (int i = 0; i < kRowSplits; i += 4) {
        if (i < n) {                            // (wave-uniform; the clamped loads of the last four are not used)
#pragma unroll
            for (int k = 0; k < 4; ++k) v[i + k] = po[min(i + k, n - 1) * (kD / 2)];
        }
    }
    int c0 = 2 * lane, c1 = 2 * lane + 1;
    if (a.perm_v) {
        c0 = a.perm_v[kvh * kD + c0] & (kD - 1);         // masked: the store stays inside the row
        c1 = a.perm_v[kvh * kD + c1] & (kD - 1);
    }
    // adds 32 or fewer partial results, (m, l) of one per lane and two channels of each in v, to what is merged so far
    float M = -INFINITY, den = 0.f, n0 = 0.f, n1 = 0.f;
    auto merge = [&](const float2 t, const int count) {
        const float M_new = fmaxf(M, wave_max(t.x));
        const float ref = M_new > -INFINITY ? M_new : 0.f;
        const float w = exp2f(t.x - ref);                // 0 for a split without cached tokens
        const float was = exp2f(M - ref);
        den = den * was + wave_sum(w * t.y);
        n0 *= was;
        n1 *= was;
        M = M_new;
#pragma unroll
        for (int i = 0; i < kRowSplits; i += 4) {
            if (i < count) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (k > 0 && i + k >= count) break;      // (not by a weight of 0: a sum beyond fp32 is infinite)
                    const float wi = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w), i + k));
                    n0 = fmaf(wi, v[i + k].x, n0);
                    n1 = fmaf(wi, v[i + k].y, n1);
                }
            }
        }
    };
    if (SHARED && at >= 0) {
        // other rows, and more than 32 of them for a long sequence among short ones
        const kvbfp::spans::Parts p = kvbfp::spans::shared_parts(a, at, count_all, h);
        for (int i0 = 0; i0 < p.n; i0 += kRowSplits) {
            const int count = min(p.n - i0, kRowSplits);
            const int64_t r0 = p.first + i0 * p.step;
            const float2 t = lane < count ? ((const float2*)a.part_ml)[r0 + lane * p.step] : make_float2(-INFINITY, 0.f);
#pragma unroll
            for (int i = 0; i < kRowSplits; i += 4) {
                if (i < count) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) v[i + k] = ((const float2*)(a.part_o + (r0 + min(i + k, count - 1) * p.step) * kD))[lane];
                }
            }
            merge(t, count);
        }
    } else {
        merge(ml, n);
    }
    out_s[wave][c0] = den > 0.f ? n0 / den : 0.f;
    out_s[wave][c1] = den > 0.f ? n1 / den : 0.f;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const float r0 = out_s[wave][2 * lane], r1 = out_s[wave][2 * lane + 1];
    const int64_t oi = kvbfp::query_row(a, b, kvh, h % a.G) * kD + 2 * lane;
    if (dt == KVBFP_F32) {
        ((float*)a.out)[oi] = r0;
        ((float*)a.out)[oi + 1] = r1;
    } else {
        const uint16_t h0 = dt == KVBFP_F16 ? __builtin_bit_cast(unsigned short, (_Float16)r0) : narrow_bf16(r0);
        const uint16_t h1 = dt == KVBFP_F16 ? __builtin_bit_cast(unsigned short, (_Float16)r1) : narrow_bf16(r1);
        uint16_t* const p = (uint16_t*)a.out + oi;
        if (((uintptr_t)a.out & 3u) == 0) {
            *(uint32_t*)p = (uint32_t)h0 | ((uint32_t)h1 << 16);
        } else {
            p[0] = h0;
            p[1] = h1;
        }
    }
}

int log2_exact(int v) {
    int l = 0;
    while ((1 << l) < v) ++l;
    return l;
}

}  // namespace

using namespace kvbfp;

extern "C" {

// Workspace: the partial results of the splits, and behind them the table of places (DecodeArgs::places) where it may be used.
static size_t rows_bytes(const kvbfp_layout* L, int32_t n_q_heads, int32_t n_splits) {
    return (size_t)L->batch * (size_t)n_q_heads * (size_t)n_splits * (size_t)(kD + 2) * sizeof(float);
}
static size_t places_bytes(const kvbfp_layout* L) { return (size_t)L->batch * 2 * sizeof(int32_t); }
// Tiles of a sequence above which the workgroups are shared out by the lengths (0: nowhere).  A split of the longest sequence
// has T / n_splits tiles, and with B sequences sharing out leaves it at best a B-th of them; what it has to save for that to
// pay (`tiles`) depends on the time of a tile, see share_from.
static int64_t share_above(const kvbfp_layout* L, int32_t n_splits, int64_t max_len, int log2_tile, float tiles) {
    if (L->batch < 2 || L->batch > kvbfp::kMaxShared || n_splits < 2) return 0;
    const int64_t above = (int64_t)(tiles * (float)n_splits * (float)L->batch / (float)(L->batch - 1));
    return ((max_len + (1 << log2_tile) - 1) >> log2_tile) > above ? above : 0;
}
// Lengths log-uniform from 16, one call, kept -> shared out: 4-bit mantissas 3 x 16384 tokens, 32 kv-heads (saves 5.3 tiles)
// 22.5 -> 25.4 us, 8 x 16384 (4.7) 17.1 -> 19.0, 12 x 16384 (7.3) 22.7 -> 20.7, 48 x 4096 (7.8) 22.2 -> 19.4; 8 bits 20 x 1024
// (1.3) 15.1 -> 14.6, 20 x 2048 (2.5) 19.1 -> 15.5; rotation 20 x 1024 (1.3) 24.8 -> 23.3, 8 x 4096 (1.8) 23.4 -> 20.1; fp32 8 x
// 4096 (1.2) 14.8 -> 15.0, 20 x 2048 (1.9) 19.6 -> 17.6; 12 heads 3 x 4096 (1.3) 15.9 -> 18.7, 8 x 2048 (1.8) 15.9 -> 15.2;
// 128 heads, tiles of 64, 3 x 8192 (4.1) 37.9 -> 40.1, 20 x 1024 (5.1) 41.3 -> 39.7.  With more than 16 splits the longest
// sequence gets more places than the combine pass merges at once: 8 bits 3 x 16384 (2.0) 19.1 -> 22.2, 12 heads 3 x 8192 (2.0)
// 20.9 -> 24.2.
static float share_from(bool f32, int mant_bits, int G, bool rope, int32_t n_splits) {
    if (G > 32 && !rope && !f32) return 4.2f;
    if (!rope && !f32 && G <= 8 && mant_bits == 4) return 6.0f;
    if (n_splits > 16) return 2.1f;
    if (f32 && G <= 4) return 1.85f;
    return G > 8 && !rope && !f32 ? 1.5f : 1.2f;
}

size_t kvbfp_decode_workspace_bytes(const kvbfp_layout* L, int32_t n_q_heads, int64_t max_len) {
    clear_error();
    if (check_device_layout(L) != KVBFP_OK) return 0;
    if (n_q_heads <= 0 || n_q_heads % L->n_kv_heads != 0 || max_len <= 0 || max_len > L->max_seq) {
        fail(KVBFP_ERR_INVALID_ARG, "decode_workspace_bytes: bad n_q_heads/max_len");
        return 0;
    }
    const SplitPlan sp = plan_splits(L, n_q_heads, max_len);
    // (a pass that takes fewer splits than these has room for the table anyway)
    const int G = n_q_heads / L->n_kv_heads;
    const int log2_tile = G > 8 ? plan_wide(G, 1, 1, 1).log2_tile : 8;
    // (the I/O type and the rotation are not known here: the least of share_from; above 32 heads one pass shares)
    const float from = G > 32 ? share_from(false, L->mant_bits, G, false, sp.n_splits) : 1.2f;
    const bool may_share = share_above(L, sp.n_splits, max_len, log2_tile, from) != 0;
    return rows_bytes(L, n_q_heads, sp.n_splits) + (may_share ? places_bytes(L) : 0);
}

// What the variants of the decode call add to the plain one; the defaults are the plain call.
struct DecodeExtras {
    int32_t q_mant_bits = 0;                 // query cast to BFP first (kvbfp_decode_attention_qbfp)
    float* kernel_ms = nullptr;              // HOST float[2]: wait and return the two kernel durations
    const void* k_new = nullptr;             // the current token, appended first (kvbfp_append_decode_attention)
    const void* v_new = nullptr;
    int64_t new_stride_b = 0, new_stride_h = 0;
    int32_t n_q_tokens = 1;                  // kvbfp_decode_attention_multi
    const float* rope_theta = nullptr;       // rotation at read (kvbfp_decode_attention_rope)
    const int32_t* rope_partner = nullptr;
    const float* rope_sign = nullptr;
    const Paging* paging = nullptr;          // L is a pool of pages (kvbfp_decode_attention_paged)
    // kvbfp_decode_attention_profile_ring: with kernel_ms, the split pass is launched `reps` times back to back over
    // the caches ring[0], ring[1], ... (cyclically) between the first two events, then the combine pass `reps`
    // times between the last two; the durations returned are per launch.
    const kvbfp_cache* ring = nullptr;
    int32_t ring_len = 0, reps = 1;
};

// fp32 I/O, 4-bit mantissas, up to four heads, one region per sequence, blocks of up to 64: splits (at most the n that the workspace has room
// for) of `units` (sequence, kv-head) pairs of `tiles` 256-token tiles; lengths: they may differ.  Two workgroups per compute unit with the
// steady tiles of decode_mfma.hip, or (true) three of the form with a branch around the requests.  Of some 14000 calls of any shape, full and ragged,
// two rounded down to one resident round are within 1 % of the better one up to 256 units, three 6 to 18 % behind: 8 kv-heads, three -> two,
// 4 x 4352 tokens 18.2 -> 17.3 us, 4 x 9216 25.0 -> 21.1, 20 x 16384 99 -> 79, lengths log-uniform 16 x 8192 25.7 -> 20.7.  (Where three are
// just enough for a tile each, they can be faster: 8 sequences log-uniform up to 35970, 2 kv-heads 19.6 and 25.2.)  But
// - 171 to 192 units leave a quarter of the places empty as two and none as three: long sequences take three (two and three as multiples of
//   the better one: 17 to 32 tiles 1.05 and 1.01, 33 to 48 1.05 and 1.00; lengths that differ, 9 to 12 1.03 and 1.02, 13 to 16 1.08 and 1.00, beyond
//   1.05 to 1.13 and 1.00).  So do 5 and 6 tiles there with lengths, whose two-tile splits by the actual lengths (kPaired) a test holds: 24.2 and 20.4 us.
// - 257 to 512 units would have a split each or two, which are more than fit: one while the longest place, which then is the longest sequence,
//   is short (three, one, two splits: 48 x 1024 25.7, 21.3, 25.7 us, ragged 19.7, 17.3, 20.8; 64 x 2048 49.3, 35.4, 43.0, ragged 32.3, 28.7,
//   29.2), two beyond (33 x 4096 55.4, 55.8, 50.3; ragged 64 x 4096 40.4, 45.6, 36.5, 64 x 16384 83.8, 139, 70.9).  Equal lengths of more than 384 units
//   always take one (64 x 8192 143.7, 116.4, 120.5).  With lengths, 301 to 384 units take their two as three workgroups per compute unit, which fit
//   (7 to 24 tiles, two and three: log-uniform 1.07 to 1.11 and 1.00 to 1.04 times the better one, uniform 1.02 to 1.08 and 1.01 to 1.06, but all
//   equal 1.00 to 1.03 and 1.04 to 1.12).
// - More than 512 likewise, one up to 4096 tokens (ragged 65 x 3000 39.6, 32.0, 35.4, 65 x 4096 43.3, 39.5, 38.0; 65 x 8192 57.7, 68.4, 49.9).  Few tiles
//   take three where these are fewer rounds (not from 769 to 1024 units): one tile 1.18 to 1.28 as two and 1.00 to 1.01 as three, two 1.03 to 1.14
//   and 1.00 to 1.02, three 1.01 to 1.03 and 1.03 to 1.06 up to 640 units, 1.02 to 1.06 and 1.01 to 1.02 from there, four 1.02 and 1.03 up to
//   1536 units, 1.03 to 1.04 and 1.02 beyond, five 1.00 to 1.02 and 1.03 to 1.18.
static bool plan_f32(int64_t units, int64_t tiles, bool lengths, int32_t& n) {
    if (units > 512) {
        if (!lengths || tiles <= 16) n = 1;
        return n == 1 && (units <= 768 || units > 1024) && tiles <= (units <= 640 ? 2 : units <= 1536 ? 3 : 4);
    }
    if (units > 256) {
        n = std::min(n, (lengths ? tiles <= units / 42 : units > 384 || tiles <= 8) ? 1 : 2);
        return n == 2 && lengths && units > 300 && units <= 384;
    }
    const int32_t fit2 = (int32_t)(512 / units), fit3 = std::min(n, (int32_t)(768 / units));
    const bool three = units * fit2 <= 384 && (tiles > (lengths ? 12 : 16) || (lengths && tiles > 2 * fit2 && kvbfp::spans::paired_splits(fit3, tiles) != fit3));
    n = three ? fit3 : std::min(n, fit2);
    return three;
}

// Rotation at read in fp32, more than four heads, no lengths: splits (at most n) of `workgroups` (sequence, kv-head, four heads) of `tiles`
// 256-token tiles, two resident per compute unit.  Those with the shortest of up to two rounds, a round being half a tile's time and the tiles of a
// workgroup: of some 3300 calls none is slower than with a launch for every four heads, where one round at most (two where it would
// be less than two splits) was up to 13 % slower (17 x 8 units x 8 heads of 700 tokens, 8 bits 40.2 us, now 33.2; 12 x 8 x 5 heads of
// 9000 tokens 166 and 143).
static int32_t plan_rope_groups(int64_t workgroups, int64_t tiles, int32_t n) {
    int32_t best = 1;
    int64_t best_time = INT64_MAX;
    for (int32_t i = 1; i <= n; ++i) {
        const int64_t rounds = (i * workgroups + 511) / 512, time = rounds * (1 + 2 * ((tiles + i - 1) / i));
        if ((i > 1 && rounds > 2) || time >= best_time) continue;
        best = i;
        best_time = time;
    }
    return best;
}

static int decode_impl(const kvbfp_layout* L, const kvbfp_cache* cache, int32_t n_q_heads,
                       const void* q, kvbfp_dtype dtype, const int32_t* seq_len_dev,
                       int64_t max_len, float softmax_scale, const int32_t* perm_k,
                       const int32_t* perm_v, void* out, void* workspace, size_t workspace_bytes,
                       void* hip_stream, const DecodeExtras& x = DecodeExtras{}) {
    const int32_t q_mant_bits = x.q_mant_bits, n_q_tokens = x.n_q_tokens;
    float* const kernel_ms = x.kernel_ms;
    const void* const k_new = x.k_new;
    const void* const v_new = x.v_new;
    const int64_t new_stride_b = x.new_stride_b, new_stride_h = x.new_stride_h;
    const float* const rope_theta = x.rope_theta;
    const int32_t* const rope_partner = x.rope_partner;
    const float* const rope_sign = x.rope_sign;
    const Paging* const paging = x.paging;
    clear_error();
    kvbfp_layout logical;
    const kvbfp_layout* pool = L;
    if (paging) {
        if (int rc = check_paging(pool, *paging, &logical)) return rc;
        L = &logical;             // from here on: what the sequences look like
    }
    const bool rope = rope_theta || rope_partner || rope_sign;
    if (rope && !(rope_theta && rope_partner && rope_sign))
        return fail(KVBFP_ERR_INVALID_ARG, "decode_attention_rope: rope_theta, rope_partner and rope_sign are all needed");
    if (rope && (q_mant_bits != 0 || n_q_tokens != 1 || k_new || v_new))
        return fail(KVBFP_ERR_UNSUPPORTED, "decode_attention_rope: plain single-token decode only");
    if (n_q_tokens < 1 || n_q_tokens > 64)
        return fail(KVBFP_ERR_INVALID_ARG, "decode_attention: n_q_tokens = %d (1..64)", n_q_tokens);
    if (q_mant_bits != 0 && q_mant_bits != 4 && q_mant_bits != 8)
        return fail(KVBFP_ERR_INVALID_ARG, "decode_attention: q_mant_bits = %d (0, 4 or 8)", q_mant_bits);
    if (int rc = check_device_layout(L)) return rc;
    if (int rc = check_cache(cache, true, true)) return rc;
    if (!q || !out) return fail(KVBFP_ERR_INVALID_ARG, "decode_attention: q/out is NULL");
    if (dtype_size(dtype) == 0) return fail(KVBFP_ERR_INVALID_ARG, "decode_attention: unknown dtype %d", (int)dtype);
    if (n_q_heads <= 0 || n_q_heads % L->n_kv_heads != 0)
        return fail(KVBFP_ERR_INVALID_ARG, "decode_attention: n_q_heads %d not a multiple of n_kv_heads %d",
                    n_q_heads, L->n_kv_heads);
    if (max_len <= 0 || max_len > L->max_seq)
        return fail(KVBFP_ERR_INVALID_ARG, "decode_attention: max_len %lld outside (0, max_seq=%lld]",
                    (long long)max_len, (long long)L->max_seq);
    if (!std::isfinite(softmax_scale))
        return fail(KVBFP_ERR_INVALID_ARG, "decode_attention: softmax_scale is not finite");
    // from here on "heads" are virtual heads: every query token brings its own set (see DecodeArgs)
    const int32_t real_heads = n_q_heads;
    n_q_heads *= n_q_tokens;
    // (the partial results alone will do: without room for the table nothing is shared out)
    const size_t need = kvbfp_decode_workspace_bytes(L, n_q_heads, max_len) ? rows_bytes(L, n_q_heads, plan_splits(L, n_q_heads, max_len).n_splits) : 0;
    if (!workspace || workspace_bytes < need)
        return fail(KVBFP_ERR_WORKSPACE, "decode_attention: workspace of %zu bytes needed, %zu given", need,
                    workspace ? workspace_bytes : (size_t)0);
    if ((uintptr_t)workspace % 256 != 0)
        return fail(KVBFP_ERR_WORKSPACE, "decode_attention: workspace must be 256-byte aligned");
    if ((int64_t)L->batch > 65535 || (int64_t)n_q_heads > 65535)
        return fail(KVBFP_ERR_UNSUPPORTED, "decode_attention: batch/heads exceed the grid limits");

    SplitPlan sp = plan_splits(L, n_q_heads, max_len);       // what the workspace is sized for
    DecodeArgs a{};
    a.k_mant = cache->k_mant; a.k_exp = cache->k_exp; a.v_mant = cache->v_mant; a.v_exp = cache->v_exp;
    a.q = q; a.out = out; a.seq_len = seq_len_dev; a.perm_k = perm_k; a.perm_v = perm_v;
    a.part_o = (float*)workspace;
    a.max_seq = L->max_seq; a.max_len = max_len;
    a.H_kv = L->n_kv_heads; a.H_q = n_q_heads; a.G = n_q_heads / L->n_kv_heads;
    a.log2_block = log2_exact(L->block);
    a.n_q_tokens = n_q_tokens; a.real_Hq = real_heads; a.real_G = real_heads / L->n_kv_heads;
    a.q_mant_bits = q_mant_bits;
    a.scale_log2e = softmax_scale * 1.4426950408889634f;
    a.rope_theta = rope_theta; a.rope_partner = rope_partner; a.rope_sign = rope_sign;
    if (paging) {
        a.block_table = paging->block_table; a.table_stride = paging->table_stride;
        a.n_pages = pool->batch;
        a.log2_page = log2_exact((int)pool->max_seq);
    }

    hipStream_t s = (hipStream_t)hip_stream;
    const int gg = (a.G + kHeadsPerWg - 1) / kHeadsPerWg;
    if ((int64_t)a.H_kv * gg > 65535)
        return fail(KVBFP_ERR_UNSUPPORTED, "decode_attention: too many heads for the grid");
    auto aligned16 = [](const void* p) { return ((uintptr_t)p & 15u) == 0; };
    // Matrix-core passes (not with the rotation at read): up to 8 (virtual) heads of a kv-head per launch; larger groups with
    // fp32 I/O take several launches over head subsets (the cache is then read once per subset), up to 4 of them.
    // (mantissa planes are 16-byte aligned, checked above; exponent planes that are not go to the general
    // pass, which reads them byte by byte)
    const bool fast = !rope && a.G <= 32 && aligned16(a.k_exp) && aligned16(a.v_exp);
    // More heads than one launch of those takes, 16-bit I/O: all of them in one pass that decodes a row once.  8 sequences x
    // 12000 tokens x 8 kv-heads, call time before (16 heads per launch of an LDS pipeline for 4 bits and blocks of 16 / 32,
    // 8 heads otherwise, from 33 heads the general pass) -> now: 16 heads, blocks of 32 48 -> 46 us, of 16 62 -> 47 us, of 64
    // 67 -> 45 us, 8 bits 95 -> 65 us; 32 heads 90 -> 50 us, 8 bits 168 -> 68 us; 64 heads 1135 -> 69 us.
    const bool wide = !rope && a.G > 8 && dtype != KVBFP_F32 && aligned16(a.k_exp) && aligned16(a.v_exp);
    const WidePlan wp = plan_wide(a.G, (int64_t)L->batch * L->n_kv_heads, max_len, sp.n_splits);
    if (wide) sp.n_splits = wp.n_splits;
    const int log2_tile = wide ? wp.log2_tile : 8;
    // rotation at read: 4-bit mantissas with 16-bit I/O go through binary16 operands, everything else through fp32 ones
    // (8 sequences x 16384 tokens, 4 bits, bf16: 48 us, 65 in fp32).  More than 32 heads have fp32 products, as they always had; in one launch they
    // also take less time over short sequences than a launch for every four heads would (64 heads, 1 x 1000 tokens 18.4 us).
    const bool rope_halves = rope && dtype != KVBFP_F32 && L->mant_bits == 4 && a.G <= 32 && aligned16(a.k_exp) && aligned16(a.v_exp);
    // One resident round: the workgroups that fit the compute units together (three each, two of the passes for 8-bit mantissas,
    // for more than four heads with fp32 I/O and for the rotation, whose workgroups hold a 64 KB table in LDS) and not a few more, which
    // would run alone after the others.  8 kv-heads, 8000 tokens, one call with the splits rounded up -> down: 10 sequences 26.5 -> 23.0 us, 13 29.4 ->
    // 26.5, 30 51.3 -> 49.8; 8 bits, 7 sequences 33.8 -> 28.5; rotation, 7 sequences 50.4 -> 39.0.  Not down to one split: lengths
    // that differ need two to be shared out (50 ragged sequences 32.6 us with two, 45.1 with one), and 65 equal ones took
    // 105.8 against 117.9 us (50 equal ones would be 6 % faster with one).
    const bool f32_steady = fast && dtype == KVBFP_F32 && L->mant_bits == 4 && a.G <= 4 && !paging && L->block != 128;
    bool f32_three = false;
    if (rope || (fast && !wide)) {
        // (workgroups of a split: the fp32 rotation has all groups of four heads in one launch)
        const int64_t units = (int64_t)L->batch * L->n_kv_heads * (rope && !rope_halves ? gg : 1);
        const bool two = rope || L->mant_bits == 8 || (dtype == KVBFP_F32 && a.G > 4);
        const int64_t round = 256 * (two ? 2 : 3) / units;
        if (f32_steady) f32_three = plan_f32(units, (max_len + 255) / 256, seq_len_dev != nullptr, sp.n_splits);
        else if (rope && !rope_halves && gg > 1 && !seq_len_dev) sp.n_splits = plan_rope_groups(units, (max_len + 255) / 256, sp.n_splits);
        else if (round >= 2 && sp.n_splits > round) sp.n_splits = (int32_t)round;
        else if (rope && round < 2) sp.n_splits = (int32_t)std::min<int64_t>(sp.n_splits, (512 + units - 1) / units);
    }
    // Short sequences, 16-bit I/O: one workgroup of eight wavefronts a sequence and kv-head instead of splits and a combine pass, as
    // long as the tiles of 512 tokens that it takes one after the other cost less than that launch.  With many units the splits
    // are busy for longer, so the line moves up with them; beyond 256 units the workgroups would not be spread evenly over the
    // compute units.  8 kv-heads, one call in a graph, splits -> one workgroup: 4 bits, 8 x 512 9.5 -> 7.3, 16 x 1536 14.0 -> 11.3, 24 x 2048
    // 16.6 -> 13.6, ragged 14.8 -> 13.7 (24 x 3072 16.6 -> 16.9); 5 to 8 heads, 16 x 1024 15.2 -> 13.8, 24 x 1536 ragged 18.6 -> 16.1; 8 bits,
    // 8 x 512 10.0 -> 8.8, 16 x 1024 14.4 -> 13.1, 24 x 1536 ragged 17.3 -> 15.5.  With few units a tile for every wavefront always pays (0.80 to 0.93
    // of the time), and of a second round one that costs little: 4 bits up to 768 tokens (up to 64 units 0.85 to 0.97; 5 to 8 heads 0.96 to
    // 1.02), not 8 bits (0.95 to 1.07, 5 to 8 heads 1.11) unless the three tiles of 256 tokens are more workgroups than compute units (from 86 units
    // on 0.83 to 0.95, 5 to 8 heads 0.93 to 1.03; four tiles up to 128 units 0.99 to 1.09, beyond them 0.82 to 0.91 and ragged 0.93 to 1.13).  4
    // bits up to four heads from there to 1024 tokens: 0.92 to 1.06 in a graph, over pages up to 1.09, and 0.88 to 0.97 and up to 1.04 as single calls,
    // of which the host makes one launch in less time (5 to 8 heads 1.02 to 1.13 either way).  One line whatever the
    // query's cast and whether over pages, which are within 6 % of each other and return the bits of a region.
    int waves = 4;
    if (fast && !wide && dtype != KVBFP_F32 && sp.n_splits > 1) {
        const int64_t units = (int64_t)L->batch * L->n_kv_heads;
        const bool p4 = L->mant_bits == 4, one_group = a.G <= 4;
        const int64_t few_units = !p4 ? 512 : one_group ? 1024 : 768;
        const int64_t by_units = p4 ? (one_group ? 12 : 10) * units : units < 86 ? 0 : units <= 128 ? 768 : 7 * units;
        if (units <= 256 && max_len <= std::max(few_units, by_units)) {
            sp.n_splits = 1;
            waves = 8;
        }
    }
    // Where up to half of the splits would take a second tile, all take two instead and there are fewer of them (to set up, to run
    // beside each other and to merge).  8 kv-heads, one call, as many splits as fit -> two tiles each: fp32 4 x 8192 tokens (24 splits for 32
    // tiles) 21.9 -> 20.5 us, 6 x 5000 25.5 -> 21.3; 4 bits 6 x 5000 17.1 -> 15.2, 1 x 30000 16.8 -> 15.9, 8 bits 2 x 9000 18.4 ->
    // 17.8; with more than half no more: 4 bits 8 x 5000 (12 splits for 20) 16.6 -> 17.1, 8 bits 32 kv-heads 1 x 7500 (16 for 30) 17.1 -> 18.0;
    // nor with the rotation: 4 x 5600 23.5 and 23.3, 6 x 3000 21.1 -> 22.8.
    // Lengths on the device may be anything up to max_len.  Of 0.6 to 0.8 of it the fewer splits take two tiles where the others took
    // one: 8 bits 2 x 9000 15.7 -> 17.6, 8 heads 8 x 2500 18.8 -> 21.8, fp32 8 heads 4 x 5600 19.4 -> 22.9.  So 8 bits keep
    // their splits there, and fp32 I/O with 4 bits launches them all and decides by the length of each sequence (4 x 8192: 20.9 where they are max_len,
    // 18.6 against 20.5 at 0.6; 6 x 5000, whose 6 idle splits of 16 leave some of the dies with less work than others, 24.8).  16-bit I/O with 4 bits
    // goes by max_len: 3 % less to 7 % more at 0.6 to 0.8 (32 kv-heads 2 x 4000 12.7 -> 13.2, 16-token pages 2 x 15000 16.1 -> 17.1), 4 to
    // 14 % less at max_len, 20 % less to 8 % more below a half.
    if (fast && !wide && !(f32_steady && !f32_three)) {
        const int32_t paired = kvbfp::spans::paired_splits(sp.n_splits, (max_len + 255) / 256);
        if (!seq_len_dev || (L->mant_bits == 4 && dtype != KVBFP_F32)) sp.n_splits = paired;
        else if (L->mant_bits == 4 && paired != sp.n_splits) a.direct = kvbfp::kPaired;
    }
    a.n_splits = sp.n_splits;
    // by the lengths where there are any (not in the general pass) and the workspace has room for the table
    const size_t rows = rows_bytes(L, n_q_heads, sp.n_splits);
    if ((fast || wide || rope) && seq_len_dev && workspace_bytes >= rows + places_bytes(L)) {
        a.share_above = (int32_t)share_above(L, sp.n_splits, max_len, log2_tile, share_from(dtype == KVBFP_F32, L->mant_bits, a.G, rope, sp.n_splits));
        a.places = (int32_t*)((char*)workspace + rows);
    }
    // One split: nothing to merge, the split pass writes the output itself and the combine pass is not launched: an appended
    // step over 250 tokens 15.6 -> 8.2 us, 128 sequences x 1000 tokens (1024 units) 36.6 -> 33.0 us.  (Not in the passes for
    // many heads: their merge has no registers to spare, 20 heads over 12000 tokens 44.7 -> 45.7 us with the branch in it.)
    if (sp.n_splits == 1 && (rope || (fast && !wide))) a.direct = 1;
    a.part_ml = a.part_o + (size_t)L->batch * n_q_heads * sp.n_splits * kD;
    const dim3 grid1((unsigned)sp.n_splits, (unsigned)(a.H_kv * gg), (unsigned)L->batch);
    a.g_base = 0;
    a.g_cnt = a.G < 8 ? a.G : 8;
    // The current token (kvbfp_append_decode_attention): cast inside the LDS split pass, else by the
    // cache-write kernel ahead of the split pass.  Either way it lands at position seq_len - 1.
    if (k_new || v_new) {
        if (!k_new || !v_new) return fail(KVBFP_ERR_INVALID_ARG, "append_decode_attention: k_new and v_new are both needed");
        if (n_q_tokens != 1) return fail(KVBFP_ERR_UNSUPPORTED, "append_decode_attention: one query token only");
        if (new_stride_b < 0 || new_stride_h < 0)
            return fail(KVBFP_ERR_INVALID_ARG, "append_decode_attention: negative stride");
        // Inside the LDS split pass the cast is done by the one wavefront that reads the new row, off
        // the path of everybody else; elsewhere the cache-write kernel goes first, as in the two calls.
        // (the pass for many heads: where one workgroup serves all heads of a kv-head)
        const bool in_kernel = wide ? wp.row_tiles == 1 : (fast && dtype != KVBFP_F32);
        if (in_kernel) {
            a.k_new = k_new; a.v_new = v_new; a.new_stride_b = new_stride_b; a.new_stride_h = new_stride_h;
        } else {
            if (int rc = kvbfp::quantize_append_impl(pool, cache, k_new, v_new, dtype, 1, new_stride_b, 0, new_stride_h,
                                                     max_len - 1, seq_len_dev, max_len, perm_k, perm_v, hip_stream,
                                                     paging))
                return rc;
        }
    }
    // Optional timing of the two launches (kvbfp_decode_attention_profile): events on the same stream.
    hipEvent_t ev[3] = {nullptr, nullptr, nullptr};
    if (kernel_ms) {
        for (auto& e : ev)
            if (hipEventCreate(&e) != hipSuccess) {
                for (auto& made : ev)
                    if (made) (void)hipEventDestroy(made);
                return fail(KVBFP_ERR_HIP, "decode_attention_profile: hipEventCreate failed");
            }
        (void)hipEventRecord(ev[0], s);
    }
    hipError_t err = hipSuccess;
    auto launch_split = [&]() {
        if (wide) {
            err = launch_decode_split_wide(a, L->mant_bits, (int)dtype, L->block, L->batch, wp, s);
        } else if (fast) {
            for (int g0 = 0; g0 < a.G && err == hipSuccess; g0 += a.g_cnt) {      // 8 heads per launch
                a.g_base = g0;
                a.g_cnt = a.G - g0 < 8 ? a.G - g0 : 8;
                err = L->mant_bits == 4 ? launch_decode_split_mfma(a, (int)dtype, L->block, L->batch, waves, f32_three || a.direct == kvbfp::kPaired, s)
                                        : launch_decode_split_mfma_p8(a, (int)dtype, L->block, L->batch, waves, s);
                a.k_new = a.v_new = nullptr;       // the current token is cast by the first launch only
            }
        } else if (rope_halves) {                                                  // four heads per launch
            for (int g0 = 0; g0 < a.G && err == hipSuccess; g0 += 4) {
                a.g_base = g0;
                a.g_cnt = a.G - g0 < 4 ? a.G - g0 : 4;
                err = launch_decode_split_rope(a, (int)dtype, L->block, L->batch, s);
            }
        } else if (rope) {
            err = launch_decode_split_rope_f32(a, L->mant_bits, (int)dtype, L->block, L->batch, s);
        } else {
            if (L->mant_bits == 4) decode_split_generic<4><<<grid1, kTile, 0, s>>>(a, (int)dtype);
            else decode_split_generic<8><<<grid1, kTile, 0, s>>>(a, (int)dtype);
            err = hipGetLastError();
        }
    };
    const int reps = (kernel_ms && x.ring && x.ring_len > 0 && x.reps > 1) ? x.reps : 1;
    for (int r = 0; r < reps && err == hipSuccess; ++r) {
        if (reps > 1) {
            const kvbfp_cache& c = x.ring[r % x.ring_len];
            a.k_mant = c.k_mant; a.k_exp = c.k_exp; a.v_mant = c.v_mant; a.v_exp = c.v_exp;
        }
        launch_split();
    }
    if (kernel_ms) (void)hipEventRecord(ev[1], s);
    for (int r = 0; r < reps && err == hipSuccess && a.direct != 1; ++r) {
        // few (batch, head) pairs with many splits: 32 channels per workgroup (16 slices x 8 loads cover 128 splits)
        if (sp.n_splits > 32 && (int64_t)n_q_heads * L->batch < 256) {
            const dim3 grid2((unsigned)n_q_heads, (unsigned)L->batch, kD / 32);
            if (a.share_above) decode_combine<8, 32, true><<<grid2, kCombineThreads, 0, s>>>(a, (int)dtype);
            else decode_combine<8, 32, false><<<grid2, kCombineThreads, 0, s>>>(a, (int)dtype);
        } else if (sp.n_splits <= kRowSplits) {
            const dim3 grid2((unsigned)((n_q_heads * L->batch + 3) / 4));
            if (a.share_above) decode_combine_rows<true><<<grid2, 256, 0, s>>>(a, (int)dtype, L->batch);
            else decode_combine_rows<false><<<grid2, 256, 0, s>>>(a, (int)dtype, L->batch);
        } else {
            const dim3 grid2((unsigned)n_q_heads, (unsigned)L->batch, 1);
            if (a.share_above) decode_combine<32, kD, true><<<grid2, kCombineThreads, 0, s>>>(a, (int)dtype);
            else decode_combine<32, kD, false><<<grid2, kCombineThreads, 0, s>>>(a, (int)dtype);
        }
        err = hipGetLastError();
    }
    if (kernel_ms) {
        (void)hipEventRecord(ev[2], s);
        hipError_t e2 = hipEventSynchronize(ev[2]);
        if (e2 == hipSuccess) e2 = hipEventElapsedTime(&kernel_ms[0], ev[0], ev[1]);
        if (e2 == hipSuccess) e2 = hipEventElapsedTime(&kernel_ms[1], ev[1], ev[2]);
        kernel_ms[0] /= (float)reps;
        kernel_ms[1] /= (float)reps;
        for (auto& e : ev) (void)hipEventDestroy(e);
        if (err == hipSuccess) err = e2;
    }
    if (err != hipSuccess) return fail(KVBFP_ERR_HIP, "decode_attention: %s", hipGetErrorString(err));
    return KVBFP_OK;
}

int kvbfp_decode_attention(const kvbfp_layout* L, const kvbfp_cache* cache, int32_t n_q_heads,
                           const void* q, kvbfp_dtype dtype, const int32_t* seq_len_dev,
                           int64_t max_len, float softmax_scale, const int32_t* perm_k,
                           const int32_t* perm_v, void* out, void* workspace,
                           size_t workspace_bytes, void* hip_stream) {
    return decode_impl(L, cache, n_q_heads, q, dtype, seq_len_dev, max_len, softmax_scale, perm_k, perm_v, out,
                       workspace, workspace_bytes, hip_stream);
}

int kvbfp_decode_attention_qbfp(const kvbfp_layout* L, const kvbfp_cache* cache, int32_t n_q_heads,
                                const void* q, kvbfp_dtype dtype, const int32_t* seq_len_dev,
                                int64_t max_len, float softmax_scale, const int32_t* perm_k,
                                const int32_t* perm_v, int32_t q_mant_bits, void* out, void* workspace,
                                size_t workspace_bytes, void* hip_stream) {
    DecodeExtras x;
    x.q_mant_bits = q_mant_bits;
    return decode_impl(L, cache, n_q_heads, q, dtype, seq_len_dev, max_len, softmax_scale, perm_k, perm_v, out,
                       workspace, workspace_bytes, hip_stream, x);
}

int kvbfp_append_decode_attention(const kvbfp_layout* L, const kvbfp_cache* cache, int32_t n_q_heads,
                                  const void* k_new, const void* v_new, int64_t new_stride_b,
                                  int64_t new_stride_h, const void* q, kvbfp_dtype dtype,
                                  const int32_t* seq_len_dev, int64_t max_len, float softmax_scale,
                                  const int32_t* perm_k, const int32_t* perm_v, int32_t q_mant_bits,
                                  void* out, void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!k_new || !v_new) {
        clear_error();
        return fail(KVBFP_ERR_INVALID_ARG, "append_decode_attention: k_new/v_new is NULL");
    }
    DecodeExtras x;
    x.q_mant_bits = q_mant_bits;
    x.k_new = k_new; x.v_new = v_new; x.new_stride_b = new_stride_b; x.new_stride_h = new_stride_h;
    return decode_impl(L, cache, n_q_heads, q, dtype, seq_len_dev, max_len, softmax_scale, perm_k, perm_v, out,
                       workspace, workspace_bytes, hip_stream, x);
}

int kvbfp_decode_attention_multi(const kvbfp_layout* L, const kvbfp_cache* cache, int32_t n_q_heads,
                                 int32_t n_q_tokens, const void* q, kvbfp_dtype dtype,
                                 const int32_t* seq_len_dev, int64_t max_len, float softmax_scale,
                                 const int32_t* perm_k, const int32_t* perm_v, int32_t q_mant_bits, void* out,
                                 void* workspace, size_t workspace_bytes, void* hip_stream) {
    DecodeExtras x;
    x.q_mant_bits = q_mant_bits;
    x.n_q_tokens = n_q_tokens;
    return decode_impl(L, cache, n_q_heads, q, dtype, seq_len_dev, max_len, softmax_scale, perm_k, perm_v, out,
                       workspace, workspace_bytes, hip_stream, x);
}

int kvbfp_decode_attention_rope(const kvbfp_layout* L, const kvbfp_cache* cache, int32_t n_q_heads,
                                const void* q, kvbfp_dtype dtype, const int32_t* seq_len_dev,
                                int64_t max_len, float softmax_scale, const int32_t* perm_k,
                                const int32_t* perm_v, const float* rope_theta, const int32_t* rope_partner,
                                const float* rope_sign, void* out, void* workspace, size_t workspace_bytes,
                                void* hip_stream, float* kernel_ms) {
    if (!rope_theta || !rope_partner || !rope_sign) {
        clear_error();
        return fail(KVBFP_ERR_INVALID_ARG, "decode_attention_rope: rope_theta/rope_partner/rope_sign is NULL");
    }
    DecodeExtras x;
    x.kernel_ms = kernel_ms;
    x.rope_theta = rope_theta; x.rope_partner = rope_partner; x.rope_sign = rope_sign;
    return decode_impl(L, cache, n_q_heads, q, dtype, seq_len_dev, max_len, softmax_scale, perm_k, perm_v, out,
                       workspace, workspace_bytes, hip_stream, x);
}

size_t kvbfp_decode_workspace_bytes_paged(const kvbfp_layout* pool, int64_t table_stride, int32_t batch,
                                          int32_t n_q_heads, int64_t max_len) {
    clear_error();
    static const int32_t placeholder = 0;      // only its address is looked at here
    const Paging pg{&placeholder, table_stride, batch};
    kvbfp_layout logical;
    if (check_paging(pool, pg, &logical) != KVBFP_OK) return 0;
    return kvbfp_decode_workspace_bytes(&logical, n_q_heads, max_len);
}

int kvbfp_decode_attention_paged(const kvbfp_layout* pool, const kvbfp_cache* cache, const int32_t* block_table,
                                 int64_t table_stride, int32_t batch, int32_t n_q_heads, const void* q,
                                 kvbfp_dtype dtype, const int32_t* seq_len_dev, int64_t max_len,
                                 float softmax_scale, const int32_t* perm_k, const int32_t* perm_v,
                                 int32_t q_mant_bits, void* out, void* workspace, size_t workspace_bytes,
                                 void* hip_stream, float* kernel_ms) {
    const Paging pg{block_table, table_stride, batch};
    DecodeExtras x;
    x.q_mant_bits = q_mant_bits;
    x.kernel_ms = kernel_ms;
    x.paging = &pg;
    return decode_impl(pool, cache, n_q_heads, q, dtype, seq_len_dev, max_len, softmax_scale, perm_k, perm_v, out,
                       workspace, workspace_bytes, hip_stream, x);
}

int kvbfp_append_decode_attention_paged(const kvbfp_layout* pool, const kvbfp_cache* cache,
                                        const int32_t* block_table, int64_t table_stride, int32_t batch,
                                        int32_t n_q_heads, const void* k_new, const void* v_new,
                                        int64_t new_stride_b, int64_t new_stride_h, const void* q, kvbfp_dtype dtype,
                                        const int32_t* seq_len_dev, int64_t max_len, float softmax_scale,
                                        const int32_t* perm_k, const int32_t* perm_v, int32_t q_mant_bits, void* out,
                                        void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!k_new || !v_new) {
        clear_error();
        return fail(KVBFP_ERR_INVALID_ARG, "append_decode_attention_paged: k_new/v_new is NULL");
    }
    const Paging pg{block_table, table_stride, batch};
    DecodeExtras x;
    x.q_mant_bits = q_mant_bits;
    x.k_new = k_new; x.v_new = v_new; x.new_stride_b = new_stride_b; x.new_stride_h = new_stride_h;
    x.paging = &pg;
    return decode_impl(pool, cache, n_q_heads, q, dtype, seq_len_dev, max_len, softmax_scale, perm_k, perm_v, out,
                       workspace, workspace_bytes, hip_stream, x);
}

int kvbfp_decode_attention_multi_paged(const kvbfp_layout* pool, const kvbfp_cache* cache,
                                       const int32_t* block_table, int64_t table_stride, int32_t batch,
                                       int32_t n_q_heads, int32_t n_q_tokens, const void* q, kvbfp_dtype dtype,
                                       const int32_t* seq_len_dev, int64_t max_len, float softmax_scale,
                                       const int32_t* perm_k, const int32_t* perm_v, int32_t q_mant_bits, void* out,
                                       void* workspace, size_t workspace_bytes, void* hip_stream) {
    const Paging pg{block_table, table_stride, batch};
    DecodeExtras x;
    x.q_mant_bits = q_mant_bits;
    x.n_q_tokens = n_q_tokens;
    x.paging = &pg;
    return decode_impl(pool, cache, n_q_heads, q, dtype, seq_len_dev, max_len, softmax_scale, perm_k, perm_v, out,
                       workspace, workspace_bytes, hip_stream, x);
}

// ---- kvbfp_decode_attention_noalloc: the partial results of the splits live in a file-scope device
// array instead of a caller's workspace.  Every GPU holds its own copy of the array; its address on a
// device is asked for once, with that device current, and kept.
// (the table of places has room of its own: what fits the scratch is a matter of the partial results)
constexpr size_t kScratchBytes = KVBFP_NOALLOC_SCRATCH_BYTES + kvbfp::kMaxShared * 2 * sizeof(int32_t);
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (nullptr + recorded error on failure).
void* scratch_on_current_device() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        fail(KVBFP_ERR_HIP, "decode_attention_noalloc: cannot identify the current device");
        return nullptr;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            fail(KVBFP_ERR_HIP, "decode_attention_noalloc: hipGetSymbolAddress: %s", hipGetErrorString(e));
            return nullptr;
        }
        g_scratch_ptr[dev] = p;
    }
    return g_scratch_ptr[dev];
}
}  // namespace

int kvbfp_decode_attention_noalloc(const kvbfp_layout* L, const kvbfp_cache* cache, int32_t n_q_heads,
                                   const void* q, kvbfp_dtype dtype, const int32_t* seq_len_dev,
                                   int64_t max_len, float softmax_scale, const int32_t* perm_k,
                                   const int32_t* perm_v, int32_t q_mant_bits, void* out, void* hip_stream) {
    clear_error();
    // the size check comes first: a geometry that does not fit is refused before anything else happens
    const size_t need = kvbfp_decode_workspace_bytes(L, n_q_heads, max_len) ? rows_bytes(L, n_q_heads, plan_splits(L, n_q_heads, max_len).n_splits) : 0;
    if (need == 0) return fail(KVBFP_ERR_INVALID_ARG, "decode_attention_noalloc: bad layout, n_q_heads or max_len");
    if (need > (size_t)KVBFP_NOALLOC_SCRATCH_BYTES)
        return fail(KVBFP_ERR_WORKSPACE,
                    "decode_attention_noalloc: this geometry needs %zu bytes of split partials, the built-in "
                    "scratch holds %zu; use kvbfp_decode_attention with a workspace",
                    need, (size_t)KVBFP_NOALLOC_SCRATCH_BYTES);
    void* const ws = scratch_on_current_device();
    if (!ws) return KVBFP_ERR_HIP;
    DecodeExtras x;
    x.q_mant_bits = q_mant_bits;
    return decode_impl(L, cache, n_q_heads, q, dtype, seq_len_dev, max_len, softmax_scale, perm_k, perm_v, out, ws,
                       kScratchBytes, hip_stream, x);
}

int kvbfp_decode_attention_profile(const kvbfp_layout* L, const kvbfp_cache* cache, int32_t n_q_heads,
                                   const void* q, kvbfp_dtype dtype, const int32_t* seq_len_dev,
                                   int64_t max_len, float softmax_scale, const int32_t* perm_k,
                                   const int32_t* perm_v, int32_t q_mant_bits, void* out, void* workspace,
                                   size_t workspace_bytes, void* hip_stream, float* kernel_ms) {
    if (!kernel_ms) {
        clear_error();
        return fail(KVBFP_ERR_INVALID_ARG, "decode_attention_profile: kernel_ms is NULL");
    }
    DecodeExtras x;
    x.q_mant_bits = q_mant_bits;
    x.kernel_ms = kernel_ms;
    return decode_impl(L, cache, n_q_heads, q, dtype, seq_len_dev, max_len, softmax_scale, perm_k, perm_v, out,
                       workspace, workspace_bytes, hip_stream, x);
}

int kvbfp_decode_attention_profile_ring(const kvbfp_layout* L, const kvbfp_cache* caches, int32_t n_caches,
                                        int32_t n_launches, int32_t n_q_heads, const void* q, kvbfp_dtype dtype,
                                        const int32_t* seq_len_dev, int64_t max_len, float softmax_scale,
                                        const int32_t* perm_k, const int32_t* perm_v, int32_t q_mant_bits, void* out,
                                        void* workspace, size_t workspace_bytes, void* hip_stream, float* kernel_ms) {
    clear_error();
    if (!kernel_ms) return fail(KVBFP_ERR_INVALID_ARG, "decode_attention_profile_ring: kernel_ms is NULL");
    if (!caches || n_caches <= 0 || n_launches <= 0 || n_launches > 4096)
        return fail(KVBFP_ERR_INVALID_ARG, "decode_attention_profile_ring: caches / n_caches / n_launches (1..4096)");
    for (int i = 0; i < n_caches; ++i)
        if (int rc = check_cache(&caches[i], true, true)) return rc;
    DecodeExtras x;
    x.q_mant_bits = q_mant_bits;
    x.kernel_ms = kernel_ms;
    x.ring = caches; x.ring_len = n_caches; x.reps = n_launches;
    return decode_impl(L, &caches[0], n_q_heads, q, dtype, seq_len_dev, max_len, softmax_scale, perm_k, perm_v, out,
                       workspace, workspace_bytes, hip_stream, x);
}

}  // extern "C"
