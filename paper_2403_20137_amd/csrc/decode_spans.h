// Which tokens a workgroup of the split pass takes, and which partial results the combine pass merges (internal).
//
// The grid has n_splits workgroups per (sequence, kv-head).  With sequences of one length, split s of sequence b is
// blockIdx (s, ., b) and takes the tiles s, s + n_splits, ... of the sequence; so it is where the host passes no lengths.
// With lengths that differ, that leaves the workgroups of a short sequence without work while those of the longest one
// carry n_splits-ths of it: 48 sequences spread log-uniformly from 64 to 16384 tokens (8 kv-heads, two splits, 16-token pages,
// 168 MB) took 74 us a call, as many tokens in equal lengths 40.  There (a.spread, set by the host where a sequence can have more tiles than splits) the
// n_splits * B workgroups of a kv-head are one list: a sequence of T tiles gets n = ceil(T / c) of them, c the smallest
// value found for which the list is long enough.  Every wavefront of either pass works c out for itself from the
// lengths, one sequence per lane, which takes less time than any exchange between workgroups; equal tile counts (one
// compare) keep the first form (51.9 us a call on 8 x 32769 tokens with lengths passed, 51.8 without the look at them).  The
// call above takes 46 us: the longest place has 9 tiles, 6.3 would be even.  The partial results of place x of the list are the rows x * H_q + h, and the l of every row
// (also of a place without work) carries a sign bit there, by which the combine pass knows the form without having
// waited for the lengths.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "decode_args.h"
#include "kvbfp.h"

namespace kvbfp {
namespace spans {

struct Span {
    int b, split, n;            // sequence; this workgroup takes its tiles split, split + n, split + 2 n, ...
    int64_t L;                  // cached tokens of the sequence
    int64_t row0, row_step;     // partial results of head h: row0 + h * row_step
    bool listed;                // the lengths differ: a place of the list
    // bit 31 set or cleared whatever l is: a NaN, from inputs that are not finite, comes with either sign
    __device__ float mark(float l) const {
        const uint32_t m = __float_as_uint(l) & 0x7FFFFFFFu;
        return __uint_as_float(listed ? m | 0x80000000u : m);
    }
    __device__ int64_t row(int64_t h) const { return row0 + h * row_step; }
};

__device__ __forceinline__ int64_t clamped_len(const DecodeArgs& a, int64_t len) {
    return len < 0 ? 0 : (len > a.max_len ? a.max_len : len);
}
// The lengths of the first 64 sequences, one per lane: requested ahead of a kernel's other loads (they return in order, and
// nothing can start without them).
__device__ __forceinline__ int request_lengths(const DecodeArgs& a, int batch) {
    return a.spread ? a.seq_len[min((int)(threadIdx.x & 63), batch - 1)] : 0;
}
// tiles of the sequence this lane looks at in the group of 64 that starts at b0 (0 beyond the last one)
__device__ __forceinline__ int lane_tiles(const DecodeArgs& a, int len0, int batch, int b0, int lane, int log2_tile) {
    const int b = b0 + lane;
    if (b >= batch) return 0;
    return (int)((clamped_len(a, b0 == 0 ? len0 : a.seq_len[b]) + ((1 << log2_tile) - 1)) >> log2_tile);
}
// inclusive prefix sum over the 64 lanes
__device__ __forceinline__ int wave_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);      // row_shr 1, 2, 4, 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);      // lane 15 of rows 0, 2 to rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);      // lane 31 to rows 2, 3
    return v;
}
// places of a sequence of T tiles at 1 / c = inv
__device__ __forceinline__ int places(int T, float inv) {
    return T == 0 ? 0 : min(T, max(1, (int)ceilf((float)T * inv - 1.0f / 1024.0f)));
}
// 1 / c, or 0 where all sequences have as many tiles as each other
__device__ __forceinline__ float inverse_share(const DecodeArgs& a, int len0, int batch, int lane, int log2_tile) {
    const int t0 = lane_tiles(a, len0, batch, 0, lane, log2_tile);
    const int first = __builtin_amdgcn_readfirstlane(t0);
    bool same = t0 == first || lane >= batch;
    int total = t0;
    for (int b0 = 64; b0 < batch; b0 += 64) {
        const int t = lane_tiles(a, len0, batch, b0, lane, log2_tile);
        same = same && (t == first || b0 + lane >= batch);
        total += t;
    }
    if (__builtin_amdgcn_ballot_w64(!same) == 0) return 0.f;
    const int list = a.n_splits * batch;
    total = __builtin_amdgcn_readlane(wave_scan(total), 63);
    // total / list is the least it can be; in steps of 1/16 the list suffices soon after (at the latest with the
    // longest sequence's tiles, one place each)
    float c = fmaxf(1.0f, (float)total / (float)list);
    for (;;) {
        const float inv = 1.0f / c;
        int sum = places(t0, inv);
        for (int b0 = 64; b0 < batch; b0 += 64) sum += places(lane_tiles(a, len0, batch, b0, lane, log2_tile), inv);
        if (__builtin_amdgcn_readlane(wave_scan(sum), 63) <= list) return inv;
        c *= 1.0625f;
    }
}

// The work of this workgroup (grid (n_splits, ., B)); false: none, and the marks of its `heads` heads from `h0` on are written.
__device__ __forceinline__ bool take(const DecodeArgs& a, int len0, int log2_tile, int h0, int heads, Span& s) {
    s.b = blockIdx.z;
    s.split = blockIdx.x;
    s.n = a.n_splits;
    s.row0 = (int64_t)s.b * a.H_q * a.n_splits + s.split;
    s.row_step = a.n_splits;
    s.listed = false;
    if (a.spread) {
        const int batch = gridDim.z, lane = threadIdx.x & 63;
        const float inv = inverse_share(a, len0, batch, lane, log2_tile);
        if (inv != 0.f) {
            const int x = blockIdx.z * a.n_splits + blockIdx.x;
            s.listed = true;
            s.row0 = (int64_t)x * a.H_q;
            s.row_step = 1;
            int before = 0;
            for (int b0 = 0; b0 < batch; b0 += 64) {
                const int n = places(lane_tiles(a, len0, batch, b0, lane, log2_tile), inv);
                const int upto = before + wave_scan(n);
                const uint64_t m = __builtin_amdgcn_ballot_w64(x < upto);
                if (m != 0) {
                    const int l = __builtin_ctzll(m);
                    s.b = b0 + l;
                    s.n = __builtin_amdgcn_readlane(n, l);
                    s.split = x - (__builtin_amdgcn_readlane(upto, l) - s.n);
                    s.L = clamped_len(a, b0 == 0 ? __builtin_amdgcn_readlane(len0, l) : a.seq_len[s.b]);
                    return true;
                }
                before = __builtin_amdgcn_readlane(upto, 63);
            }
            for (int i = threadIdx.x; i < heads; i += blockDim.x) {
                float* const ml = a.part_ml + s.row(h0 + i) * 2;
                ml[0] = -INFINITY;
                ml[1] = s.mark(0.f);
            }
            return false;
        }
    }
    s.L = !a.seq_len ? a.max_len : clamped_len(a, a.spread && gridDim.z <= 64 ? __builtin_amdgcn_readlane(len0, s.b) : a.seq_len[s.b]);
    return true;
}

// The partial results of (sequence b, head h): n rows first, first + step, ...
struct Parts {
    int64_t first, step;
    int n;
};
__device__ __forceinline__ Parts parts_of(const DecodeArgs& a, int b, int h) {
    return Parts{((int64_t)b * a.H_q + h) * a.n_splits, 1, a.n_splits};
}
// the same where the marks say that the lengths differ
__device__ __forceinline__ Parts listed_parts(const DecodeArgs& a, int batch, int b, int h, int log2_tile) {
    Parts p;
    const int lane = threadIdx.x & 63;
    const int len0 = request_lengths(a, batch);
    const float inv = inverse_share(a, len0, batch, lane, log2_tile);
    int before = 0;
    for (int b0 = 0;; b0 += 64) {
        const int n = places(lane_tiles(a, len0, batch, b0, lane, log2_tile), inv);
        const int upto = before + wave_scan(n);
        if (b < b0 + 64) {
            p.n = __builtin_amdgcn_readlane(n, b - b0);
            p.first = (int64_t)(__builtin_amdgcn_readlane(upto, b - b0) - p.n) * a.H_q + h;
            p.step = a.H_q;
            return p;
        }
        before = __builtin_amdgcn_readlane(upto, 63);
    }
}

// One split (a.direct): the merged o of channel c (cache order) of virtual head s of kv-head kvh, normalised by l and
// rounded once to the output's type, goes where the combine pass would put it.
__device__ __forceinline__ void write_output(const DecodeArgs& a, int dt, int b, int kvh, int s, int c, float o, float l) {
    const int to = a.perm_v ? (a.perm_v[kvh * 128 + c] & 127) : c;       // masked: the store stays inside the row
    const int64_t i = query_row(a, b, kvh, s) * 128 + to;
    const float r = l > 0.f ? o / l : 0.f;
    if (dt == KVBFP_F32) {
        ((float*)a.out)[i] = r;
    } else if (dt == KVBFP_F16) {
        ((uint16_t*)a.out)[i] = __builtin_bit_cast(unsigned short, (_Float16)r);
    } else {
        uint32_t u = __float_as_uint(r);
        u += 0x7FFFu + ((u >> 16) & 1u);
        ((uint16_t*)a.out)[i] = (uint16_t)(u >> 16);
    }
}

}  // namespace spans
}  // namespace kvbfp
