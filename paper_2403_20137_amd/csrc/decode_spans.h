// Which tokens a workgroup of the split pass takes, and which partial results the combine pass merges (internal).
//
// The grid has n_splits workgroups per (sequence, kv-head).  With sequences of one length, split s of sequence b is
// blockIdx (s, ., b) and takes the tiles s, s + n_splits, ... of the sequence; so it is where the host passes no lengths.
// With lengths that differ, that leaves the workgroups of a short sequence without work while those of the longest one
// carry n_splits-ths of it: 48 sequences spread log-uniformly from 64 to 16384 tokens (8 kv-heads, two splits, 16-token pages,
// 168 MB) took 74 us a call, as many tokens in equal lengths 40.  There the n_splits * B workgroups of a kv-head are one
// list: a sequence of T tiles gets n = ceil(T / c) of them, c the smallest value found for which the list is long enough.
// Every wavefront of the split pass works c out for itself from the lengths, which takes less time than any exchange between
// workgroups.  The partial results of place x of the list are the rows x * H_q + h, and the workgroups (0, 0, b) leave the
// place and count of sequence b (or that nothing was shared out) in a.places for the combine pass.
//
// Sharing out costs 2 to 4 us: the search, more workgroups with a set-up, and in the combine pass a round trip for the table
// ahead of the rows.  So sequences keep their splits, decided on the lengths, where all have as many tiles as each other or
// none has more than a.share_above of them (which the host sets by the pass, with the figures there).
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
    int row0, row_step;         // partial results of head h: row0 + h * row_step (a row is 520 bytes: fewer than 2^31 fit memory)
    __device__ int64_t row(int h) const { return row0 + h * row_step; }
};

__device__ __forceinline__ int64_t clamped_len(const DecodeArgs& a, int64_t len) {
    return len < 0 ? 0 : (len > a.max_len ? a.max_len : len);
}
// The lengths of up to 64 sequences, one per lane: requested ahead of a kernel's other loads (they return in order, and
// nothing can start without them).
__device__ __forceinline__ int request_lengths(const DecodeArgs& a, int batch) {
    return a.share_above ? a.seq_len[min((int)(threadIdx.x & 63), batch - 1)] : 0;
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
// 1 / c for the tiles of this lane's K sequences (from K * lane on), or 0 where the sequences keep their splits
template <int K>
__device__ __forceinline__ float inverse_share(const DecodeArgs& a, const int (&tiles)[K], int batch) {
    const int lane = threadIdx.x & 63;
    const int first = __builtin_amdgcn_readfirstlane(tiles[0]);
    bool differ = false, longer = false;
    int total = 0;
#pragma unroll
    for (int g = 0; g < K; ++g) {
        differ = differ || (tiles[g] != first && K * lane + g < batch);
        longer = longer || tiles[g] > a.share_above;
        total += tiles[g];
    }
    if (__builtin_amdgcn_ballot_w64(differ) == 0 || __builtin_amdgcn_ballot_w64(longer) == 0) return 0.f;
    const int list = a.n_splits * batch;
    total = __builtin_amdgcn_readlane(wave_scan(total), 63);
    // c0 = total / list is the least it can be, and 2 c0 is enough: there are fewer than total / c + batch places then, and
    // the list has two per sequence or more.  The smallest of c0 * 2^(k/16) that does, by halves.
    const float inv0 = __builtin_amdgcn_rcpf(fmaxf(1.0f, (float)total / (float)list));
    auto fits = [&](float inv) {
        int sum = 0;
#pragma unroll
        for (int g = 0; g < K; ++g) sum += places(tiles[g], inv);
        return __builtin_amdgcn_readlane(wave_scan(sum), 63) <= list;
    };
    if (fits(inv0)) return inv0;
    int lo = 1, hi = 16;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (fits(inv0 * __builtin_amdgcn_exp2f((float)mid * -0.0625f))) hi = mid;
        else lo = mid + 1;
    }
    return inv0 * __builtin_amdgcn_exp2f((float)hi * -0.0625f);
}

// Where up to half of the splits would take a second tile, all take two instead and there are fewer of them: how many, for a
// sequence of so many tiles (when, and the figures: attention.hip).
__host__ __device__ __forceinline__ int paired_splits(int n, int64_t tiles) {
    return n < tiles && 2 * tiles <= 3 * (int64_t)n ? (int)((tiles + 1) / 2) : n;
}
// The same by the actual length (kPaired): the grid has all splits, and those that are not needed have nothing to do.
__device__ __forceinline__ void pair_up(const DecodeArgs& a, int log2_tile, Span& s) {
    if (a.direct != kPaired) return;
    const int tiles = (int)((s.L + ((1 << log2_tile) - 1)) >> log2_tile);
    s.n = paired_splits(a.n_splits, tiles);
    if (s.split >= s.n) s.split = tiles;        // beyond the end
}

// take() with K sequences per lane; len0: request_lengths
template <bool PAIR, int K>
__device__ __forceinline__ bool take_shared(const DecodeArgs& a, int len0, int log2_tile, Span& s) {
    const int batch = gridDim.z, lane = threadIdx.x & 63;
    int len[K], tiles[K], n[K];
#pragma unroll
    for (int g = 0; g < K; ++g) len[g] = K == 1 ? len0 : a.seq_len[min(K * lane + g, batch - 1)];
#pragma unroll
    for (int g = 0; g < K; ++g)
        tiles[g] = K * lane + g < batch ? (int)((clamped_len(a, len[g]) + ((1 << log2_tile) - 1)) >> log2_tile) : 0;
    const float inv = inverse_share<K>(a, tiles, batch);
    const bool writer = blockIdx.x == 0 && blockIdx.y == 0;
    if (inv == 0.f) {
        if (writer && threadIdx.x == 0) a.places[2 * s.b] = -1;
        s.L = clamped_len(a, K == 1 ? __builtin_amdgcn_readlane(len0, s.b) : a.seq_len[s.b]);
        if (PAIR) pair_up(a, log2_tile, s);
        return true;
    }
    int mine = 0;
#pragma unroll
    for (int g = 0; g < K; ++g) mine += n[g] = places(tiles[g], inv);
    const int upto = wave_scan(mine);
    if (writer) {
        const int of = s.b / K;
        int at = __builtin_amdgcn_readlane(upto - mine, of), count = 0;
#pragma unroll
        for (int g = 0; g < K; ++g) {
            const int here = __builtin_amdgcn_readlane(n[g], of);
            if (K * of + g < s.b) at += here;
            if (K * of + g == s.b) count = here;
        }
        if (threadIdx.x == 0) {
            a.places[2 * s.b] = at;
            a.places[2 * s.b + 1] = count;
        }
    }
    const int x = blockIdx.z * a.n_splits + blockIdx.x;
    s.row0 = x * a.H_q;
    s.row_step = 1;
    const uint64_t m = __builtin_amdgcn_ballot_w64(x < upto);
    if (m == 0) return false;                   // beyond the last place: its rows are not read
    const int of = __builtin_ctzll(m);
    int at = __builtin_amdgcn_readlane(upto - mine, of);
    bool found = false;
#pragma unroll
    for (int g = 0; g < K; ++g) {
        const int here = __builtin_amdgcn_readlane(n[g], of);
        if (!found && x < at + here) {
            found = true;
            s.b = K * of + g;
            s.n = here;
            s.split = x - at;
            s.L = clamped_len(a, __builtin_amdgcn_readlane(len[g], of));
        }
        at += here;
    }
    return true;
}

// The work of this workgroup (grid (n_splits, ., B)); false: none.  SHARE false: for calls without share_above; PAIR: for the
// pass that may have kPaired.
template <bool SHARE = true, bool PAIR = false>
__device__ __forceinline__ bool take(const DecodeArgs& a, int len0, int log2_tile, Span& s) {
    s.b = blockIdx.z;
    s.split = blockIdx.x;
    s.n = a.n_splits;
    s.row0 = s.b * a.H_q * a.n_splits + s.split;
    s.row_step = a.n_splits;
    if (SHARE && a.share_above) {
        if (gridDim.z <= 64) return take_shared<PAIR, 1>(a, len0, log2_tile, s);
        if (gridDim.z <= 256) return take_shared<PAIR, 4>(a, len0, log2_tile, s);
        return take_shared<PAIR, kMaxShared / 64>(a, len0, log2_tile, s);
    }
    s.L = !a.seq_len ? a.max_len : clamped_len(a, a.seq_len[s.b]);
    if (PAIR) pair_up(a, log2_tile, s);
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
// the same where the workgroups were shared out: at, n as the split pass left them in a.places
__device__ __forceinline__ Parts shared_parts(const DecodeArgs& a, int at, int n, int h) {
    return Parts{(int64_t)at * a.H_q + h, a.H_q, n};
}

// The arguments of a split kernel (its first parameter) again, for what comes after its main loop: read there, they are not
// held in scalar registers through it, where those that do not fit take vector registers.  Blocks of 32, two groups of four
// heads over pages: the three wavefronts per SIMD leave 168, and 4 were spilled; 8 heads, 8 x 8192 tokens 27.2 -> 26.3 us.
__device__ __forceinline__ const DecodeArgs& arguments_again() {
    const __attribute__((address_space(4))) DecodeArgs* p = (const __attribute__((address_space(4))) DecodeArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));                 // (not the same to the compiler)
    return *(const DecodeArgs*)p;
}

// One split (a.direct = 1): the merged o of channel c (cache order) of virtual head s of kv-head kvh, normalised by l and
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
