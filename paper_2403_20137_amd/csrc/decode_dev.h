// Device helpers shared by the matrix-core decode kernels (internal).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>
#include <utility>

#include "kvbfp.h"

namespace kvbfp {
namespace dev {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));

// f(std::integral_constant<int, 0>{}), ..., f(std::integral_constant<int, N - 1>{}): arrays it indexes stay in registers
template <class F, int... I>
__device__ __forceinline__ void static_for(std::integer_sequence<int, I...>, F&& f) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) { static_for(std::make_integer_sequence<int, N>{}, f); }

constexpr int kD = 128;
constexpr int kWaves = 4;
constexpr int kSuper = 64;   // tokens per wavefront iteration (4 MFMA column tiles of 16)
// The conversions produce cached values as value * 2^-kShift, with kShift chosen per mantissa width so
// that the conversion's scale operand is the stored exponent byte itself (kShift4, kShift8 in the kernel
// files).  The inverse factor rides on the other operand of each product (the query for scores, the
// probabilities for outputs), so the fp32 accumulators hold true-scale numbers: nothing is lost at either
// end of the fp32 range that the bf16 operand format can hold.

template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, 0xF, 0xF, false));
}
// all-reduce over the 16 lanes of a DPP row
__device__ __forceinline__ float row_max(float v) {
    v = fmaxf(v, dpp_f<0xB1>(v));
    v = fmaxf(v, dpp_f<0x4E>(v));
    v = fmaxf(v, dpp_f<0x141>(v));
    v = fmaxf(v, dpp_f<0x140>(v));
    return v;
}
__device__ __forceinline__ float row_sum(float v) {
    v += dpp_f<0xB1>(v);
    v += dpp_f<0x4E>(v);
    v += dpp_f<0x141>(v);
    v += dpp_f<0x140>(v);
    return v;
}

__device__ __forceinline__ float load_as_float(const void* p, int dt, int64_t i) {
    if (dt == KVBFP_F32) return ((const float*)p)[i];
    const uint32_t h = ((const uint16_t*)p)[i];
    if (dt == KVBFP_F16) return (float)__builtin_bit_cast(_Float16, (unsigned short)h);
    return __uint_as_float(h << 16);
}

// 2^x by the hardware instruction alone (1 ulp; results below 2^-126 come out as 0 instead of as
// denormals, which is all a softmax weight relative to the running maximum needs; 2^-inf = 0).
__device__ __forceinline__ float exp2_raw(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ bf16x8 join(bf16x2 a, bf16x2 b, bf16x2 c, bf16x2 d) {
    bf16x8 r;
    r[0] = a[0]; r[1] = a[1]; r[2] = b[0]; r[3] = b[1];
    r[4] = c[0]; r[5] = c[1]; r[6] = d[0]; r[7] = d[1];
    return r;
}

// scale operand of the conversions: only the exponent field is looked at, and it is the stored exponent byte
__device__ __forceinline__ float scale_operand(uint32_t E) { return __uint_as_float(E << 23); }
// 8 sign-magnitude nibbles -> FP8 bytes: the nibble s|mmm widened to the byte s0000mmm is the FP8-E4M3 subnormal (-1)^s m 2^-9
__device__ __forceinline__ void spread4(uint32_t w, uint32_t& lo, uint32_t& hi) {
    lo = ((w << 4) & 0x80808080u) | (w & 0x07070707u);          // even nibbles
    hi = (w & 0x80808080u) | ((w >> 4) & 0x07070707u);          // odd nibbles
}
// 4 sign-magnitude bytes s mmmm lll -> s000mmmm (worth eight times as much) and s0000lll, both valid FP8-E4M3 numbers (the subnormals
// and the first binade share one spacing: s000xxxx reads as +-x 2^-9 for x = 0..15)
__device__ __forceinline__ void spread8(uint32_t w, uint32_t& hi, uint32_t& lo) {
    hi = ((w >> 3) & 0x0F0F0F0Fu) | (w & 0x80808080u);
    lo = w & 0x87878787u;
}
// 8 nibbles -> 8 bf16 values in slot order [c0,c2,c4,c6,c1,c3,c5,c7]
struct Unpacked4 { bf16x2 p[4]; };
__device__ __forceinline__ Unpacked4 unpack8_p4(uint32_t w, float scale) {
    uint32_t lo, hi;
    spread4(w, lo, hi);
    Unpacked4 u;
    u.p[0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, scale, false);      // (c0, c2)
    u.p[1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, scale, true);       // (c4, c6)
    u.p[2] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, scale, false);      // (c1, c3)
    u.p[3] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, scale, true);       // (c5, c7)
    return u;
}
// 4 bytes -> hi pieces (c0,c1), (c2,c3) and lo pieces (c0,c1), (c2,c3) as bf16 pairs; the hi piece takes 8 times the scale
struct Pieces8 { bf16x2 h01, h23, l01, l23; };
__device__ __forceinline__ Pieces8 unpack4_p8(uint32_t w, float s_hi, float s_lo) {
    uint32_t hi, lo;
    spread8(w, hi, lo);
    Pieces8 r;
    r.h01 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, s_hi, false);
    r.h23 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, s_hi, true);
    r.l01 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, s_lo, false);
    r.l23 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, s_lo, true);
    return r;
}
// channel offset inside a dword of MFMA slot x (4-bit mantissas)
__device__ __forceinline__ int slot_channel(int x) { return (x < 4) ? 2 * x : 2 * (x - 4) + 1; }
// Lane (j, row) of a wavefront, row = lane / 16, holds M[row][r] in v[r].  Afterwards v[r] holds M[r][row]:
// first the 2 x 2 blocks are exchanged between the two halves of the wavefront, then single rows
// between neighbouring 16-lane rows.
__device__ __forceinline__ void transpose_rows(u32x4& v) {
    const auto a = __builtin_amdgcn_permlane32_swap(v[0], v[2], false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(v[1], v[3], false, false);
    const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
    const auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
    v[0] = c[0]; v[1] = c[1]; v[2] = d[0]; v[3] = d[1];
}

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also waits for every outstanding
// vector-memory operation of the wavefront, which a kernel with cache rows in flight cannot afford
// during its set-up.
__device__ __forceinline__ void lds_only_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Casts the queries in q_s[n_heads][128] (cache channel order, fp32, unscaled) to Block Floating Point
// in place: blocks of 2^log2_block channels, `bits`-bit sign-magnitude mantissas, the shared exponent
// chosen by the same rule as for cached rows (Sec. II-B, Eq. (1); Sec. III: the activations of the
// score product are BFP as well).  The decoded values are written back, so what follows is a product
// of exact small integers per block.  amax_s: n_heads * 8 words of LDS scratch.  Called by every
// thread of the workgroup after q_s is complete (barrier before); ends with a barrier (LDS only).
__device__ __forceinline__ void bfp_round_queries(float* q_s, uint32_t* amax_s, int n_heads, int log2_block, int bits) {
    const int tid = threadIdx.x, nt = blockDim.x;
    for (int i = tid; i < n_heads * 8; i += nt) amax_s[i] = 0u;
    lds_only_barrier();
    for (int i = tid; i < n_heads * kD; i += nt)
        atomicMax(&amax_s[(i / kD) * 8 + ((i % kD) >> log2_block)], __float_as_uint(q_s[i]) & 0x7FFFFFFFu);
    lds_only_barrier();
    for (int i = tid; i < n_heads * kD; i += nt) {
        const uint32_t amax = amax_s[(i / kD) * 8 + ((i % kD) >> log2_block)];
        const uint32_t bumped = (amax + (1u << (24 - bits))) >> 23;
        const int E = amax == 0 ? 0 : (int)max(bumped, 1u);
        const int e = E - 127 - (bits - 2);
        q_s[i] = ldexpf(rintf(ldexpf(q_s[i], -e)), e);     // both scalings exact; rintf rounds to nearest even
    }
    lds_only_barrier();
}

// x - n pi / 2 for the nearest whole n, and n modulo 4.  The sum with 1.5 * 2^52 rounds to whole numbers and has them in its lowest bits.
__device__ __forceinline__ double pi_half_remainder(double x, int& quarter) {
    const double whole = fma(x, 0.63661977236758134308, 6755399441055744.0);
    const double n = whole - 6755399441055744.0;
    quarter = (int)__double_as_longlong(whole) & 3;
    return fma(-n, 6.12323399573676603587e-17, fma(-n, 1.57079632679489655800, x));
}
// (cs, sn) of the remainder -> of the whole angle
template <class T>
__device__ __forceinline__ void add_quarters(int quarter, T cs, T sn, T& c, T& s) {
    const bool swap = quarter & 1;
    const T ca = swap ? sn : cs, sa = swap ? cs : sn;
    c = (quarter == 1 || quarter == 2) ? -ca : ca;
    s = quarter >= 2 ? -sa : sa;
}
// Cosine and sine of t * th in double precision: the product of a token index below 2^29 with a 24-bit number is exact, what
// is left of it after multiples of pi / 2 (in two parts) is within pi / 4, and there the Taylor series up to r^15 and r^16 are off by
// less than 2^-54.  Some 40 instructions, without the branches of the library's sincos.  Angles of up to 2^50: beyond, the multiple is
// rounded.
__device__ __forceinline__ void phasor(double t, double th, double& c, double& s) {
    int quarter;
    const double r = pi_half_remainder(t * th, quarter);
    const double z = r * r;
    double a = fma(z, -1.0 / 1307674368000.0, 1.0 / 6227020800.0);
    a = fma(z, a, -1.0 / 39916800.0);
    a = fma(z, a, 1.0 / 362880.0);
    a = fma(z, a, -1.0 / 5040.0);
    a = fma(z, a, 1.0 / 120.0);
    a = fma(z, a, -1.0 / 6.0);
    const double sn = fma(r * z, a, r);
    double b = fma(z, 1.0 / 20922789888000.0, -1.0 / 87178291200.0);
    b = fma(z, b, 1.0 / 479001600.0);
    b = fma(z, b, -1.0 / 3628800.0);
    b = fma(z, b, 1.0 / 40320.0);
    b = fma(z, b, -1.0 / 720.0);
    b = fma(z, b, 1.0 / 24.0);
    b = fma(z, b, -0.5);
    add_quarters(quarter, fma(z, b, 1.0), sn, c, s);
}
// The same to fp32: the remainder as two fp32 numbers, the series up to r^9 and r^10 (3e-9).
__device__ __forceinline__ void phasor(double t, double th, float& c, float& s) {
    int quarter;
    const double rd = pi_half_remainder(t * th, quarter);
    const float r = (float)rd, rest = (float)(rd - (double)r), z = r * r;
    float a = fmaf(z, 1.f / 362880.f, -1.f / 5040.f);
    a = fmaf(z, a, 1.f / 120.f);
    a = fmaf(z, a, -1.f / 6.f);
    float b = fmaf(z, -1.f / 3628800.f, 1.f / 40320.f);
    b = fmaf(z, b, -1.f / 720.f);
    b = fmaf(z, b, 1.f / 24.f);
    b = fmaf(z, b, -0.5f);
    const float cs = 1.f + fmaf(-rest, r, z * b);
    add_quarters(quarter, cs, r + fmaf(r * z, a, rest * cs), c, s);
}
// the phasor (c, s) turned by (dc, ds)
__device__ __forceinline__ void turn(double& c, double& s, double dc, double ds) {
    const double n = fma(c, dc, -(s * ds));
    s = fma(s, dc, c * ds);
    c = n;
}

}  // namespace dev
}  // namespace kvbfp
