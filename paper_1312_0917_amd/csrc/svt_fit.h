// Fit helpers shared by the kernels of libsvt: packed 16-bit dot products, the exact split
// offset, division by small numbers and the record stores.
//
// The fit of section II is p_j = sum_l f[j][l] x_l + q_j followed by the fixed-point shift.
// Constants are int16 and coordinates int13, so the five products of one row are three packed
// 16-bit dot products (v_dot2_i32_i16) once the coordinates of layers (0,1) and (2,3) are
// paired.  The offset is split exactly as q = qh * 2^s + ql with 0 <= ql < 2^s: ql seeds the
// accumulator, so the sum stays inside int32, and
//     floor((S + q) / 2^s) = qh + floor((S + ql) / 2^s)       (exact for every integer S).
#pragma once

#include "svt_common.h"

namespace svt {

constexpr int kRecNone = 0;  // no per-combination records (kept-only output)
constexpr int kRecFit = 1;   // p0..p2 and chi2
constexpr int kRecRows = 2;  // also the constraint rows c0..c2 (each pointer may be null)

typedef short v2s __attribute__((ext_vector_type(2)));

// a.lo * b.lo + a.hi * b.hi + c on signed 16-bit halves (v_dot2_i32_i16, no clamping).
__device__ __forceinline__ int32_t dot2(int32_t a, int32_t b, int32_t c) {
    return __builtin_amdgcn_sdot2(__builtin_bit_cast(v2s, a), __builtin_bit_cast(v2s, b), c,
                                  false);
}

// floor(k / n) for 0 <= k < 2^15 and 1 <= n <= 64 with m = ceil(2^23 / n) < 2^24, using the
// full-rate 24-bit multiply: (k * 2^9) * m / 2^32 = k * m / 2^23 and k * (m * n - 2^23) <
// 2^15 * 64 < 2^23, so the high word is exactly floor(k / n) (n = 1 included).
__device__ __forceinline__ uint32_t div_small(uint32_t k, uint32_t m) {
    const uint64_t p = static_cast<uint64_t>((k << 9) & 0xFFFFFFu) * static_cast<uint64_t>(m & 0xFFFFFFu);
    return static_cast<uint32_t>(p >> 32);  // v_mul_hi_u32_u24
}

// a * b for a, b < 2^24 (low 32 bits) on the full-rate 24-bit multiplier
__device__ __forceinline__ uint32_t mul_u24(uint32_t a, uint32_t b) {
    uint32_t r;
    asm("v_mul_u32_u24 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

__host__ __device__ constexpr uint32_t magic_of(uint32_t n) {
    return static_cast<uint32_t>(((1u << 23) + n - 1) / n);
}

// 16-byte stores marked non-temporal: the per-combination records are written once and read
// by nothing later in the pass, so they should not displace the staged inputs in the caches.
typedef int32_t nt_i32x4 __attribute__((ext_vector_type(4)));
typedef int64_t nt_i64x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void store_nt(int32_t *p, const int32_t *v) {
    const nt_i32x4 x = {v[0], v[1], v[2], v[3]};
    __builtin_nontemporal_store(x, reinterpret_cast<nt_i32x4 *>(p));
}
__device__ __forceinline__ void store_nt(int64_t *p, int64_t a, int64_t b) {
    const nt_i64x2 x = {a, b};
    __builtin_nontemporal_store(x, reinterpret_cast<nt_i64x2 *>(p));
}

__device__ __forceinline__ int32_t pack16(int32_t lo, int32_t hi) {
    return static_cast<int32_t>((static_cast<uint32_t>(lo) & 0xFFFFu) |
                                (static_cast<uint32_t>(hi) << 16));
}

struct Fit {
    int32_t v[6];
    int64_t chi2;
};

// Arithmetic forms of the fit, all exact (same values as the int64 definition):
//   kFitSplit  q = qh * 2^s + ql, ql seeds each row, qh is added after the shift;
//   kFitNarrow the whole offset seeds each row and the chi-square is summed in 32 bits.  Valid
//              for a constant set whose bounds narrow_ok() accepts: every row's sum stays in
//              int32 for any int13 coordinates, and every chi-square component has |c| < 2^15,
//              so c^2 < 2^30 and the sum of three is below 2^32.
constexpr int kFitSplit = 0;
constexpr int kFitNarrow = 1;

// Whether a constant set allows kFitNarrow: with |x_l| <= 2^12 the row sum S_j + q_j lies in
// [-B_j, B_j] for B_j = 2^12 * sum_l |f_jl| + |q_j|; int32 needs B_j < 2^31, and the shifted
// value floor((S_j + q_j) / 2^s) then has magnitude at most (B_j >> s) + 1, which must stay
// below 2^15 for the chi-square rows (j = 3..5).  f holds the set's 30 constants row-major.
__device__ __forceinline__ bool narrow_ok(const int32_t *f, const int32_t *q, int32_t shift) {
    bool ok = true;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        int64_t sf = 0;
#pragma unroll
        for (int l = 0; l < 5; ++l) sf += f[5 * j + l] < 0 ? -f[5 * j + l] : f[5 * j + l];
        const int64_t b = (sf << 12) + (q[j] < 0 ? -static_cast<int64_t>(q[j]) : q[j]);
        ok &= b < (1ll << 31);
        if (j >= 3) ok &= (b >> shift) + 1 < (1ll << 15);
    }
    return ok;
}

// a * b + c on the full-rate 24-bit signed multiplier (low 32 bits of the result)
__device__ __forceinline__ int32_t mad_i24(int32_t a, int32_t b, int32_t c) {
    int32_t r;
    asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

}  // namespace svt
