// Second reads of a row by one wavefront, for rows whose sums left the range
// that the first pass accepts.
#pragma once

#include "tr_internal.h"
#include "tr_wave.h"

namespace tr {

// Element j of a row as fp32 (exact widening), for the re-read paths.
template <bool BF16>
__device__ __forceinline__ float elem(const char* row, int j)
{
    if constexpr (BF16) return __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(row)[j] << 16);
    else return reinterpret_cast<const float*>(row)[j];
}

// 2^-e for a positive m, e the exponent that puts m 2^-e in [0.5, 1), limited
// to [-125, 126] so that 2^-e is a normal number (m 2^-e then lies in
// [2^-24, 4) for every finite m > 0).
__device__ __forceinline__ float binade_scale(float m)
{
    int e;
    (void)frexpf(m, &e);
    e = e < -125 ? -125 : (e > 126 ? 126 : e);
    return ldexpf(1.f, -e);
}

__device__ __forceinline__ float wave_max_nonneg(float v)
{
    // non-negative floats order like their bit patterns
    return __uint_as_float(wave_max_u32(__float_as_uint(v)));
}

__device__ __forceinline__ float wave_min_nonneg(float v)
{
    return __uint_as_float(~wave_max_u32(~__float_as_uint(v)));
}

struct CRow {
    float s;
    bool nonfinite;   // some element of x' or x'' is a NaN or infinite
};

// Eq. (6) from a second read of the two rows, each scaled by the power of two
// of its own maximum |x| (s is invariant to both), in fp32 fused
// multiply-adds.  A zero vector gives s = 0.
template <bool BF16>
__device__ __noinline__ CRow cos_reread(const char* pr, const char* qr, int Dc, int lane)
{
    float mp = 0.f, mq = 0.f;
    bool bad = false;
    for (int j = lane; j < Dc; j += kWave) {
        const float u = fabsf(elem<BF16>(pr, j)), v = fabsf(elem<BF16>(qr, j));
        mp = fmaxf(mp, u);
        mq = fmaxf(mq, v);
        bad = bad || !(u <= 3.40282347e38f) || !(v <= 3.40282347e38f);   // NaN or infinite
    }
    CRow r{0.f, __any(bad) != 0};
    const float xp = wave_max_nonneg(mp), xq = wave_max_nonneg(mq);
    if (!(xp > 0.f) || !(xq > 0.f)) return r;
    const float sp = binade_scale(xp), sq = binade_scale(xq);
    float dot = 0.f, n1 = 0.f, n2 = 0.f;
    for (int j = lane; j < Dc; j += kWave) {
        const float u = elem<BF16>(pr, j) * sp, v = elem<BF16>(qr, j) * sq;
        dot = fmaf(u, v, dot);
        n1 = fmaf(u, u, n1);
        n2 = fmaf(v, v, n2);
    }
    dot = wave_sum_f32(dot);
    n1 = wave_sum_f32(n1);
    n2 = wave_sum_f32(n2);
    r.s = dot / (sqrtf(n1) * sqrtf(n2));
    return r;
}

// The squared norms of Eq. (6)'s first pass between which its sums stand:
// products that underflow (or denormal inputs) move s by less than 2^-40 and
// nothing overflowed.  Any other row is read again.
__device__ __forceinline__ bool cos_in_range(float n1, float n2)
{
    return n1 >= 0x1p-60f && n2 >= 0x1p-60f && n1 <= 3.40282347e38f && n2 <= 3.40282347e38f;
}

}  // namespace tr
