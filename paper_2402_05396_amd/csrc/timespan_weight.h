// The weight of an entry `delta` ticks before the query, max(1, floor(2^32 / delta)), by a single-precision reciprocal
// that may be off by one unit in its last place either way.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

// delta > kLastLargeDelta, so the quotient is at most kSmallWeight. The reciprocal of (float)delta gives it within
// 2^-22 of itself (conversion, the reciprocal's one unit in the last place, the product); scaled
// down by 2^-21 it gives the quotient or one less, and the exact remainder says which. NEAR: delta < 2^24,
// where the quotient is at least 256 and one full-rate 24-bit multiply-add does for the remainder.
constexpr uint32_t kLastLargeDelta = 65536;      // its quotient is 2^16 itself: with it a tile of ties would sum to 2^32
constexpr uint32_t kSmallWeight = (uint32_t)(((uint64_t)1 << 32) / (kLastLargeDelta + 1));
static_assert(kSmallWeight == 65535, "the quotient of every larger delta is below 2^16");
template <bool NEAR> __host__ __device__ inline uint32_t quotient_by_reciprocal(uint32_t delta, float reciprocal) {
    const uint32_t q = (uint32_t)(4294967296.0f * (1.0f - 4.76837158203125e-7f) * reciprocal);
    if (NEAR) return q + ((int32_t)((q & 0xffffffu) * (delta & 0xffffffu) + delta) <= 0 ? 1u : 0u);   // (q + 1) delta is at most 2^32 (it is within delta of it)
    const uint32_t rest = 0u - q * delta;                                 // 2^32 - q delta, below 2 delta; wraps only for delta > 2^31
    const uint32_t w = q + (rest >= delta ? 1u : 0u);
    return w > 1u ? w : 1u;                                               // (where the quotient is 1 in any case)
}
// Any delta >= 1; the quotient has up to 33 bits. The first estimate is at most 2^-20 of it too small (or one,
// where that is less), so that the remainder is below 2^13 + 2 delta; the remainder's own quotient, found the same
// way, is exact or one too small.
__host__ __device__ inline uint64_t weight_by_reciprocal(uint32_t delta, float reciprocal) {
    const float r = (1.0f - 4.76837158203125e-7f) * reciprocal;
    const uint32_t q = (uint32_t)(4294967296.0f * r);
    const uint32_t rest = 0u - q * delta;                 // 2^32 - q delta; wraps only for delta > 2^31 (q == 0)
    const uint32_t more = (uint32_t)((float)rest * r), left = rest - more * delta;
    const uint64_t w = (uint64_t)q + (more + (left >= delta ? 1u : 0u));
    return w > 1u ? w : 1u;
}
