// Device helpers shared by the sampling kernels: the counter-based random
// generator and the lane-group primitives. Internal header; every translation
// unit that includes it gets its own copy.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "taser_internal.h"

namespace {

// ---- Philox4x32-10 (Salmon et al., SC'11) --------------------------------
// WIDE: the two products as 64-bit ones, one v_mad_u64_u32 each, where separate low and high products are
// two quarter-rate instructions. The weighted finders and the window's selection are faster so (40 000 roots, 10
// of 25: 22.3 -> 21.6 us), the uniform finder is not (60 000 roots, k = 10: 16.6 -> 17.1).
template <bool WIDE> __device__ __forceinline__ void philox_round(uint32_t (&c)[4], uint32_t k0, uint32_t k1) {
    uint32_t lo0, hi0, lo1, hi1;
    if (WIDE) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c[0], p1 = (uint64_t)0xCD9E8D57u * c[2];
        lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32), lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
    } else {
        lo0 = 0xD2511F53u * c[0], hi0 = __umulhi(0xD2511F53u, c[0]);
        lo1 = 0xCD9E8D57u * c[2], hi1 = __umulhi(0xCD9E8D57u, c[2]);
    }
    const uint32_t a = hi1 ^ c[1] ^ k0;
    const uint32_t b = hi0 ^ c[3] ^ k1;
    c[0] = a; c[1] = lo1; c[2] = b; c[3] = lo0;
}

// 64 random bits for (seed, hop, root index, slot).
template <bool WIDE> __device__ __forceinline__ uint64_t philox_draw(uint32_t seed_lo, uint32_t seed_hi, uint32_t hop,
                                                                     uint64_t root, uint32_t slot) {
    uint32_t c[4] = {(uint32_t)root, (uint32_t)(root >> 32), slot, hop};
    uint32_t k0 = seed_lo, k1 = seed_hi;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        philox_round<WIDE>(c, k0, k1);
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return ((uint64_t)c[1] << 32) | c[0];
}
__device__ __forceinline__ uint64_t draw64(uint32_t seed_lo, uint32_t seed_hi, uint32_t hop, uint64_t root, uint32_t slot) {
    return philox_draw<false>(seed_lo, seed_hi, hop, root, slot);
}
__device__ __forceinline__ uint64_t draw64_wide(uint32_t seed_lo, uint32_t seed_hi, uint32_t hop, uint64_t root, uint32_t slot) {
    return philox_draw<true>(seed_lo, seed_hi, hop, root, slot);
}

// floor(u * n / 2^64) for a 32-bit n: the high word of the 96-bit product.
__device__ __forceinline__ uint32_t mulhi_64x32(uint64_t u, uint32_t n) {
    const uint64_t low = (uint64_t)(uint32_t)u * n;                    // contributes its high word as a carry
    return (uint32_t)(((u >> 32) * n + (low >> 32)) >> 32);
}

// ---- group helpers ---------------------------------------------------------
// A wavefront is split into 64/G groups of G consecutive lanes (G = 16, 32 or
// 64), one root per group. `sub` is a lane's index inside its group.
template <int G> __device__ __forceinline__ uint64_t group_bits(uint64_t wave_ballot, int group) {
    if (G == 64) return wave_ballot;
    return (wave_ballot >> (group * G)) & (((uint64_t)1 << G) - 1);
}
// Lane (inside the group) of the lowest set bit of the group's part, -1 if there is none.
template <int G> __device__ __forceinline__ int group_first(uint64_t wave_ballot, int group) {
    if (G == 64) return __ffsll((long long)wave_ballot) - 1;
    const uint32_t lo = (uint32_t)wave_ballot, hi = (uint32_t)(wave_ballot >> 32);
    if (G == 32) return __ffs((int)(group ? hi : lo)) - 1;
    return __ffs((int)(((group & 2) ? hi : lo) >> (16 * (group & 1)) & 0xffffu)) - 1;
}
template <int G> __device__ __forceinline__ uint32_t group_get(uint32_t v, int sub_lane) {
    return (uint32_t)__shfl((int)v, sub_lane, G);
}
template <int G> __device__ __forceinline__ uint64_t group_get64(uint64_t v, int sub_lane) {
    return ((uint64_t)group_get<G>((uint32_t)(v >> 32), sub_lane) << 32) | group_get<G>((uint32_t)v, sub_lane);
}

// The 64-bit value of the lane a DPP control points at, 0 where there is no such lane or the
// row is masked out: one cross-lane move per half, a few cycles each, no trip through LDS.
// CTRL: 0x110 + n = the lane n places below inside a row of 16 lanes; 0x142 / 0x143 = lane 15 of
// the row below / lane 31, broadcast to a whole row. Every lane of the wave must be active.
template <int CTRL, int ROW_MASK> __device__ __forceinline__ uint64_t dpp_take64(uint64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROW_MASK, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, ROW_MASK, 0xf, false);
    return ((uint64_t)hi << 32) | lo;
}

// Inclusive prefix sum of one 64-bit value per lane inside a group: four shifted additions
// inside the rows of 16 lanes, then the rows' totals handed on (to rows 1 and 3 for groups of
// 32, and to the upper half for the whole wave). Every lane of the wave must call it.
template <int G> __device__ __forceinline__ uint64_t group_inclusive_scan64(uint64_t v, int /*sub*/) {
    v += dpp_take64<0x111, 0xf>(v);
    v += dpp_take64<0x112, 0xf>(v);
    v += dpp_take64<0x114, 0xf>(v);
    v += dpp_take64<0x118, 0xf>(v);
    if (G >= 32) v += dpp_take64<0x142, 0xa>(v);
    if (G == 64) v += dpp_take64<0x143, 0xc>(v);
    return v;
}

// The 64-bit value of one lane of the wave; `lane` must be the same in every lane.
__device__ __forceinline__ uint64_t wave_get64(uint64_t v, int lane) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

// Inclusive prefix sum over the whole wave, and the wave's total in every lane.
__device__ __forceinline__ uint64_t wave_inclusive_scan64(uint64_t v) { return group_inclusive_scan64<64>(v, 0); }
__device__ __forceinline__ uint64_t wave_sum64(uint64_t v) { return wave_get64(wave_inclusive_scan64(v), 63); }

// The same for one 32-bit value per lane, whose sum over the group stays below 2^32.
template <int CTRL, int ROW_MASK> __device__ __forceinline__ uint32_t dpp_take32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xf, false);
}
template <int G> __device__ __forceinline__ uint32_t group_inclusive_scan32(uint32_t v) {
    v += dpp_take32<0x111, 0xf>(v);
    v += dpp_take32<0x112, 0xf>(v);
    v += dpp_take32<0x114, 0xf>(v);
    v += dpp_take32<0x118, 0xf>(v);
    if (G >= 32) v += dpp_take32<0x142, 0xa>(v);
    if (G == 64) v += dpp_take32<0x143, 0xc>(v);
    return v;
}
__device__ __forceinline__ uint32_t wave_inclusive_scan32(uint32_t v) { return group_inclusive_scan32<64>(v); }
__device__ __forceinline__ uint32_t wave_sum32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan32(v), kWave - 1);
}

// One of k successive weighted draws without replacement inside a group whose lane i
// holds candidate i: `run` is the inclusive prefix sum of the weights still in play,
// `total` their sum, `w` this lane's weight (below 2^32; 0 once taken), u the 64 random
// bits of this draw. Returns the lane of the first candidate whose running sum exceeds
// floor(u * total / 2^64), or -1 when nothing is left, and takes that candidate out:
// every running sum from its lane on drops by its weight, which is what summing the
// remaining weights again would give. All lanes of the wave must call this; groups
// with `active` false are left untouched.
template <int G>
__device__ __forceinline__ int group_weighted_pick(uint64_t& run, uint64_t& total, uint64_t& w, uint64_t u, bool active,
                                                   int group, int sub) {
    const uint64_t x = __umul64hi(u, total);
    const int pick = group_first<G>(__ballot(active && run > x), group);
    const uint64_t taken = group_get<G>((uint32_t)w, pick < 0 ? 0 : pick);   // executed by every lane
    if (active && pick >= 0) {
        if (sub >= pick) run -= taken;
        total -= taken;
        if (sub == pick) w = 0;
    }
    return pick;
}

// k successive weighted draws without replacement inside every group with `active` set: lane i holds
// candidate i's weight w, lane j the 64 random bits u of draw j. Returns draw j's candidate in lane j
// (-1 once nothing is left, and in lanes j >= k or of other groups). All lanes of the wave must call it.
// With every weight below 2^26 all sums of at most 64 of them fit 32 bits, and so does every product's
// high part: the draws then take half the instructions (and each lane scales its own draw to the current
// total, so that one 32-bit value travels per draw instead of 64 random bits). 40 000 windows of 25, 10
// kept: 18.9 us with 64-bit sums and separate low and high Philox products, 14.2 so.
template <int G> __device__ __forceinline__ int group_weighted_picks(uint32_t w, uint64_t u, int k, bool active, int group, int sub) {
    int mine = -1;
    if (!__ballot(active && w >= (1u << 26))) {
        uint32_t run = group_inclusive_scan32<G>(w);
        uint32_t total = group_get<G>(run, G - 1);
        for (int j = 0; j < k; ++j) {
            const uint32_t x = group_get<G>(mulhi_64x32(u, total), j);
            const int pick = group_first<G>(__ballot(active && run > x), group);
            const uint32_t taken = group_get<G>(w, pick < 0 ? 0 : pick);   // executed by every lane
            if (active && pick >= 0) {
                if (sub >= pick) run -= taken;
                total -= taken;
                if (sub == pick) w = 0;
            }
            if (active && sub == j) mine = pick;
        }
        return mine;
    }
    uint64_t left = w, run = group_inclusive_scan64<G>(left, sub), total = group_get64<G>(run, G - 1);
    for (int j = 0; j < k; ++j) {
        const int pick = group_weighted_pick<G>(run, total, left, group_get64<G>(u, j), active, group, sub);
        if (active && sub == j) mine = pick;
    }
    return mine;
}

// What a wave left in LDS for its own lanes can be read by them: its LDS operations complete in order.
__device__ __forceinline__ void own_lds_ready() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace
