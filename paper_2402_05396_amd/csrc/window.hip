// Candidate-window products of the adaptive sampler on gfx950.
//
// TASER (arXiv 2402.05396) samples in two levels (Sec. 3 overview, Alg. 1): a
// static finder returns m candidates per root, a small network turns them into
// probabilities q(j|i), and n of the m are kept. Two integer inputs of that
// network depend only on the candidate window (Sec. 3.2): freq(u_j), how often
// candidate j's node appears among the candidates, and the identity encoding
// IE[j][l] = 1 if u_j = u_l. The second draw of Alg. 1 then selects by one
// weight per (root, candidate).
//
// The kernels use a group of G = 16, 32 or 64 lanes per root (G >= m), one lane per candidate; the
// selection for many roots eight lanes per root.
#include <type_traits>

#include "sampling_device.h"
#include "taser_internal.h"

namespace {

constexpr int kThreads = 256;

// Candidates [0, n) of a window, as bits of the mask's part that begins at candidate `from`.
__device__ __forceinline__ uint32_t first_bits(int n, int from) {
    const int k = n - from;
    return k >= 32 ? ~0u : k <= 0 ? 0u : (1u << k) - 1u;
}

// freq + identity. Lane j of a group holds u_j; the group's u are broadcast from LDS, four at a time, and
// every lane shifts the outcomes of its comparisons into a bit mask over l of the candidates equal to it;
// freq is the mask's population count. The m x m identity bytes are those masks, one bit per byte: the
// masks of the block's roots go into LDS as one string of bits, and the block's range of the output is
// written from it 16 bytes at a time (4 bits times 0x204081 are 4 bytes), whatever m and the alignment.
// Bound by its output: 40 000 windows of 25 (33 MB in all) take 9.1 to 10.4 us, 6.4 at the rate of a large copy; with one lane shuffle per
// comparison and per output byte it was 24 us of vector and LDS instructions.
// ROOTS of a block: so many that their matrices are whole 16-byte pieces, of which none is shared by two blocks and written by
// bytes: 8 where m is even, 16 where it is odd. us by 8 / by 16, windows of 25: 600 3.32 2.97, 8 000 4.61 4.20, 40 000 9.79 9.21; of
// 32: 600 2.72 2.81, 8 000 4.06 4.30, 40 000 9.32 9.81. Up to 16 candidates have 16 lanes, and 16 roots in 256 threads; with 64 lanes
// per root 16 would be 1 024 threads (2 000 windows of 64 5.9 us, of 4 roots 4.5).
// PAST: the pieces go past the caches. With odd m most blocks end inside a 128-byte line, and the parts of a line that go past the caches
// are late where there is little to write: us through the caches / past them, windows of 9: 2 000 2.26 2.54, 40 000 4.01 4.43; of 25:
// 2 000 2.82 3.10, 8 000 3.80 4.19, 16 000 (10 MB) 5.49 5.55, 40 000 9.84 9.19. So there it is done from 12 MB on; with even m always: windows of
// 32, 2 000 2.96 2.95, 16 000 6.40 5.61, 40 000 10.99 9.21.
constexpr int64_t kPastFrom = 12 << 20;
template <int G, int ROOTS, bool PAST>
__global__ __launch_bounds__(ROOTS * G) void candidate_encodings_kernel(
    const int32_t* __restrict__ nbr, const int32_t* __restrict__ count, int64_t num_roots, int m, int32_t* __restrict__ freq,
    uint8_t* __restrict__ identity) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
    constexpr int kRoots = ROOTS, kThreads = ROOTS * G;
    constexpr int kWords = kRoots * G * G / 32 + 1;     // bits of their identity matrices, and a word to read past the end
    constexpr int kParts = G > 32 ? 2 : 1;              // 32-bit parts of a mask
    __shared__ __align__(16) int32_t cand[kThreads];
    __shared__ uint32_t bits[kWords];
    const int group = threadIdx.x / G, sub = threadIdx.x % G;
    const int64_t root0 = (int64_t)blockIdx.x * kRoots, q = root0 + group;
    const bool live = q < num_roots;
    int c = 0;
    if (live) {
        c = count[q];
        c = c < 0 ? 0 : (c > m ? m : c);
    }
    const bool mine_valid = sub < c;
    int32_t u = -1;
    if (mine_valid) u = nbr[q * m + sub];
    cand[threadIdx.x] = u;
    for (int i = threadIdx.x; i < kWords; i += kThreads) bits[i] = 0;
    __syncthreads();

    uint32_t same[kParts];   // bit l: candidate l is valid and names the same node as mine
#pragma unroll
    for (int p = 0; p < kParts; ++p) {
        same[p] = 0;
        const i32x4* from = reinterpret_cast<const i32x4*>(cand + group * G + 32 * p);
#pragma unroll
        for (int i = (G < 32 ? G : 32) / 4 - 1; i >= 0; --i) {
            if (32 * p + 4 * i >= m) continue;          // uniform
            const i32x4 v = from[i];
            same[p] = 2u * same[p] + (uint32_t)(v.w == u);
            same[p] = 2u * same[p] + (uint32_t)(v.z == u);
            same[p] = 2u * same[p] + (uint32_t)(v.y == u);
            same[p] = 2u * same[p] + (uint32_t)(v.x == u);
        }
        same[p] = mine_valid ? same[p] & first_bits(c, 32 * p) : 0u;
    }
    if (live && sub < m) {
        int n = __popc(same[0]);
        if (kParts == 2) n += __popc(same[kParts - 1]);
        freq[q * m + sub] = n;
    }

    if (identity == nullptr) return;   // uniform for the whole grid
    if (sub < m) {
        const uint32_t at = (uint32_t)(group * m + sub) * (uint32_t)m;   // this row's place in the string of bits
        const uint32_t shift = at & 31u;
#pragma unroll
        for (int p = 0; p < kParts; ++p) {
            if (!same[p]) continue;
            atomicOr(&bits[at / 32u + p], same[p] << shift);
            if (shift) atomicOr(&bits[at / 32u + p + 1], same[p] >> (32u - shift));
        }
    }
    __syncthreads();
    const int64_t roots_here = num_roots - root0 < kRoots ? num_roots - root0 : kRoots;
    const uint32_t length = (uint32_t)roots_here * (uint32_t)(m * m);               // bytes of the block's range
    const uint64_t base = (uint64_t)(uintptr_t)identity + (uint64_t)root0 * (uint64_t)(m * m);
    const uint32_t head = (uint32_t)(base & 15u);                                   // bytes between the aligned start and base
    uint8_t* const aligned = reinterpret_cast<uint8_t*>(base - head);
    for (uint32_t off = threadIdx.x * 16u; off < head + length; off += kThreads * 16u) {
        if (off >= head && off + 16u <= head + length) {
            const uint32_t b = off - head;
            const uint32_t x = __builtin_amdgcn_alignbit(bits[b / 32u + 1u], bits[b / 32u], b & 31u);
            u32x4 v;
            v.x = __umul24(x & 15u, 0x204081u) & 0x01010101u;
            v.y = __umul24((x >> 4) & 15u, 0x204081u) & 0x01010101u;
            v.z = __umul24((x >> 8) & 15u, 0x204081u) & 0x01010101u;
            v.w = __umul24((x >> 12) & 15u, 0x204081u) & 0x01010101u;
            if (PAST) __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(aligned + off));
            else *reinterpret_cast<u32x4*>(aligned + off) = v;
        } else {   // the range's first or last bytes
            for (uint32_t o = off; o < off + 16u; o += 4u) {
                if (o >= head && o + 4u <= head + length) {
                    const uint32_t b = o - head;
                    const uint32_t x = __builtin_amdgcn_alignbit(bits[b / 32u + 1u], bits[b / 32u], b & 31u) & 15u;
                    *reinterpret_cast<uint32_t*>(aligned + o) = __umul24(x, 0x204081u) & 0x01010101u;
                } else {
                    for (uint32_t e = o; e < o + 4u; ++e)
                        if (e >= head && e < head + length) aligned[e] = (uint8_t)((bits[(e - head) / 32u] >> ((e - head) & 31u)) & 1u);
                }
            }
        }
    }
}

// n of m by per-slot weights: lane i of a group holds the weight of candidate i.
// The running sums of the weights are taken once; each of the k rounds scales one
// 64-bit draw to the remaining total, picks the first lane whose running sum exceeds
// it and takes that lane's weight out of the sums after it (group_weighted_picks). Lane j
// keeps round j's pick, so the outputs are written coalesced at the end.
template <int G>
__global__ __launch_bounds__(kThreads) void select_weighted_kernel(
    const uint32_t* __restrict__ weight, const int32_t* __restrict__ count, int64_t num_roots, int m, int k,
    uint32_t seed_lo, uint32_t seed_hi, uint32_t hop, int32_t* __restrict__ sel, int32_t* __restrict__ out_count,
    const int32_t* __restrict__ c_nbr, const int32_t* __restrict__ c_eid, const int64_t* __restrict__ c_ts,
    int32_t* __restrict__ k_nbr, int32_t* __restrict__ k_eid, int64_t* __restrict__ k_ts) {
    constexpr int kGroups = kWave / G;
    const int lane = threadIdx.x & (kWave - 1);
    const int group = lane / G, sub = lane % G;
    const int64_t q = ((int64_t)blockIdx.x * (kThreads / kWave) + (threadIdx.x >> 6)) * kGroups + group;
    const bool live = q < num_roots;

    int c = 0;
    if (live) {
        c = count[q];
        c = c < 0 ? 0 : (c > m ? m : c);
    }
    uint32_t w = 0;
    if (sub < c) w = weight[q * m + sub];
    const bool draw = c > k;
    const int filled = draw ? k : c;
    int32_t my_pick = (!draw && sub < c) ? sub : -1;   // slot `sub` of the output
    if (__ballot(draw)) {
        uint64_t u = 0;
        if (draw && sub < k) u = draw64_wide(seed_lo, seed_hi, hop, (uint64_t)q, (uint32_t)sub);
        const int pick = group_weighted_picks<G>(w, u, k, draw, group, sub);   // -1 only if every remaining weight is 0
        if (draw) my_pick = pick;
    }
    if (live && sub < k) {
        const int64_t at = q * k + sub;
        sel[at] = my_pick;
        if (k_nbr) {
            const bool ok = my_pick >= 0;
            const int64_t from = q * m + (ok ? my_pick : 0);
            k_nbr[at] = ok ? c_nbr[from] : -1;
            k_eid[at] = ok ? c_eid[from] : -1;
            k_ts[at] = ok ? c_ts[from] : 0;
        }
    }
    if (live && sub == 0) out_count[q] = filled;
}

// ---- octets: eight lanes per root, eight roots per wave -----------------------------------------------------
// With a lane per candidate a wave of 32-lane groups spends the instructions of every draw on two roots. Here lane
// `sub` of a root's octet holds its candidates sub * C to sub * C + C - 1, and a wave's instructions serve eight. All
// exchanges are DPP moves inside rows of sixteen lanes: neighbors, pairs of neighbors (quad_perm), and the other quad of
// the octet (row_half_mirror, where the quad's lanes agree).
template <typename T, int CTRL> __device__ __forceinline__ T lanes_take(T v) {
    if constexpr (sizeof(T) == 8) return (T)dpp_take64<CTRL, 0xf>((uint64_t)v);
    else return (T)dpp_take32<CTRL, 0xf>((uint32_t)v);
}
template <typename T> __device__ __forceinline__ T octet_sum(T v) {
    v += lanes_take<T, 0xB1>(v);
    v += lanes_take<T, 0x4E>(v);
    return v + lanes_take<T, 0x141>(v);
}
template <typename T> __device__ __forceinline__ T octet_max(T v) {
    T o = lanes_take<T, 0xB1>(v);
    v = v > o ? v : o;
    o = lanes_take<T, 0x4E>(v);
    v = v > o ? v : o;
    o = lanes_take<T, 0x141>(v);
    return v > o ? v : o;
}
// The value of the octet's lane AT.
template <int AT, typename T> __device__ __forceinline__ T octet_get(T v, int sub) {
    const T quad = lanes_take<T, (AT & 3) * 0x55>(v), other = lanes_take<T, 0x141>(quad);
    return (sub >> 2) == (AT >> 2) ? quad : other;
}
__device__ __forceinline__ uint32_t scaled_draw(uint64_t u, uint32_t total) { return mulhi_64x32(u, total); }
__device__ __forceinline__ uint64_t scaled_draw(uint64_t u, uint64_t total) { return __umul64hi(u, total); }

// One draw: `run` the running sums of the weights still in play, x below their total. Returns the candidate whose
// running sum first exceeds x (8 C where there is none), and takes it out.
template <int C, typename T> __device__ __forceinline__ uint32_t octet_draw(T (&run)[C], T& total, T x) {
    // entries that do not exceed x come first: their number is the candidate, and its weight what lies between the
    // largest of their sums and the smallest of the others'
    uint32_t below = 0;
    T low = 0, high = ~(T)0;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        below += run[i] <= x ? 1u : 0u;
        low = run[i] <= x ? run[i] : low;
    }
#pragma unroll
    for (int i = C - 1; i >= 0; --i) high = run[i] > x ? run[i] : high;
    below = octet_sum(below);
    low = octet_max(low);
    high = (T)~octet_max((T)~high);
    const T taken = below < 8u * C ? high - low : (T)0;
#pragma unroll
    for (int i = 0; i < C; ++i) run[i] -= run[i] > x ? taken : (T)0;
    total -= taken;
    return below;
}

// k successive draws without replacement for every octet: draw j's candidate (-1 once nothing is left) goes to
// picks[j], which is the octet's own. All lanes of the wave must call it.
template <int C, typename T>
__device__ __forceinline__ void octet_picks(const uint32_t (&w)[C], int k, uint32_t seed_lo, uint32_t seed_hi, uint32_t hop, uint64_t root, int sub,
                                            int8_t* picks) {
    T run[C], sum = 0;
#pragma unroll
    for (int i = 0; i < C; ++i) run[i] = sum += w[i];
    T upto = sum;    // over the octet's lanes up to this one
    T o = lanes_take<T, 0x111>(upto);
    upto += sub >= 1 ? o : (T)0;
    o = lanes_take<T, 0x112>(upto);
    upto += sub >= 2 ? o : (T)0;
    o = lanes_take<T, 0x114>(upto);
    upto += sub >= 4 ? o : (T)0;
#pragma unroll
    for (int i = 0; i < C; ++i) run[i] += upto - sum;
    T total = octet_max(upto);
#pragma unroll 1
    for (int j0 = 0; j0 < k; j0 += 8) {
        const uint64_t u = draw64_wide(seed_lo, seed_hi, hop, root, (uint32_t)(j0 + sub));   // lane sub's is draw j0 + sub
        auto one = [&](auto at) {
            constexpr int AT = decltype(at)::value;
            if (j0 + AT < k) {   // uniform
                const T x = octet_get<AT>(scaled_draw(u, total), sub);
                const uint32_t pick = octet_draw<C, T>(run, total, x);
                if (sub == AT) picks[j0 + AT] = pick < 8u * C ? (int8_t)pick : (int8_t)-1;
            }
        };
        one(std::integral_constant<int, 0>{});
        one(std::integral_constant<int, 1>{});
        one(std::integral_constant<int, 2>{});
        one(std::integral_constant<int, 3>{});
        one(std::integral_constant<int, 4>{});
        one(std::integral_constant<int, 5>{});
        one(std::integral_constant<int, 6>{});
        one(std::integral_constant<int, 7>{});
    }
}

// The same for whatever weights: in 32 bits where all sums of the wave's roots fit them.
template <int C>
__device__ __forceinline__ void octet_weighted_picks(const uint32_t (&w)[C], int k, bool active, uint32_t seed_lo, uint32_t seed_hi, uint32_t hop,
                                                     uint64_t root, int sub, int8_t* picks) {
    uint32_t any = 0;
#pragma unroll
    for (int i = 0; i < C; ++i) any |= w[i];
    if (!__ballot(active && any >= (1u << 26))) octet_picks<C, uint32_t>(w, k, seed_lo, seed_hi, hop, root, sub, picks);   // at most 64 of them
    else octet_picks<C, uint64_t>(w, k, seed_lo, seed_hi, hop, root, sub, picks);
}

// The same for many roots: an octet of lanes per root draws (octet_weighted_picks); the slots of a wave's eight roots
// are then written flat, so that all lanes load and store whatever k is. Bound by vector instructions like the other one, but
// with fewer of them where that one has one or two roots per wave; its chain of dependent steps is longer, so it is for
// numbers of roots that fill the chip, and not for windows that are all kept. us of the other one / of this one, 2 000,
// 8 000, 40 000 roots: 10 of 16 candidates 3.9 4.3, 4.1 4.7, 9.0 8.9; 10 of 25 3.9 4.6, 5.0 4.9, 13.7 10.4; 24 of 25
// 5.8 6.8, 7.9 7.3, 23.8 18.1; 20 of 49 5.5 7.7, 9.8 8.1, 33.4 21.0; 64 of 64 2.7 5.6, 4.2 6.5, 16.6 17.8.
//
// An octet costs its wave as much as eight do, and most roots of a sparse graph have no more than k candidates and draw
// nothing. So where few draw, each of them gets a lane per candidate as in the other kernel, G = 8 C lanes: with windows of
// up to 32 the drawing roots of a wave if they are two at most, with longer ones, whose octets have the longer chain, those
// of a block if they are four at most, one per wave; more than that are packed into octets. us of the other one, of octets
// for every root, and so, 120 000 roots of which one in 8 / one in 30 has more than k candidates: 10 of 25 15.8 18.3 12.3,
// 11.0 13.2 8.6; 32 of 64 40.1 63.0 32.1, 27.9 41.9 18.1; 60 of 64 60.1 112 55.2, 36.5 74.5 30.3; 16 000 roots: 10 of 25
// 5.5 5.3 5.3, 5.3 5.3 5.4; 32 of 64 10.9 13.5 10.3, 8.8 13.3 9.0; 60 of 64 17.7 23.3 22.4, 13.5 22.9 15.1.
constexpr int64_t kOctetRoots = 8000;
constexpr int kSelectRoots = kWave / 8;                            // of a wave
constexpr int kBlockRoots = kThreads / kWave * kSelectRoots;      // of a block

// One draw after the other for the roots `root` (of the block) of those of the wave's groups that are active.
template <int G>
__device__ __forceinline__ void group_draws(const uint32_t* __restrict__ weight, int64_t root, int at, int candidates, bool active, int m, int k,
                                            uint32_t seed_lo, uint32_t seed_hi, uint32_t hop, int group, int slot, int8_t* picks) {
    uint32_t w = 0;
    if (active && slot < candidates) w = weight[root * m + slot];
    uint64_t u = 0;
    if (active && slot < k) u = draw64_wide(seed_lo, seed_hi, hop, (uint64_t)root, (uint32_t)slot);
    const int pick = group_weighted_picks<G>(w, u, k, active, group, slot);
    if (active && slot < k) picks[at * k + slot] = (int8_t)pick;
}
template <int C>
__device__ __forceinline__ void octet_draws(const uint32_t* __restrict__ weight, int64_t root, int at, int candidates, bool active, int m, int k,
                                            uint32_t seed_lo, uint32_t seed_hi, uint32_t hop, int sub, int8_t* picks) {
    uint32_t w[C];
#pragma unroll
    for (int i = 0; i < C; ++i) {
        w[i] = 0;
        if (active && sub * C + i < candidates) w[i] = weight[root * m + sub * C + i];
    }
    octet_weighted_picks<C>(w, k, active, seed_lo, seed_hi, hop, (uint64_t)root, sub, picks + (active ? at : kBlockRoots) * k);
}

template <int C>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8))) void select_weighted_octets_kernel(
    const uint32_t* __restrict__ weight, const int32_t* __restrict__ count, int64_t num_roots, int m, int k, uint32_t magic_k,
    uint32_t seed_lo, uint32_t seed_hi, uint32_t hop, int32_t* __restrict__ sel, int32_t* __restrict__ out_count,
    const int32_t* __restrict__ c_nbr, const int32_t* __restrict__ c_eid, const int64_t* __restrict__ c_ts,
    int32_t* __restrict__ k_nbr, int32_t* __restrict__ k_eid, int64_t* __restrict__ k_ts) {
    constexpr int G = 8 * C, kGroups = kWave / G, kWaves = kThreads / kWave;
    __shared__ int8_t picks[(kBlockRoots + 1) * TASER_MAX_K];   // the last row is for octets that have no root
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6, octet = lane >> 3, sub = lane & 7;
    const int64_t b0 = (int64_t)blockIdx.x * kBlockRoots, q0 = b0 + wave * kSelectRoots, q = q0 + octet;   // the block's first root, the wave's, the octet's
    const int here = num_roots - q0 >= kSelectRoots ? kSelectRoots : num_roots > q0 ? (int)(num_roots - q0) : 0;
    const int mine = wave * kSelectRoots + octet, group = lane / G, slot = lane % G;
    int c = 0;
    if (octet < here) {
        c = count[q];
        c = c < 0 ? 0 : (c > m ? m : c);
    }
    const uint64_t draws = __ballot(sub == 0 && c > k);   // a bit per root that draws
    if constexpr (C == 4) {
        if (__popcll(draws) > kGroups) {
            octet_draws<C>(weight, q, mine, c, c > k, m, k, seed_lo, seed_hi, hop, sub, picks);
        } else if (draws) {
            const int first = (__ffsll((long long)draws) - 1) >> 3, last = (63 - __clzll((long long)draws)) >> 3, r = group == 0 ? first : last;
            group_draws<G>(weight, q0 + r, wave * kSelectRoots + r, __shfl(c, r * 8, kWave), group == 0 || last != first, m, k, seed_lo, seed_hi, hop,
                           group, slot, picks);
        }
        own_lds_ready();
    } else {
        __shared__ uint8_t counts[kBlockRoots], drawing[kBlockRoots];   // candidates of the block's roots; those that draw, in order
        __shared__ int draws_of_wave[kWaves];
        if (sub == 0) counts[mine] = (uint8_t)c;
        if (lane == 0) draws_of_wave[wave] = __popcll(draws);
        __syncthreads();
        int before = 0, all = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            if (w < wave) before += draws_of_wave[w];
            all += draws_of_wave[w];
        }
        all = __builtin_amdgcn_readfirstlane(all);
        if (all > 0) {   // uniform over the block, like the next
            const bool own = all == kBlockRoots;   // every octet keeps its root: nothing passes from wave to wave
            if (!own) {
                if (sub == 0 && c > k) drawing[before + __popcll(draws & (((uint64_t)1 << lane) - 1))] = (uint8_t)mine;
                __syncthreads();
            }
            const bool packed = all > kWaves * kGroups;
            const int n = packed ? mine : wave + group * kWaves;   // of the roots that draw
            const int at = own ? mine : drawing[n < all ? n : 0], candidates = own ? c : counts[at];
            if (packed) {
                if (wave * kSelectRoots < all) octet_draws<C>(weight, b0 + at, at, candidates, n < all, m, k, seed_lo, seed_hi, hop, sub, picks);
            } else if (wave < all) {
                group_draws<G>(weight, b0 + at, at, candidates, n < all, m, k, seed_lo, seed_hi, hop, group, slot, picks);
            }
            if (own) own_lds_ready();
            else __syncthreads();
        }
    }
    if (octet < here && sub == 0) out_count[q] = c > k ? k : c;
    const uint32_t slots = (uint32_t)(here * k);
    for (uint32_t s0 = 0; s0 < slots; s0 += kWave) {
        const uint32_t s = s0 + (uint32_t)lane;
        uint32_t r = k == 1 ? s : __umulhi(s, magic_k);        // exact: s < 2^10, k <= 64
        const uint32_t j = s - r * (uint32_t)k;
        if (r > kSelectRoots - 1) r = kSelectRoots - 1;        // past the wave's slots
        const int of_root = __shfl(c, (int)r * 8, kWave);      // (all lanes take part)
        if (s >= slots) continue;
        const int pick = of_root > k ? picks[wave * kSelectRoots * k + s] : (int)j < of_root ? (int)j : -1;
        const int64_t at = q0 * k + s;
        sel[at] = pick;
        if (k_nbr) {
            const bool ok = pick >= 0;
            const int64_t from = (q0 + r) * m + (ok ? pick : 0);
            k_nbr[at] = ok ? c_nbr[from] : -1;
            k_eid[at] = ok ? c_eid[from] : -1;
            k_ts[at] = ok ? c_ts[from] : 0;
        }
    }
}

template <int G> unsigned grid_for(int64_t n) {
    constexpr int roots_per_block = (kThreads / kWave) * (kWave / G);
    return (unsigned)((n + roots_per_block - 1) / roots_per_block);
}

}  // namespace

extern "C" int taser_candidate_encodings(const int32_t* nbr, const int32_t* count, int64_t num_roots, int32_t m,
                                         int32_t* freq, uint8_t* identity, void* hip_stream) {
    if (num_roots < 0) return taser_fail(TASER_E_ARG, "candidate_encodings: num_roots = %lld", (long long)num_roots);
    if (m < 1 || m > TASER_MAX_M) return taser_fail(TASER_E_RANGE, "candidate_encodings: m = %d outside [1, %d]", m, TASER_MAX_M);
    if (num_roots * (int64_t)m >= ((int64_t)1 << 31))
        return taser_fail(TASER_E_RANGE, "candidate_encodings: num_roots * m must stay below 2^31");
    if (num_roots == 0) return TASER_OK;
    if (!nbr || !count || !freq) return taser_fail(TASER_E_ARG, "candidate_encodings: null nbr, count or freq");
    taser_clear_stale_hip_error();
    hipStream_t stream = (hipStream_t)hip_stream;
    TaserProfileSpan span(stream, "candidate_encodings");
    const bool past = m % 2 == 0 || num_roots * m * m >= kPastFrom;   // num_roots * m is below 2^31
    const int lanes = m <= 16 ? 16 : m <= 32 ? 32 : 64, roots = lanes == 64 ? 4 : lanes == 32 && m % 2 == 0 ? 8 : 16;
    const auto kernel = lanes == 64   ? (past ? candidate_encodings_kernel<64, 4, true> : candidate_encodings_kernel<64, 4, false>)
                        : roots == 8  ? candidate_encodings_kernel<32, 8, true>
                        : lanes == 32 ? (past ? candidate_encodings_kernel<32, 16, true> : candidate_encodings_kernel<32, 16, false>)
                                      : (past ? candidate_encodings_kernel<16, 16, true> : candidate_encodings_kernel<16, 16, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)((num_roots + roots - 1) / roots)), dim3(roots * lanes), 0, stream, nbr, count, num_roots, m, freq, identity);
    TASER_HIP_TRY(hipGetLastError());
    return TASER_OK;
}

extern "C" int taser_select_weighted(const uint32_t* weight, const int32_t* count, int64_t num_roots, int32_t m,
                                     int32_t k, uint64_t seed, uint32_t hop, int32_t* sel, int32_t* out_count,
                                     const taser_hop_out* candidates, const taser_hop_out* kept, void* hip_stream) {
    if (num_roots < 0) return taser_fail(TASER_E_ARG, "select_weighted: num_roots = %lld", (long long)num_roots);
    if (m < 1 || m > TASER_MAX_M) return taser_fail(TASER_E_RANGE, "select_weighted: m = %d outside [1, %d]", m, TASER_MAX_M);
    if (k < 1 || k > TASER_MAX_K) return taser_fail(TASER_E_RANGE, "select_weighted: k = %d outside [1, %d]", k, TASER_MAX_K);
    if (num_roots * (int64_t)(m > k ? m : k) >= ((int64_t)1 << 31))
        return taser_fail(TASER_E_RANGE, "select_weighted: num_roots * max(m, k) must stay below 2^31");
    if ((candidates == nullptr) != (kept == nullptr))
        return taser_fail(TASER_E_ARG, "select_weighted: candidates and kept go together");
    if (num_roots == 0) return TASER_OK;
    if (!weight || !count || !sel || !out_count) return taser_fail(TASER_E_ARG, "select_weighted: null weight, count, sel or out_count");
    if (kept && (!candidates->nbr || !candidates->eid || !candidates->ts || !kept->nbr || !kept->eid || !kept->ts))
        return taser_fail(TASER_E_ARG, "select_weighted: null nbr/eid/ts buffer in candidates or kept");
    taser_clear_stale_hip_error();
    hipStream_t stream = (hipStream_t)hip_stream;
    const int32_t *c_nbr = nullptr, *c_eid = nullptr;
    const int64_t* c_ts = nullptr;
    int32_t *k_nbr = nullptr, *k_eid = nullptr;
    int64_t* k_ts = nullptr;
    if (kept) {
        c_nbr = candidates->nbr; c_eid = candidates->eid; c_ts = candidates->ts;
        k_nbr = kept->nbr; k_eid = kept->eid; k_ts = kept->ts;
    }
    const uint32_t s_lo = (uint32_t)seed, s_hi = (uint32_t)(seed >> 32);
    const int lanes = m > k ? m : k;
    TaserProfileSpan span(stream, "select_weighted");
    if (m > 16 && m > k && num_roots >= kOctetRoots) {
        const auto kernel = m <= 32 ? select_weighted_octets_kernel<4> : select_weighted_octets_kernel<8>;
        constexpr int roots_per_block = kThreads / kWave * kSelectRoots;
        const uint32_t magic_k = k > 1 ? (uint32_t)((((uint64_t)1 << 32) + (uint32_t)k - 1) / (uint32_t)k) : 0u;
        hipLaunchKernelGGL(kernel, dim3((unsigned)((num_roots + roots_per_block - 1) / roots_per_block)), dim3(kThreads), 0, stream, weight, count,
                           num_roots, m, k, magic_k, s_lo, s_hi, hop, sel, out_count, c_nbr, c_eid, c_ts, k_nbr, k_eid, k_ts);
    } else if (lanes <= 16)
        hipLaunchKernelGGL((select_weighted_kernel<16>), dim3(grid_for<16>(num_roots)), dim3(kThreads), 0, stream, weight, count, num_roots, m, k, s_lo, s_hi, hop, sel, out_count, c_nbr, c_eid, c_ts, k_nbr, k_eid, k_ts);
    else if (lanes <= 32)
        hipLaunchKernelGGL((select_weighted_kernel<32>), dim3(grid_for<32>(num_roots)), dim3(kThreads), 0, stream, weight, count, num_roots, m, k, s_lo, s_hi, hop, sel, out_count, c_nbr, c_eid, c_ts, k_nbr, k_eid, k_ts);
    else
        hipLaunchKernelGGL((select_weighted_kernel<64>), dim3(grid_for<64>(num_roots)), dim3(kThreads), 0, stream, weight, count, num_roots, m, k, s_lo, s_hi, hop, sel, out_count, c_nbr, c_eid, c_ts, k_nbr, k_eid, k_ts);
    TASER_HIP_TRY(hipGetLastError());
    return TASER_OK;
}
