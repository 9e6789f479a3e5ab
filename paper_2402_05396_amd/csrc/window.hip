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
// Both kernels use a group of G = 16, 32 or 64 lanes per root (G >= m), one
// lane per candidate.
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
// Bound by its output: 40 000 windows of 25 (33 MB in all) take 12 us; with one lane shuffle per comparison
// and per output byte it was 24 us of vector and LDS instructions.
template <int G>
__global__ __launch_bounds__(kThreads) void candidate_encodings_kernel(
    const int32_t* __restrict__ nbr, const int32_t* __restrict__ count, int64_t num_roots, int m, int32_t* __restrict__ freq,
    uint8_t* __restrict__ identity) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
    constexpr int kRoots = kThreads / G;                // roots of a block
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
            *reinterpret_cast<u32x4*>(aligned + off) = v;
        } else {   // the range's first or last bytes
            for (uint32_t o = off; o < off + 16u; ++o)
                if (o >= head && o < head + length) aligned[o] = (uint8_t)((bits[(o - head) / 32u] >> ((o - head) & 31u)) & 1u);
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
    if (m <= 16)
        hipLaunchKernelGGL((candidate_encodings_kernel<16>), dim3(grid_for<16>(num_roots)), dim3(kThreads), 0, stream, nbr, count, num_roots, m, freq, identity);
    else if (m <= 32)
        hipLaunchKernelGGL((candidate_encodings_kernel<32>), dim3(grid_for<32>(num_roots)), dim3(kThreads), 0, stream, nbr, count, num_roots, m, freq, identity);
    else
        hipLaunchKernelGGL((candidate_encodings_kernel<64>), dim3(grid_for<64>(num_roots)), dim3(kThreads), 0, stream, nbr, count, num_roots, m, freq, identity);
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
    if (lanes <= 16)
        hipLaunchKernelGGL((select_weighted_kernel<16>), dim3(grid_for<16>(num_roots)), dim3(kThreads), 0, stream, weight, count, num_roots, m, k, s_lo, s_hi, hop, sel, out_count, c_nbr, c_eid, c_ts, k_nbr, k_eid, k_ts);
    else if (lanes <= 32)
        hipLaunchKernelGGL((select_weighted_kernel<32>), dim3(grid_for<32>(num_roots)), dim3(kThreads), 0, stream, weight, count, num_roots, m, k, s_lo, s_hi, hop, sel, out_count, c_nbr, c_eid, c_ts, k_nbr, k_eid, k_ts);
    else
        hipLaunchKernelGGL((select_weighted_kernel<64>), dim3(grid_for<64>(num_roots)), dim3(kThreads), 0, stream, weight, count, num_roots, m, k, s_lo, s_hi, hop, sel, out_count, c_nbr, c_eid, c_ts, k_nbr, k_eid, k_ts);
    TASER_HIP_TRY(hipGetLastError());
    return TASER_OK;
}
