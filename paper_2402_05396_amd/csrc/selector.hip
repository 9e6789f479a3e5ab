// Adaptive mini-batch selection on gfx950 (TASER, arXiv 2402.05396, Sec. 3.1):
// an importance score per training edge, batches drawn with probability
// proportional to the scores, the scores of a batch overwritten after the
// iteration.
//
// An iteration changes only a batch's worth of scores, so nothing here is
// linear in the number of training edges per iteration: the scores carry two
// levels of partial sums (1024 scores per level-1 sum, 1024 level-1 sums per
// level-2 sum) that an update adjusts by the difference it makes, and a draw
// descends the three levels with one wavefront: at most 32 rows of 64 values of
// the top level for 2^31 edges, one for a million, then one group of 1024 values
// of each lower level, read at once.
#include <new>

#include "edge_hash.h"
#include "sampling_device.h"
#include "taser_internal.h"

struct taser_selector {
    int64_t n;          // training edges
    int64_t n1, n2;     // level-1 and level-2 sums
    uint32_t* score;    // device uint32[n]
    uint64_t* sum1;     // device uint64[n1]: sum of score[1024*i .. 1024*i+1023]
    uint64_t* sum2;     // device uint64[n2]: sum of sum1[1024*i .. 1024*i+1023]
    int32_t* owner;     // device int32[n], -1 between calls: latest batch position that names an edge
};

namespace {

constexpr int kThreads = 256;
constexpr int kFan = 1024;             // values per partial sum
constexpr uint32_t kDrawTag = 0x4253454Cu;

// First index i in [begin, end) whose running sum over a[begin..i] exceeds x, by
// one wavefront, 64 values per step; x is reduced by the sum before a[i]. The
// caller guarantees that the whole range sums to more than x. Wave-uniform.
// Used for the top level, whose length varies.
template <typename T>
__device__ __forceinline__ int64_t wave_descend(const T* __restrict__ a, int64_t begin, int64_t end, uint64_t& x,
                                                int lane) {
    uint64_t before = 0;
    for (int64_t row = begin; row < end; row += kWave) {
        const int64_t i = row + lane;
        const uint64_t v = i < end ? (uint64_t)a[i] : 0;
        const uint64_t inc = wave_inclusive_scan64(v);
        const uint64_t hit = __ballot(before + inc > x);
        if (hit) {
            const int first = __ffsll((long long)hit) - 1;
            x -= before + wave_get64(inc - v, first);
            return row + first;
        }
        before += wave_get64(inc, kWave - 1);
    }
    return end - 1;   // not reached while the guarantee holds
}

// Totals over the wave of R values per lane (rows of a group), 4 at a time: lanes exchange halves so that every
// quarter of the wave ends up with one row's sums, 22 instructions for a row where a prefix sum takes 25. v[4 i]
// then holds rows 4 i .. 4 i + 3, which total_of_row takes out.
template <int R> __device__ __forceinline__ void fold_rows(uint64_t (&v)[R]) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    auto join = [](u32x2 lo, u32x2 hi) { return (((uint64_t)hi.x << 32) | lo.x) + (((uint64_t)hi.y << 32) | lo.y); };
    auto halves = [&](uint64_t a, uint64_t b) {     // lower half of the wave: a's sums, upper half: b's
        const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
        return join(u32x2{lo[0], lo[1]}, u32x2{hi[0], hi[1]});
    };
    auto quarters = [&](uint64_t a, uint64_t b) {   // of each half: a's sums, then b's
        const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)a, (uint32_t)b, false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
        return join(u32x2{lo[0], lo[1]}, u32x2{hi[0], hi[1]});
    };
#pragma unroll
    for (int i = 0; i < R; i += 4) {
        uint64_t t = quarters(halves(v[i], v[i + 1]), halves(v[i + 2], v[i + 3]));
        t += dpp_take64<0x128, 0xf>(t);             // rotations inside 16 lanes
        t += dpp_take64<0x124, 0xf>(t);
        t += dpp_take64<0x122, 0xf>(t);
        t += dpp_take64<0x121, 0xf>(t);
        v[i] = t;
    }
}
template <int R> __device__ __forceinline__ uint64_t total_of_row(const uint64_t (&folded)[R], int r) {
    return wave_get64(folded[r & ~3], (r & 1) * 32 + (r & 2) * 8);
}

// The same for one group of up to 1024 values starting at a[begin], all its loads in flight together. The
// group is read in rows of 64 x 16 bytes, one piece per lane, so that a load covers whole lines (with 16
// neighboring values per lane every load touched 64 lines). The row is found first, from the rows' totals, then
// the lane by a prefix sum over that row alone, then the value. Draws from 1 M, 40 M, 500 M scores, us a launch with 16
// neighboring values per lane / a prefix sum over every row / so: 600 draws 6.3 5.3 7.4 / 5.1 4.6 6.8 / 4.8 4.2 6.5,
// 100 000 draws 193 119 175 / 136 130 200 / 88 83 141.
template <typename T> struct Group {
    static constexpr int kVec = 16 / (int)sizeof(T);          // values per piece: 4 or 2
    static constexpr int kRows = kFan / (kWave * kVec);       // 4 or 8
    T v[kRows][kVec];
};
template <typename T>
__device__ __forceinline__ void load_group(const T* __restrict__ a, int64_t begin, int64_t end, int lane, Group<T>& group) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    constexpr int kVec = Group<T>::kVec, kRows = Group<T>::kRows;
    auto& v = group.v;
    const int64_t mine = begin + (int64_t)lane * kVec;
    if (begin + kFan <= end) {   // a whole group (wave-uniform); `begin` is a multiple of 1024 values, so the address is aligned
        u32x4 raw[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r) raw[r] = *reinterpret_cast<const u32x4*>(a + mine + r * kWave * kVec);
        __builtin_memcpy(v, raw, sizeof(v));
    } else {
#pragma unroll
        for (int r = 0; r < kRows; ++r)
#pragma unroll
            for (int i = 0; i < kVec; ++i) v[r][i] = mine + r * kWave * kVec + i < end ? a[mine + r * kWave * kVec + i] : (T)0;
    }
}
template <typename T> __device__ __forceinline__ int64_t pick_in_group(const Group<T>& group, int64_t begin, uint64_t& x) {
    constexpr int kVec = Group<T>::kVec, kRows = Group<T>::kRows;
    const auto& v = group.v;
    uint64_t own[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        own[r] = 0;
#pragma unroll
        for (int i = 0; i < kVec; ++i) own[r] += (uint64_t)v[r][i];
    }
    fold_rows(own);
    // the row where the running sum passes x; the last one while the guarantee does not hold
    int row = kRows - 1;
    uint64_t before = 0, rest = x;
    T pick[kVec];
#pragma unroll
    for (int i = 0; i < kVec; ++i) pick[i] = v[kRows - 1][i];
    bool open = true;
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        const uint64_t total = total_of_row(own, r);
        const bool here = open && (r == kRows - 1 || before + total > x);   // wave-uniform
        if (here) {
            row = r;
            rest = x - before;
#pragma unroll
            for (int i = 0; i < kVec; ++i) pick[i] = v[r][i];
            open = false;
        }
        before += total;
    }
    uint64_t pick_own = 0;
#pragma unroll
    for (int i = 0; i < kVec; ++i) pick_own += (uint64_t)pick[i];
    const uint64_t pick_inc = wave_inclusive_scan64(pick_own);
    const uint64_t hit = __ballot(pick_inc > rest);
    const int first = hit ? __ffsll((long long)hit) - 1 : kWave - 1;   // hit is never 0 while the guarantee holds
    rest -= wave_get64(pick_inc - pick_own, first);                    // what is left inside that lane
    int found = kVec - 1;
    bool done = false;
#pragma unroll
    for (int i = 0; i < kVec; ++i) {
        const uint64_t value = wave_get64((uint64_t)pick[i], first);
        if (!done) {
            if (value > rest) {
                found = i;
                done = true;
            } else {
                rest -= value;
            }
        }
    }
    x = rest;
    return begin + (int64_t)row * (kWave * kVec) + (int64_t)first * kVec + found;
}

// One block per partial sum: out[b] = sum of in[1024*b .. 1024*b+1023].
template <typename T>
__global__ __launch_bounds__(kThreads) void partial_sums_kernel(const T* __restrict__ in, int64_t n,
                                                                uint64_t* __restrict__ out) {
    __shared__ uint64_t part[kThreads / kWave];
    const int64_t base = (int64_t)blockIdx.x * kFan;
    uint64_t s = 0;
    for (int j = threadIdx.x; j < kFan; j += kThreads)
        if (base + j < n) s += (uint64_t)in[base + j];
    s = wave_sum64(s);
    if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t t = 0;
        for (int w = 0; w < kThreads / kWave; ++w) t += part[w];
        out[blockIdx.x] = t;
    }
}

__global__ __launch_bounds__(kThreads) void fill_u32_kernel(uint32_t* __restrict__ a, int64_t n, uint32_t v) {
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) a[i] = v;
}

// One wavefront per draw. What does not depend on the draw is on its way before its random number is worked out: the top level
// (of 64 sums at most, 64 M edges, it stays in the lanes) and, where that is one sum, the level below. (From 10^6 scores, us of the
// launch: 2 000 draws 6.2 with the three levels read one after the other behind the random number, 5.6 so; a call of 8 000 10.4
// and 9.5, of 100 000 89 and 76; from 60 M 82 and 76.)
__global__ __launch_bounds__(kThreads) void batch_draw_kernel(const uint32_t* __restrict__ score, int64_t n,
                                                              const uint64_t* __restrict__ sum1, int64_t n1,
                                                              const uint64_t* __restrict__ sum2, int64_t n2, int64_t b,
                                                              uint32_t seed_lo, uint32_t seed_hi, uint64_t iteration,
                                                              int32_t* __restrict__ out) {
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t j = (int64_t)blockIdx.x * (kThreads / kWave) + (threadIdx.x >> 6);
    if (j >= b) return;   // wave-uniform
    const uint64_t top = lane < n2 ? sum2[lane] : 0;
    Group<uint64_t> group;
    if (n2 == 1) load_group(sum1, 0, n1, lane, group);   // (uniform)
    const uint64_t u = draw64(seed_lo, seed_hi, kDrawTag, iteration, (uint32_t)j);
    uint64_t inc = top, total;
    if (n2 > kWave) {
        for (int64_t i = kWave + lane; i < n2; i += kWave) inc += sum2[i];
        total = wave_sum64(inc);
    } else {
        inc = wave_inclusive_scan64(top);
        total = wave_get64(inc, kWave - 1);
    }
    if (total == 0) {
        if (lane == 0) out[j] = -1;
        return;
    }
    uint64_t x = __umul64hi(u, total);
    int64_t i2 = 0;
    if (n2 > kWave) {
        i2 = wave_descend(sum2, 0, n2, x, lane);
    } else if (n2 > 1) {
        i2 = __ffsll((long long)__ballot(inc > x)) - 1;   // x < total: there is one
        x -= wave_get64(inc - top, (int)i2);
    }
    if (n2 > 1) load_group(sum1, i2 * kFan, (i2 + 1) * kFan < n1 ? (i2 + 1) * kFan : n1, lane, group);
    const int64_t i1 = pick_in_group(group, i2 * kFan, x);
    Group<uint32_t> scores;
    load_group(score, i1 * kFan, (i1 + 1) * kFan < n ? (i1 + 1) * kFan : n, lane, scores);
    const int64_t e = pick_in_group(scores, i1 * kFan, x);
    if (lane == 0) out[j] = (int32_t)e;
}

// Moves the partial sums by one edge's difference per lane (0: nothing), modulo 2^64. A whole wavefront calls it.
__device__ __forceinline__ void move_sums(int32_t e, uint64_t diff, int lane, uint64_t* __restrict__ sum1, uint64_t* __restrict__ sum2) {
    if (diff) atomicAdd((unsigned long long*)&sum1[e / kFan], (unsigned long long)diff);
    // A million edges share one level-2 sum: thousands of atomics on one address would
    // run one after the other. Lanes of a wavefront that change the same level-2 sum
    // as its first changing lane add up first and issue a single atomic.
    const uint64_t changing = __ballot(diff != 0);
    if (changing == 0) return;   // wave-uniform
    const int leader = __ffsll((long long)changing) - 1;
    const int32_t top = diff ? e / (kFan * kFan) : -1;
    const int32_t leader_top = __shfl(top, leader, kWave);
    const uint64_t together = wave_sum64(top == leader_top ? diff : 0);
    if (lane == leader) {
        if (together) atomicAdd((unsigned long long*)&sum2[leader_top], (unsigned long long)together);
    } else if (diff && top != leader_top) {
        atomicAdd((unsigned long long*)&sum2[top], (unsigned long long)diff);
    }
}

// Update of a large batch, step 1: for every named edge remember the latest batch position that names it.
__global__ __launch_bounds__(kThreads) void claim_kernel(const int32_t* __restrict__ idx, int64_t b, int64_t n,
                                                         int32_t* __restrict__ owner) {
    const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (j >= b) return;
    const int32_t e = idx[j];
    if (e >= 0 && e < n) atomicMax(&owner[e], (int32_t)j);
}

// Update, step 2: that position writes its value, moves the partial sums by the
// difference (integer adds: any order gives the same sums) and releases the edge.
__global__ __launch_bounds__(kThreads) void apply_kernel(const int32_t* __restrict__ idx,
                                                         const uint32_t* __restrict__ value, int64_t b, int64_t n,
                                                         uint32_t* __restrict__ score, uint64_t* __restrict__ sum1,
                                                         uint64_t* __restrict__ sum2, int32_t* __restrict__ owner) {
    const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int lane = threadIdx.x & (kWave - 1);
    uint64_t diff = 0;   // modulo 2^64: adding it is the signed change
    int32_t e = -1;
    if (j < b) {
        e = idx[j];
        if (e >= 0 && e < n && owner[e] == (int32_t)j) {
            const uint32_t old = score[e], now = value[j];
            score[e] = now;
            owner[e] = -1;
            diff = (uint64_t)now - (uint64_t)old;
        }
    }
    move_sums(e, diff, lane, sum1, sum2);
}

// The whole update of a batch of at most 768 by one block: which position names an edge last is settled in
// a hash table in LDS instead of the array of owners, so the chain of dependent reads is index -> score, in
// one launch instead of two (us a call, million edges: 100 positions 3.4 -> 2.5, 600 4.3 -> 2.4). The random reads and adds
// of one compute unit take longer the more there are: by 8 blocks (next kernel) 600 / 800 / 1 000 positions are 2.5 /
// 2.5 / 2.6, by one 2.4 / 2.7 / 3.1.
constexpr int kOneBlockThreads = 1024, kOneBlockBatch = 768;

__global__ __launch_bounds__(kOneBlockThreads) void update_one_block_kernel(const int32_t* __restrict__ idx, const uint32_t* __restrict__ value,
                                                                            int32_t b, uint32_t slots, int64_t n, uint32_t* __restrict__ score,
                                                                            uint64_t* __restrict__ sum1, uint64_t* __restrict__ sum2) {
    __shared__ int32_t edge[2 * kOneBlockThreads];   // `slots` >= 2 b of them in use; -1: free
    __shared__ int32_t last[2 * kOneBlockThreads];   // latest position that names it
    const int32_t j = (int32_t)threadIdx.x;
    for (uint32_t s = threadIdx.x; s < slots; s += kOneBlockThreads) {
        edge[s] = -1;
        last[s] = -1;
    }
    int32_t e = j < b ? idx[j] : -1;
    const uint32_t now = j < b ? value[j] : 0;
    if (e >= n) e = -1;
    const uint32_t old = e >= 0 ? score[e] : 0;   // every read lies before the barrier, every write after it
    __syncthreads();
    uint32_t slot = 0;
    if (e >= 0) {
        slot = edge_hash((uint32_t)e) & (slots - 1);
        for (;;) {   // at most half the slots are taken: ends at the edge or at a free one
            const int32_t was = atomicCAS(&edge[slot], -1, e);
            if (was == -1 || was == e) break;
            slot = (slot + 1) & (slots - 1);
        }
        atomicMax(&last[slot], j);
    }
    __syncthreads();
    uint64_t diff = 0;
    if (e >= 0 && last[slot] == j) {
        score[e] = now;
        diff = (uint64_t)now - (uint64_t)old;
    }
    move_sums(e, diff, (int)(threadIdx.x & (kWave - 1)), sum1, sum2);
}

// The update of a batch of up to kClassBatch positions in one launch of several blocks: every block reads the whole
// batch and takes the edges whose hash begins with its number, so that who names an edge last is settled inside a
// block, as above, and no score is another block's. A block's table holds the batch even if all of it were its own. The level-2
// sums' changes are added up per block first (a million edges share one). us a call, million edges, against the two
// launches above: 1 500 positions 4.3 -> 2.8, 3 000 4.5 -> 3.8, 4 096 4.7 -> 4.1; with twice the table for 6 000 4.7 -> 6.3,
// so larger batches stay with two.
constexpr int kClassBatch = 4 * kOneBlockThreads;
constexpr int kClassTops = 64;   // level-2 sums that fit the block's own (64 M edges)

template <int kPer>   // positions per thread
__global__ __launch_bounds__(kOneBlockThreads) void update_classes_kernel(const int32_t* __restrict__ idx, const uint32_t* __restrict__ value,
                                                                          int32_t b, int class_bits, int64_t n, uint32_t* __restrict__ score,
                                                                          uint64_t* __restrict__ sum1, uint64_t* __restrict__ sum2, int n2) {
    constexpr uint32_t kSlots = 2 * kPer * kOneBlockThreads;
    __shared__ int32_t edge[kSlots];                 // -1: free
    __shared__ int32_t last[kSlots];                 // latest position that names it
    __shared__ unsigned long long top_sum[kClassTops];
    const int lane = threadIdx.x & (kWave - 1);
    int32_t e[kPer];
    uint32_t slot[kPer], old[kPer], now[kPer];
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        const int32_t j = r * kOneBlockThreads + (int32_t)threadIdx.x;
        e[r] = j < b ? idx[j] : -1;
        now[r] = j < b ? value[j] : 0;               // (read here, few of them are needed: behind the barriers it is one more wait)
    }
    for (uint32_t s = threadIdx.x; s < kSlots; s += kOneBlockThreads) {
        edge[s] = -1;
        last[s] = -1;
    }
    if (threadIdx.x < kClassTops) top_sum[threadIdx.x] = 0;
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        slot[r] = edge_hash((uint32_t)e[r]);
        if (e[r] >= n || slot[r] >> (32 - class_bits) != blockIdx.x) e[r] = -1;
        old[r] = e[r] >= 0 ? score[e[r]] : 0;        // the block's own edges: every read lies before the barriers, every write after them
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        if (e[r] >= 0) {
            slot[r] &= kSlots - 1;
            for (;;) {   // at most half the slots are taken: ends at the edge or at a free one
                const int32_t was = atomicCAS(&edge[slot[r]], -1, e[r]);
                if (was == -1 || was == e[r]) break;
                slot[r] = (slot[r] + 1) & (kSlots - 1);
            }
            atomicMax(&last[slot[r]], r * kOneBlockThreads + (int32_t)threadIdx.x);
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
        const int32_t j = r * kOneBlockThreads + (int32_t)threadIdx.x;
        uint64_t diff = 0;
        if (e[r] >= 0 && last[slot[r]] == j) {
            score[e[r]] = now[r];
            diff = (uint64_t)now[r] - (uint64_t)old[r];
        }
        if (diff) atomicAdd((unsigned long long*)&sum1[e[r] / kFan], (unsigned long long)diff);
        const uint64_t changing = __ballot(diff != 0);
        if (changing == 0) continue;                 // wave-uniform
        const int leader = __ffsll((long long)changing) - 1;
        const int32_t top = diff ? e[r] / (kFan * kFan) : -1;
        const int32_t leader_top = __shfl(top, leader, kWave);
        const uint64_t together = wave_sum64(top == leader_top ? diff : 0);
        if (lane == leader) atomicAdd(&top_sum[leader_top], (unsigned long long)together);
        else if (diff && top != leader_top) atomicAdd(&top_sum[top], (unsigned long long)diff);
    }
    __syncthreads();
    if ((int)threadIdx.x < n2 && top_sum[threadIdx.x]) atomicAdd((unsigned long long*)&sum2[threadIdx.x], top_sum[threadIdx.x]);
}

void free_all(taser_selector* s) {
    if (!s) return;
    (void)hipFree(s->score);
    (void)hipFree(s->sum1);
    (void)hipFree(s->sum2);
    (void)hipFree(s->owner);
    delete s;
}

void rebuild_sums(taser_selector* s, hipStream_t stream) {
    hipLaunchKernelGGL((partial_sums_kernel<uint32_t>), dim3((unsigned)s->n1), dim3(kThreads), 0, stream, s->score, s->n, s->sum1);
    hipLaunchKernelGGL((partial_sums_kernel<uint64_t>), dim3((unsigned)s->n2), dim3(kThreads), 0, stream, s->sum1, s->n1, s->sum2);
}

}  // namespace

extern "C" int taser_selector_init(const uint32_t* scores, int64_t n, uint32_t initial_score, void* hip_stream,
                                   taser_selector** out) {
    if (!out) return taser_fail(TASER_E_ARG, "selector_init: null out");
    *out = nullptr;
    if (n < 1 || n >= ((int64_t)1 << 31)) return taser_fail(TASER_E_RANGE, "selector_init: n = %lld outside [1, 2^31)", (long long)n);
    taser_clear_stale_hip_error();
    hipStream_t stream = (hipStream_t)hip_stream;
    taser_selector* s = new (std::nothrow) taser_selector();
    if (!s) return taser_fail(TASER_E_OOM, "selector_init: out of host memory");
    s->n = n;
    s->n1 = (n + kFan - 1) / kFan;
    s->n2 = (s->n1 + kFan - 1) / kFan;
    hipError_t e = hipMalloc(&s->score, (size_t)n * sizeof(uint32_t));
    if (e == hipSuccess) e = hipMalloc(&s->sum1, (size_t)s->n1 * sizeof(uint64_t));
    if (e == hipSuccess) e = hipMalloc(&s->sum2, (size_t)s->n2 * sizeof(uint64_t));
    if (e == hipSuccess) e = hipMalloc(&s->owner, (size_t)n * sizeof(int32_t));
    if (e == hipSuccess) {
        if (scores) e = hipMemcpyAsync(s->score, scores, (size_t)n * sizeof(uint32_t), hipMemcpyDeviceToDevice, stream);
        else hipLaunchKernelGGL(fill_u32_kernel, dim3(1024), dim3(kThreads), 0, stream, s->score, n, initial_score);
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(fill_u32_kernel, dim3(1024), dim3(kThreads), 0, stream, (uint32_t*)s->owner, n, 0xFFFFFFFFu);
        rebuild_sums(s, stream);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) {
        free_all(s);
        return taser_fail_hip(e, "selector_init");
    }
    *out = s;
    return TASER_OK;
}

extern "C" int taser_selector_draw(const taser_selector* s, int64_t b, uint64_t seed, uint64_t iteration,
                                   int32_t* batch, void* hip_stream) {
    if (!s) return taser_fail(TASER_E_ARG, "selector_draw: null selector");
    if (b < 0 || b >= ((int64_t)1 << 31)) return taser_fail(TASER_E_RANGE, "selector_draw: b = %lld outside [0, 2^31)", (long long)b);
    if (b == 0) return TASER_OK;
    if (!batch) return taser_fail(TASER_E_ARG, "selector_draw: null batch");
    taser_clear_stale_hip_error();
    hipStream_t stream = (hipStream_t)hip_stream;
    TaserProfileSpan span(stream, "selector_draw");
    const int64_t blocks = (b + kThreads / kWave - 1) / (kThreads / kWave);
    hipLaunchKernelGGL(batch_draw_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, stream, s->score, s->n, s->sum1,
                       s->n1, s->sum2, s->n2, b, (uint32_t)seed, (uint32_t)(seed >> 32), iteration, batch);
    TASER_HIP_TRY(hipGetLastError());
    return TASER_OK;
}

extern "C" int taser_selector_update(taser_selector* s, const int32_t* batch, const uint32_t* new_scores, int64_t b,
                                     void* hip_stream) {
    if (!s) return taser_fail(TASER_E_ARG, "selector_update: null selector");
    if (b < 0 || b >= ((int64_t)1 << 31)) return taser_fail(TASER_E_RANGE, "selector_update: b = %lld outside [0, 2^31)", (long long)b);
    if (b == 0) return TASER_OK;
    if (!batch || !new_scores) return taser_fail(TASER_E_ARG, "selector_update: null batch or new_scores");
    taser_clear_stale_hip_error();
    hipStream_t stream = (hipStream_t)hip_stream;
    TaserProfileSpan span(stream, "selector_update");
    if (b <= kOneBlockBatch) {
        uint32_t slots = 2;
        while (slots < 2 * (uint32_t)b) slots *= 2;
        hipLaunchKernelGGL(update_one_block_kernel, dim3(1), dim3(kOneBlockThreads), 0, stream, batch, new_scores, (int32_t)b, slots, s->n, s->score,
                           s->sum1, s->sum2);
    } else if (b <= kClassBatch && s->n2 <= kClassTops) {
        const int bits = b <= 2048 ? 3 : 4;   // about 250 positions a block
        const auto kernel = b <= 2048 ? update_classes_kernel<2> : update_classes_kernel<4>;
        hipLaunchKernelGGL(kernel, dim3(1u << bits), dim3(kOneBlockThreads), 0, stream, batch, new_scores, (int32_t)b, bits, s->n, s->score,
                           s->sum1, s->sum2, (int)s->n2);
    } else {
        const unsigned blocks = (unsigned)((b + kThreads - 1) / kThreads);
        hipLaunchKernelGGL(claim_kernel, dim3(blocks), dim3(kThreads), 0, stream, batch, b, s->n, s->owner);
        hipLaunchKernelGGL(apply_kernel, dim3(blocks), dim3(kThreads), 0, stream, batch, new_scores, b, s->n, s->score,
                           s->sum1, s->sum2, s->owner);
    }
    TASER_HIP_TRY(hipGetLastError());
    return TASER_OK;
}

extern "C" int taser_selector_scores(const taser_selector* s, uint32_t* scores, uint64_t* total, void* hip_stream) {
    if (!s) return taser_fail(TASER_E_ARG, "selector_scores: null selector");
    taser_clear_stale_hip_error();
    hipStream_t stream = (hipStream_t)hip_stream;
    if (scores) TASER_HIP_TRY(hipMemcpyAsync(scores, s->score, (size_t)s->n * sizeof(uint32_t), hipMemcpyDeviceToDevice, stream));
    if (total) {
        // sum of the level-2 sums, read back: at most 2048 values
        uint64_t host2[2048];
        TASER_HIP_TRY(hipMemcpyAsync(host2, s->sum2, (size_t)s->n2 * sizeof(uint64_t), hipMemcpyDeviceToHost, stream));
        TASER_HIP_TRY(hipStreamSynchronize(stream));
        uint64_t t = 0;
        for (int64_t i = 0; i < s->n2; ++i) t += host2[i];
        *total = t;
    }
    return TASER_OK;
}

extern "C" int taser_selector_size(const taser_selector* s, int64_t* n) {
    if (!s || !n) return taser_fail(TASER_E_ARG, "selector_size: null argument");
    *n = s->n;
    return TASER_OK;
}

extern "C" void taser_selector_free(taser_selector* s) { free_all(s); }
