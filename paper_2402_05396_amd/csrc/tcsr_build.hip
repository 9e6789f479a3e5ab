// taser_tcsr_build: the T-CSR of TASER (arXiv 2402.05396, Sec. 3.3): every
// node's outgoing entries contiguous and ordered by timestamp, ties by input
// position. Built on the device by a stable least-significant-digit radix
// sort over the composite key (node, ts):
//   * the key has only the bits that matter: those of the timestamp between the
//     lowest and the highest bit in which the timestamps differ (none at all when
//     the input is already time-sorted, which is how event streams arrive), then
//     those of the node id. They are cut into equal digits of at most 9 bits, so a
//     digit may hold the top of the one and the bottom of the other;
//   * one pass = per-tile digit histogram -> per-digit scan over the tiles ->
//     stable scatter. Inside a tile the stable rank of an item among equal digits
//     comes from wave ballots (which lanes hold my digit, how many of them are
//     below me) plus per-wave running counters in LDS, so no atomics decide an
//     output position;
//   * the 16-byte record {ts, nbr, eid} the sampler reads travels with the key,
//     so the last pass leaves the final layout in place. The first pass reads the
//     caller's columns directly: nothing is packed beforehand;
//   * indptr is read off the sorted node column (no atomics, no histogram);
//   * input in no order of at most 1.5 M entries is cut into buckets by sampled keys instead, which a workgroup each sorts
//     in LDS (sort_bucket_kernel): two passes over memory however many bits the keys have;
//   * time-sorted input with node ids of two digits and timestamps that span less than 2^32 (136 years of seconds, 49
//     days of milliseconds) has two passes of its own that move fewer bytes (node_scatter_kernel), and its indptr comes
//     from the scanned histogram.
// All device memory is one storage block (what the graph keeps) and one scratch
// block, either the caller's (taser_tcsr_build_in) or allocated here.
#include <new>

#include "pinned_info.h"
#include "sampling_device.h"
#include "taser_internal.h"

namespace {

constexpr int kThreads = 256;
constexpr int kMaxDigitBits = 9;
constexpr int kBins = 1 << kMaxDigitBits;
constexpr int kSortThreads = 512;                 // block of the sorting kernels: as many threads as digit values
constexpr int kSortWaves = kSortThreads / kWave;
static_assert(kSortThreads == kBins, "one digit per thread");
constexpr int kSmallItems = 4, kLargeItems = 8;   // items per thread of a tile (see items_for)

// Bits [s, s + bits) of the composite key, for s inside the timestamp's part (with from_ts) or above it.
struct DigitSpec {
    int from_ts;           // the digit has timestamp bits
    int ts_shift;          // where they start in the (sign-biased) timestamp
    uint32_t ts_mask;      // and how many of them there are
    int node_left;         // node bits above them: shift to the left (31: none fit)
    int node_right;        // without timestamp bits: shift of the node id to the right
    int bits;
};

__device__ __forceinline__ uint64_t biased(int64_t ts) { return (uint64_t)ts ^ 0x8000000000000000ull; }

__device__ __forceinline__ uint32_t digit_of(const DigitSpec& d, int64_t ts, int32_t node) {
    const uint32_t v = d.from_ts ? (((uint32_t)(biased(ts) >> d.ts_shift) & d.ts_mask) | ((uint32_t)node << d.node_left))
                                 : (uint32_t)node >> d.node_right;
    return v & ((1u << d.bits) - 1u);
}

// Where a pass finds its items: the caller's columns (first pass) or the records and node keys of
// the pass before.
struct Items {
    const TaserRec* rec;
    const int32_t* key;    // node ids
    const int32_t* dst;    // columns (rec == nullptr)
    const int64_t* ts;
    const int32_t* eid;    // may be null: the position
};

// Histogram of a tile in LDS: a digit's counter has kCopies copies, one per lane modulo kCopies, so
// that equal digits of one wave instruction (popular nodes) meet at fewer addresses. Thread t clears
// and adds up digit t's.
constexpr uint32_t kCopies = 4;
template <uint32_t kOf = kCopies> __device__ __forceinline__ void clear_digit(uint32_t* bins) {
    for (uint32_t c = 0; c < kOf; ++c) bins[threadIdx.x * kOf + c] = 0;
}
template <uint32_t kOf = kCopies> __device__ __forceinline__ uint32_t count_of_digit(const uint32_t* bins) {
    uint32_t sum = 0;
    for (uint32_t c = 0; c < kOf; ++c) sum += bins[threadIdx.x * kOf + c];
    return sum;
}

// Inspects the input before the sort is planned: partial[4 * block + ...]: [0] != 0: a node id
// outside [0, num_nodes); [1] != 0: timestamps not non-decreasing in input order; [2] / [3]: OR /
// AND of the biased timestamps (bits in which they agree need no sorting). On the way it counts
// every tile's node ids by their lowest digit, hist[tile * bins + bin] as radix_hist_kernel
// would: time-sorted input is sorted by the node digits only, and its first pass then needs no
// histogram kernel. It reads 12 of an entry's 20 bytes and writes nothing per entry: 0.17 ms for
// 64 M entries (4.5 TB/s, with 4- and 8-byte loads 0.177 ms), where packing the columns into records here, and
// reading them back in the first pass, took 0.50.
// On the way it also takes `samples` (if not null) out of every tile, one of each kStratum places, for rank_samples_kernel.
struct Sample {
    int64_t ts;
    int32_t node;
    uint32_t pos;
};
struct Samples {
    Sample* at;        // null: none wanted
    uint32_t* rank;    // set to 0
};
constexpr uint32_t kStratum = 256;   // of a small tile: one wave's run of four entries per lane
__device__ __forceinline__ uint32_t sample_place(uint32_t sample) {   // in its stratum
    uint32_t h = sample * 0x9E3779B1u;
    h ^= h >> 15;
    h *= 0x85EBCA77u;
    return (h >> 13) % kStratum;
}
constexpr unsigned kInspectBlocks = 1024;   // 4 per compute unit; the fold below is one block over their words
struct __attribute__((packed, aligned(4))) FourNodes {
    int32_t v[4];
};
struct __attribute__((packed, aligned(8))) TwoTimes {
    int64_t a, b;
};
template <int kItems>
__global__ __launch_bounds__(kSortThreads) void inspect_kernel(const int32_t* __restrict__ src, const int64_t* __restrict__ ts,
                                                           int64_t n, int32_t num_nodes,
                                                           unsigned long long* __restrict__ partial, int low_bits,
                                                           uint32_t* __restrict__ hist, uint32_t num_tiles, const Samples samples) {
    constexpr int kTile = kSortThreads * kItems;
    constexpr uint32_t kStrata = kTile / kStratum;
    __shared__ uint32_t bins[kBins * kCopies];
    const uint32_t low_mask = (1u << low_bits) - 1u, copy = threadIdx.x % kCopies;
    unsigned long long any_or = 0, all_and = ~0ull;
    int bad = 0, unsorted = 0;
    for (uint32_t tile = blockIdx.x; tile < num_tiles; tile += gridDim.x) {
        clear_digit(bins);
        __syncthreads();
        const int64_t tile0 = (int64_t)tile * kTile;
        const bool whole = tile0 + kTile < n;   // uniform: every item of the tile has a successor
        const uint32_t last = whole ? (uint32_t)kTile : (uint32_t)(n - 1 - tile0);   // place of the array's last item, if it is here
        const int32_t* const tile_src = src + tile0;
        const int64_t* const tile_ts = ts + tile0;
        if (whole) {   // a thread takes runs of four entries, in wide loads (the columns are aligned to their elements only)
            FourNodes s[kItems / 4];
            TwoTimes t[kItems / 4][2];
            int64_t t_end[kItems / 4];                          // the entry after the wave's last run; the others have it in a lane
#pragma unroll
            for (int u = 0; u < kItems / 4; ++u) {
                const uint32_t i = (threadIdx.x + u * kSortThreads) * 4u;
                s[u] = *reinterpret_cast<const FourNodes*>(tile_src + i);
                t[u][0] = *reinterpret_cast<const TwoTimes*>(tile_ts + i);
                t[u][1] = *reinterpret_cast<const TwoTimes*>(tile_ts + i + 2);
                t_end[u] = 0;
                if ((threadIdx.x & (kWave - 1)) == kWave - 1) t_end[u] = tile_ts[i + 4];
            }
#pragma unroll
            for (int u = 0; u < kItems / 4; ++u) {
                const int64_t x[4] = {t[u][0].a, t[u][0].b, t[u][1].a, t[u][1].b};
                const uint32_t next_lo = __shfl_down((uint32_t)(uint64_t)x[0], 1, kWave), next_hi = __shfl_down((uint32_t)((uint64_t)x[0] >> 32), 1, kWave);
                int64_t next = (int64_t)(((uint64_t)next_hi << 32) | next_lo);
                if ((threadIdx.x & (kWave - 1)) == kWave - 1) next = t_end[u];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    bad |= (uint32_t)s[u].v[j] >= (uint32_t)num_nodes;   // negative ids included
                    unsorted |= (j < 3 ? x[j + 1] : next) < x[j];
                    any_or |= biased(x[j]);
                    all_and &= biased(x[j]);
                    atomicAdd(&bins[((uint32_t)s[u].v[j] & low_mask) * kCopies + copy], 1u);
                }
                if (kItems == kSmallItems && samples.at) {
                    const uint32_t sample = tile * kStrata + threadIdx.x * 4u / kStratum, place = sample_place(sample);
                    if (threadIdx.x * 4u % kStratum == place / 4u * 4u) {
                        const uint32_t j = place % 4u;
                        samples.rank[sample] = 0;
                        samples.at[sample] = Sample{j == 0 ? x[0] : j == 1 ? x[1] : j == 2 ? x[2] : x[3], j == 0 ? s[u].v[0] : j == 1 ? s[u].v[1] : j == 2 ? s[u].v[2] : s[u].v[3],
                                                 (uint32_t)tile0 + threadIdx.x * 4u + j};
                    }
                }
            }
        } else {
            if (kItems == kSmallItems && samples.at && threadIdx.x < kStrata) {
                const uint32_t sample = tile * kStrata + threadIdx.x, at = threadIdx.x * kStratum + sample_place(sample), i = at < last ? at : last;
                samples.rank[sample] = 0;
                samples.at[sample] = Sample{tile_ts[i], tile_src[i], (uint32_t)tile0 + i};
            }
            for (uint32_t i = threadIdx.x; i <= last; i += kSortThreads) {
                const int32_t node = tile_src[i];
                const int64_t x = tile_ts[i];
                bad |= (uint32_t)node >= (uint32_t)num_nodes;
                unsorted |= tile_ts[i < last ? i + 1 : i] < x;
                any_or |= biased(x);
                all_and &= biased(x);
                atomicAdd(&bins[((uint32_t)node & low_mask) * kCopies + copy], 1u);
            }
        }
        __syncthreads();
        if (threadIdx.x <= low_mask) hist[((size_t)tile << low_bits) + threadIdx.x] = count_of_digit(bins);
        // (each thread clears the counters it has just read)
    }
    for (int d = 1; d < kWave; d <<= 1) {
        any_or |= __shfl_xor(any_or, d, kWave);
        all_and &= __shfl_xor(all_and, d, kWave);
    }
    __shared__ unsigned long long w_or[kSortWaves], w_and[kSortWaves];
    __shared__ int w_bad[kSortWaves], w_unsorted[kSortWaves];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const unsigned long long any_bad = __ballot(bad), any_unsorted = __ballot(unsorted);
    if (lane == 0) {
        w_or[wave] = any_or;
        w_and[wave] = all_and;
        w_bad[wave] = any_bad != 0;
        w_unsorted[wave] = any_unsorted != 0;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long o = 0, a = ~0ull;
        int b = 0, u = 0;
        for (int w = 0; w < kSortWaves; ++w) {
            o |= w_or[w];
            a &= w_and[w];
            b |= w_bad[w];
            u |= w_unsorted[w];
        }
        partial[4 * blockIdx.x + 0] = (unsigned long long)b;
        partial[4 * blockIdx.x + 1] = (unsigned long long)u;
        partial[4 * blockIdx.x + 2] = o;
        partial[4 * blockIdx.x + 3] = a;
    }
}

// One block: info[0..3] = the `blocks` per-block word groups of inspect_kernel combined; where the input is in time
// order info[2] and info[3] are the first and the last timestamp instead.
__global__ __launch_bounds__(kSortThreads) void fold_info_kernel(const unsigned long long* __restrict__ partial, uint32_t blocks,
                                                             const int64_t* __restrict__ ts, int64_t n, unsigned long long* __restrict__ info) {
    __shared__ unsigned long long part[4][kSortWaves];
    unsigned long long v[4] = {0, 0, 0, ~0ull};
    for (uint32_t b = threadIdx.x; b < blocks; b += kSortThreads) {
        v[0] |= partial[4 * (size_t)b + 0];
        v[1] |= partial[4 * (size_t)b + 1];
        v[2] |= partial[4 * (size_t)b + 2];
        v[3] &= partial[4 * (size_t)b + 3];
    }
    for (int d = 1; d < kWave; d <<= 1) {
        for (int j = 0; j < 3; ++j) v[j] |= __shfl_xor(v[j], d, kWave);
        v[3] &= __shfl_xor(v[3], d, kWave);
    }
    if ((threadIdx.x & (kWave - 1)) == 0)
        for (int j = 0; j < 4; ++j) part[j][threadIdx.x >> 6] = v[j];
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kSortWaves; ++w) {
            for (int j = 0; j < 3; ++j) v[j] |= part[j][w];
            v[3] &= part[3][w];
        }
        if (!v[1]) {
            v[2] = (unsigned long long)ts[0];
            v[3] = (unsigned long long)ts[n - 1];
        }
        for (int j = 0; j < 4; ++j) info[j] = v[j];
    }
}

// Tile of a workgroup of the scatter: workgroups go to the chip's eight L2 partitions round-robin;
// each partition takes a contiguous eighth of the tiles, so that the short runs of one digit that
// its workgroups write one after the other into neighboring addresses (16 records per tile on
// average for 256 digits) meet in its L2 and leave as whole lines. With tile = workgroup index
// those pieces came from eight different L2s as partial lines (5.8 -> 3.6 ms for the 256-digit
// pass over 382 M entries). The grid is rounded up to a multiple of kPartitions; tiles >=
// num_tiles do not exist.
constexpr uint32_t kPartitions = 8;
__device__ __forceinline__ uint32_t tile_of_block(uint32_t block, uint32_t num_tiles) {
    const uint32_t per_part = (num_tiles + kPartitions - 1) / kPartitions;
    return (block % kPartitions) * per_part + block / kPartitions;
}
inline unsigned pass_grid(unsigned num_tiles) { return (num_tiles + kPartitions - 1) / kPartitions * kPartitions; }

// hist[tile * bins + bin] = items of the tile whose digit is bin. (One row per tile: with one row
// per digit value every counter went to a line of its own, and the kernel took 0.11 ms for 64 M
// keys, with that and the copies of the counters 0.07.)
template <int kItems>
__global__ __launch_bounds__(kSortThreads) void radix_hist_kernel(const Items in, int64_t n, DigitSpec d,
                                                              uint32_t* __restrict__ hist) {
    constexpr int kTile = kSortThreads * kItems;
    __shared__ uint32_t bins[kBins * kCopies];
    const uint32_t tile = blockIdx.x;   // (the partition-wise order of the scatter below does not pay here)
    const uint32_t copy = threadIdx.x % kCopies;
    clear_digit(bins);
    __syncthreads();
    const int64_t tile0 = (int64_t)tile * kTile;
    if (!d.from_ts && in.rec && tile0 + kTile <= n) {
        // a whole tile of node keys: which thread counts which item does not matter, so every thread
        // takes runs of four keys with 16-byte loads (tile0 is a multiple of the tile size and the
        // keys of a pass start an aligned part of the scratch block), all loads in flight together
        typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
        const i32x4* quads = reinterpret_cast<const i32x4*>(in.key + tile0);
        i32x4 v[kItems / 4];
#pragma unroll
        for (int r = 0; r < kItems / 4; ++r) v[r] = quads[r * kSortThreads + threadIdx.x];
#pragma unroll
        for (int r = 0; r < kItems / 4; ++r) {
            atomicAdd(&bins[digit_of(d, 0, v[r].x) * kCopies + copy], 1u);
            atomicAdd(&bins[digit_of(d, 0, v[r].y) * kCopies + copy], 1u);
            atomicAdd(&bins[digit_of(d, 0, v[r].z) * kCopies + copy], 1u);
            atomicAdd(&bins[digit_of(d, 0, v[r].w) * kCopies + copy], 1u);
        }
    } else {
        constexpr int kPer = 4;
        for (int round = 0; round < kItems / kPer; ++round) {
            const int64_t i0 = tile0 + (int64_t)round * (kPer * kSortThreads) + threadIdx.x;
            int64_t t[kPer];
            int32_t node[kPer];
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                const int64_t i = i0 + u * kSortThreads;
                const int64_t at = i < n ? i : n - 1;
                t[u] = d.from_ts ? (in.rec ? in.rec[at].ts : in.ts[at]) : 0;
                node[u] = in.key[at];
            }
#pragma unroll
            for (int u = 0; u < kPer; ++u)
                if (i0 + u * kSortThreads < n) atomicAdd(&bins[digit_of(d, t[u], node[u]) * kCopies + copy], 1u);
        }
    }
    __syncthreads();
    if (threadIdx.x < (1u << d.bits)) hist[((size_t)tile << d.bits) + threadIdx.x] = count_of_digit(bins);
}

// Per digit value: hist[...][bin] becomes its own exclusive scan over the tiles, and total[bin] the
// digit's count (the scatter adds up the totals below its digits itself, which saves the two further
// launches of a scan over the whole table). A block owns kScanCols digit values, that is a 32-byte
// piece of every row; its 128 groups of lanes each take a run of consecutive tiles, sum it, and go
// over it again with what came before. One launch, bound by the latency of its few loads: 6 us for
// 656 rows of 512. From kChunkedTiles rows on there is too little of it in flight (15 600 rows of
// 256: 0.11 ms) and two launches over chunks of rows do the same (0.014 ms).
constexpr uint32_t kChunkedTiles = 2048;
constexpr int kScanThreads = 1024, kScanCols = 8, kScanGroups = kScanThreads / kScanCols;
__global__ __launch_bounds__(kScanThreads) void bin_scan_kernel(uint32_t* __restrict__ hist, uint32_t num_tiles, int bits,
                                                                uint32_t* __restrict__ total) {
    __shared__ uint32_t wave_total[kScanThreads / kWave][kScanCols];
    constexpr int kAhead = 8;
    const uint32_t col = threadIdx.x % kScanCols, group = threadIdx.x / kScanCols;
    const uint32_t bin = blockIdx.x * kScanCols + col;
    const bool live = bin < (1u << bits);
    const uint32_t per_group = (num_tiles + kScanGroups - 1) / kScanGroups;
    uint32_t r0 = group * per_group, r1 = r0 + per_group;
    if (r1 > num_tiles) r1 = num_tiles;
    if (!live || r0 > r1) r0 = r1;
    uint32_t* const a = hist + bin;
    uint32_t sum = 0, v[kAhead];
    for (uint32_t r = r0; r < r1; r += kAhead) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) v[u] = r + u < r1 ? a[(size_t)(r + u) << bits] : 0u;
#pragma unroll
        for (int u = 0; u < kAhead; ++u) sum += v[u];
    }
    const bool held = per_group <= (uint32_t)kAhead;   // uniform: v is still all of the group's rows
    // exclusive over the groups: a wave holds 64 / kScanCols of them, kScanCols lanes apart
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    uint32_t inc = sum;
#pragma unroll
    for (int d = kScanCols; d < kWave; d <<= 1) {
        const uint32_t y = __shfl_up(inc, d, kWave);
        if (lane >= d) inc += y;
    }
    if (lane >= kWave - kScanCols) wave_total[wave][col] = inc;
    __syncthreads();
    uint32_t run = inc - sum, all = 0;
#pragma unroll
    for (int w = 0; w < kScanThreads / kWave; ++w) {
        const uint32_t x = wave_total[w][col];
        if (w < wave) run += x;
        all += x;
    }
    if (live && group == 0) total[bin] = all;
    for (uint32_t r = r0; r < r1; r += kAhead) {
        if (!held) {
#pragma unroll
            for (int u = 0; u < kAhead; ++u) v[u] = r + u < r1 ? a[(size_t)(r + u) << bits] : 0u;
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            if (r + u < r1) a[(size_t)(r + u) << bits] = run;
            run += v[u];
        }
    }
}

// The same over chunks of rows: a block of the first kernel sums one chunk for 64 digit values (a row
// piece of 256 bytes per wave instruction), a block of the second adds up the chunks before its own
// and scans it. At most kMaxChunks chunks, so that adding up stays short.
constexpr uint32_t kMaxChunks = 256;
constexpr int kChunkWaves = kThreads / kWave;
__global__ __launch_bounds__(kThreads) void chunk_sum_kernel(const uint32_t* __restrict__ hist, uint32_t num_tiles, int bits,
                                                             uint32_t rows_per_chunk, uint32_t* __restrict__ chunk_sum) {
    __shared__ uint32_t part[kChunkWaves][kWave];
    const uint32_t lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const uint32_t bin = blockIdx.x * kWave + lane, bins = 1u << bits;
    const uint32_t r0 = blockIdx.y * rows_per_chunk, r1 = r0 + rows_per_chunk < num_tiles ? r0 + rows_per_chunk : num_tiles;
    uint32_t sum = 0;
    if (bin < bins) {
#pragma unroll 8
        for (uint32_t r = r0 + wave; r < r1; r += kChunkWaves) sum += hist[((size_t)r << bits) + bin];
    }
    part[wave][lane] = sum;
    __syncthreads();
    if (wave == 0 && bin < bins) {
        for (int w = 1; w < kChunkWaves; ++w) sum += part[w][lane];
        chunk_sum[(size_t)blockIdx.y * bins + bin] = sum;
    }
}

__global__ __launch_bounds__(kThreads) void chunk_scan_kernel(uint32_t* __restrict__ hist, uint32_t num_tiles, int bits,
                                                              uint32_t rows_per_chunk, const uint32_t* __restrict__ chunk_sum,
                                                              uint32_t* __restrict__ total) {
    __shared__ uint32_t part[2][kChunkWaves][kWave];
    const uint32_t lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const uint32_t bin = blockIdx.x * kWave + lane, bins = 1u << bits;
    const bool live = bin < bins;
    // the chunk's rows, a quarter per wave; the chunks before it, every fourth per wave
    const uint32_t c0 = blockIdx.y * rows_per_chunk, c1 = c0 + rows_per_chunk < num_tiles ? c0 + rows_per_chunk : num_tiles;
    const uint32_t per_wave = (rows_per_chunk + kChunkWaves - 1) / kChunkWaves;
    uint32_t r0 = c0 + wave * per_wave, r1 = r0 + per_wave;
    if (r0 > c1) r0 = c1;
    if (r1 > c1) r1 = c1;
    uint32_t before = 0, own = 0;
    if (live) {
#pragma unroll 8
        for (uint32_t c = wave; c < blockIdx.y; c += kChunkWaves) before += chunk_sum[(size_t)c * bins + bin];
#pragma unroll 8
        for (uint32_t r = r0; r < r1; ++r) own += hist[((size_t)r << bits) + bin];
    }
    part[0][wave][lane] = before;
    part[1][wave][lane] = own;
    __syncthreads();
    uint32_t run = 0;
    for (uint32_t w = 0; w < (uint32_t)kChunkWaves; ++w) {
        run += part[0][w][lane];
        if (w < wave) run += part[1][w][lane];
    }
    if (!live) return;
    constexpr uint32_t kAhead = 8;
    for (uint32_t r = r0; r < r1; r += kAhead) {
        uint32_t v[kAhead];
#pragma unroll
        for (uint32_t u = 0; u < kAhead; ++u) v[u] = r + u < r1 ? hist[((size_t)(r + u) << bits) + bin] : 0u;
#pragma unroll
        for (uint32_t u = 0; u < kAhead; ++u) {
            if (r + u < r1) hist[((size_t)(r + u) << bits) + bin] = run;
            run += v[u];
        }
    }
    if (c1 == num_tiles && wave == kChunkWaves - 1) total[bin] = run;   // the last rows' running sum
}

// Exclusive prefix sum of one value per thread over the block of a sorting kernel. `wave_sum` is
// written before and read after the one barrier inside.
__device__ __forceinline__ uint32_t scan_digits(uint32_t own, uint32_t* wave_sum) {
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const uint32_t inc = wave_inclusive_scan32(own);
    if (lane == kWave - 1) wave_sum[wave] = inc;
    __syncthreads();
    uint32_t before = 0;
    for (int w = 0; w < wave; ++w) before += wave_sum[w];
    return before + inc - own;
}

// Stable rank of a lane's item among its wave's items with the same digit, in the rows of 64 so far: `seen` of the
// rows before plus the lanes below it in this one. counts: the wave's, one per digit.
__device__ __forceinline__ uint32_t rank_in_wave(uint32_t dg, bool valid, int bits, uint16_t* counts) {
    // lanes of this row that hold the same digit as me: per bit a ballot, and of the lanes left those that agree
    const uint64_t all = __ballot(valid);
    uint32_t same_lo = (uint32_t)all, same_hi = (uint32_t)(all >> 32);
#pragma unroll
    for (int b = 0; b < kMaxDigitBits; ++b) {
        if (b < bits) {   // uniform
            const uint32_t mine = (uint32_t)((int32_t)(dg << (31 - b)) >> 31);   // my bit, everywhere
            const uint64_t has = __ballot(mine != 0);
            same_lo &= ~((uint32_t)has ^ mine);
            same_hi &= ~((uint32_t)(has >> 32) ^ mine);
        }
    }
    const uint32_t before_me = __builtin_amdgcn_mbcnt_hi(same_hi, __builtin_amdgcn_mbcnt_lo(same_lo, 0u));
    uint32_t seen = 0;
    if (valid) seen = counts[dg];            // equal for all lanes of a digit
    if (valid && before_me == 0) counts[dg] = (uint16_t)(seen + (uint32_t)(__popc(same_lo) + __popc(same_hi)));
    __builtin_amdgcn_wave_barrier();         // keep the LDS counter update of this row ahead of the next row's read
    return seen + before_me;
}

// The ranks of a tile's items are known, wave_count says how many of every digit each wave has. Thread t, for digit t:
// wave_count[w] becomes the place in the ordered tile of wave w's first item of it, `base` (global position of the
// tile's first item of the digit) what has to be added to a place of the digit.
__device__ __forceinline__ void places_of_digit(uint16_t (*wave_count)[kBins], uint32_t* base, uint32_t* scan_tmp) {
    const uint32_t own = threadIdx.x;
    uint32_t in_wave[kSortWaves], all = 0;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) {
        in_wave[w] = wave_count[w][own];
        all += in_wave[w];
    }
    const uint32_t start = scan_digits(all, scan_tmp);
    base[own] -= start;
    uint32_t run = start;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) {
        wave_count[w][own] = (uint16_t)run;
        run += in_wave[w];
    }
}

// Stable scatter of one tile. offs / total = the scanned histogram: this tile's first item with
// digit `bin` goes to (sum of total[] below bin) + offs[tile * bins + bin]. The tile is
// first put in digit order in LDS (stable: rank among equal digits = ballots
// inside a row of 64 + running per-wave counters + the waves before), then
// written out in that order, so that consecutive lanes write consecutive
// addresses of one digit's run instead of 64 scattered records. The ordered tile
// passes through LDS in slices of at most kPart items (every item knows its place in
// the order; a slice takes the items whose place falls into it): a whole tile of 4096
// records and keys, 80 KB, would leave room for one block per compute unit, a slice of
// half of it for two, which the registers allow (a third block, at 80 registers with spills: 0.62 and
// 0.53 ms for the two passes over 64 M entries instead of 0.52 and 0.49). 20 bytes in and 20 out per
// entry at 5 TB/s, the rate of a large copy.
// `level1` (last pass only, else null): see the write-out.
constexpr int kMaxPart = 2048;
template <bool kColumns, int kItems>
__global__ __launch_bounds__(kSortThreads) __attribute__((amdgpu_waves_per_eu(4))) void radix_scatter_kernel(
    const Items in, int64_t n, DigitSpec d, const uint32_t* __restrict__ offs, const uint32_t* __restrict__ total,
    uint32_t num_tiles, TaserRec* __restrict__ rec_out, int32_t* __restrict__ key_out, int64_t* __restrict__ level1) {
    constexpr int kTile = kSortThreads * kItems;
    constexpr int kPart = kTile < kMaxPart ? kTile : kMaxPart;
    __shared__ uint16_t wave_count[kSortWaves][kBins];   // items of each wave per digit, then the place of its first one
    __shared__ uint32_t block_base[kBins];           // what makes a place of a digit a global position
    __shared__ uint32_t scan_tmp[2][kSortWaves];
    __shared__ TaserRec tile_rec[kPart];
    __shared__ int32_t tile_key[kPart];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const uint32_t tile = tile_of_block(blockIdx.x, num_tiles);
    if (tile >= num_tiles) return;
    const int64_t tile0 = (int64_t)tile * kTile;
    const uint32_t count = n - tile0 < kTile ? (uint32_t)(n - tile0) : (uint32_t)kTile;   // items of this tile
    const uint32_t mine = (uint32_t)wave * (kWave * kItems) + (uint32_t)lane;               // place of this lane's first item: rows
                                                                                             // of 64 consecutive items per wave

    TaserRec item_rec[kItems];
    int32_t item_key[kItems];
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const uint32_t i = mine + r * kWave;
        if (i < count) {
            item_key[r] = (in.key + tile0)[i];
            if (kColumns) item_rec[r] = TaserRec{(in.ts + tile0)[i], (in.dst + tile0)[i], in.eid ? (in.eid + tile0)[i] : (int32_t)(tile0 + i)};
            else item_rec[r] = (in.rec + tile0)[i];
        }
    }
    const uint32_t own = threadIdx.x;   // the digit value this thread looks after
    {
        const bool live = own < (1u << d.bits);
        const uint32_t all = live ? total[own] : 0u;
        const uint32_t before = live ? offs[((size_t)tile << d.bits) + own] : 0u;
        for (int w = 0; w < kSortWaves; ++w) wave_count[w][own] = 0;
        block_base[own] = scan_digits(all, scan_tmp[0]) + before;   // (its barrier also covers the counters)
    }

    uint32_t rank[kItems];   // among the tile's items of its digit, the digit above bit 16 (one register for both)
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const bool valid = mine + r * kWave < count;
        const uint32_t dg = valid ? digit_of(d, item_rec[r].ts, item_key[r]) : 0u;
        rank[r] = rank_in_wave(dg, valid, d.bits, wave_count[wave]) | (dg << 16);
    }
    __syncthreads();
    places_of_digit(wave_count, block_base, scan_tmp[1]);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kItems; ++r)   // rank becomes the item's place in the ordered tile
        if (mine + r * kWave < count) rank[r] = (rank[r] & 0xffffu) + wave_count[wave][rank[r] >> 16];
    for (uint32_t part0 = 0; part0 < count; part0 += kPart) {
#pragma unroll
        for (int r = 0; r < kItems; ++r) {
            const uint32_t at = rank[r] - part0;   // wraps far beyond kPart for places before this slice
            if (mine + r * kWave < count && at < (uint32_t)kPart) {
                tile_rec[at] = item_rec[r];
                tile_key[at] = item_key[r];
            }
        }
        __syncthreads();
#pragma unroll 2
        for (int r = 0; r < kPart / kSortThreads; ++r) {
            const uint32_t j = (uint32_t)r * kSortThreads + threadIdx.x;   // place inside the slice
            if (part0 + j < count) {
                const TaserRec rr = tile_rec[j];
                const int32_t kk = tile_key[j];
                const uint32_t dg = digit_of(d, rr.ts, kk);
                const uint32_t to = block_base[dg] + (part0 + j);
                rec_out[to] = rr;
                key_out[to] = kk;
                // the last pass knows the final positions: it also leaves level 1 of the search index
                // (the timestamp of the last record of every run of 16, and of the array's last record)
                if (level1 && ((to & 15u) == 15u || (int64_t)to == n - 1)) level1[to >> 4] = rr.ts;
            }
        }
        __syncthreads();   // the slice is free again
    }
}

// indptr[v] = first position whose node id is >= v, from the sorted node column: position p starts
// the lists of the nodes in (key[p - 1], key[p]]. A thread looks at four consecutive positions (one
// 16-byte load; `key` is the start of an allocation) plus the key before them. Ranges of more than kWideGap
// nodes without entries, the one behind the last entry for instance, are written by a wave, of more than kLongGap by the whole
// block: by their thread alone they are a serial chain, 26 ns a store, and the whole launch waits for it. Builds among 300 000
// nodes of which the last tenth has no entries, in order of time: 2 000 entries 911 -> 127 us, 20 000 853 -> 91, 1.34 M 886 -> 116;
// of no entries, 57 instead of 7 740. (By the block from 256 on: 2 000 entries 160; by a wave from 16 or 32 on: up to 5 % slower
// where such ranges are many, 5 000 entries of 300 000 nodes 117 and 113 us, 110 so.)
constexpr int32_t kWideGap = 64, kLongGap = kThreads * 8;
__global__ __launch_bounds__(kThreads) void indptr_kernel(const int32_t* __restrict__ key, int64_t n,
                                                          int32_t num_nodes, int64_t* __restrict__ indptr, const uint32_t* __restrict__ failed) {
    if (failed && *failed) return;   // the column is not in order
    typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
    __shared__ int32_t from[kThreads * 4], to[kThreads * 4];   // gaps: the wide ones from the front, the long ones from the back
    __shared__ uint16_t at[kThreads * 4];                      // the position within the block that ends one
    __shared__ uint32_t n_wide, n_long;
    if (threadIdx.x == 0) n_wide = n_long = 0;
    __syncthreads();
    const int64_t block0 = (int64_t)blockIdx.x * kThreads * 4, p0 = block0 + threadIdx.x * 4;
    if (p0 <= n) {
        int32_t k[5];   // k[0] = the key before p0, k[1 + j] = key at p0 + j (num_nodes from position n on)
        k[0] = p0 > 0 ? key[p0 - 1] : -1;
        if (p0 + 4 <= n) {
            const i32x4 v = *reinterpret_cast<const i32x4*>(key + p0);
            k[1] = v.x; k[2] = v.y; k[3] = v.z; k[4] = v.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) k[1 + j] = p0 + j < n ? key[p0 + j] : num_nodes;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (p0 + j > n) break;
            const int64_t gap = (int64_t)k[1 + j] - k[j];
            if (gap > kWideGap) {
                const uint32_t i = gap > kLongGap ? kThreads * 4u - 1u - atomicAdd(&n_long, 1u) : atomicAdd(&n_wide, 1u);
                from[i] = k[j] + 1;
                to[i] = k[1 + j];
                at[i] = (uint16_t)(threadIdx.x * 4 + j);
            } else
                for (int32_t v = k[j] + 1; v <= k[1 + j]; ++v) indptr[v] = p0 + j;
        }
    }
    __syncthreads();
    const uint32_t lane = threadIdx.x & (kWave - 1), n_mine = n_wide;
    for (uint32_t i = threadIdx.x >> 6; i < n_mine; i += kThreads / kWave) {
        const int64_t p = block0 + at[i], end = to[i];
        for (int64_t v = (int64_t)from[i] + lane; v <= end; v += kWave) indptr[v] = p;
    }
    for (uint32_t i = kThreads * 4u - n_long; i < kThreads * 4u; ++i) {
        const int64_t p = block0 + at[i], end = to[i];
        for (int64_t v = (int64_t)from[i] + threadIdx.x; v <= end; v += kThreads) indptr[v] = p;
    }
}

// ---- time-sorted input, two node digits ------------------------------------------------------
// How event streams arrive, with node ids of 10 to 18 bits. The entries only go by their node: by its low digit first
// (an exact histogram of it came with the inspection), then by the rest. Between the two passes an entry is 12 bytes
// (the timestamp as a 32-bit distance from the first one, where the whole range allows it) and the rest of its
// node id in 2: 20 bytes in, 14 out, 2 for the second histogram, 14 in and 16 out, where the passes below move 20 at
// every step and another 4 twice for the sorted node column. The lists' starts come from the scanned second histogram
// instead of that column. 64 M entries, 17 000 nodes, against the passes below: first pass 508 -> 450 us, second histogram
// 68 -> 39, second pass 487 -> 384, starts 61 -> 8.
struct NarrowRec {
    uint32_t ts;
    int32_t nbr, eid;
};

// kFirst: from the caller's columns to narrow records by the low `bits` bits of the node id; else from those to the
// graph's records by the other bits. Otherwise as radix_scatter_kernel. Bound by the memory (34 and 30 bytes per entry at
// 4.8 and 5.0 TB/s; a large copy moves 5.2), as long as three blocks fit a compute unit: with the 84 registers that the
// compiler takes by itself there are two, and the passes took 551 and 494 us. The low digit is the shorter one where the
// node id has an odd number of bits: the first pass, whose runs of a digit are short in any input, gains what the second
// loses (6, 7, 8 of 15 bits: 852, 842, 852 us for both).
template <bool kFirst, int kItems>
__global__ __launch_bounds__(kSortThreads) __attribute__((amdgpu_waves_per_eu(6))) void node_scatter_kernel(
    const Items in, const NarrowRec* __restrict__ narrow_in, const uint16_t* __restrict__ rest_in, int64_t ts_first, int64_t n, int bits,
    const uint32_t* __restrict__ offs, const uint32_t* __restrict__ total, uint32_t num_tiles, NarrowRec* __restrict__ narrow_out,
    uint16_t* __restrict__ rest_out, TaserRec* __restrict__ rec_out, int64_t* __restrict__ level1) {
    constexpr int kTile = kSortThreads * kItems;
    constexpr int kPart = 1024;
    __shared__ uint16_t wave_count[kSortWaves][kBins];   // as in radix_scatter_kernel
    __shared__ uint32_t block_base[kBins];
    __shared__ uint32_t scan_tmp[2][kSortWaves];
    __shared__ NarrowRec tile_rec[kPart];
    __shared__ uint32_t tile_key[kPart];                 // the digit, and above bit 9 the rest of the node id
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const uint32_t tile = tile_of_block(blockIdx.x, num_tiles);
    if (tile >= num_tiles) return;
    const int64_t tile0 = (int64_t)tile * kTile;
    const uint32_t count = n - tile0 < kTile ? (uint32_t)(n - tile0) : (uint32_t)kTile;
    const uint32_t mine = (uint32_t)wave * (kWave * kItems) + (uint32_t)lane;

    uint32_t item_ts[kItems], key[kItems];
    int32_t item_nbr[kItems], item_eid[kItems];
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const uint32_t i = mine + r * kWave;
        if (i < count) {
            if (kFirst) {
                const uint32_t node = (uint32_t)(in.key + tile0)[i];
                key[r] = (node & ((1u << bits) - 1u)) | (node >> bits << kMaxDigitBits);
                item_ts[r] = (uint32_t)((uint64_t)(in.ts + tile0)[i] - (uint64_t)ts_first);
                item_nbr[r] = (in.dst + tile0)[i];
                item_eid[r] = in.eid ? (in.eid + tile0)[i] : (int32_t)(tile0 + i);
            } else {
                key[r] = (rest_in + tile0)[i];
                const NarrowRec* from = narrow_in + tile0 + i;
                item_ts[r] = from->ts;
                item_nbr[r] = from->nbr;
                item_eid[r] = from->eid;
            }
        }
    }
    const uint32_t own = threadIdx.x;   // the digit value this thread looks after
    {
        const bool live = own < (1u << bits);
        const uint32_t all = live ? total[own] : 0u;
        const uint32_t before = live ? offs[((size_t)tile << bits) + own] : 0u;
        for (int w = 0; w < kSortWaves; ++w) wave_count[w][own] = 0;
        block_base[own] = scan_digits(all, scan_tmp[0]) + before;   // (its barrier also covers the counters)
    }
    uint32_t place[kItems];
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const bool valid = mine + r * kWave < count;
        place[r] = rank_in_wave(valid ? key[r] & (kBins - 1u) : 0u, valid, bits, wave_count[wave]);
    }
    __syncthreads();
    places_of_digit(wave_count, block_base, scan_tmp[1]);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kItems; ++r)
        if (mine + r * kWave < count) place[r] += wave_count[wave][key[r] & (kBins - 1u)];
    for (uint32_t part0 = 0; part0 < count; part0 += kPart) {
#pragma unroll
        for (int r = 0; r < kItems; ++r) {
            const uint32_t at = place[r] - part0;
            if (mine + r * kWave < count && at < (uint32_t)kPart) {
                tile_rec[at] = NarrowRec{item_ts[r], item_nbr[r], item_eid[r]};
                tile_key[at] = key[r];
            }
        }
        __syncthreads();
#pragma unroll 2
        for (int r = 0; r < kPart / kSortThreads; ++r) {
            const uint32_t j = (uint32_t)r * kSortThreads + threadIdx.x;
            if (part0 + j < count) {
                const NarrowRec x = tile_rec[j];
                const uint32_t k = tile_key[j], dg = k & (kBins - 1u);
                const uint32_t to = block_base[dg] + (part0 + j);
                if (kFirst) {
                    narrow_out[to] = x;
                    rest_out[to] = (uint16_t)(k >> kMaxDigitBits);
                } else {
                    const int64_t ts = (int64_t)((uint64_t)ts_first + x.ts);
                    rec_out[to] = TaserRec{ts, x.nbr, x.eid};
                    if ((to & 15u) == 15u || (int64_t)to == n - 1) level1[to >> 4] = ts;
                }
            }
        }
        __syncthreads();
    }
}

// hist[tile * bins + bin] of the second digit, from its column. The entries of a tile share their low digit, and often a popular
// node has most of them: bound by LDS atomics on few addresses, hence eight copies of every counter (64 M entries: 4, 8, 16
// copies 49, 39, 50 us).
constexpr uint32_t kRestCopies = 8;
template <int kItems>
__global__ __launch_bounds__(kSortThreads) void rest_hist_kernel(const uint16_t* __restrict__ rest, int64_t n, int bits,
                                                             uint32_t* __restrict__ hist) {
    constexpr int kTile = kSortThreads * kItems;
    __shared__ uint32_t bins[kBins * kRestCopies];
    const uint32_t copy = threadIdx.x % kRestCopies;
    clear_digit<kRestCopies>(bins);
    __syncthreads();
    const int64_t tile0 = (int64_t)blockIdx.x * kTile;
    if (tile0 + kTile <= n) {   // every thread takes kItems neighbors (the column starts an aligned part of the scratch block)
        typedef uint16_t Some __attribute__((ext_vector_type(kItems)));
        const Some v = reinterpret_cast<const Some*>(rest + tile0)[threadIdx.x];
#pragma unroll
        for (int r = 0; r < kItems; ++r) atomicAdd(&bins[v[r] * kRestCopies + copy], 1u);
    } else {
        for (int64_t i = tile0 + threadIdx.x; i < n; i += kSortThreads) atomicAdd(&bins[rest[i] * kRestCopies + copy], 1u);
    }
    __syncthreads();
    if (threadIdx.x < (1u << bits)) hist[((size_t)blockIdx.x << bits) + threadIdx.x] = count_of_digit<kRestCopies>(bins);
}

// Where every list starts. Block b: the nodes whose low digit is b; thread t: the one of them whose rest is t.
// Before it lie the items with a smaller rest and, of those with its rest, the ones that the first pass left before the
// first item of low digit b: the tiles before that item's (the scanned histogram) and a part of its own tile.
template <int kItems>
__global__ __launch_bounds__(kSortThreads) void list_starts_kernel(const uint32_t* __restrict__ low_total, const uint16_t* __restrict__ rest,
                                                               int64_t n, int low_bits, int rest_bits, const uint32_t* __restrict__ offs,
                                                               const uint32_t* __restrict__ total, uint32_t num_tiles, int32_t num_nodes,
                                                               int64_t* __restrict__ indptr) {
    constexpr uint32_t kTile = kSortThreads * kItems;
    __shared__ uint32_t bins[kBins * kCopies];
    __shared__ uint32_t scan_tmp[2][kSortWaves];
    __shared__ uint32_t low_start;
    const uint32_t own = threadIdx.x, low = blockIdx.x, copy = threadIdx.x % kCopies;
    clear_digit(bins);
    const uint32_t low_before = scan_digits(own < (1u << low_bits) ? low_total[own] : 0u, scan_tmp[0]);
    if (own == low) low_start = low_before;
    __syncthreads();
    const uint32_t tile = low_start / kTile, part = low_start % kTile;
    for (uint32_t i = own; i < part; i += kSortThreads) atomicAdd(&bins[rest[(size_t)tile * kTile + i] * kCopies + copy], 1u);
    const bool live = own < (1u << rest_bits);
    const uint32_t all = live ? total[own] : 0u;
    const uint32_t tiles_before = !live ? 0u : tile < num_tiles ? offs[((size_t)tile << rest_bits) + own] : all;
    const uint32_t smaller = scan_digits(all, scan_tmp[1]);   // (its barrier also covers the counting)
    const uint32_t node = (own << low_bits) | low;
    if (live && node < (uint32_t)num_nodes) indptr[node] = (int64_t)smaller + tiles_before + count_of_digit(bins);
    if (low == 0 && own == 0) indptr[num_nodes] = n;
}

// ---- input in no order, few entries ------------------------------------------------------------
// The passes above move every entry once per digit, four times for 36 bits of key, and a pass over few entries is three
// launches that do not fill the chip. Here the entries are moved once into buckets of some 2 000 to 3 000 neighbors in the final
// order, and once more by a workgroup per bucket that sorts it in LDS. The buckets' limits are quantiles of the samples that
// the inspection took (eight per 2 048 entries), with the position as the key's last digit, so that equal keys divide as well.
// The largest bucket passes 2.7 times the mean, which is what LDS has room for at most, in some of a thousand inputs of the
// largest size; then the passes above do it all behind it (1.57 M entries 244 us, by the passes alone 169; 20 000 155 and 107). 1.34 M
// entries, 36 bits of key, with the plain view: 183 us by 17 launches, so 157 by 10 (kernels: samples' ranks 10, buckets 13, scan 5,
// scatter 16, sort 41, which is what the largest bucket takes).
// Builds by digits / by buckets, us: 2 000 entries of 300 nodes over 2^24 ticks 92 / 60, 20 000 of 17 000 nodes 108 / 88, 200 000
// 121 / 90, 700 000 146 / 108, 1 570 000 172 / 138; over 2^32 ticks 194 / 144. With so few bits that the passes are three at most
// it is a draw from half a million entries on: 1.34 M entries of 300 nodes over 1 000 ticks 113 / 121, of 17 000 121 / 120,
// 700 000 104 / 95 and 108 / 100, 200 000 87 / 81 and 91 / 84. The bits of a whole key and the place in a bucket have to fit one word.
constexpr int64_t kBucketEntries = (int64_t)3 << 19;   // of the whole input
constexpr int64_t kOneBucketEntries = 4096;            // with no more there is one, and nothing to cut
constexpr int kLocalThreads = 1024, kLocalWaves = kLocalThreads / kWave, kLocalItems = 8, kLocalMost = kLocalThreads * kLocalItems;
constexpr int kLocalIndexBits = 13, kLocalDigitBits = 8, kLocalBins = 1 << kLocalDigitBits;
static_assert(kLocalMost == 1 << kLocalIndexBits, "an item's place in its bucket");
inline bool buckets_pay(int64_t n, int key_bits) {
    return n <= kBucketEntries && key_bits <= 64 - kLocalIndexBits && (key_bits > 3 * kMaxDigitBits || n <= (int64_t)1 << 19);
}
static_assert(kLocalThreads == 4 * kLocalBins && kLocalWaves == 16, "four waves' counts of a digit per thread");

// The sort key: the timestamp bits that differ, the node id above them; below 2^63.
struct KeySpec {
    int ts_low, ts_bits;
    __device__ __forceinline__ uint64_t of(int64_t ts, int32_t node) const {
        return ((uint64_t)(uint32_t)node << ts_bits) | ((biased(ts) >> ts_low) & (((uint64_t)1 << ts_bits) - 1u));
    }
};

// rank[i] += how many samples are below sample i (equal keys: in the order of their positions). A lane per sample, a sixteenth of the
// others per wave; the samples of equally spaced ranks are the limits of the buckets. (A sort of them by one workgroup takes longer than the
// rest of the build.)
constexpr uint32_t kRankParts = 16;  // workgroups per 64 samples
__global__ __launch_bounds__(kThreads) void rank_samples_kernel(const Sample* __restrict__ samples, uint32_t num_samples, const KeySpec spec,
                                                               uint32_t* __restrict__ rank, uint32_t* __restrict__ failed) {
    constexpr uint32_t kWaves = kThreads / kWave;
    __shared__ uint32_t part[kWaves][kWave];
    const uint32_t lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const uint32_t own0 = blockIdx.x * kWave;
    auto key_of = [&](uint32_t i) {   // past the last one: above all
        if (i >= num_samples) return ~(uint64_t)0;
        const Sample s = samples[i];
        return spec.of(s.ts, s.node);
    };
    const uint64_t mine = key_of(own0 + lane);
    uint32_t below = 0;
    for (uint32_t j0 = (blockIdx.y * kWaves + wave) * kWave; j0 < num_samples; j0 += kRankParts * kWaves * kWave) {
        const uint64_t theirs = key_of(j0 + lane), limit = j0 < own0 ? mine + 1u : mine;
#pragma unroll 8
        for (int t = 0; t < kWave; ++t) below += wave_get64(theirs, t) < limit ? 1u : 0u;
        if (j0 == own0)
            for (int t = 0; t < kWave; ++t) below += wave_get64(theirs, t) == mine && t < (int)lane ? 1u : 0u;
    }
    part[wave][lane] = below;
    __syncthreads();
    if (wave == 0 && own0 + lane < num_samples) {
        for (uint32_t w = 1; w < kWaves; ++w) below += part[w][lane];
        atomicAdd(&rank[own0 + lane], below);
    }
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *failed = 0;
}

// Every entry's bucket, and how many of a tile's entries each bucket gets (as radix_hist_kernel).
// Bucket b > 0 begins at the first entry whose (key, position) is not below those of the sample of rank b S / buckets.
constexpr uint32_t kMostSamples = (uint32_t)(kBucketEntries / kStratum);
__global__ __launch_bounds__(kSortThreads) void bucket_hist_kernel(const Items in, int64_t n, const KeySpec spec, const Sample* __restrict__ samples,
                                                               const uint32_t* __restrict__ rank, uint32_t num_samples, uint32_t buckets, int bits,
                                                               uint16_t* __restrict__ bucket, uint32_t* __restrict__ hist, uint64_t* __restrict__ first_key) {
    constexpr int kItems = kSmallItems, kTile = kSortThreads * kItems;
    __shared__ uint64_t split_key[kBins];
    __shared__ uint32_t split_pos[kBins];
    __shared__ uint32_t bins[kBins * kCopies];
    __shared__ uint16_t of_rank[kMostSamples];
    const uint32_t copy = threadIdx.x % kCopies;
    clear_digit(bins);
    for (uint32_t i = threadIdx.x; i < num_samples; i += kSortThreads) of_rank[rank[i]] = (uint16_t)i;
    __syncthreads();
    uint64_t limit = ~(uint64_t)0;   // the splitters that there are not are above every entry
    uint32_t limit_pos = 0xffffffffu;
    if (threadIdx.x + 1u < buckets) {
        const Sample x = samples[of_rank[(threadIdx.x + 1u) * num_samples / buckets]];   // below 2^23
        limit = spec.of(x.ts, x.node);
        limit_pos = x.pos;
    }
    split_key[threadIdx.x] = limit;
    if (blockIdx.x == 0) {   // the least key that bucket b may hold; behind the last one, one that none has
        if (threadIdx.x < buckets) first_key[threadIdx.x + 1u] = limit;
        if (threadIdx.x == 0) first_key[0] = 0;
    }
    split_pos[threadIdx.x] = limit_pos;
    const int64_t tile0 = (int64_t)blockIdx.x * kTile;
    uint64_t key[kItems];
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const int64_t i = tile0 + r * kSortThreads + threadIdx.x, at = i < n ? i : n - 1;
        key[r] = spec.of(in.ts[at], in.key[at]);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const int64_t i = tile0 + r * kSortThreads + threadIdx.x;
        uint32_t b = 0;
#pragma unroll
        for (uint32_t half = kBins / 2; half > 0; half /= 2) {
            const uint64_t k = split_key[b + half - 1u];
            if (k < key[r] || (k == key[r] && split_pos[b + half - 1u] <= (uint32_t)i)) b += half;
        }
        if (i < n) {
            bucket[i] = (uint16_t)b;
            atomicAdd(&bins[b * kCopies + copy], 1u);
        }
    }
    __syncthreads();
    if (threadIdx.x < (1u << bits)) hist[((size_t)blockIdx.x << bits) + threadIdx.x] = count_of_digit(bins);
}

// Stable scatter of one tile by the entries' buckets. As radix_scatter_kernel.
__global__ __launch_bounds__(kSortThreads) void bucket_scatter_kernel(const Items in, const uint16_t* __restrict__ bucket, int64_t n, int bits,
                                                                  const uint32_t* __restrict__ offs, const uint32_t* __restrict__ total,
                                                                  uint32_t num_tiles, TaserRec* __restrict__ rec_out, int32_t* __restrict__ key_out) {
    constexpr int kItems = kSmallItems, kTile = kSortThreads * kItems, kPart = 1024;
    __shared__ uint16_t wave_count[kSortWaves][kBins];
    __shared__ uint32_t block_base[kBins];
    __shared__ uint32_t scan_tmp[2][kSortWaves];
    __shared__ TaserRec tile_rec[kPart];
    __shared__ int32_t tile_key[kPart];
    __shared__ uint16_t tile_bucket[kPart];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const uint32_t tile = tile_of_block(blockIdx.x, num_tiles);
    if (tile >= num_tiles) return;
    const int64_t tile0 = (int64_t)tile * kTile;
    const uint32_t count = n - tile0 < kTile ? (uint32_t)(n - tile0) : (uint32_t)kTile;
    const uint32_t mine = (uint32_t)wave * (kWave * kItems) + (uint32_t)lane;
    TaserRec item_rec[kItems];
    int32_t item_key[kItems];
    uint32_t dg[kItems];
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const uint32_t i = mine + r * kWave;
        dg[r] = 0;
        if (i < count) {
            dg[r] = (bucket + tile0)[i];
            item_key[r] = (in.key + tile0)[i];
            item_rec[r] = TaserRec{(in.ts + tile0)[i], (in.dst + tile0)[i], in.eid ? (in.eid + tile0)[i] : (int32_t)(tile0 + i)};
        }
    }
    const uint32_t own = threadIdx.x;
    {
        const bool live = own < (1u << bits);
        const uint32_t all = live ? total[own] : 0u;
        const uint32_t before = live ? offs[((size_t)tile << bits) + own] : 0u;
        for (int w = 0; w < kSortWaves; ++w) wave_count[w][own] = 0;
        block_base[own] = scan_digits(all, scan_tmp[0]) + before;   // (its barrier also covers the counters)
    }
    uint32_t place[kItems];
#pragma unroll
    for (int r = 0; r < kItems; ++r) place[r] = rank_in_wave(dg[r], mine + r * kWave < count, bits, wave_count[wave]);
    __syncthreads();
    places_of_digit(wave_count, block_base, scan_tmp[1]);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kItems; ++r)
        if (mine + r * kWave < count) place[r] += wave_count[wave][dg[r]];
    for (uint32_t part0 = 0; part0 < count; part0 += kPart) {
#pragma unroll
        for (int r = 0; r < kItems; ++r) {
            const uint32_t at = place[r] - part0;
            if (mine + r * kWave < count && at < (uint32_t)kPart) {
                tile_rec[at] = item_rec[r];
                tile_key[at] = item_key[r];
                tile_bucket[at] = (uint16_t)dg[r];
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kPart / kSortThreads; ++r) {
            const uint32_t j = (uint32_t)r * kSortThreads + threadIdx.x;
            if (part0 + j < count) {
                const uint32_t to = block_base[tile_bucket[j]] + (part0 + j);
                rec_out[to] = tile_rec[j];
                key_out[to] = tile_key[j];
            }
        }
        __syncthreads();
    }
}

// One bucket into the final order: its entries' keys, less the bucket's least, with the place in the bucket below them, are
// sorted by stable passes of at most eight bits in LDS (over the bits in which the bucket's limits differ: two to four passes for 36
// bits of key and 500 buckets), then the records are fetched in that order. 74 KB of LDS and 64 registers: two workgroups to a
// compute unit, as long as the loads of all eight rows are not issued together (with spills 69 us, so 41).
// kColumns: the one bucket of a small input, from the caller's columns.
template <bool kColumns>
__global__ __launch_bounds__(kLocalThreads) __attribute__((amdgpu_waves_per_eu(8))) void sort_bucket_kernel(
    const Items in, int64_t n, const uint32_t* __restrict__ total, const KeySpec spec, TaserRec* __restrict__ rec_out,
    int32_t* __restrict__ key_out, int64_t* __restrict__ level1, const uint64_t* __restrict__ first_key, uint64_t all_keys,
    uint32_t* __restrict__ failed) {
    typedef uint64_t __attribute__((may_alias)) FourCounts;
    __shared__ uint64_t item[kLocalMost];
    __shared__ __align__(8) uint16_t wave_count[kLocalWaves][kLocalBins];
    __shared__ uint32_t scan_tmp[kLocalWaves];
    const uint32_t lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    uint32_t start = 0, count = (uint32_t)n;
    uint64_t least = 0, most = all_keys;
    if (kColumns) {
        if (threadIdx.x == 0) *failed = 0;
    } else {   // the buckets before this one
        uint32_t before = threadIdx.x < blockIdx.x ? total[threadIdx.x] : 0u;   // (at most kBins of them)
        count = total[blockIdx.x];
        least = first_key[blockIdx.x];
        most = first_key[blockIdx.x + 1u];
        if (most > all_keys) most = all_keys;
        if (count == 0) return;
        before = wave_sum32(before);
        if (lane == 0) scan_tmp[wave] = before;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kBins / kWave; ++w) start += scan_tmp[w];
    }
    if (count > (uint32_t)kLocalMost) {   // uniform
        if (threadIdx.x == 0) *failed = 1;
        return;
    }
    const int key_bits = most > least ? 64 - __clzll((long long)(most - least)) : 0;   // at most 64 - kLocalIndexBits
    const uint32_t per = (count + kLocalThreads - 1) / kLocalThreads;   // rows of 64 of each wave
    const uint32_t mine = wave * per * kWave + lane;
    uint64_t v[kLocalItems];
#pragma unroll
    for (uint32_t r = 0; r < (uint32_t)kLocalItems; ++r) {
        v[r] = 0;
        const uint32_t i = mine + r * kWave;
        if (r < per && i < count) {
            v[r] = ((spec.of(kColumns ? in.ts[i] : in.rec[start + i].ts, in.key[start + i]) - least) << kLocalIndexBits) | i;
            if (key_bits == 0) item[i] = v[r];
        }
        if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // the loads of four rows together: of all, the registers would spill
    }
    const int passes = (key_bits + kLocalDigitBits - 1) / kLocalDigitBits, digit_bits = passes ? (key_bits + passes - 1) / passes : 0;
    const uint32_t digit_mask = (1u << digit_bits) - 1u;
    for (int pass = 0, shift = kLocalIndexBits; pass < passes; ++pass, shift += digit_bits) {
        for (uint32_t c = threadIdx.x; c < (uint32_t)(kLocalWaves * kLocalBins / 4); c += kLocalThreads) reinterpret_cast<FourCounts*>(&wave_count[0][0])[c] = 0;
        __syncthreads();
        uint32_t place[kLocalItems];
#pragma unroll
        for (uint32_t r = 0; r < (uint32_t)kLocalItems; ++r) {
            if (r >= per) continue;   // uniform
            const bool valid = mine + r * kWave < count;
            const uint32_t dg = valid ? (uint32_t)(v[r] >> shift) & digit_mask : 0u;
            place[r] = rank_in_wave(dg, valid, digit_bits, wave_count[wave]);
        }
        __syncthreads();
        // how many of a digit a wave has becomes the place of its first one; a thread has four waves' of a digit
        const uint32_t digit = threadIdx.x / 4u, w0 = threadIdx.x % 4u * 4u;
        uint32_t here[4], all = 0;
#pragma unroll
        for (uint32_t w = 0; w < 4; ++w) {
            here[w] = wave_count[w0 + w][digit];
            all += here[w];
        }
        const uint32_t inc = wave_inclusive_scan32(all);
        if (lane == kWave - 1) scan_tmp[wave] = inc;
        __syncthreads();
        uint32_t run = inc - all;
#pragma unroll
        for (uint32_t w = 0; w < (uint32_t)kLocalWaves; ++w) run += w < wave ? scan_tmp[w] : 0u;
#pragma unroll
        for (uint32_t w = 0; w < 4; ++w) {
            wave_count[w0 + w][digit] = (uint16_t)run;
            run += here[w];
        }
        __syncthreads();
#pragma unroll
        for (uint32_t r = 0; r < (uint32_t)kLocalItems; ++r)
            if (r < per && mine + r * kWave < count) item[place[r] + wave_count[wave][(uint32_t)(v[r] >> shift) & digit_mask]] = v[r];
        __syncthreads();
        if (pass + 1 < passes) {
#pragma unroll
            for (uint32_t r = 0; r < (uint32_t)kLocalItems; ++r)
                if (r < per && mine + r * kWave < count) v[r] = item[mine + r * kWave];
        }
    }
    if (key_bits == 0) __syncthreads();
    for (uint32_t j = threadIdx.x; j < count; j += kLocalThreads) {
        const uint32_t from = start + ((uint32_t)item[j] & (kLocalMost - 1u)), to = start + j;
        const TaserRec r = kColumns ? TaserRec{in.ts[from], in.dst[from], in.eid ? in.eid[from] : (int32_t)from} : in.rec[from];
        rec_out[to] = r;
        key_out[to] = (int32_t)((least + (item[j] >> kLocalIndexBits)) >> spec.ts_bits);
        if ((to & 15u) == 15u || (int64_t)to == n - 1) level1[to >> 4] = r.ts;
    }
}

// The plain arrays of a graph, indptr among them: views of small graphs are bound by launches (2 000 to 670 000 entries with a
// copy of indptr of its own 15.2 us, so 12.8).
__global__ __launch_bounds__(kThreads) void unpack_kernel(const TaserRec* __restrict__ rec, int64_t n, const int64_t* __restrict__ indptr, int64_t starts,
                                                          int64_t* __restrict__ o_indptr, int32_t* __restrict__ nbr, int64_t* __restrict__ ts,
                                                          int32_t* __restrict__ eid) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < starts) o_indptr[i] = indptr[i];
    if (i >= n) return;
    const TaserRec r = rec[i];
    if (nbr) nbr[i] = r.nbr;
    if (ts) ts[i] = r.ts;
    if (eid) eid[i] = r.eid;
}

inline unsigned blocks_for(int64_t n, int per_block) { return (unsigned)((n + per_block - 1) / per_block); }

// Levels 2 and up of the search index from level 1, which the last pass wrote: entry i of level l is
// the level-1 entry of the last run of 16 records it covers. One launch for all of them.
struct UpperLevels {
    int64_t* out[kTimeIndexLevels - 1];    // level 2 first
    int64_t end[kTimeIndexLevels - 1];     // running sum of their lengths
};
__global__ __launch_bounds__(kThreads) void time_index_upper_kernel(const int64_t* __restrict__ level1, int64_t len1,
                                                                    UpperLevels up, const uint32_t* __restrict__ failed,
                                                                    unsigned long long* __restrict__ report) {
    const int64_t g = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (g == 0 && failed) *report = *failed;
    int64_t begin = 0;
#pragma unroll
    for (int l = 0; l < kTimeIndexLevels - 1; ++l) {
        if (g >= begin && g < up.end[l]) {
            const int64_t last = ((g - begin + 1) << (4 * (l + 1))) - 1;
            up.out[l][g - begin] = level1[last < len1 ? last : len1 - 1];
        }
        begin = up.end[l];
    }
}

// ---- the two memory blocks of a build ----------------------------------------------
// Items per thread of a tile: the large tile's longer runs per digit are what the scatter's writes
// want, but with few entries its tiles do not fill 256 compute units and a pass takes the latency of
// one tile. Whole builds, 2048- / 4096-item tiles, unsorted input: 20 k entries 112 / 120 us, 1.34 M
// 160 / 163, 3 M 249 / 236, 12 M 717 / 677; sorted input 70 / 77, 91 / 97, 124 / 125, 319 / 316.
constexpr int64_t kSmallEntries = (int64_t)1 << 21;
inline int items_for(int64_t n) { return n <= kSmallEntries ? kSmallItems : kLargeItems; }

constexpr int kInfoWords = 5;   // the inspection's four, and whether the buckets could not be sorted
struct Layout {
    size_t indptr, rec, level[kTimeIndexLevels], storage;                                   // what the graph keeps
    size_t src, dst, ts, eid, tmp_rec, key[2], hist, total, chunk_sum, partial, info, scratch;         // what the build needs
    // (inputs that may be cut into buckets have too few tiles for chunk_sum: samples and splitters are in its place)
    int64_t level_len[kTimeIndexLevels];
    uint32_t tiles;
};

Layout layout_of(int64_t n, int32_t num_nodes, bool copy_input) {
    Layout l = {};
    size_t at = 0;
    auto take = [&at](size_t bytes) {
        const size_t here = at;
        at += (bytes + 255) / 256 * 256;
        return here;
    };
    l.indptr = take(((size_t)num_nodes + 1) * sizeof(int64_t));
    // kSearchSlack entries behind the records and behind every level: the search reads whole groups of 16
    l.rec = take((size_t)(n + kSearchSlack) * sizeof(TaserRec));
    int64_t below = n;
    for (int i = 0; i < kTimeIndexLevels; ++i) {
        l.level_len[i] = below = (below + 15) / 16;
        l.level[i] = take((size_t)(below + kSearchSlack) * sizeof(int64_t));
    }
    l.storage = at;
    at = 0;
    l.tiles = blocks_for(n, kSortThreads * items_for(n));
    if (copy_input) {
        l.src = take((size_t)n * sizeof(int32_t));
        l.dst = take((size_t)n * sizeof(int32_t));
        l.ts = take((size_t)n * sizeof(int64_t));
        l.eid = take((size_t)n * sizeof(int32_t));
    }
    l.tmp_rec = take((size_t)n * sizeof(TaserRec));
    l.key[0] = take((size_t)n * sizeof(int32_t));
    l.key[1] = take((size_t)n * sizeof(int32_t));
    l.hist = take((size_t)kBins * l.tiles * sizeof(uint32_t));
    l.total = take(kBins * sizeof(uint32_t));
    l.chunk_sum = take((size_t)kMaxChunks * kBins * sizeof(uint32_t));
    l.partial = take((size_t)kInspectBlocks * 4 * sizeof(unsigned long long));
    l.info = take(kInfoWords * sizeof(unsigned long long));
    l.scratch = at;
    return l;
}

int check_build_sizes(const char* what, int64_t num_entries, int32_t num_nodes, uint32_t flags) {
    if (num_entries < 0 || num_entries >= 0x7fffffffLL) return taser_fail(TASER_E_RANGE, "%s: num_entries = %lld outside [0, 2^31 - 1)", what, (long long)num_entries);
    if (num_nodes < 1 || num_nodes == 0x7fffffff) return taser_fail(TASER_E_RANGE, "%s: num_nodes = %d outside [1, 2^31 - 1)", what, num_nodes);
    if (flags & ~(uint32_t)TASER_INPUT_ON_DEVICE) return taser_fail(TASER_E_ARG, "%s: unknown flags 0x%x", what, flags);
    return TASER_OK;
}

// hist becomes its exclusive scan per digit over the tiles, total the digits' counts.
void launch_scan(const Layout& l, int bits, uint32_t* hist, uint32_t* total, uint32_t* chunk_sum, hipStream_t stream) {
    TaserProfileSpan span(stream, "tcsr_scan");
    if (l.tiles >= kChunkedTiles) {
        const uint32_t by_count = (l.tiles + kMaxChunks - 1) / kMaxChunks, rows = by_count > 64 ? by_count : 64;
        const dim3 grid(((1u << bits) + kWave - 1) / kWave, (l.tiles + rows - 1) / rows);
        hipLaunchKernelGGL(chunk_sum_kernel, grid, dim3(kThreads), 0, stream, hist, l.tiles, bits, rows, chunk_sum);
        hipLaunchKernelGGL(chunk_scan_kernel, grid, dim3(kThreads), 0, stream, hist, l.tiles, bits, rows, chunk_sum, total);
    } else {
        hipLaunchKernelGGL(bin_scan_kernel, dim3(((1u << bits) + kScanCols - 1) / kScanCols), dim3(kScanThreads), 0, stream, hist,
                           l.tiles, bits, total);
    }
}

// Time-sorted input whose node digit of `low_bits` bits is counted in hist and whose others are `rest_bits`: both passes
// and indptr.
static_assert(kInspectBlocks * 4 * sizeof(unsigned long long) >= kBins * sizeof(uint32_t), "total[1] of launch_sorted");
template <int kItems>
void launch_sorted(const Layout& l, const Items& in, int64_t ts_first, int64_t n, int32_t num_nodes, int low_bits, int rest_bits, uint8_t* scratch,
                   TaserRec* rec, int64_t* level1, int64_t* indptr, hipStream_t stream) {
    uint32_t* hist = reinterpret_cast<uint32_t*>(scratch + l.hist);
    // the second digit's totals go where the inspection's words were, which have been read
    uint32_t* total[2] = {reinterpret_cast<uint32_t*>(scratch + l.total), reinterpret_cast<uint32_t*>(scratch + l.partial)};
    uint32_t* chunk_sum = reinterpret_cast<uint32_t*>(scratch + l.chunk_sum);
    NarrowRec* narrow = reinterpret_cast<NarrowRec*>(scratch + l.tmp_rec);   // 12 of its 16 bytes per entry
    uint16_t* rest = reinterpret_cast<uint16_t*>(scratch + l.key[0]);
    launch_scan(l, low_bits, hist, total[0], chunk_sum, stream);
    {
        TaserProfileSpan span(stream, "tcsr_radix_scatter");
        hipLaunchKernelGGL((node_scatter_kernel<true, kItems>), dim3(pass_grid(l.tiles)), dim3(kSortThreads), 0, stream, in, nullptr, nullptr, ts_first, n,
                           low_bits, hist, total[0], l.tiles, narrow, rest, nullptr, nullptr);
    }
    {
        TaserProfileSpan span(stream, "tcsr_radix_hist");
        hipLaunchKernelGGL((rest_hist_kernel<kItems>), dim3(l.tiles), dim3(kSortThreads), 0, stream, rest, n, rest_bits, hist);
    }
    launch_scan(l, rest_bits, hist, total[1], chunk_sum, stream);
    {
        TaserProfileSpan span(stream, "tcsr_radix_scatter");
        hipLaunchKernelGGL((node_scatter_kernel<false, kItems>), dim3(pass_grid(l.tiles)), dim3(kSortThreads), 0, stream, in, narrow, rest, ts_first, n,
                           rest_bits, hist, total[1], l.tiles, nullptr, nullptr, rec, level1);
    }
    TaserProfileSpan span(stream, "tcsr_indptr");
    hipLaunchKernelGGL((list_starts_kernel<kItems>), dim3(1u << low_bits), dim3(kSortThreads), 0, stream, total[0], rest, n, low_bits, rest_bits,
                       hist, total[1], l.tiles, num_nodes, indptr);
}

// Input in no order that is cut into buckets: everything up to the records and the sorted node column.
struct BucketScratch {
    Sample at[kMostSamples];
    uint64_t first_key[kBins + 1];
    uint32_t rank[kMostSamples];
    uint32_t failed;   // a bucket could not be sorted
};
static_assert(sizeof(BucketScratch) <= (size_t)kMaxChunks * kBins * sizeof(uint32_t), "in place of chunk_sum");
static_assert(kBucketEntries <= kSmallEntries && kBucketEntries / (kSortThreads * kSmallItems) < kChunkedTiles, "small tiles, one scan launch");
inline BucketScratch* bucket_scratch(const Layout& l, uint8_t* scratch) { return reinterpret_cast<BucketScratch*>(scratch + l.chunk_sum); }
void launch_buckets(const Layout& l, const Items& columns, int64_t n, int node_bits, const KeySpec& spec, uint8_t* scratch, TaserRec* rec, int64_t* level1, hipStream_t stream) {
    uint32_t* hist = reinterpret_cast<uint32_t*>(scratch + l.hist);
    uint32_t* total = reinterpret_cast<uint32_t*>(scratch + l.total);
    int32_t* key_out = reinterpret_cast<int32_t*>(scratch + l.key[1]);
    BucketScratch* own = bucket_scratch(l, scratch);
    const uint64_t all_keys = ((uint64_t)1 << (spec.ts_bits + node_bits)) - 1u;
    if (n <= kOneBucketEntries) {
        TaserProfileSpan span(stream, "tcsr_sort_buckets");
        hipLaunchKernelGGL((sort_bucket_kernel<true>), dim3(1), dim3(kLocalThreads), 0, stream, columns, n, nullptr, spec, rec, key_out, level1, nullptr,
                           all_keys, &own->failed);
        return;
    }
    const uint32_t buckets = l.tiles < (uint32_t)kBins ? l.tiles : (uint32_t)kBins, samples = l.tiles * (uint32_t)(kSortThreads * kSmallItems / kStratum);
    {
        TaserProfileSpan span(stream, "tcsr_rank_samples");
        hipLaunchKernelGGL(rank_samples_kernel, dim3((samples + kWave - 1) / kWave, kRankParts), dim3(kThreads), 0, stream, own->at, samples, spec, own->rank,
                           &own->failed);
    }
    int bits = 1;
    while ((1u << bits) < buckets) ++bits;
    uint16_t* bucket = reinterpret_cast<uint16_t*>(scratch + l.key[1]);   // read before the sorted column is written
    TaserRec* tmp_rec = reinterpret_cast<TaserRec*>(scratch + l.tmp_rec);
    int32_t* tmp_key = reinterpret_cast<int32_t*>(scratch + l.key[0]);
    {
        TaserProfileSpan span(stream, "tcsr_radix_hist");
        hipLaunchKernelGGL(bucket_hist_kernel, dim3(l.tiles), dim3(kSortThreads), 0, stream, columns, n, spec, own->at, own->rank, samples, buckets,
                           bits, bucket, hist, own->first_key);
    }
    launch_scan(l, bits, hist, total, nullptr, stream);
    {
        TaserProfileSpan span(stream, "tcsr_radix_scatter");
        hipLaunchKernelGGL(bucket_scatter_kernel, dim3(pass_grid(l.tiles)), dim3(kSortThreads), 0, stream, columns, bucket, n, bits, hist, total, l.tiles,
                           tmp_rec, tmp_key);
    }
    TaserProfileSpan span(stream, "tcsr_sort_buckets");
    const Items in = {tmp_rec, tmp_key, nullptr, nullptr, nullptr};
    hipLaunchKernelGGL((sort_bucket_kernel<false>), dim3(buckets), dim3(kLocalThreads), 0, stream, in, n, total, spec, rec, key_out, level1, own->first_key, all_keys,
                       &own->failed);
}

template <int kItems>
void launch_pass(const Layout& l, const Items& in, int64_t n, const DigitSpec& d, bool hist_known, uint32_t* hist, uint32_t* total, uint32_t* chunk_sum,
                 TaserRec* rec_out, int32_t* key_out, int64_t* level1, hipStream_t stream) {
    if (!hist_known) {
        TaserProfileSpan span(stream, "tcsr_radix_hist");
        hipLaunchKernelGGL((radix_hist_kernel<kItems>), dim3(l.tiles), dim3(kSortThreads), 0, stream, in, n, d, hist);
    }
    launch_scan(l, d.bits, hist, total, chunk_sum, stream);
    TaserProfileSpan span(stream, "tcsr_radix_scatter");
    if (in.rec)
        hipLaunchKernelGGL((radix_scatter_kernel<false, kItems>), dim3(pass_grid(l.tiles)), dim3(kSortThreads), 0, stream, in, n, d, hist,
                           total, l.tiles, rec_out, key_out, level1);
    else
        hipLaunchKernelGGL((radix_scatter_kernel<true, kItems>), dim3(pass_grid(l.tiles)), dim3(kSortThreads), 0, stream, in, n, d, hist,
                           total, l.tiles, rec_out, key_out, level1);
}

// The build itself, in `storage` and `scratch` (l.storage and l.scratch bytes of device memory, 256-byte
// aligned). Synchronizes the stream before it returns TASER_OK.
int build_in(const Layout& l, const int32_t* src, const int32_t* dst, const int64_t* ts, const int32_t* eid, int64_t n,
             int32_t num_nodes, uint32_t flags, hipStream_t stream, uint8_t* storage, uint8_t* scratch, taser_tcsr** out) {
    if (!(flags & TASER_INPUT_ON_DEVICE) && n > 0) {
        TASER_HIP_TRY(hipMemcpyAsync(scratch + l.src, src, n * sizeof(int32_t), hipMemcpyHostToDevice, stream));
        TASER_HIP_TRY(hipMemcpyAsync(scratch + l.dst, dst, n * sizeof(int32_t), hipMemcpyHostToDevice, stream));
        TASER_HIP_TRY(hipMemcpyAsync(scratch + l.ts, ts, n * sizeof(int64_t), hipMemcpyHostToDevice, stream));
        if (eid) TASER_HIP_TRY(hipMemcpyAsync(scratch + l.eid, eid, n * sizeof(int32_t), hipMemcpyHostToDevice, stream));
        src = reinterpret_cast<const int32_t*>(scratch + l.src);
        dst = reinterpret_cast<const int32_t*>(scratch + l.dst);
        ts = reinterpret_cast<const int64_t*>(scratch + l.ts);
        if (eid) eid = reinterpret_cast<const int32_t*>(scratch + l.eid);
    }
    const bool small = items_for(n) == kSmallItems;
    int64_t* indptr = reinterpret_cast<int64_t*>(storage + l.indptr);
    TaserRec* rec = reinterpret_cast<TaserRec*>(storage + l.rec);
    int64_t* level1 = reinterpret_cast<int64_t*>(storage + l.level[0]);
    uint32_t* hist = reinterpret_cast<uint32_t*>(scratch + l.hist);
    uint32_t* total = reinterpret_cast<uint32_t*>(scratch + l.total);
    uint32_t* chunk_sum = reinterpret_cast<uint32_t*>(scratch + l.chunk_sum);
    TaserTimeIndex index = {};
    index.num_entries = n;
    for (int i = 0; i < kTimeIndexLevels; ++i) {
        index.len[i] = l.level_len[i];
        index.level[i] = reinterpret_cast<int64_t*>(storage + l.level[i]);
    }
    // indptr, if it is `wanted` from the sorted node column (not where *failed says that this is in no order), and the upper index
    // levels; *report = *failed, copied to *read_back if that is not null. Waits for the stream.
    auto finish = [&](bool wanted, const int32_t* sorted_key, const uint32_t* failed, unsigned long long* report, unsigned long long* read_back) -> int {
        if (wanted) {
            TaserProfileSpan span(stream, "tcsr_indptr");
            hipLaunchKernelGGL(indptr_kernel, dim3(blocks_for(n + 1, kThreads * 4)), dim3(kThreads), 0, stream, sorted_key, n, num_nodes, indptr, failed);
        }
        if (n > 0) {
            TaserProfileSpan span(stream, "tcsr_time_index");
            UpperLevels up;
            int64_t end = 0;
            for (int i = 1; i < kTimeIndexLevels; ++i) {
                up.out[i - 1] = reinterpret_cast<int64_t*>(storage + l.level[i]);
                up.end[i - 1] = end += l.level_len[i];
            }
            hipLaunchKernelGGL(time_index_upper_kernel, dim3(blocks_for(end, kThreads)), dim3(kThreads), 0, stream, level1, l.level_len[0], up, failed, report);
        }
        TASER_HIP_TRY(hipGetLastError());
        if (read_back) TASER_HIP_TRY(hipMemcpyAsync(read_back, report, sizeof(*report), hipMemcpyDeviceToHost, stream));
        TASER_HIP_TRY(hipStreamSynchronize(stream));
        return TASER_OK;
    };

    if (n == 0) {
        const int rc = finish(true, nullptr, nullptr, nullptr, nullptr);
        if (rc != TASER_OK) return rc;
    } else {
        // ---- what the input looks like
        int node_bits = 0;
        while (((int64_t)1 << node_bits) < (int64_t)num_nodes) ++node_bits;
        // equal digits of at most kMaxDigitBits bits (one pass at least: it is what packs the records)
        auto width_of = [](int bits) {
            const int passes = (bits + kMaxDigitBits - 1) / kMaxDigitBits;
            return passes > 0 ? (bits + passes - 1) / passes : 1;
        };
        const bool two_digits = node_bits > kMaxDigitBits && node_bits <= 2 * kMaxDigitBits;   // of the node id
        const int low_bits = two_digits ? node_bits / 2 : width_of(node_bits);                  // counted by the inspection
        unsigned long long info[kInfoWords] = {0, 0, 0, ~0ull, 0};
        unsigned long long* partial = reinterpret_cast<unsigned long long*>(scratch + l.partial);
        PinnedInfo pinned;
        unsigned long long* d_info = pinned.words ? pinned.words : reinterpret_cast<unsigned long long*>(scratch + l.info);
        pinned.launched(stream);
        Samples wanted = {};
        if (n <= kBucketEntries) wanted = Samples{bucket_scratch(l, scratch)->at, bucket_scratch(l, scratch)->rank};
        {
            TaserProfileSpan span(stream, "tcsr_inspect");
            const unsigned grid = l.tiles < kInspectBlocks ? l.tiles : kInspectBlocks;
            if (small)
                hipLaunchKernelGGL((inspect_kernel<kSmallItems>), dim3(grid), dim3(kSortThreads), 0, stream, src, ts, n, num_nodes, partial,
                                   low_bits, hist, l.tiles, wanted);
            else
                hipLaunchKernelGGL((inspect_kernel<kLargeItems>), dim3(grid), dim3(kSortThreads), 0, stream, src, ts, n, num_nodes, partial,
                                   low_bits, hist, l.tiles, wanted);
            hipLaunchKernelGGL(fold_info_kernel, dim3(1), dim3(kSortThreads), 0, stream, partial, grid, ts, n, d_info);
        }
        TASER_HIP_TRY(hipGetLastError());
        if (!pinned.words) TASER_HIP_TRY(hipMemcpyAsync(info, d_info, 4 * sizeof(info[0]), hipMemcpyDeviceToHost, stream));
        TASER_HIP_TRY(hipStreamSynchronize(stream));
        pinned.settled();
        if (pinned.words)
            for (int j = 0; j < 4; ++j) info[j] = __atomic_load_n(&pinned.words[j], __ATOMIC_RELAXED);
        if (info[0]) return taser_fail(TASER_E_RANGE, "tcsr_build: a src node id is outside [0, %d)", num_nodes);
        int ts_low = 0, ts_bits = 0;
        if (info[1]) {
            const unsigned long long differ = info[2] & ~info[3];   // not 0: the timestamps are not all equal
            ts_low = __builtin_ctzll(differ);
            ts_bits = 64 - __builtin_clzll(differ) - ts_low;
        }
        const Items columns = {nullptr, src, dst, ts, eid};
        const bool in_node_digits = two_digits && !info[1] && info[3] - info[2] < (1ull << 32);
        bool done = false;
        if (in_node_digits) {
            if (small) launch_sorted<kSmallItems>(l, columns, (int64_t)info[2], n, num_nodes, low_bits, node_bits - low_bits, scratch, rec, level1, indptr, stream);
            else launch_sorted<kLargeItems>(l, columns, (int64_t)info[2], n, num_nodes, low_bits, node_bits - low_bits, scratch, rec, level1, indptr, stream);
            const int rc = finish(false, nullptr, nullptr, nullptr, nullptr);
            if (rc != TASER_OK) return rc;
            done = true;
        } else if (info[1] && buckets_pay(n, ts_bits + node_bits)) {
            pinned.launched(stream);
            launch_buckets(l, columns, n, node_bits, KeySpec{ts_low, ts_bits}, scratch, rec, level1, stream);
            const int rc = finish(true, reinterpret_cast<const int32_t*>(scratch + l.key[1]), &bucket_scratch(l, scratch)->failed, d_info + 4,
                                  pinned.words ? nullptr : &info[4]);
            if (rc != TASER_OK) return rc;
            pinned.settled();
            if (pinned.words) info[4] = __atomic_load_n(&pinned.words[4], __ATOMIC_RELAXED);
            done = info[4] == 0;
        }

        // ---- one stable pass per digit; the last one writes the graph's own records
        if (!done) {
            const int key_bits = ts_bits + node_bits;
            const int width = width_of(key_bits);
            const int passes = key_bits > 0 ? (key_bits + width - 1) / width : 1;
            // without timestamp digits the first digit is the one that inspect_kernel counted, also where the others are wider by a
            // bit (64 M entries over 2^45 ticks, 131 000 nodes: 1.56 ms with equal digits and a count of their own, 1.44 so)
            const int first_width = ts_bits ? width : low_bits;
            TaserRec* tmp_rec = reinterpret_cast<TaserRec*>(scratch + l.tmp_rec);
            Items in = columns;
            for (int pass = 0; pass < passes; ++pass) {
                const int s = pass ? first_width + (pass - 1) * width : 0, most = pass ? width : first_width;
                DigitSpec d = {};
                d.bits = key_bits - s < most ? key_bits - s : most;
                if (d.bits < 1) d.bits = 1;               // a single node and sorted input: every digit is 0
                if (s < ts_bits) {
                    const int have = ts_bits - s;         // timestamp bits from here on
                    d.from_ts = 1;
                    d.ts_shift = ts_low + s;
                    d.ts_mask = (1u << (have < d.bits ? have : d.bits)) - 1u;
                    d.node_left = have < 31 ? have : 31;
                } else {
                    d.node_right = s - ts_bits;
                }
                const bool last = pass + 1 == passes;
                TaserRec* rec_out = ((passes - 1 - pass) & 1) ? tmp_rec : rec;
                int32_t* key_out = reinterpret_cast<int32_t*>(scratch + l.key[pass & 1]);
                const bool hist_known = pass == 0 && ts_bits == 0;
                if (small) launch_pass<kSmallItems>(l, in, n, d, hist_known, hist, total, chunk_sum, rec_out, key_out, last ? level1 : nullptr, stream);
                else launch_pass<kLargeItems>(l, in, n, d, hist_known, hist, total, chunk_sum, rec_out, key_out, last ? level1 : nullptr, stream);
                in = Items{rec_out, key_out, nullptr, nullptr, nullptr};
            }
            const int rc = finish(true, in.key, nullptr, nullptr, nullptr);
            if (rc != TASER_OK) return rc;
        }
    }

    taser_tcsr* g = new (std::nothrow) taser_tcsr();
    if (!g) return taser_fail(TASER_E_OOM, "tcsr_build: host allocation failed");
    *g = taser_tcsr{};
    g->num_entries = n;
    g->num_nodes = num_nodes;
    g->indptr = indptr;
    g->rec = rec;
    g->time_index = index;
    *out = g;
    return TASER_OK;
}

}  // namespace

extern "C" int taser_tcsr_build(const int32_t* src, const int32_t* dst, const int64_t* ts,
                                const int32_t* eid, int64_t num_entries, int32_t num_nodes,
                                uint32_t flags, void* hip_stream, taser_tcsr** out) {
    if (!out) return taser_fail(TASER_E_ARG, "tcsr_build: null out");
    *out = nullptr;
    const int bad = check_build_sizes("tcsr_build", num_entries, num_nodes, flags);
    if (bad != TASER_OK) return bad;
    if (num_entries > 0 && (!src || !dst || !ts)) return taser_fail(TASER_E_ARG, "tcsr_build: null src/dst/ts");
    taser_clear_stale_hip_error();
    taser_resolve_device_constants();
    const Layout l = layout_of(num_entries, num_nodes, !(flags & TASER_INPUT_ON_DEVICE));
    void *storage = nullptr, *scratch = nullptr;
    hipError_t e = hipMalloc(&storage, l.storage);
    if (e == hipSuccess) e = hipMalloc(&scratch, l.scratch);
    int rc = e == hipSuccess ? TASER_OK : taser_fail_hip(e, "tcsr_build: hipMalloc");
    if (rc == TASER_OK)
        rc = build_in(l, src, dst, ts, eid, num_entries, num_nodes, flags, (hipStream_t)hip_stream, static_cast<uint8_t*>(storage),
                      static_cast<uint8_t*>(scratch), out);
    (void)hipFree(scratch);
    if (rc == TASER_OK) (*out)->owned_storage = storage;
    else (void)hipFree(storage);
    return rc;
}

extern "C" int taser_tcsr_build_bytes(int64_t num_entries, int32_t num_nodes, uint32_t flags, uint64_t* storage_bytes,
                                      uint64_t* scratch_bytes) {
    const int bad = check_build_sizes("tcsr_build_bytes", num_entries, num_nodes, flags);
    if (bad != TASER_OK) return bad;
    const Layout l = layout_of(num_entries, num_nodes, !(flags & TASER_INPUT_ON_DEVICE));
    if (storage_bytes) *storage_bytes = l.storage;
    if (scratch_bytes) *scratch_bytes = l.scratch;
    return TASER_OK;
}

extern "C" int taser_tcsr_build_in(const int32_t* src, const int32_t* dst, const int64_t* ts,
                                   const int32_t* eid, int64_t num_entries, int32_t num_nodes,
                                   uint32_t flags, void* hip_stream, void* storage, uint64_t storage_bytes,
                                   void* scratch, uint64_t scratch_bytes, taser_tcsr** out) {
    if (!out) return taser_fail(TASER_E_ARG, "tcsr_build_in: null out");
    *out = nullptr;
    const int bad = check_build_sizes("tcsr_build_in", num_entries, num_nodes, flags);
    if (bad != TASER_OK) return bad;
    if (num_entries > 0 && (!src || !dst || !ts)) return taser_fail(TASER_E_ARG, "tcsr_build_in: null src/dst/ts");
    const Layout l = layout_of(num_entries, num_nodes, !(flags & TASER_INPUT_ON_DEVICE));
    if (!storage || !scratch) return taser_fail(TASER_E_ARG, "tcsr_build_in: null storage or scratch");
    if (((uintptr_t)storage | (uintptr_t)scratch) & 255) return taser_fail(TASER_E_ARG, "tcsr_build_in: storage and scratch must be 256-byte aligned");
    if (storage_bytes < l.storage || scratch_bytes < l.scratch)
        return taser_fail(TASER_E_RANGE, "tcsr_build_in: %llu bytes of storage and %llu of scratch are needed", (unsigned long long)l.storage,
                          (unsigned long long)l.scratch);
    taser_clear_stale_hip_error();
    taser_resolve_device_constants();
    const int rc = build_in(l, src, dst, ts, eid, num_entries, num_nodes, flags, (hipStream_t)hip_stream, static_cast<uint8_t*>(storage),
                            static_cast<uint8_t*>(scratch), out);
    if (rc != TASER_OK) {
        (void)hipStreamSynchronize((hipStream_t)hip_stream);   // what was launched before the error still uses the caller's blocks
        (void)hipGetLastError();
    } else if (hipGetDevice(&(*out)->device) != hipSuccess) {
        (*out)->device = -1;
    }
    return rc;
}

extern "C" int taser_tcsr_size(const taser_tcsr* g, int64_t* num_entries, int32_t* num_nodes) {
    if (!g) return taser_fail(TASER_E_ARG, "tcsr_size: null graph");
    if (num_entries) *num_entries = g->num_entries;
    if (num_nodes) *num_nodes = g->num_nodes;
    return TASER_OK;
}

extern "C" int taser_tcsr_view(const taser_tcsr* g, int64_t* indptr, int32_t* nbr, int64_t* ts, int32_t* eid,
                               void* hip_stream) {
    if (!g) return taser_fail(TASER_E_ARG, "tcsr_view: null graph");
    taser_clear_stale_hip_error();
    hipStream_t stream = (hipStream_t)hip_stream;
    const int64_t starts = indptr ? (int64_t)g->num_nodes + 1 : 0, entries = nbr || ts || eid ? g->num_entries : 0;
    if (starts > 0 || entries > 0) {
        hipLaunchKernelGGL(unpack_kernel, dim3(blocks_for(starts > entries ? starts : entries, kThreads)), dim3(kThreads), 0, stream,
                           g->rec, entries, g->indptr, starts, indptr, nbr, ts, eid);
        TASER_HIP_TRY(hipGetLastError());
    }
    return TASER_OK;
}

extern "C" void taser_tcsr_free(taser_tcsr* g) {
    if (!g) return;
    if (g->owned_storage) {
        (void)hipFree(g->owned_storage);
    } else {
        // the storage is the caller's and may go to other uses as soon as this returns: wait, as hipFree
        // does, for whatever still reads it on any stream of the graph's device
        int current = -1;
        const bool other = g->device >= 0 && hipGetDevice(&current) == hipSuccess && current != g->device;
        if (other) (void)hipSetDevice(g->device);
        (void)hipDeviceSynchronize();
        if (other) (void)hipSetDevice(current);
    }
    (void)hipFree(g->ts_low);
    delete g;
}
