// Temporal neighbor finding on gfx950: one group of 16, 32 or 64 lanes of a
// wavefront per root (the smallest that holds the k slots, or the m candidates
// of the weighted policy).
//
// What is computed follows TASER (arXiv 2402.05396) Sec. 2.1 (temporal
// neighborhood, uniform / most-recent finders), Alg. 2 (pivot search, then one
// neighbor per slot) and the layer loop of Alg. 1 (kept neighbors become the
// next hop's roots; n of m candidates drawn by given probabilities).
//
// How it is computed differs from Alg. 2's block-per-root / single-thread
// binary search / shared-memory bitmap with atomic retry:
//   * the pivot is found by a cooperative 16-ary descent through a small index
//     of the timestamps: every level 16 lanes of a root read 16 neighboring
//     entries (one 128-byte line) and a ballot gives the child, so a 2^25-entry
//     list needs 7 dependent reads of one line each instead of 25 scattered ones;
//   * selection without replacement is a partial Fisher-Yates shuffle whose
//     random draws come from a counter-based generator keyed by
//     (seed, hop, root index, slot). No atomics, no retries: the result is a
//     pure function of the inputs, independent of scheduling;
//   * weighted selection keeps the candidate window in registers (one lane per
//     candidate) and uses integer prefix sums across the group's lanes;
//   * large hops of the most-recent finder search with four lanes per root and
//     hand out the slots of a wave's 16 roots flat (see quads_pay);
//   * the inverse-timespan finder, whose weights depend on the query time, sums
//     the whole valid list, by entries or by weights (see its kernel).
#include <mutex>

#include "gather_kernel.h"
#include "sampling_device.h"
#include "taser_internal.h"
#include "timespan_weight.h"

namespace {

// Number of entries in [lo, hi) with ts < t, for a time-sorted list [lo, hi) of the
// record array: the first position p* in [lo, hi] that is not "before", where
// before(p) = p < lo, or p < hi and ts[p] < t (monotone over the whole array).
// The search descends the levels of the time index. Entry i of level L stands for
// the positions [i 16^L, (i+1) 16^L) and holds the timestamp of the last of them;
// p* lies in the first entry whose last position is not before. A group starts at
// the lowest level at which its list touches at most 16 entries, then reads one
// aligned block of 16 entries (one 128-byte line) per level down to the records
// themselves (level 0). 16 lanes of the group probe; whether a position is below
// lo or at/after hi is known without reading it. Groups of one wave start at
// different levels under one wave-uniform loop. lo, hi, t are uniform inside a
// group; every lane of the wave must call this.
// R independent lists per group are searched side by side (their loads of a level are
// issued together): the kernel is bound by how many dependent reads are in flight.
// Positions are 32-bit: a graph has fewer than 2^31 entries, and the last position an index entry
// stands for, ((i + 1) << 4 L) - 1 with i < ceil(n / 16^L), stays below n + 16^L < 2^32.
template <int G, int R>
__device__ __forceinline__ void group_cutoff(const TaserRec* __restrict__ rec, const TaserTimeIndex& index,
                                             const uint32_t (&lo)[R], const uint32_t (&hi)[R], const int64_t (&t)[R],
                                             int group, int sub, uint32_t (&cnt)[R]) {
    const uint32_t n = (uint32_t)index.num_entries;
    int top[R];
    uint32_t at[R];   // entry of the current level that holds p*
#pragma unroll
    for (int r = 0; r < R; ++r) {
        // lowest level at which the list touches at most 16 entries: (hi >> 4 L) - (lo >> 4 L) is
        // floor((hi - lo) / 16^L) or one more, so it is the first L with hi - lo < 16^(L + 1), or the next
        const uint32_t d = hi[r] - lo[r];
        const int bits = d ? 32 - __clz((int)d) : 0;
        int L = bits ? (bits + 3) / 4 - 1 : 0;                          // <= 7 for d < 2^31
        if ((hi[r] >> (4 * L)) - (lo[r] >> (4 * L)) > 15u) ++L;         // never beyond 7: positions below 2^31 differ by < 8 there
        top[r] = L;
        at[r] = 0;
    }
#pragma unroll
    for (int L = kTimeIndexLevels; L >= 0; --L) {
        bool any = false;
#pragma unroll
        for (int r = 0; r < R; ++r) any |= L <= top[r];
        if (!__ballot(any)) continue;   // no list of this wave is at this level yet
        const uint32_t len = L == 0 ? n : (uint32_t)index.len[L - 1];
        uint32_t first[R], probe[R];
        bool known_before[R], read[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {   // what to read
            const bool active = L <= top[r];
            first[r] = at[r] * 16u;
            uint32_t width = 16;
            if (L == top[r]) {
                first[r] = lo[r] >> (4 * L);
                width = (hi[r] >> (4 * L)) - first[r] + 1u;
            }
            known_before[r] = false;
            read[r] = false;
            probe[r] = first[r] + (uint32_t)sub;
            if (active && (uint32_t)sub < width && probe[r] < len) {
                uint32_t pos = ((probe[r] + 1u) << (4 * L)) - 1u;       // last position the entry stands for
                if (pos >= n) pos = n - 1u;
                if (pos < lo[r]) known_before[r] = true;
                else if (pos < hi[r]) read[r] = true;
                if (L == 0) probe[r] = pos;
            }
        }
        int64_t ts[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {   // the reads of all lists, back to back
            ts[r] = 0;
            if (read[r]) ts[r] = L == 0 ? rec[probe[r]].ts : index.level[L - 1][probe[r]];
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const bool before = known_before[r] || (read[r] && ts[r] < t[r]);
            const uint32_t c = (uint32_t)__popcll(group_bits<G>(__ballot(before), group));   // before is monotone in the lane
            if (L <= top[r]) at[r] = first[r] + c;
        }
    }
    // `at` is p*, except past the array's last, partial entry, where it overshoots hi
#pragma unroll
    for (int r = 0; r < R; ++r) cnt[r] = (at[r] < hi[r] ? at[r] : hi[r]) - lo[r];
}

template <int G>
__device__ __forceinline__ int64_t group_cutoff(const TaserRec* __restrict__ rec, const TaserTimeIndex& index,
                                                int64_t lo, int64_t hi, int64_t t, int group, int sub) {
    const uint32_t lo1[1] = {(uint32_t)lo}, hi1[1] = {(uint32_t)hi};
    const int64_t t1[1] = {t};
    uint32_t cnt1[1];
    group_cutoff<G, 1>(rec, index, lo1, hi1, t1, group, sub, cnt1);
    return (int64_t)cnt1[0];
}

__device__ __forceinline__ void store_slot(int32_t* o_nbr, int32_t* o_eid, int64_t* o_ts,
                                           int64_t at, const TaserRec& r) {
    o_nbr[at] = r.nbr;
    o_eid[at] = r.eid;
    o_ts[at] = r.ts;
}

constexpr int kThreads = 256;

// Selection for the R roots of a group whose cutoffs are known. Leaves, in lane `sub` of the
// group, the record of output slot `sub` of every root (padding from slot `filled` on). Written in
// stages over all R roots, so that the loads of one stage (the last k records; the candidate window
// and then its weights; the uniformly drawn records) are in flight for all of them together, with
// the draws' arithmetic in between. Every lane of the wave must call it.
template <int POLICY, int G, int R>
__device__ __forceinline__ void select_slots(
    const TaserRec* __restrict__ rec, int64_t q0, const uint32_t (&lo)[R], const uint32_t (&cnt)[R], int group, int sub, int k,
    uint32_t seed_lo, uint32_t seed_hi, uint32_t hop, int m, const uint32_t* __restrict__ edge_weight,
    TaserRec (&out)[R], int (&filled)[R]) {
    const TaserRec pad = {0, -1, -1};

    // All lanes of the wave walk through the same code; what a group does not need is masked.
    if (POLICY == TASER_RECENT) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            filled[r] = (int)(cnt[r] < (uint32_t)k ? cnt[r] : (uint32_t)k);
            out[r] = pad;
            if (sub < filled[r]) out[r] = rec[lo[r] + cnt[r] - 1u - (uint32_t)sub];
        }
    } else if (POLICY == TASER_UNIFORM) {
        // cnt <= k: everything, most recent first. Otherwise a partial Fisher-Yates
        // over the virtual array a[x] = x, x in [0, cnt): step j draws pos_j in
        // [j, cnt), takes a[pos_j] and puts a[j] there; lane j of the group owns step j.
        uint32_t at[R];   // list position of this lane's slot
        bool some[R];     // false: padding
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const bool shuffle = cnt[r] > (uint32_t)k;
            filled[r] = shuffle ? k : (int)cnt[r];
            uint32_t pos = 0, val = 0, idx = 0;
            if (shuffle && sub < k) {
                const uint64_t u = draw64(seed_lo, seed_hi, hop, (uint64_t)(q0 + r), (uint32_t)sub);
                pos = (uint32_t)sub + mulhi_64x32(u, cnt[r] - (uint32_t)sub);
            }
            if (__ballot(shuffle)) {
                if (G <= 32) {
                    // Every lane resolves its own step from the positions all steps drew (no values
                    // need to travel): a[x] at step j is x unless an earlier step wrote x; the latest
                    // such step i put there what position i held at step i, which is the same question
                    // for (i, i). Chains are short: one pass when no two steps of a root collide.
                    uint32_t drawn[G];
#pragma unroll
                    for (int i = 0; i < G; ++i) drawn[i] = group_get<G>(pos, i);
                    uint32_t x = pos;
                    int before = sub;                       // only steps below this one count
                    bool open = shuffle && sub < k;
                    while (__ballot(open)) {
                        int found = -1;
#pragma unroll
                        for (int i = 0; i < G; ++i)
                            if (i < before && drawn[i] == x) found = i;   // ascending: the latest match stays
                        if (open) {
                            if (found < 0) {
                                open = false;
                            } else {
                                x = (uint32_t)found;
                                before = found;
                            }
                        }
                    }
                    idx = x;
                } else {
                    // lane j of the group owns step j; it remembers the position it overwrote (pos) and
                    // the value it put there (val); a lookup of a[x] at step j is the val of the latest
                    // earlier step that wrote x, else x itself
                    for (int j = 0; j < k; ++j) {
                        const uint32_t x = group_get<G>(pos, j);
                        const bool earlier = sub < j;
                        const uint64_t hit_x = group_bits<G>(__ballot(earlier && pos == x), group);
                        const uint64_t hit_j = group_bits<G>(__ballot(earlier && pos == (uint32_t)j), group);
                        // the shuffles are executed by every lane; lanes without a hit read lane 0 and drop it
                        const uint32_t v_x = group_get<G>(val, hit_x ? 63 - __clzll((long long)hit_x) : 0);
                        const uint32_t v_j = group_get<G>(val, hit_j ? 63 - __clzll((long long)hit_j) : 0);
                        if (sub == j) {
                            idx = hit_x ? v_x : x;
                            val = hit_j ? v_j : (uint32_t)j;
                        }
                    }
                }
            }
            at[r] = 0;
            some[r] = false;
            if (sub < k) {
                if (shuffle) {
                    at[r] = idx;
                    some[r] = true;
                } else if (sub < filled[r]) {
                    at[r] = cnt[r] - 1u - (uint32_t)sub;
                    some[r] = true;
                }
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            out[r] = pad;
            if (some[r]) out[r] = rec[lo[r] + at[r]];
        }
    } else {
        // Candidate window: lane i of the group holds candidate i (the i-th most recent);
        // lane j notes which candidate draw j picked and fetches it from that lane at the end.
        TaserRec mine[R];
        uint32_t w[R];
        int c[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            c[r] = (int)(cnt[r] < (uint32_t)m ? cnt[r] : (uint32_t)m);
            mine[r] = pad;
            if (sub < c[r]) mine[r] = rec[lo[r] + cnt[r] - 1u - (uint32_t)sub];
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            w[r] = 0;
            if (sub < c[r]) w[r] = edge_weight[mine[r].eid];
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const bool draw = c[r] > k;
            filled[r] = draw ? k : c[r];
            int my_pick = (!draw && sub < c[r]) ? sub : -1;
            if (__ballot(draw)) {
                uint64_t u = 0;
                if (draw && sub < k) u = draw64_wide(seed_lo, seed_hi, hop, (uint64_t)(q0 + r), (uint32_t)sub);
                const int pick = group_weighted_picks<G>(w[r], u, k, draw, group, sub);
                if (draw) my_pick = pick;
            }
            const int from = my_pick < 0 ? 0 : my_pick;   // the shuffles are executed by every lane
            const int32_t p_nbr = (int32_t)group_get<G>((uint32_t)mine[r].nbr, from);
            const int32_t p_eid = (int32_t)group_get<G>((uint32_t)mine[r].eid, from);
            const int64_t p_ts = (int64_t)group_get64<G>((uint64_t)mine[r].ts, from);
            out[r] = pad;
            if (my_pick >= 0 && sub < k) out[r] = TaserRec{p_ts, p_nbr, p_eid};
        }
    }
}

// What a hop kernel needs to also write the feature rows of the edges it sampled
// (Sec. 3.4 slices them right after Alg. 2 found the neighbors): the table, and the dense
// output of this hop, one row per slot in slot order. The launcher guarantees: row_bytes a
// multiple of 4 and >= 16, table and pitch 4-byte aligned, `out` 16-byte aligned, and the
// rows of one wavefront's roots a multiple of 16 bytes.
struct RowCopy {
    const uint8_t* table;
    int64_t table_rows, pitch_bytes;
    uint8_t* out;
    const uint8_t* zeros;    // 16 zero bytes
    uint32_t row_bytes;
    uint32_t magic;          // ceil(2^32 / row_bytes)
    uint32_t step_rows, step_rest;   // 1024 = step_rows * row_bytes + step_rest
};

// The rows of one wavefront's roots form one contiguous, 16-byte aligned range of the
// output: `rows_here` rows whose edge ids the wave has just left in `wave_eid` (LDS, slot
// order). The range is copied as a flat stream, 16 bytes per lane and 1 KiB per wave
// instruction, kInFlight of them in flight; a lane finds the row of its first chunk by one
// division and of the following ones by stepping. A chunk inside one row is one 16-byte
// load (4-byte aligned); one that crosses a row end takes two. Padding slots and ids
// outside the table give zero rows.
template <int kInFlight>
__device__ __forceinline__ void copy_wave_rows(const RowCopy& rc, const int32_t* wave_eid, uint32_t rows_here,
                                               int64_t first_row, int lane) {
    using namespace taser_gather;
    const uint32_t bytes_here = rows_here * rc.row_bytes;
    uint8_t* const out = rc.out + first_row * (int64_t)rc.row_bytes;
    uint32_t o = (uint32_t)lane * 16u;
    uint32_t row = __umulhi(o, rc.magic);
    uint32_t off = o - row * rc.row_bytes;
    for (uint32_t base = 0; base < bytes_here; base += kInFlight * 1024u) {
        uint32_t c_o[kInFlight], c_row[kInFlight], c_off[kInFlight];
        bool whole[kInFlight], cross[kInFlight];
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) {
            c_o[u] = o;
            c_row[u] = row;
            c_off[u] = off;
            const bool live = o < bytes_here;
            whole[u] = live && off + 16u <= rc.row_bytes;
            cross[u] = live && !whole[u];
            o += 1024u;
            row += rc.step_rows;
            off += rc.step_rest;
            if (off >= rc.row_bytes) {
                off -= rc.row_bytes;
                ++row;
            }
        }
        u32x4 vals[kInFlight], tail[kInFlight], head[kInFlight];
        uint32_t keep[kInFlight];   // dwords of a crossing chunk that belong to the row it starts in (1..3)
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) {
            const uint32_t r = c_row[u] < rows_here ? c_row[u] : rows_here - 1u;
            const int32_t id = wave_eid[r];
            const bool ok = id >= 0 && id < rc.table_rows;
            const uint8_t* src = rc.table + (int64_t)(ok ? id : 0) * rc.pitch_bytes;
            vals[u] = ((GlobalChunk16Ptr)(whole[u] && ok ? src + c_off[u] : rc.zeros))->v;
            // A chunk that crosses a row end is the last dwords of this row followed by the first of
            // the next one (rows hold at least 16 bytes): the last 16 bytes of the one and the first
            // 16 of the other, read by the crossing lanes only and put together below.
            keep[u] = (rc.row_bytes - c_off[u]) >> 2;
            tail[u] = head[u] = u32x4{0u, 0u, 0u, 0u};
            if (cross[u]) {
                const int32_t id1 = r + 1u < rows_here ? wave_eid[r + 1u] : -1;   // past the range: never stored
                const bool ok1 = id1 >= 0 && id1 < rc.table_rows;
                tail[u] = ((GlobalChunk16Ptr)(ok ? src + (rc.row_bytes - 16u) : rc.zeros))->v;
                head[u] = ((GlobalChunk16Ptr)(ok1 ? rc.table + (int64_t)id1 * rc.pitch_bytes : rc.zeros))->v;
            }
        }
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) {
            // dwords 4 - keep .. 7 - keep of (tail, head), by selects in every lane
            const u32x4 t = tail[u], h = head[u];
            const bool k1 = keep[u] == 1u, k2 = keep[u] == 2u;
            const uint32_t d0 = k1 ? t.w : k2 ? t.z : t.y;
            const uint32_t d1 = k1 ? h.x : k2 ? t.w : t.z;
            const uint32_t d2 = k1 ? h.y : k2 ? h.x : t.w;
            const uint32_t d3 = k1 ? h.z : k2 ? h.y : h.x;
            if (cross[u]) vals[u] = u32x4{d0, d1, d2, d3};
        }
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) {
            if (c_o[u] + 16u <= bytes_here) {
                __builtin_nontemporal_store(vals[u], reinterpret_cast<u32x4*>(out + c_o[u]));
            } else if (c_o[u] < bytes_here) {
                const uint32_t w[4] = {vals[u].x, vals[u].y, vals[u].z, vals[u].w};
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (c_o[u] + 4u * i < bytes_here) *reinterpret_cast<uint32_t*>(out + c_o[u] + 4u * i) = w[i];
            }
        }
    }
}

// G lanes per root: G >= k, and G >= m for the weighted policy. A group serves kRootsPerGroup
// consecutive roots: their searches run side by side, their selections stage by stage. Two pay for
// the most-recent finder on large hops that the kernel below does not take (lists of two entries, 32
// slots, 160 000 roots: 26.2 us with one, 21.8 with two); the uniform and weighted finders, whose time
// is mostly the arithmetic of their draws, gain nothing from them.
// With ROWS (one root per group; how many wave instructions of the copy are in flight) a wavefront then also copies
// the table rows of the edges it sampled into the hop's dense row output: the finder is bound by instruction issue and
// dependent reads, the copy by memory bandwidth, and in one kernel the wavefronts of a
// compute unit that search overlap with those that copy.
template <int POLICY, int G, int kRootsPerGroup, int ROWS>
__global__ __launch_bounds__(kThreads) void sample_hop_kernel(
    const int64_t* __restrict__ indptr, const TaserRec* __restrict__ rec, const TaserTimeIndex index,
    const int32_t* __restrict__ roots, const int64_t* __restrict__ times, int64_t num_roots,
    int32_t num_nodes, int k, uint32_t seed_lo, uint32_t seed_hi, uint32_t hop, int m, const uint32_t* __restrict__ edge_weight,
    int32_t* __restrict__ o_nbr, int32_t* __restrict__ o_eid, int64_t* __restrict__ o_ts,
    int32_t* __restrict__ o_count, const RowCopy rows) {
    static_assert(!ROWS || kRootsPerGroup == 1, "the row copy takes one root per group");
    constexpr int kGroups = kWave / G;                         // groups per wave
    const int lane = threadIdx.x & (kWave - 1);
    const int group = lane / G, sub = lane % G;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t wave_q0 = ((int64_t)blockIdx.x * (kThreads / kWave) + wave) * (kGroups * kRootsPerGroup);   // first root of the wave
    const int64_t q0 = wave_q0 + group * kRootsPerGroup;

    uint32_t lo[kRootsPerGroup], hi[kRootsPerGroup], cnt[kRootsPerGroup];   // positions fit 32 bits: fewer than 2^31 entries
    int64_t t[kRootsPerGroup];
    int32_t v[kRootsPerGroup];
#pragma unroll
    for (int r = 0; r < kRootsPerGroup; ++r) {
        lo[r] = hi[r] = 0;
        t[r] = 0;
        v[r] = q0 + r < num_roots ? roots[q0 + r] : -1;
    }
#pragma unroll
    for (int r = 0; r < kRootsPerGroup; ++r) {
        if (v[r] >= 0 && v[r] < num_nodes) {   // anything else is a root without neighbors
            t[r] = times[q0 + r];
            lo[r] = (uint32_t)indptr[v[r]];
            hi[r] = (uint32_t)indptr[v[r] + 1];
        }
    }
    group_cutoff<G, kRootsPerGroup>(rec, index, lo, hi, t, group, sub, cnt);   // 0 for dead roots (lo == hi)
    TaserRec slot[kRootsPerGroup];
    int filled[kRootsPerGroup];
    select_slots<POLICY, G, kRootsPerGroup>(rec, q0, lo, cnt, group, sub, k, seed_lo, seed_hi, hop, m, edge_weight, slot, filled);
#pragma unroll
    for (int r = 0; r < kRootsPerGroup; ++r) {
        if (q0 + r < num_roots) {
            if (sub < k) store_slot(o_nbr, o_eid, o_ts, (q0 + r) * k + sub, slot[r]);
            if (sub == 0) o_count[q0 + r] = filled[r];
        }
    }
    if constexpr (ROWS > 0) {
        __shared__ int32_t eid_of_row[kThreads / kWave][kWave];   // per wave: k ids per group, slot order (kGroups * k <= 64)
        if (sub < k) eid_of_row[wave][group * k + sub] = slot[0].eid;
        // only this wave reads them back: its LDS operations complete in order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        int64_t roots_here = num_roots - wave_q0;
        if (roots_here > kGroups) roots_here = kGroups;
        if (roots_here > 0) copy_wave_rows<ROWS>(rows, eid_of_row[wave], (uint32_t)roots_here * (uint32_t)k, wave_q0 * k, lane);
    }
}

// ---- inverse-timespan finder -------------------------------------------------
// Weight of an entry at time ts for a query at t > ts: max(1, floor(2^32 / delta)), delta = t - ts.
// Entries with delta >= 2^32 weigh 1 and are the first `ones` of a list; of the others the low words of
// the timestamps say all: delta = (low word of t) - (low word of ts), in 32 bits.
template <bool NEAR> __device__ __forceinline__ uint32_t quotient_of_delta(uint32_t delta) {
    return quotient_by_reciprocal<NEAR>(delta, __builtin_amdgcn_rcpf((float)delta));
}
__device__ __forceinline__ uint64_t weight_of_delta(uint32_t delta) { return weight_by_reciprocal(delta, __builtin_amdgcn_rcpf((float)delta)); }

constexpr int kMaxTiles = 16 * kWave;             // tile sums of a block, divided among its roots
constexpr int kSamples = 512;                     // of a far part, per root
constexpr int kListThreads = 256;                 // block of the finder that reads whole lists
constexpr int kListWaves = kListThreads / kWave;

// What is known about a root. Its valid entries are cut into up to three parts: the entries 2^32 and more before the
// query, [0, far_begin), where they are many, which all weigh 1; a far part, [far_begin, first), whose weights are
// below w_end; and a near part, [first, cnt). The first part is one tile that is never read: its sum is its number of
// entries. The far part is described by its weights: the entries of weight w are one run of the list, found by a search,
// so that a lane's work is a weight and not an entry. The near part is read entry by entry, in rows of 64.
struct ListQuery {
    uint32_t lo, cnt;            // its list begins at record lo; cnt valid entries
    uint32_t ones;               // entries [0, ones) are 2^32 or more before the query
    uint32_t t_low;              // low word of the query time
    uint32_t far_begin;          // first entry of the far part: `ones` where they are a tile of their own, else 0
    uint32_t first;              // first entry of the near part
    uint32_t tile_shift;         // near part: log2 of the rows of a tile
    uint32_t stride;             // far part: entries between two samples
    uint32_t together;           // 1: its tiles are summed by all wavefronts of the block, 0: by its own
    uint32_t w_first, w_end;     // far part: weight of its first entry, and the first weight of the near part
    uint32_t batches;            // batches of kBatch weights per far tile
    uint32_t far_tiles, tiles;   // tiles before the near part's, the one of the `ones` included, and all of them
    uint32_t k;                  // the call's
    uint32_t near;               // every delta of the near part is below 2^24 (then none of it is among the `ones`)
    __device__ uint32_t ones_tiles() const { return far_begin ? 1u : 0u; }   // tile 0 is the entries before far_begin
};
struct __attribute__((packed, aligned(4))) Low4 {
    uint32_t w[4];
};
constexpr uint32_t kBatch = kWave - 1;   // weights of a far batch: the last lane only says where the last run ends

// A query as the whole wave read it from LDS, in scalar registers.
__device__ __forceinline__ ListQuery uniform(const ListQuery& v) {
    auto get = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); };
    return ListQuery{get(v.lo), get(v.cnt), get(v.ones), get(v.t_low), get(v.far_begin), get(v.first), get(v.tile_shift), get(v.stride), get(v.together),
                     get(v.w_first), get(v.w_end),
                     get(v.batches), get(v.far_tiles), get(v.tiles), get(v.k), get(v.near)};
}

// delta of entry p (its low word loaded as `low`), 0xFFFFFFFF (weight 1) for the first `ones`.
template <bool NEAR> __device__ __forceinline__ uint32_t delta_of(const ListQuery& q, uint32_t p, uint32_t low) {
    return !NEAR && p < q.ones ? 0xFFFFFFFFu : q.t_low - low;
}

// The sums over the wave of eight 32-bit values per lane, value l % 8 in lane l: three exchanges in which a lane
// keeps half of its values and adds the other lane's half of the same ones, then the eighths of the wave.
__device__ __forceinline__ uint32_t wave_sums_of_8(const uint32_t (&a)[8], int lane) {
    const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4;
    uint32_t b[4], c[2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        b[i] = (b0 ? a[2 * i + 1] : a[2 * i]) +
               (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(b0 ? a[2 * i] : a[2 * i + 1]), 0xB1, 0xf, 0xf, true);   // quad_perm [1, 0, 3, 2]
#pragma unroll
    for (int i = 0; i < 2; ++i)
        c[i] = (b1 ? b[2 * i + 1] : b[2 * i]) +
               (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(b1 ? b[2 * i] : b[2 * i + 1]), 0x4E, 0xf, 0xf, true);   // quad_perm [2, 3, 0, 1]
    const int give = (int)(b2 ? c[0] : c[1]);
    int got = __builtin_amdgcn_update_dpp(0, give, 0x104, 0xf, 0x5, false);   // row_shl:4 into the banks below,
    got = __builtin_amdgcn_update_dpp(got, give, 0x114, 0xf, 0xA, false);     // row_shr:4 into those above
    uint32_t d = (b2 ? c[1] : c[0]) + (uint32_t)got;
    d += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)d, 0x128, 0xf, 0xf, true);   // row_ror:8
    d += __shfl_xor(d, 16, kWave);
    d += __shfl_xor(d, 32, kWave);
    return d;
}
// The same, added up over every 2^shift (at most 8) neighboring values: correct in lanes whose low `shift` bits are 0.
__device__ __forceinline__ uint64_t tile_sums_of_8(const uint32_t (&a)[8], uint32_t shift, int lane) {
    uint64_t s = wave_sums_of_8(a, lane);
    for (uint32_t i = 0; i < shift; ++i) s += __shfl_xor(s, 1 << i, kWave);
    return s;
}

// A row whose deltas are this large has a sum below 2^32.
constexpr uint32_t kRowSumDelta = 128;
static_assert((((uint64_t)1 << 32) / kRowSumDelta) * kWave < ((uint64_t)1 << 32), "a row's sum");

// Sums of the near part's tiles, by units of kGroup rows (or of one tile, where that is more): units
// first, first + step, ... The rows of a group are loaded together.
constexpr uint32_t kGroup = 8;
template <bool NEAR>
__device__ __forceinline__ void sum_near_tiles(const ListQuery& q, const uint32_t* __restrict__ low, uint32_t first, uint32_t step,
                                               uint64_t* tile_sum, int lane) {
    const uint32_t rows = (q.cnt - q.first + kWave - 1) / kWave, per = 1u << q.tile_shift;
    const uint32_t unit = per < kGroup ? kGroup : per;
    for (uint32_t u0 = first * unit; u0 < rows; u0 += step * unit) {
        uint64_t sum = 0;        // of a tile of more than a group
        const uint32_t u1 = u0 + unit < rows ? u0 + unit : rows;
        for (uint32_t r = u0; r < u1; r += kGroup) {
            const uint32_t p0 = q.first + r * kWave;
            uint32_t v[kGroup];
            const bool whole = p0 + kGroup * kWave <= q.cnt;
            if (whole) {
                const uint32_t* at = low + p0 + (uint32_t)lane;
#pragma unroll
                for (uint32_t i = 0; i < kGroup; ++i) v[i] = at[i * kWave];
            } else {
#pragma unroll
                for (uint32_t i = 0; i < kGroup; ++i) {
                    const uint32_t p = p0 + i * kWave + (uint32_t)lane;
                    v[i] = r + i < u1 ? low[p < q.cnt ? p : q.cnt - 1u] : 0u;   // (uniform) a row that there is
                }
            }
            // (uniform) the last deltas are the smallest; half rows and rows with sums beyond 32 bits take the last path
            const uint32_t least = delta_of<NEAR>(q, p0 + (kGroup - 1) * kWave + (uint32_t)lane, v[kGroup - 1]);
            bool split = false;
            uint32_t high[kGroup];       // of a weight, above its low 16 bits
            if (whole && !__ballot(least <= kLastLargeDelta)) {
#pragma unroll
                for (uint32_t i = 0; i < kGroup; ++i) v[i] = quotient_of_delta<NEAR>(delta_of<NEAR>(q, p0 + i * kWave + (uint32_t)lane, v[i]));
            } else if (whole && !__ballot(least < kRowSumDelta)) {
#pragma unroll
                for (uint32_t i = 0; i < kGroup; ++i) v[i] = (uint32_t)weight_of_delta(delta_of<NEAR>(q, p0 + i * kWave + (uint32_t)lane, v[i]));
            } else {
#pragma unroll
                for (uint32_t i = 0; i < kGroup; ++i) {
                    uint32_t w_low = 0, w_high = 0;
                    if (r + i < u1) {    // uniform, like the next
                        const uint32_t p = p0 + i * kWave + (uint32_t)lane, delta = delta_of<NEAR>(q, p, v[i]);
                        const bool valid = p < q.cnt;
                        if (__ballot(valid && delta <= kLastLargeDelta)) {
                            split = true;
                            const uint64_t w = weight_of_delta(delta);
                            w_low = valid ? (uint32_t)w & 0xffffu : 0u;
                            w_high = valid ? (uint32_t)(w >> 16) : 0u;
                        } else {
                            const uint32_t w = quotient_of_delta<NEAR>(delta);
                            w_low = valid ? w : 0u;
                        }
                    }
                    v[i] = w_low;
                    high[i] = w_high;
                }
            }
            if (per <= kGroup) {         // whole tiles: rows' sums in the lanes, then the tiles'
                uint64_t s = tile_sums_of_8(v, q.tile_shift, lane);
                if (split) s += tile_sums_of_8(high, q.tile_shift, lane) << 16;
                if ((uint32_t)lane < u1 - r && (uint32_t)lane < kGroup && ((uint32_t)lane & (per - 1u)) == 0)
                    tile_sum[q.far_tiles + ((r + (uint32_t)lane) >> q.tile_shift)] = s;
            } else {
                uint64_t s = 0;          // eight weights below 2^26 each: 64 lanes of them do not fit 32 bits
                uint32_t lane_sum = 0;
#pragma unroll
                for (uint32_t i = 0; i < kGroup; ++i) lane_sum += v[i];
                s = (uint64_t)wave_sum32(lane_sum & 0xffffu) + ((uint64_t)wave_sum32(lane_sum >> 16) << 16);
                if (split) {
                    uint32_t h = 0;      // 8 x 2^17 per lane
#pragma unroll
                    for (uint32_t i = 0; i < kGroup; ++i) h += high[i];
                    s += (uint64_t)wave_sum32(h) << 16;
                }
                sum += s;
            }
        }
        if (per > kGroup && lane == 0) tile_sum[q.far_tiles + (u0 >> q.tile_shift)] = sum;
    }
}

// Row r of the near part, entries picked by the draws before number j left out (lane e of my_pick: draw e's
// entry): finds the first entry whose running sum, `before` it included, exceeds x.
// Returns its lane and its weight, or -1 and adds the row's sum to `before`.
__device__ __forceinline__ int pick_in_row(const ListQuery& q, uint32_t low, uint32_t r, uint64_t x, uint64_t& before, int j,
                                           uint32_t my_pick, int lane, uint64_t& pick_w) {
    const uint32_t p0 = q.first + r * kWave, p = p0 + lane;
    const uint32_t delta = delta_of<false>(q, p, low);
    bool valid = p < q.cnt;
    for (uint64_t taken = __ballot(lane < j && my_pick - p0 < (uint32_t)kWave); taken; taken &= taken - 1) {
        const uint32_t gone = (uint32_t)__builtin_amdgcn_readlane((int)my_pick, __ffsll((long long)taken) - 1);
        if (p == gone) valid = false;
    }
    const uint64_t rest = x - before;                        // x >= before
    if (!__ballot(delta < kRowSumDelta)) {                   // (uniform)
        const uint32_t w = valid ? (uint32_t)weight_of_delta(delta) : 0u;
        const uint32_t inc = wave_inclusive_scan32(w);
        const uint64_t hit = __ballot((uint64_t)inc > rest);
        if (hit) {
            const int first = __ffsll((long long)hit) - 1;
            pick_w = (uint32_t)__builtin_amdgcn_readlane((int)w, first);
            return first;
        }
        before += (uint32_t)__builtin_amdgcn_readlane((int)inc, kWave - 1);
    } else {
        const uint64_t w = valid ? weight_of_delta(delta) : 0u;
        const uint64_t inc = wave_inclusive_scan64(w);
        const uint64_t hit = __ballot(inc > rest);
        if (hit) {
            const int first = __ffsll((long long)hit) - 1;
            pick_w = wave_get64(w, first);
            return first;
        }
        before += wave_get64(inc, kWave - 1);
    }
    return -1;
}

// Far part: where the entries of weight w and more begin, that is how many entries have a delta above
// floor(2^32 / w). w_first is the weight of the part's first entry. The samples (the deltas of every stride-th entry, in LDS) say between
// which two, the list itself the rest: three probes a step, sixteen neighbors in the last. Probes behind the far
// part read an entry of the near part or the list's last one, which is not above unless the whole list is.
__device__ __forceinline__ uint32_t run_begin(const ListQuery& q, const uint32_t* __restrict__ low, const uint32_t* sample, uint32_t w) {
    const uint32_t most = (uint32_t)weight_of_delta(w < 2u ? 2u : w < kLastLargeDelta ? w : kLastLargeDelta);   // floor(2^32 / w)
    uint32_t at = 0;
#pragma unroll
    for (uint32_t half = kSamples / 2; half > 0; half /= 2)
        if (sample[at + half - 1u] > most) at += half;
    at = q.ones + at * q.stride;             // one sample is left out: the last one stands for the end of the far part
    for (uint32_t len = q.stride; len > 16u;) {
        const uint32_t part = (len + 3u) / 4u;
        uint32_t v[3];
#pragma unroll
        for (uint32_t i = 0; i < 3; ++i) {
            const uint32_t p = at + (i + 1u) * part - 1u;
            v[i] = low[p < q.cnt ? p : q.cnt - 1u];
        }
        uint32_t c = 0;
#pragma unroll
        for (uint32_t i = 0; i < 3; ++i) c += q.t_low - v[i] > most ? 1u : 0u;
        at += c * part;
        len = part;
    }
    if (at > q.cnt - 16u) at = q.cnt - 16u;  // (a list with a far part has kFarEntries entries and more)
    const Low4* p = reinterpret_cast<const Low4*>(low + at);
    Low4 v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = p[i];
    uint32_t d[16];                          // the neighbors, halved in registers
#pragma unroll
    for (int i = 0; i < 16; ++i) d[i] = v[i / 4].w[i % 4];
    uint32_t c = 0;
#pragma unroll
    for (int half = 8; half > 0; half /= 2) {
        const uint32_t upper = q.t_low - d[half - 1] > most ? 0xFFFFFFFFu : 0u;   // a mask, or the selects become searches for an index
        c += upper & (uint32_t)half;
#pragma unroll
        for (int i = 0; i < half; ++i) d[i] = (upper & d[half + i]) | (~upper & d[i]);
    }
    at += c + (q.t_low - d[0] > most ? 1u : 0u);
    return w <= q.w_first ? q.far_begin : w >= q.w_end || at > q.first ? q.first : at;
}

// The runs of one batch of a far tile: lane l < kBatch has the entries [begin, end) of weight w.
struct Runs {
    uint32_t w, begin, end;
};
__device__ __forceinline__ Runs far_runs(const ListQuery& q, const uint32_t* __restrict__ low, const uint32_t* sample, uint32_t batch, int lane) {
    Runs r;
    r.w = q.w_first + batch * kBatch + (uint32_t)lane;
    r.begin = run_begin(q, low, sample, r.w);
    r.end = __shfl_down(r.begin, 1, kWave);
    if (lane == kWave - 1) r.end = r.begin;
    return r;
}

__device__ __forceinline__ uint64_t far_tile_weight(const ListQuery& q, const uint32_t* __restrict__ low, const uint32_t* sample, uint32_t tile, int lane) {
    if (tile < q.ones_tiles()) return q.far_begin;
    tile -= q.ones_tiles();
    uint64_t s = 0;
    #pragma unroll 1
    for (uint32_t b = tile * q.batches; b < (tile + 1u) * q.batches; ++b) {
        const Runs r = far_runs(q, low, sample, b, lane);
        s += (uint64_t)(r.end - r.begin) * r.w;
    }
    return wave_sum64(s);
}

// Entry number nth of a run that begins at `begin`, entries picked by the draws before number j left out.
__device__ __forceinline__ uint32_t pick_in_run(uint32_t begin, uint32_t nth, int j, uint32_t my_pick, int lane) {
    uint32_t pick = begin + nth;
    for (;;) {   // ends: pick only grows, and is at most begin + nth + j
        const uint32_t skipped = (uint32_t)__popcll(__ballot(lane < j && my_pick >= begin && my_pick <= pick));
        if (begin + nth + skipped == pick) return pick;
        pick = begin + nth + skipped;
    }
}

// As pick_in_row, for a whole far tile: returns the entry.
__device__ __forceinline__ uint32_t pick_in_far_tile(const ListQuery& q, const uint32_t* __restrict__ low, const uint32_t* sample, uint32_t tile,
                                                     uint64_t x, uint64_t before, int j, uint32_t my_pick, int lane, uint64_t& pick_w) {
    if (tile < q.ones_tiles()) {   // (tile 0, before which there is nothing)
        pick_w = 1;
        return pick_in_run(0u, (uint32_t)x, j, my_pick, lane);
    }
    tile -= q.ones_tiles();
    #pragma unroll 1
    for (uint32_t b = tile * q.batches; b < (tile + 1u) * q.batches; ++b) {
        const Runs r = far_runs(q, low, sample, b, lane);
        uint32_t left = r.end - r.begin;
        const uint32_t b0 = (uint32_t)__builtin_amdgcn_readlane((int)r.begin, 0), b1 = (uint32_t)__builtin_amdgcn_readlane((int)r.begin, kWave - 1);
        for (uint64_t taken = __ballot(lane < j && my_pick >= b0 && my_pick < b1); taken; taken &= taken - 1) {
            const uint32_t gone = (uint32_t)__builtin_amdgcn_readlane((int)my_pick, __ffsll((long long)taken) - 1);
            if (gone >= r.begin && gone < r.end) --left;
        }
        const uint64_t inc = wave_inclusive_scan64((uint64_t)left * r.w);
        const uint64_t hit = __ballot(inc > x - before);
        if (hit) {
            const int at = __ffsll((long long)hit) - 1;
            const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)r.w, at);
            const uint32_t begin = (uint32_t)__builtin_amdgcn_readlane((int)r.begin, at);
            const uint64_t rest = x - before - (at ? wave_get64(inc, at - 1) : 0);
            const uint32_t nth = (rest >> 32) ? (uint32_t)(rest / w) : (uint32_t)rest / w;   // of the run's entries that are left
            pick_w = w;
            return pick_in_run(begin, nth, j, my_pick, lane);
        }
        before += wave_get64(inc, kWave - 1);
    }
    return q.cnt - 1u;   // (never while the sums are consistent)
}

// The k successive draws of one root, by one wavefront. The tile sums become running sums within groups of
// 64 tiles (in LDS, where the sums were) and over the groups (group g's in lane g): a draw compares x with
// both, re-reads only the tile it lands in, and the pick's weight leaves every running sum from its tile on,
// which is what summing the remaining weights again would give. Lane j returns draw j's entry.
__device__ __forceinline__ uint32_t draw_entries(const ListQuery& q, const uint32_t* __restrict__ low, const uint32_t* sample, uint64_t* tile_sum,
                                                 uint64_t u, int lane) {
    const uint32_t rows = (q.cnt - q.first + kWave - 1) / kWave;
    const int groups = (int)((q.tiles + kWave - 1) / kWave);
    uint64_t group_run = 0, total = 0;
#pragma unroll 1
    for (int g = 0; g < groups; ++g) {
        const uint32_t tile = (uint32_t)(g * kWave + lane);
        const uint64_t inc = wave_inclusive_scan64(tile < q.tiles ? tile_sum[tile] : 0);
        tile_sum[tile] = inc;               // (every root has a multiple of kWave)
        total += wave_get64(inc, kWave - 1);
        if (lane >= g) group_run = total;   // lane g: the sum of the groups up to g; beyond the last one: all
    }
    uint32_t my_pick = 0;
#pragma unroll 1
    for (int j = 0; j < (int)q.k; ++j) {
        const uint64_t x = __umul64hi(wave_get64(u, j), total);
        // the tile whose running sum first exceeds x, and the sum before it. There always is one while the sums
        // are consistent (x < total); the last lane or tile otherwise, which keeps the reads in bounds.
        const uint64_t in_group = __ballot(group_run > x);
        int g = in_group ? __ffsll((long long)in_group) - 1 : groups - 1;
        if (g > groups - 1) g = groups - 1;
        uint64_t before = g > 0 ? wave_get64(group_run, g - 1) : 0;
        own_lds_ready();
        uint64_t run = tile_sum[g * kWave + lane];
        const uint64_t in_tile = __ballot(run > x - before);
        const int t = in_tile ? __ffsll((long long)in_tile) - 1 : kWave - 1;
        if (t > 0) before += wave_get64(run, t - 1);
        uint32_t tile = (uint32_t)(g * kWave + t);
        if (tile > q.tiles - 1u) tile = q.tiles - 1u;
        uint32_t pick = q.cnt - 1u;     // same remark
        uint64_t pick_w = 0;
        if (tile < q.far_tiles) {
            pick = pick_in_far_tile(q, low, sample, tile, x, before, j, my_pick, lane, pick_w);
        } else {   // inside the tile, row by row
            const uint32_t r0 = (tile - q.far_tiles) << q.tile_shift, end = r0 + (1u << q.tile_shift), r1 = end < rows ? end : rows;
            for (uint32_t r = r0; r < r1; ++r) {
                const uint32_t p = q.first + r * kWave + (uint32_t)lane;
                const int at = pick_in_row(q, low[p < q.cnt ? p : q.cnt - 1u], r, x, before, j, my_pick, lane, pick_w);
                if (at >= 0) {
                    pick = q.first + r * kWave + (uint32_t)at;
                    break;
                }
            }
        }
        if (lane == j) my_pick = pick;
        total -= pick_w;
        if (lane >= g) group_run -= pick_w;
        if (lane >= t) tile_sum[g * kWave + lane] = run - pick_w;
    }
    return my_pick;
}

// Sums of a wave's share of the tiles.
__device__ __forceinline__ void sum_tiles(const ListQuery& q, const uint32_t* __restrict__ ts_low, const uint32_t* sample, uint32_t first,
                                          uint32_t step, uint64_t* tile_sum, int lane) {
    const uint32_t* low = ts_low + q.lo;
    for (uint32_t tile = first; tile < q.far_tiles; tile += step) {
        const uint64_t s = far_tile_weight(q, low, sample, tile, lane);
        if (lane == 0) tile_sum[tile] = s;
    }
    if (q.near) sum_near_tiles<true>(q, low, first, step, tile_sum, lane);
    else sum_near_tiles<false>(q, low, first, step, tile_sum, lane);
}

// Entries per weight from which a list is described by its weights: a batch of 63 weights costs about 180 vector
// instructions, a row of 64 entries 16 (8, 12, 16 entries: 248, 245, 247 us for 40 000 roots over lists of 13 000
// entries). Entries per draw: a draw from the far part finds its tile's runs again, some 250 instructions more than one that
// reads a row or two. 4 000 roots over lists of 10 000 entries, timestamps within 2^31 ticks, 10 / 25 / 64 draws: without this
// term 44 80 212 us, with 150 entries per draw 44 80 143, 300 44 77 143, 1 200 45 76 143; lists of 25 000 entries, 25 draws
// within 2^26 ticks 86 85 84 95. kFarEntries: with fewer there is no far part.
constexpr float kRunEntries = 12.0f, kDrawEntries = 300.0f;
constexpr uint32_t kFarEntries = 1024 + (uint32_t)(kRunEntries + kDrawEntries);
// Entries 2^32 and more before the query from which they are a tile of their own: a row of them. Read like any others, a list
// of a million entries of which 50 are younger took 0.39 ms for 200 roots, so 0.010; 4 000 roots over lists of 1 000 entries,
// 1 % of them younger, ten draws 28.9 us, so 20.0 (with a line at 256 entries the same, at 1 024 28.9).
constexpr uint32_t kManyOnes = 64;
constexpr uint32_t kWaveRows = 48, kFewRows = 8;   // a list of no more rows is one wavefront's work, beside other roots and in a block of its own

// Roots per block of kListWaves wavefronts. With as many roots as wavefronts none of these is idle while lists are
// short or while draws are made, with one the longest lists are spread widest. One / two / four roots per block, ten draws
// each, over lists of one length and over lists by a power law (exponent 0.9), of 20, 400 and 4 000 entries on average, us:
//   2 000 roots:  14.6 14.7 14.8   32.6 39.3 40.1    15.0 15.1 15.2   41.2 47.2 51.7    20.1 22.9 24.4   50.9 60.0 77.0
//   4 000 roots:  21.9 18.6 18.6   39.6 48.9 48.8    26.3 19.0 18.9   51.7 57.3 61.9    31.4 28.7 29.5   66.5 72.7 85.8
//   6 000 roots:  26.6 24.8 23.3   47.3 49.6 46.7    33.1 28.6 23.7   62.7 66.9 82.1    41.0 38.7 35.9   84.7 89.5  103
//   12 000 roots: 40.3 37.0 34.6   70.7 71.0 75.9    56.4 47.5 39.6    101  101 95.5    70.0 62.7 57.0    137  137  139
int list_roots_per_block(int64_t entries, int64_t nodes, int64_t roots) {
    if (entries < 256 * nodes) return roots < 4000 ? 1 : 4;
    return roots < 6000 ? 1 : roots < 12000 ? 2 : 4;
}

// What a block holds in LDS: the queries, the samples of its roots, the tile sums. As little as it takes: with one root and all
// four wavefronts' samples, 16.6 KB, fewer blocks are resident (3 000 roots over lists of 300 entries 25.0 us, so 19.8).
static_assert(kListWaves * sizeof(ListQuery) % sizeof(uint64_t) == 0, "the tile sums' alignment");
inline unsigned list_lds_bytes(int per_block) {
    return kListWaves * sizeof(ListQuery) + per_block * kSamples * sizeof(uint32_t) + kMaxTiles * sizeof(uint64_t);
}

// How a list of cnt > k valid entries is cut up, into at most max_tiles tiles. By one wavefront. Where the cuts lie changes the
// time and never a result: approximate quotients and roots do.
__device__ __forceinline__ ListQuery plan_list(const TaserRec* __restrict__ rec, const TaserTimeIndex& index, int64_t lo, int64_t hi,
                                               int64_t t, uint32_t cnt, int k, uint32_t alone_rows, uint32_t max_tiles, int lane) {
    ListQuery q = {};
    q.lo = (uint32_t)lo;
    q.cnt = cnt;
    q.t_low = (uint32_t)(uint64_t)t;
    q.k = (uint32_t)k;
    q.batches = 1u;
    uint64_t longest = (uint64_t)t - (uint64_t)rec[lo].ts;   // of all deltas
    // delta >= 2^32 is ts < t - (2^32 - 1); t is at least 2^32 above the smallest timestamp here
    if (longest >> 32) q.ones = (uint32_t)group_cutoff<kWave>(rec, index, lo, hi, t - 0xFFFFFFFFll, 0, lane);
    if (q.ones >= kManyOnes) {
        q.far_begin = q.first = q.ones;
        q.far_tiles = 1;
    }
    const uint32_t rest = cnt - q.far_begin;
    if (q.far_begin && rest >= kFarEntries) longest = (uint64_t)t - (uint64_t)rec[lo + q.ones].ts;
    if (cnt - q.ones >= kFarEntries && longest > kLastLargeDelta) {
        const float every = (float)longest * __builtin_amdgcn_rcpf((float)rest);   // time between two entries
        float from = __builtin_amdgcn_sqrtf(kRunEntries * 4294967296.0f * every);   // around it a weight has kRunEntries entries
        if (from < (float)(kLastLargeDelta + 1u)) from = (float)(kLastLargeDelta + 1u);
        const uint32_t w_first = longest >> 32 ? 1u : quotient_of_delta<false>((uint32_t)longest);
        uint32_t w_end = (uint32_t)(4294967296.0f * __builtin_amdgcn_rcpf(from));
        if (w_end > kSmallWeight) w_end = kSmallWeight;
        const float far = (float)rest * (1.0f - from * __builtin_amdgcn_rcpf((float)longest));  // entries, were they spread evenly
        if (w_end > w_first && far > kRunEntries * (float)(w_end - w_first) + 1024.0f + kDrawEntries * (float)k) {
            // weights below w_end are deltas above floor(2^32 / w_end), which is less than `longest`
            const uint32_t first = (uint32_t)group_cutoff<kWave>(rec, index, lo, hi, t - (int64_t)weight_of_delta(w_end), 0, lane);
            if ((first - q.far_begin) / (uint32_t)kRunEntries > w_end - w_first) {
                q.first = first;
                q.w_first = w_first;
                q.w_end = w_end;
                const uint32_t batches = (w_end - w_first + kBatch - 1) / kBatch;
                const uint32_t most = max_tiles / 2u - 1u;     // (a tile is left for the `ones`)
                q.batches = (batches + most - 1u) / most;
                q.far_tiles = q.ones_tiles() + (batches + q.batches - 1) / q.batches;
                q.stride = (first - q.ones + kSamples - 1) / kSamples;
                longest = first < cnt ? (uint64_t)t - (uint64_t)rec[lo + first].ts : 1;
            }
        }
    }
    q.near = longest < (1u << 24);
    // Rows per tile: every tile costs the summing a wave-wide reduction, every draw re-reads about half
    // a tile with a wave-wide scan per row; the sum is smallest near sqrt(rows / k). The tiling
    // never changes a result, only the cost. (64 draws, timestamps within 30 000 ticks, with 128 tiles for the near part
    // whatever the block's roots, and with all that the block has: 600 roots over lists of 100 000 entries 330 and 156 us, 200
    // over lists of a million 2.45 and 0.65 ms.)
    const uint32_t rows = (cnt - q.first + kWave - 1) / kWave;
    uint32_t per = (uint32_t)(__builtin_amdgcn_sqrtf((float)rows * __builtin_amdgcn_rcpf((float)k)) * 1.00001f);
    q.tile_shift = per > 1u ? 31u - (uint32_t)__clz((int)per) : 0u;
    while (((uint64_t)(max_tiles - q.far_tiles) << q.tile_shift) < rows) ++q.tile_shift;
    per = 1u << q.tile_shift;
    q.together = rows + 4u * q.far_tiles * q.batches > alone_rows;
    q.tiles = q.far_tiles + (rows + per - 1) / per;
    return q;
}

// The weights 1/(t - ts) depend on the query, so the whole valid list counts for every root. What an entry adds to
// the sums is a whole number that changes slowly far from the query: entries between floor(2^32 / (w + 1)) and
// floor(2^32 / w) before it all weigh w. Where a weight has kRunEntries entries and more, the list is summed by
// weights (the far part: a search per weight), elsewhere by entries (from a plain array of the timestamps' low words, a
// quarter of the bytes of the records). A block of four wavefronts: each finds the cutoff of a root and cuts up its
// list; all of them sum the long lists' tiles; then each wavefront sums its own list if it is short, and makes its
// root's draws. Bound by vector instructions (82 % of the issue slots): 16 per 64 entries, 180 per 63 weights, about 90 per
// draw. Two hops of 10 from 4 000 roots (0.41 G weights, 0.22 G of them in far parts): 0.62 ms when every entry was weighed
// and one root had a block, 0.32 so. Eight wavefronts per SIMD take 96 scalar registers, which is what the attribute asks
// for (0.36 ms with seven).
__global__ __launch_bounds__(kListThreads) __attribute__((amdgpu_waves_per_eu(8))) void sample_hop_inverse_timespan_kernel(
    const int64_t* __restrict__ indptr, const TaserRec* __restrict__ rec, const uint32_t* __restrict__ ts_low,
    const TaserTimeIndex index, const int32_t* __restrict__ roots,
    const int64_t* __restrict__ times, int64_t num_roots, int per_block, int32_t num_nodes, int k, uint32_t seed_lo, uint32_t seed_hi,
    uint32_t hop, int32_t* __restrict__ o_nbr, int32_t* __restrict__ o_eid, int64_t* __restrict__ o_ts,
    int32_t* __restrict__ o_count) {
    extern __shared__ uint64_t list_lds[];   // list_lds_bytes(per_block)
    ListQuery* const query = reinterpret_cast<ListQuery*>(list_lds);
    uint32_t (*const sample)[kSamples] = reinterpret_cast<uint32_t (*)[kSamples]>(query + kListWaves);
    uint64_t* const tile_sums = reinterpret_cast<uint64_t*>(sample + per_block);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t root = (int64_t)blockIdx.x * per_block + wave;
    const uint32_t max_tiles = (uint32_t)kMaxTiles >> (per_block >> 1);   // of a root: per_block is 1, 2 or 4
    if (lane == 0) query[wave].tiles = query[wave].together = 0;   // nothing (more) to do for this wave's root
    if (wave < per_block && root < num_roots) {
        int64_t lo = 0, hi = 0, t = 0;
        const int32_t v = roots[root];
        if (v >= 0 && v < num_nodes) {
            t = times[root];
            lo = indptr[v];
            hi = indptr[v + 1];
        }
        const int cnt = __builtin_amdgcn_readfirstlane((int)group_cutoff<kWave>(rec, index, lo, hi, t, 0, lane));   // below 2^31
        if (cnt <= k) {          // everything, most recent first
            const TaserRec pad = {0, -1, -1};
            if (lane < k) store_slot(o_nbr, o_eid, o_ts, root * k + lane, lane < cnt ? rec[lo + cnt - 1 - lane] : pad);
            if (lane == 0) o_count[root] = cnt;
        } else {
            const ListQuery q = uniform(plan_list(rec, index, lo, hi, t, (uint32_t)cnt, k, per_block == 1 ? kFewRows : kWaveRows, max_tiles, lane));
            if (lane == 0) query[wave] = q;
            if (q.far_tiles > q.ones_tiles()) {
                uint32_t s[kSamples / kWave];
#pragma unroll
                for (uint32_t i = 0; i < kSamples / kWave; ++i) {
                    const uint64_t p = (uint64_t)(i * kWave + (uint32_t)lane + 1u) * q.stride - 1u + q.ones;
                    s[i] = ts_low[q.lo + (p < q.first ? (uint32_t)p : q.first - 1u)];
                }
#pragma unroll
                for (uint32_t i = 0; i < kSamples / kWave; ++i) sample[wave][i * kWave + (uint32_t)lane] = q.t_low - s[i];
            }
        }
    }
    // the long lists by all waves, then every wave its own
    __syncthreads();
#pragma unroll 1
    for (int w = 0; w < per_block; ++w) {
        if (!__builtin_amdgcn_readfirstlane((int)query[w].together)) continue;
        const ListQuery q = uniform(query[w]);
        sum_tiles(q, ts_low, sample[w], (uint32_t)wave, kListWaves, tile_sums + w * max_tiles, lane);
    }
    __syncthreads();
    if (wave >= per_block) return;
    const ListQuery q = uniform(query[wave]);
    if (q.tiles == 0) return;
    uint64_t* const tile_sum = tile_sums + wave * max_tiles;
    if (!q.together) {
        sum_tiles(q, ts_low, sample[wave], 0, 1, tile_sum, lane);
        own_lds_ready();
    }
    uint64_t u = 0;
    if (lane < k) u = draw64_wide(seed_lo, seed_hi, hop, (uint64_t)root, (uint32_t)lane);
    const uint32_t pick = draw_entries(q, ts_low + q.lo, sample[wave], tile_sum, u, lane);
    if (lane < k) store_slot(o_nbr, o_eid, o_ts, root * k + lane, rec[q.lo + pick]);
    if (lane == 0) o_count[root] = k;
}

__global__ __launch_bounds__(kThreads) void timestamps_low_kernel(const TaserRec* __restrict__ rec, int64_t n,
                                                                  uint32_t* __restrict__ ts_low) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n) ts_low[i] = (uint32_t)(uint64_t)rec[i].ts;
}

// The low words of a graph's timestamps, an array made on the first call that needs it. The
// call that makes it waits for the fill, so later calls on any stream find it ready.
std::mutex g_ts_low_mutex;
int ensure_ts_low(const taser_tcsr* g_const, hipStream_t stream) {
    taser_tcsr* g = const_cast<taser_tcsr*>(g_const);   // a cache inside the handle, not a change of the graph
    std::lock_guard<std::mutex> lock(g_ts_low_mutex);
    if (g->ts_low || g->num_entries == 0) return TASER_OK;
    uint32_t* p = nullptr;
    TASER_HIP_TRY(hipMalloc((void**)&p, (size_t)g->num_entries * sizeof(uint32_t)));
    hipLaunchKernelGGL(timestamps_low_kernel, dim3((unsigned)((g->num_entries + kThreads - 1) / kThreads)), dim3(kThreads),
                       0, stream, g->rec, g->num_entries, p);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) {
        (void)hipFree(p);
        return taser_fail_hip(e, "sample_temporal: building the timestamp array");
    }
    g->ts_low = p;
    return TASER_OK;
}

// ---- most-recent finder, large hops: four lanes per search ---------------------------
// A 16-lane search spends its instructions on four roots per wave, and a hop of 10^5 roots puts 30 such
// waves on every SIMD. Here a quad of lanes searches for one root, each lane comparing four neighboring
// entries of a level (the same 128-byte line per level): 16 roots per wave for little more than the
// instructions of four, and all waves resident at once. The slots are then handed out flat, k of them per
// root whatever k is, so that all lanes load and store. What is left is the latency of one chain of reads.
// The uniform finder, searched the same way, gains nothing (60 000 roots 16.6 / 16.0 us, 6 000 roots 6.2 / 12.1): its
// draws are then three rounds one after the other.
//
// Where it pays: the longer the lists, the longer the search that it makes cheaper; the more of its 16, 32 or 64 lanes
// a root's slots fill in the other kernel, the less there is to gain. Time of this kernel over the other one's, k = 10,
// 16, 25, 64, for graphs of 2, 100, 13 300 entries per node on average (the other one with two roots per group from
// 65 536 roots on):
//   16 384 roots:  1.15 1.22 1.21 1.28   1.10 1.16 1.12 1.10   1.06 1.10 1.03 1.00
//   24 576 roots:  1.13 1.19 1.06 1.05   1.04 1.09 0.95 0.93   0.94 0.98 0.88 0.87
//   32 768 roots:  1.08 1.21 0.97 0.94   1.00 1.06 0.91 0.90   0.89 1.00 0.79 0.86
//   65 536 roots:  1.03 1.14 0.93 0.85   0.98 1.01 0.90 0.96   0.82 0.89 0.84 0.87
//   640 000 roots: 1.13 1.23 0.82 0.75   0.97 1.08 0.96 0.83   0.89 0.95 0.86 0.85
// (13 300 entries, k = 10: 120 000 roots 18.8 us by 16 lanes, 13.7 by 4.) Hence a line per group size and length of
// list: the fewest roots, and how many eighths of its lanes a root's slots may fill (k = 4 takes 0.92 to 0.96 on the
// shortest lists, k = 5 up to 1.03).
inline bool quads_pay(int64_t entries, int64_t nodes, int64_t roots, int k, int lanes) {
    struct Line { int roots, eighths; };
    static constexpr Line lines[3][3] = {{{40960, 2}, {32768, 5}, {24576, 8}},    // 16 lanes: lists of less than 64, 256, more entries
                                         {{32768, 7}, {24576, 8}, {20480, 8}},    // 32 lanes
                                         {{32768, 8}, {24576, 8}, {16384, 8}}};   // 64 lanes
    const Line line = lines[lanes / 32][entries >= 256 * nodes ? 2 : entries >= 64 * nodes ? 1 : 0];
    return roots >= line.roots && 8 * k <= line.eighths * lanes;
}
constexpr int kQuadRoots = 16;          // roots per wave

// 16 bytes of a time-index level, 8-byte aligned.
struct __attribute__((packed, aligned(8))) TimePair {
    int64_t a, b;
};

// As group_cutoff, for the root of this lane's quad. Entry e of level L lies wholly before position p
// if e < p >> 4 L, so e is "before" if e < lo >> 4 L, or e < hi >> 4 L and its timestamp is below t. Reads
// at most 15 entries behind a level's (or the record array's) last one: the build leaves room for them,
// and what they hold does not matter (e >= hi >> 4 L).
__device__ __forceinline__ uint32_t quad_cutoff(const TaserRec* __restrict__ rec, const TaserTimeIndex& index, uint32_t lo, uint32_t hi,
                                                int64_t t, uint32_t sub) {
    const uint32_t d = hi - lo;
    const int bits = d ? 32 - __clz((int)d) : 0;
    int top = bits ? (bits + 3) / 4 - 1 : 0;                            // see group_cutoff
    if ((hi >> (4 * top)) - (lo >> (4 * top)) > 15u) ++top;
    uint32_t at = 0;
#pragma unroll
    for (int L = kTimeIndexLevels; L >= 0; --L) {
        if (!__ballot(L <= top)) continue;   // no list of this wave is at this level yet
        if (L <= top) {
            const uint32_t lo_l = lo >> (4 * L), hi_l = hi >> (4 * L);
            const uint32_t first = L == top ? lo_l : at * 16u;
            const uint32_t e = first + 4u * sub;
            int64_t ts[4];
            if (L > 0) {
                const TimePair* p = reinterpret_cast<const TimePair*>(index.level[L > 0 ? L - 1 : 0] + e);
                const TimePair x = p[0], y = p[1];
                ts[0] = x.a; ts[1] = x.b; ts[2] = y.a; ts[3] = y.b;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) ts[i] = rec[e + i].ts;
            }
            uint32_t c = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) c += (uint32_t)((e + i < hi_l && ts[i] < t) || e + i < lo_l);
            c += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, 0xB1, 0xf, 0xf, true);   // quad_perm [1, 0, 3, 2]
            c += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c, 0x4E, 0xf, 0xf, true);   // quad_perm [2, 3, 0, 1]
            at = first + c;
        }
    }
    return at - lo;
}

template <int kAhead>   // record loads of a lane in flight together
__global__ __launch_bounds__(kThreads) void sample_hop_recent_quads_kernel(
    const int64_t* __restrict__ indptr, const TaserRec* __restrict__ rec, const TaserTimeIndex index,
    const int32_t* __restrict__ roots, const int64_t* __restrict__ times, int64_t num_roots, int32_t num_nodes, int k, uint32_t magic_k,
    int32_t* __restrict__ o_nbr, int32_t* __restrict__ o_eid, int64_t* __restrict__ o_ts, int32_t* __restrict__ o_count) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t q0 = ((int64_t)blockIdx.x * (kThreads / kWave) + wave) * kQuadRoots;   // first root of the wave
    if (q0 >= num_roots) return;
    const int here = num_roots - q0 < kQuadRoots ? (int)(num_roots - q0) : kQuadRoots;    // roots of the wave
    const int quad = lane >> 2;
    uint32_t lo = 0, hi = 0;
    int64_t t = 0;
    if (quad < here) {
        const int32_t v = roots[q0 + quad];
        if (v >= 0 && v < num_nodes) {   // anything else is a root without neighbors
            t = times[q0 + quad];
            lo = (uint32_t)indptr[v];
            hi = (uint32_t)indptr[v + 1];
        }
    }
    const uint32_t cnt = quad_cutoff(rec, index, lo, hi, t, (uint32_t)lane & 3u);
    if ((lane & 3) == 0 && quad < here) o_count[q0 + quad] = (int32_t)(cnt < (uint32_t)k ? cnt : (uint32_t)k);
    // slot s of the wave is slot s % k of root s / k
    const TaserRec pad = {0, -1, -1};
    const uint32_t slots = (uint32_t)(here * k);
    for (uint32_t s0 = 0; s0 < slots; s0 += kAhead * kWave) {
        TaserRec got[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const uint32_t s = s0 + u * kWave + lane;
            uint32_t r = k == 1 ? s : __umulhi(s, magic_k);   // exact: s < 2^11, k <= 64
            const uint32_t j = s - r * (uint32_t)k;
            if (r > kQuadRoots - 1) r = kQuadRoots - 1;        // past the wave's slots
            const uint32_t r_lo = __shfl(lo, (int)r * 4, kWave), r_cnt = __shfl(cnt, (int)r * 4, kWave);
            got[u] = pad;
            if (s < slots && j < r_cnt) got[u] = rec[r_lo + r_cnt - 1u - j];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const uint32_t s = s0 + u * kWave + lane;
            if (s < slots) store_slot(o_nbr, o_eid, o_ts, q0 * k + s, got[u]);
        }
    }
}

template <int POLICY, int G, int kRootsPerGroup, int ROWS>
void launch_hop_gr(const taser_tcsr* g, const int32_t* roots, const int64_t* times, int64_t n, int k,
                   uint64_t seed, uint32_t hop, int m, const uint32_t* edge_weight, const taser_hop_out& o,
                   const RowCopy& rows, hipStream_t stream) {
    constexpr int roots_per_block = (kThreads / kWave) * (kWave / G) * kRootsPerGroup;
    const unsigned grid = (unsigned)((n + roots_per_block - 1) / roots_per_block);
    hipLaunchKernelGGL((sample_hop_kernel<POLICY, G, kRootsPerGroup, ROWS>), dim3(grid), dim3(kThreads), 0, stream, g->indptr, g->rec, g->time_index,
                       roots, times, n, g->num_nodes, k, (uint32_t)seed, (uint32_t)(seed >> 32), hop, m, edge_weight, o.nbr,
                       o.eid, o.ts, o.count, rows);
}

template <int POLICY, int G>
void launch_hop_g(const taser_tcsr* g, const int32_t* roots, const int64_t* times, int64_t n, int k,
                  uint64_t seed, uint32_t hop, int m, const uint32_t* edge_weight, const taser_hop_out& o,
                  const RowCopy* rows, hipStream_t stream) {
    // wave instructions of the copy in flight: four where a wavefront has four roots' rows to move, two (and
    // 28 registers fewer) where it has one or two roots
    if (rows) launch_hop_gr<POLICY, G, 1, (G == 16 ? 4 : 2)>(g, roots, times, n, k, seed, hop, m, edge_weight, o, *rows, stream);
    else if (POLICY == TASER_RECENT && n >= 65536) launch_hop_gr<POLICY, G, 2, 0>(g, roots, times, n, k, seed, hop, m, edge_weight, o, RowCopy{}, stream);
    else launch_hop_gr<POLICY, G, 1, 0>(g, roots, times, n, k, seed, hop, m, edge_weight, o, RowCopy{}, stream);
}

// Lanes of a wavefront that serve one root.
int group_lanes(int policy, int k, int m) {
    const int lanes = (policy == TASER_WEIGHTED && m > k) ? m : k;   // lanes a root needs
    return lanes <= 16 ? 16 : lanes <= 32 ? 32 : 64;
}

template <int POLICY>
void launch_hop(const taser_tcsr* g, const int32_t* roots, const int64_t* times, int64_t n, int k,
                uint64_t seed, uint32_t hop, int m, const uint32_t* edge_weight,
                const taser_hop_out& o, const RowCopy* rows, bool wave_per_root, hipStream_t stream) {
    static const char* const names[2][3] = {{"sample_hop_recent", "sample_hop_uniform", "sample_hop_weighted"},
                                            {"sample_rows_hop_recent", "sample_rows_hop_uniform", "sample_rows_hop_weighted"}};
    TaserProfileSpan span(stream, names[rows ? 1 : 0][POLICY]);
    const int lanes = group_lanes(POLICY, k, m);
    if (POLICY == TASER_RECENT && !rows && quads_pay(g->num_entries, g->num_nodes, n, k, lanes)) {
        constexpr int roots_per_block = kThreads / kWave * kQuadRoots;
        const unsigned grid = (unsigned)((n + roots_per_block - 1) / roots_per_block);
        const uint32_t magic_k = k > 1 ? (uint32_t)((((uint64_t)1 << 32) + (uint32_t)k - 1) / (uint32_t)k) : 0u;
        // up to 12 slots per root all loads of a wave fit three rounds; where they don't, a second batch of loads waits
        // for the stores of the first (16 slots, 24 576 roots: 5.71 us with batches of three, 5.56 with four; 64 slots,
        // 16 384 roots: 10.6 with three, 10.2 with four, 9.8 with eight)
        const auto kernel = k <= 12 ? sample_hop_recent_quads_kernel<3> : k <= 32 ? sample_hop_recent_quads_kernel<4> : sample_hop_recent_quads_kernel<8>;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kThreads), 0, stream, g->indptr, g->rec, g->time_index, roots,
                           times, n, g->num_nodes, k, magic_k, o.nbr, o.eid, o.ts, o.count);
        return;
    }
    if (rows && wave_per_root) launch_hop_gr<POLICY, 64, 1, 8>(g, roots, times, n, k, seed, hop, m, edge_weight, o, *rows, stream);
    else if (lanes == 16) launch_hop_g<POLICY, 16>(g, roots, times, n, k, seed, hop, m, edge_weight, o, rows, stream);
    else if (lanes == 32) launch_hop_g<POLICY, 32>(g, roots, times, n, k, seed, hop, m, edge_weight, o, rows, stream);
    else launch_hop_g<POLICY, 64>(g, roots, times, n, k, seed, hop, m, edge_weight, o, rows, stream);
}

// The feature table a call wants sliced along with the sampling (null table: none).
struct RowRequest {
    const void* table;
    int64_t table_rows;
    int32_t row_bytes;
    int64_t pitch_bytes;
    void* const* out;   // per hop
};

int check_sampling_arguments(const char* what, const taser_tcsr* g, const int32_t* roots, const int64_t* times,
                             int64_t num_roots, int32_t k, int32_t hops, int32_t policy, int32_t m,
                             const uint32_t* edge_weight, const taser_hop_out* out) {
    if (!g || !out) return taser_fail(TASER_E_ARG, "%s: null graph or output array", what);
    if (num_roots < 0) return taser_fail(TASER_E_ARG, "%s: num_roots = %lld", what, (long long)num_roots);
    if (num_roots > 0 && (!roots || !times)) return taser_fail(TASER_E_ARG, "%s: null roots/times", what);
    if (k < 1 || k > TASER_MAX_K) return taser_fail(TASER_E_RANGE, "%s: k = %d outside [1, %d]", what, k, TASER_MAX_K);
    if (hops < 1 || hops > TASER_MAX_HOPS) return taser_fail(TASER_E_RANGE, "%s: hops = %d outside [1, %d]", what, hops, TASER_MAX_HOPS);
    if (policy != TASER_RECENT && policy != TASER_UNIFORM && policy != TASER_WEIGHTED && policy != TASER_INVERSE_TIMESPAN)
        return taser_fail(TASER_E_ARG, "%s: unknown policy %d", what, policy);
    if (policy == TASER_WEIGHTED) {
        if (m < 1 || m > TASER_MAX_M) return taser_fail(TASER_E_RANGE, "%s: m = %d outside [1, %d]", what, m, TASER_MAX_M);
        if (!edge_weight) return taser_fail(TASER_E_ARG, "%s: weighted policy needs edge_weight", what);
    }
    int64_t n = num_roots;
    for (int h = 0; h < hops; ++h) {
        if (n > 0 && (!out[h].nbr || !out[h].eid || !out[h].ts || !out[h].count))
            return taser_fail(TASER_E_ARG, "%s: null output buffer at hop %d", what, h);
        if (n * k >= ((int64_t)1 << 31)) return taser_fail(TASER_E_RANGE, "%s: num_roots * k^hops must stay below 2^31", what);
        n *= k;
    }
    return TASER_OK;
}

// A wavefront copies the rows of its own roots only while they are few bytes: all wavefronts
// of a launch search at the same time and then copy at the same time, so the two phases add up
// instead of overlapping, and for long rows the plain gather (one launch for all hops) moves
// the same bytes faster. Measured on 2 x 10 slots per root: up to 8 KiB per wavefront the hop
// kernel's own copy is as fast or faster (64-byte rows: 41 against 49 us per batch of 4 000
// roots, 25 against 29 us with 16 lanes per root), beyond it up to 15 % slower.
constexpr int64_t kFinderCopyMaxWaveBytes = 8192;

// In a small hop a wavefront per root copies longer rows as well: one launch fewer, and with up to 8 KiB in flight a
// wavefront a root's rows are a round or two of loads. Small is one round of wavefronts (127 registers: sixteen per
// compute unit), of a last hop whose rows would otherwise be a launch of their own. One hop, k slots of `bytes`, us a
// call with two launches and with one: 300 / 1 800 / 3 000 / 4 500 roots, most recent, 10 x 688: 11.8 8.6, 12.1 8.7, 11.9
// 8.7, 14.7 14.5; uniform, 10 x 344: 12.4 8.7, 12.3 8.9, 12.0 9.2, 13.2 14.2; most recent, 20 x 1064: 12.3 10.1, 17.0 15.0,
// 24.6 22.4, 33.5 35.9; 4 096 roots, uniform, 20 x 1064: 33.1 29.7, 10 of 25, 10 x 2400: 33.1 32.5.
// With several hops the gather is one launch for all of them, and a copy in the kernels of the first hops, a few wavefronts
// with all of a root's rows each, is a step that the next hop waits for. So then the rows have to be few, of a root and in
// all: two hops from 240 / 400 roots, 10 x 1064: most recent 22.1 20.4, 24.4 26.1, uniform 22.1 21.5, 24.1 26.5; from 60 roots,
// 20 x 1064: most recent 21.4 21.8, uniform 21.3 26.5. Other finders than the most recent one pay for 64 lanes per root in
// every hop, the uniform one beyond 16 slots most of all (its draws are resolved one after the other there): three hops from 20
// roots, 10 x 1064: most recent 28.0 25.8, uniform 27.7 28.4, 10 of 25 28.1 29.8; from 10 roots, 20 x 344: most recent 27.0
// 23.9, uniform 27.4 28.8.
constexpr int64_t kSmallHopRoots = 4096, kSmallHopWaveBytes = 24576;
constexpr int64_t kSmallHopsBytes = (int64_t)28 << 20, kSmallHopsWaveBytes = 16384;   // of several hops: the last one's rows, and a root's
bool small_hop_pays(int policy, int64_t roots, int k, int hops, int row_bytes) {
    const int64_t of_root = (int64_t)k * row_bytes, all = roots * of_root;
    if (roots > kSmallHopRoots || of_root > kSmallHopWaveBytes) return false;
    if (hops == 1) return true;
    if (all > kSmallHopsBytes || of_root > kSmallHopsWaveBytes) return false;
    if (policy == TASER_RECENT) return true;
    const bool few = of_root <= kSmallHopsWaveBytes / 2;
    return policy == TASER_UNIFORM && k > 16 ? few && hops == 2 : few || hops == 2;
}

// All hops of one call. With `want`, hop h also leaves the table rows of its sampled edges in
// want->out[h]: written by the hop kernel where the shapes allow it and the rows are short, else
// by the plain gather launched after the last hop (same bytes either way), one launch for
// all hops (6 000 roots, 2 x 10 slots, 344-byte rows: the whole call 119 us with two, 115 with one).
int sample_hops(const taser_tcsr* g, const int32_t* roots, const int64_t* times, int64_t num_roots, int32_t k,
                int32_t hops, int32_t policy, uint64_t seed, int32_t m, const uint32_t* edge_weight,
                const taser_hop_out* out, const RowRequest* want, hipStream_t stream) {
    taser_clear_stale_hip_error();
    if (policy == TASER_INVERSE_TIMESPAN) {
        const int rc = ensure_ts_low(g, stream);
        if (rc != TASER_OK) return rc;
    }
    const int32_t* cur_roots = roots;
    const int64_t* cur_times = times;
    int64_t n = num_roots;
    TaserGatherPart pending[TASER_MAX_HOPS];
    int n_pending = 0;
    int64_t roots_of_last_hop = num_roots;
    for (int h = 1; h < hops; ++h) roots_of_last_hop *= k;
    for (int h = 0; h < hops && n > 0; ++h) {
        // Can this hop's kernel write the rows itself? It copies per wavefront, in aligned 16-byte
        // pieces read at 4-byte alignment: rows, pitch and table must allow that, and the rows of
        // one wavefront's roots must be whole 16-byte pieces.
        RowCopy copy{};
        const RowCopy* rows = nullptr;
        bool wave_per_root = false;
        if (want && policy != TASER_INVERSE_TIMESPAN) {
            int64_t wave_bytes = (int64_t)(kWave / group_lanes(policy, k, m)) * k * want->row_bytes;
            int64_t most = kFinderCopyMaxWaveBytes;
            if (wave_bytes > most && small_hop_pays(policy, roots_of_last_hop, k, hops, want->row_bytes)) {
                wave_per_root = true;
                wave_bytes = (int64_t)k * want->row_bytes;
                most = kSmallHopWaveBytes;
            }
            const uint64_t bits = (uint64_t)want->row_bytes | (uint64_t)want->pitch_bytes | (uint64_t)(uintptr_t)want->table;
            if (want->row_bytes >= 16 && wave_bytes <= most && (bits & 3) == 0 && (wave_bytes & 15) == 0 &&
                ((uintptr_t)want->out[h] & 15) == 0) {
                const uint8_t* zeros = taser_gather::zero_chunk();
                if (!zeros) return taser_fail(TASER_E_HIP, "sample_temporal_rows: the zero constant is not available on this device");
                const uint32_t rb = (uint32_t)want->row_bytes;
                copy = RowCopy{static_cast<const uint8_t*>(want->table), want->table_rows, want->pitch_bytes,
                               static_cast<uint8_t*>(want->out[h]), zeros, rb, (uint32_t)((((uint64_t)1 << 32) + rb - 1) / rb),
                               1024u / rb, 1024u % rb};
                rows = &copy;
            }
        }
        switch (policy) {
            case TASER_RECENT: launch_hop<TASER_RECENT>(g, cur_roots, cur_times, n, k, seed, (uint32_t)h, m, edge_weight, out[h], rows, wave_per_root, stream); break;
            case TASER_UNIFORM: launch_hop<TASER_UNIFORM>(g, cur_roots, cur_times, n, k, seed, (uint32_t)h, m, edge_weight, out[h], rows, wave_per_root, stream); break;
            case TASER_INVERSE_TIMESPAN: {
                TaserProfileSpan span(stream, "sample_hop_inverse_timespan");
                const int per_block = list_roots_per_block(g->num_entries, g->num_nodes, n);
                const unsigned grid = (unsigned)((n + per_block - 1) / per_block);   // n < 2^31
                hipLaunchKernelGGL(sample_hop_inverse_timespan_kernel, dim3(grid), dim3(kListThreads), list_lds_bytes(per_block), stream, g->indptr, g->rec,
                                   g->ts_low, g->time_index, cur_roots, cur_times, n, per_block, g->num_nodes, k, (uint32_t)seed,
                                   (uint32_t)(seed >> 32), (uint32_t)h, out[h].nbr, out[h].eid, out[h].ts, out[h].count);
                break;
            }
            default: launch_hop<TASER_WEIGHTED>(g, cur_roots, cur_times, n, k, seed, (uint32_t)h, m, edge_weight, out[h], rows, wave_per_root, stream); break;
        }
        if (want && !rows) {
            uint8_t* to = static_cast<uint8_t*>(want->out[h]);
            TaserGatherPart* last = n_pending ? &pending[n_pending - 1] : nullptr;
            if (last && last->ids + last->n == out[h].eid && static_cast<uint8_t*>(last->out) + last->n * want->row_bytes == to) last->n += n * k;
            else pending[n_pending++] = TaserGatherPart{out[h].eid, n * k, to};
        }
        cur_roots = out[h].nbr;
        cur_times = out[h].ts;
        n *= k;
    }
    TASER_HIP_TRY(hipGetLastError());
    if (n_pending == 0) return TASER_OK;
    return taser_launch_gather_parts(want->table, want->table_rows, want->row_bytes, want->pitch_bytes, pending, n_pending, stream);
}

}  // namespace

extern "C" int taser_sample_temporal(const taser_tcsr* g, const int32_t* roots, const int64_t* times,
                                     int64_t num_roots, int32_t k, int32_t hops, int32_t policy,
                                     uint64_t seed, int32_t m, const uint32_t* edge_weight,
                                     const taser_hop_out* out, void* hip_stream) {
    const int rc = check_sampling_arguments("sample_temporal", g, roots, times, num_roots, k, hops, policy, m, edge_weight, out);
    if (rc != TASER_OK) return rc;
    return sample_hops(g, roots, times, num_roots, k, hops, policy, seed, m, edge_weight, out, nullptr, (hipStream_t)hip_stream);
}

extern "C" int taser_sample_temporal_rows(const taser_tcsr* g, const int32_t* roots, const int64_t* times,
                                          int64_t num_roots, int32_t k, int32_t hops, int32_t policy,
                                          uint64_t seed, int32_t m, const uint32_t* edge_weight,
                                          const void* table, int64_t table_rows, int32_t row_bytes, int64_t pitch_bytes,
                                          const taser_hop_out* out, void* const* rows_out, void* hip_stream) {
    const char* what = "sample_temporal_rows";
    const int rc = check_sampling_arguments(what, g, roots, times, num_roots, k, hops, policy, m, edge_weight, out);
    if (rc != TASER_OK) return rc;
    if (table_rows < 0) return taser_fail(TASER_E_ARG, "%s: negative table_rows", what);
    if (row_bytes <= 0 || (row_bytes & 1)) return taser_fail(TASER_E_ARG, "%s: row_bytes = %d must be positive and even", what, row_bytes);
    if (pitch_bytes < row_bytes || (pitch_bytes & 1)) return taser_fail(TASER_E_ARG, "%s: pitch_bytes = %lld must be even and >= row_bytes", what, (long long)pitch_bytes);
    if (!table && table_rows > 0) return taser_fail(TASER_E_ARG, "%s: null table", what);
    if ((uintptr_t)table & 1) return taser_fail(TASER_E_ARG, "%s: table must be 2-byte aligned", what);
    if (!rows_out) return taser_fail(TASER_E_ARG, "%s: null rows_out", what);
    int64_t n = num_roots;
    for (int h = 0; h < hops; ++h) {
        if (n > 0 && !rows_out[h]) return taser_fail(TASER_E_ARG, "%s: null row buffer at hop %d", what, h);
        if ((uintptr_t)rows_out[h] & 1) return taser_fail(TASER_E_ARG, "%s: row buffers must be 2-byte aligned", what);
        n *= k;
    }
    const RowRequest want{table, table_rows, row_bytes, pitch_bytes, rows_out};
    return sample_hops(g, roots, times, num_roots, k, hops, policy, seed, m, edge_weight, out, &want, (hipStream_t)hip_stream);
}
