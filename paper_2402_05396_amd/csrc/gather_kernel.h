// Dense row gather: out row i <- the bytes of a source row chosen per i.
//
// The output is treated as one flat, dense stream, whatever the row length.
// Two kernels:
//   * gather_chunks_kernel (16-byte aligned output; rows a multiple of 4 bytes,
//     or of 2 bytes and at least 16 long): every thread produces 16 consecutive
//     output bytes with one aligned 16-byte non-temporal store. The 16 bytes
//     normally come from one source row and are read with a single 16-byte load
//     that only needs the rows' alignment; a thread whose bytes straddle a row
//     end falls back to 4-byte loads (2-byte rows: two 16-byte loads). A wave instruction therefore moves 1 KiB, rows of any length
//     (372 B, 1652 B, ...) fill every lane, and the dense output is written in
//     whole 128-byte lines.
//   * gather_elems_kernel: the same flat scheme with one V-wide element (2, 4
//     or 8 bytes) per thread, for outputs that are not 16-byte aligned and for
//     2-byte aligned rows where that is faster (see two_byte_chunks_pay).
// Where a row comes from is a functor, so the kernels serve both a table in
// device memory and the cache's choice of cache row / staged row / host row.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace taser_gather {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <typename V> __device__ __forceinline__ V zero_of() { return V(0); }
template <> __device__ __forceinline__ u32x2 zero_of<u32x2>() { return u32x2{0, 0}; }

constexpr int kThreads = 256;
constexpr int kUnroll = 4;
constexpr int kTile = kThreads * kUnroll;   // elements (or 16-byte chunks) per block
// Output rows a block of the chunk kernel can touch: rows of one dword, or with 2-byte units of at least 16 bytes.
constexpr int tile_rows(int unit) { return unit == 4 ? kTile * 4 + 2 : kTile + 2; }

// 16 bytes that are only known to be 4-byte (2-byte) aligned.
struct __attribute__((packed, aligned(4))) Chunk16 {
    u32x4 v;
};
struct __attribute__((packed, aligned(2))) Chunk16By2 {
    u32x4 v;
};

typedef const __attribute__((address_space(1))) Chunk16* GlobalChunk16Ptr;
typedef const __attribute__((address_space(1))) Chunk16By2* GlobalChunk16By2Ptr;
typedef const __attribute__((address_space(1))) uint32_t* GlobalU32Ptr;

template <int ALIGN> __device__ __forceinline__ u32x4 load16(const uint8_t* at) {
    return ALIGN == 2 ? ((GlobalChunk16By2Ptr)at)->v : ((GlobalChunk16Ptr)at)->v;
}

// A Source says where output row i comes from, in two steps so that the kernel
// can issue the (dependent) loads of several rows back to back:
//   key(i)          a 32-bit token read from memory (an id, a cache location);
//   address(key, i) first byte of the source row, or nullptr for a zero row.
//
// kAlign is what row size, pitch and addresses are known to share at least.
//
// A gather can run in two launches while some source rows are still on their way: PHASE 1 writes
// what needs only rows that are there, PHASE 2, launched when all of them are, the rest; between them
// every output byte is written (some dwords in both, with the same value). PHASE 0 is the whole
// gather in one launch. For that a Source also has
//   pending(key)    the row is on its way during PHASE 1;
//   resolve(key)    the token for PHASES 0 and 2 (PHASE 1 takes it as it is read);
//   late()          how many output rows PHASE 2 has to write (at most 2^32 - 1 of them counted);
//   late_skewed()   many of them are copies of the same source row.
// The owned-lines kernel can have a PHASE 3 between the two, when a part of the pending rows has arrived and the others
// are still on their way: it writes the first of them, and PHASE 2 is left with the others. For that a Source has
//   begin(phase)         called when PHASE 2 or 3 begins: how far the rows are; false where PHASE 3 has nothing to do, because all rows
//                        had arrived before it: they are PHASE 2's then;
//   resolve_first(key)   the token for PHASE 3;
//   in_phase<P>(key)     a row that PHASE P (2 or 3) writes, if it does not write everything;
//   after(key)           PHASE 3: the row is still on its way.

template <int PHASE, typename Source> __device__ __forceinline__ int32_t source_token(const Source& source, int64_t i) {
    const int32_t key = source.key(i);
    if constexpr (PHASE == 3) return source.resolve_first(key);
    else return PHASE == 1 ? key : source.resolve(key);
}

// UNIT: the size that divides rows, pitches and source addresses, 4 or 2 bytes; offsets are counted
// in it. With 2-byte units the rows are at least 16 bytes long. (One 16-byte load at any even address
// costs what an aligned one does: 1.33 M rows of 826 bytes take 0.20 ms, where a load and a store per
// 2 bytes took 0.71.)
// USE_MAGIC: floor(e / d) = umulhi(e, magic) with magic = ceil(2^32 / d), exact
// for e * d < 2^32 (the launcher checks that); otherwise a plain division.
// Beside: work for the first workgroups of the same launch (run() for `blocks` of them), or NothingBeside.
// (The gather is the kernel's own body: as an inlined function of two kernels it came out with register copies
// that waited for its loads, 0.180 instead of 0.178 ms for 1.32 M rows of 372 bytes.)
constexpr int kBesideWords = 2048;   // words of LDS that run() gets
struct NothingBeside {
    static constexpr bool kAny = false;
    static constexpr uint32_t blocks = 0;
    static __device__ __forceinline__ void run(uint32_t, int32_t*) {}
};
// Parts: further gathers from the same table in the same launch (a multi-hop call's hops each have ids and rows
// of their own; a launch for the small first hop costs as much as its rows), or OnePart.
struct OnePart {
    static constexpr bool kMore = false;
};
template <typename Source, bool USE_MAGIC, int UNIT, int PHASE, typename Beside, typename Parts>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void gather_chunks_kernel(
    Source source, uint32_t row_units, uint32_t magic, int64_t total_units, int64_t last_row, const uint8_t* __restrict__ zeros,
    uint8_t* __restrict__ out, const Beside beside, const Parts parts) {
    __shared__ int32_t tile_key[tile_rows(UNIT)];
    if (Beside::kAny && blockIdx.x < beside.blocks) {
        beside.run(blockIdx.x, tile_key);
        return;
    }
    uint32_t block = Beside::kAny ? blockIdx.x - beside.blocks : blockIdx.x;
    if constexpr (PHASE == 2)
        if (source.late() == 0) return;
    if constexpr (Parts::kMore) block = parts.enter(block, source, total_units, last_row, out);
    constexpr uint32_t kPer = 16 / UNIT;                       // units of a chunk
    const int64_t tile = (int64_t)block * (kTile * kPer);   // first output unit of this block
    int64_t row0;                                               // output row holding it
    if (tile < ((int64_t)1 << 32)) row0 = (uint32_t)tile / row_units;
    else row0 = tile / (int64_t)row_units;
    const uint32_t col0 = (uint32_t)(tile - row0 * row_units);

    // Pass 0: the tokens of every output row this tile touches, loaded once by consecutive
    // lanes into LDS. Without it each chunk's token is a wave-wide broadcast load at the head of
    // a chain of two dependent loads, and the kernel's speed follows the latency of the token
    // array (slower by a third when that array has dropped out of the memory-side cache).
    {
        int64_t tile_last = tile + kTile * kPer - 1;
        if (tile_last >= total_units) tile_last = total_units - 1;
        const uint32_t e_last = col0 + (uint32_t)(tile_last - tile);   // unit offset from the start of row0
        const int rows_here = (int)(USE_MAGIC ? __umulhi(e_last, magic) : e_last / row_units) + 1;   // <= the array
        bool late = false;
        for (int r = threadIdx.x; r < rows_here; r += kThreads) {
            const int32_t key = source_token<PHASE>(source, row0 + r);
            tile_key[r] = key;
            if (PHASE == 2) late |= source.pending(key);
        }
        if (PHASE != 2) __syncthreads();
        else if (!__syncthreads_or(late)) return;               // nothing of this tile was on its way
    }
    // Pass 1 (ALU only): output row and column of each of this thread's chunks.
    uint32_t col[kUnroll];
    int64_t row[kUnroll];
    bool whole[kUnroll], cross[kUnroll];   // inside one row / crossing a row end (neither: past the end)
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
        const uint32_t local = (threadIdx.x + u * kThreads) * kPer;
        const uint32_t e = col0 + local;                        // unit offset from the start of row0
        const uint32_t dr = USE_MAGIC ? __umulhi(e, magic) : e / row_units;
        col[u] = e - dr * row_units;
        row[u] = row0 + dr;
        const bool live = tile + local < total_units;
        whole[u] = live && col[u] + kPer <= row_units;
        cross[u] = live && !whole[u];
        if (row[u] > last_row) row[u] = last_row;               // keeps the token read below in bounds
    }
    // Pass 2: straight-line code, no branches, so that the four 16-byte row loads are in
    // flight together. A chunk with nothing to load here (zero row, row-crossing, past the
    // end) reads 16 zero bytes instead of branching around the load.
    int32_t key[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) key[u] = tile_key[row[u] - row0];
    bool write[kUnroll];   // chunks that are this phase's (a chunk with a pending row's bytes is PHASE 2's)
    u32x4 vals[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
        write[u] = PHASE == 0 || (PHASE == 2) == source.pending(key[u]);
        const uint8_t* base = PHASE == 1 && !write[u] ? nullptr : source.address(key[u], row[u]);
        const uint8_t* at = (whole[u] && write[u] && base) ? base + (size_t)col[u] * UNIT : zeros;
        vals[u] = load16<UNIT>(at);
    }
    // Pass 3 (rare): chunks that cross one or more row ends.
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
        if (!cross[u]) continue;
        const int64_t d = tile + (threadIdx.x + u * kThreads) * kPer;
        if (UNIT == 2) {
            // one row end (rows hold at least 16 bytes): the last 16 bytes of this row, the first 16 of
            // the next one, and of those 32 the 16 that start where this row has `in_row` bytes left
            const uint32_t in_row = (row_units - col[u]) * 2u;                    // 2 .. 14
            const uint8_t* base = source.address(key[u], row[u]);
            const uint8_t* next = row[u] < last_row ? source.address(tile_key[row[u] + 1 - row0], row[u] + 1) : nullptr;
            static_assert(UNIT == 4 || PHASE == 0, "2-byte rows come from tables, which are all there");
            const u32x4 t = load16<UNIT>(base ? base + (size_t)row_units * 2u - 16u : zeros);
            const u32x4 h = load16<UNIT>(next ? next : zeros);
            const uint32_t skip = 16u - in_row;                                   // bytes of t that belong to the chunk before
            const bool by2 = skip & 8u, by1 = skip & 4u, half = skip & 2u;
            const uint32_t y0 = by2 ? t.z : t.x, y1 = by2 ? t.w : t.y, y2 = by2 ? h.x : t.z, y3 = by2 ? h.y : t.w, y4 = by2 ? h.z : h.x,
                           y5 = by2 ? h.w : h.y;
            const uint32_t z0 = by1 ? y1 : y0, z1 = by1 ? y2 : y1, z2 = by1 ? y3 : y2, z3 = by1 ? y4 : y3, z4 = by1 ? y5 : y4;
            vals[u] = u32x4{half ? __builtin_amdgcn_alignbyte(z1, z0, 2) : z0, half ? __builtin_amdgcn_alignbyte(z2, z1, 2) : z1,
                            half ? __builtin_amdgcn_alignbyte(z3, z2, 2) : z2, half ? __builtin_amdgcn_alignbyte(z4, z3, 2) : z3};
            continue;
        }
        uint32_t c = col[u];
        int64_t r = row[u];
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        bool pending = false;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (c >= row_units) { c = 0; ++r; }
            if (d + i < total_units) {
                const int32_t token = tile_key[r - row0];
                if (PHASE != 0 && source.pending(token)) pending = true;
                if (PHASE != 1 || !pending) {
                    const uint8_t* base = source.address(token, r);
                    if (base) w[i] = ((GlobalU32Ptr)base)[c];
                }
            }
            ++c;
        }
        if (PHASE != 0) write[u] = (PHASE == 2) == pending;
        vals[u] = u32x4{w[0], w[1], w[2], w[3]};
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
        const int64_t d = tile + (threadIdx.x + u * kThreads) * kPer;
        if (PHASE != 0 && !write[u]) continue;
        if (d + kPer <= total_units) {
            __builtin_nontemporal_store(vals[u], reinterpret_cast<u32x4*>(out + d * UNIT));
        } else {
            const uint32_t w[4] = {vals[u].x, vals[u].y, vals[u].z, vals[u].w};
#pragma unroll
            for (int i = 0; i < (int)kPer; ++i) {
                if (d + i >= total_units) continue;
                if (UNIT == 4) reinterpret_cast<uint32_t*>(out)[d + i] = w[i];
                else reinterpret_cast<uint16_t*>(out)[d + i] = (uint16_t)(w[i / 2] >> (16 * (i & 1)));
            }
        }
    }
}

// ---- gather with source rows owned by L2 partitions ------------------------------
// The chip's L2 is split over kOwnerClasses dies, each caching what its own compute
// units read; workgroups go to the dies round-robin, so workgroup b runs on die
// b % kOwnerClasses. A source table a few times larger than one die's L2 but smaller
// than all of them together is re-read from memory again and again when every
// workgroup may read every row. Here a Source also gives every request an owner class,
// a function of the source row (so that one die reads a row, and only it), or of the
// request's position for rows so popular that they sit in every L2 anyway.
// Work is handed out in output lines of 128 bytes: a line belongs to the class of the
// output row that holds its first byte, so every line is written whole by one workgroup.
// kOwnerClasses workgroups look at the same super-tile of kOwnedTileLines lines; each
// lists the rows of its class (all per-row arithmetic done once per row, into LDS) and
// spreads the 16-byte chunks of their lines over its lanes. The chunks of a row's last
// line that lie beyond the row's end belong to the next output row and are read there.
// The assumption about where workgroups run only affects speed, never results.
constexpr int kOwnerClasses = 8;
// PHASE 2 can have few rows (the cache's misses) or most of the output; how many only the device knows, so the launch
// decides at run time.
//   * Few: one workgroup takes all of a super-tile's, so that there is something for its lanes to do. Below
//     kOwnedLateBlocks units (as many as are resident twice over) all classes take part, since one each would leave
//     compute units idle: 5 000 rows of 1652 bytes, 88 % late, 75 us with 43 workgroups, 60 with 344 (61 in PHASE 0
//     after the staging).
//   * From kWholeShare on: the whole output is written once more as in PHASE 0, every line once and by its class.
//     1.33 M rows of 1652 bytes, lookups with all, 90, 80, 70 % of the rows late, requests without skew: 1.25, 1.12,
//     1.00, 0.88 ms writing the late ones only, 1.05, 0.98, 0.92, 0.87 writing all (1.02, 0.95, 0.89, 0.84 in PHASE 0
//     after the staging). Not where a popular row is late: its class has more to do than the others, and every partition
//     has it in its L2 anyhow (power-law requests, 83 % late: 0.88 ms the late ones only, 0.98 all).
constexpr uint32_t kOwnedLateBlocks = 4096;
constexpr double kWholeShare = 0.78;
constexpr int kLateUnits = 4;             // per workgroup; with one each, 90 000 empty ones cost a lookup without misses 11 us
constexpr int kOwnedTileLines = 1536;     // 192 KiB of output per super-tile: about 1500 chunks per workgroup; smaller
                                          // tiles leave the workgroups' shares too uneven, larger ones cost LDS
                                          // (PHASE 2 takes the same time from 768 to 3072)
constexpr int kOwnedMinRowBytes = 512;
constexpr int kOwnedMaxRowBytes = 16384;
constexpr int kOwnedMaxRows = kOwnedTileLines * 128 / kOwnedMinRowBytes + 3;

// Geometry of such a launch, worked out by the host.
struct ChunkGrid {   // slots: 16-byte chunks of the most lines a row can own; the rest for dividing by that
    uint32_t slots, slot_magic, step_rows, step_rest;
};
struct OwnedLines {
    uint32_t row_bytes;
    ChunkGrid chunks, late_chunks;   // PHASES 2 and 3 take the second while they only write rows that were on their way
    int64_t total_bytes, n_rows;
    uint32_t tiles, late_classes, whole_from;   // PHASES 2 and 3: super-tiles; classes; how many late rows make it write everything
};

// In PHASE 1 only the lines of rows that are there are written, up to where a pending row begins. In
// PHASES 2 and 3 a pending row's share is the whole range from its own first byte (inside a line of the row
// before it) to the end of its last line, in PHASE 3 up to where a row begins that is still on its way.
template <typename Source, int PHASE, typename Beside>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void gather_owned_lines_kernel(
    Source source, const OwnedLines g, const uint8_t* __restrict__ zeros, uint8_t* __restrict__ out, const Beside beside) {
    if (Beside::kAny && blockIdx.x < beside.blocks) {
        __shared__ int32_t lds[Beside::kAny ? kBesideWords : 1];
        beside.run(blockIdx.x, lds);
        return;
    }
    const uint32_t block = Beside::kAny ? blockIdx.x - beside.blocks : blockIdx.x;
    __shared__ int32_t tile_key[kOwnedMaxRows + 1];
    __shared__ const uint8_t* own_base[kOwnedMaxRows];   // source row, or `zeros` with the zero flag set
    __shared__ const uint8_t* own_next[kOwnedMaxRows];   // source row of the next output row minus row_bytes (same flag rule); null: not to be written
    __shared__ uint32_t own_meta[kOwnedMaxRows];          // first line in the tile + 256 | lines << 12 | (bytes before the first line + bias) << 20
                                                          // | bit 30: this row is zeros | bit 31: the next row is zeros
    __shared__ uint32_t n_owned;

    const uint32_t row_bytes = g.row_bytes;
    const int64_t total_bytes = g.total_bytes, n_rows = g.n_rows;
    // a unit of work is a super-tile's rows of one class (or all); before PHASE 2 a workgroup has exactly one
    uint32_t classes = kOwnerClasses, units = 0;
    bool only_late = false;   // write the rows that were on their way in PHASE 1, not the others
    if constexpr (PHASE >= 2) {
        const uint32_t late = source.late();
        if (late == 0) return;
        only_late = late < g.whole_from || source.late_skewed();
        // where the whole output is written once more it is PHASE 2 that does it
        if (!source.begin(PHASE) || (PHASE == 3 && !only_late)) return;
        if (only_late) classes = g.late_classes;
        units = classes * g.tiles;
        if (block >= units) return;
    }
    const ChunkGrid chunks = only_late ? g.late_chunks : g.chunks;
    const uint32_t slots = chunks.slots;
    const int32_t bias = only_late ? 128 : 0;   // the first line of a row may then begin before the row
    for (uint32_t unit = block;;) {
        const uint32_t cls = unit % classes;
        const int64_t line0 = (int64_t)(unit / classes) * kOwnedTileLines;
        const int64_t total_lines = (total_bytes + 127) >> 7;
        const uint32_t lines_here = (uint32_t)(total_lines - line0 < kOwnedTileLines ? total_lines - line0 : kOwnedTileLines);
        const int64_t tile_byte0 = line0 * 128;
        const uint32_t tile_limit = (uint32_t)(total_bytes - tile_byte0 < (int64_t)kOwnedTileLines * 128 ? total_bytes - tile_byte0
                                                                                                      : (int64_t)kOwnedTileLines * 128);
        const int64_t r0 = tile_byte0 / row_bytes;                              // row holding the tile's first byte
        int64_t r_last = (tile_byte0 + (int64_t)lines_here * 128 - 1) / row_bytes;   // row holding its last byte
        if (r_last > n_rows - 1) r_last = n_rows - 1;
        const int rows_here = (int)(r_last - r0 + 1);                           // <= kOwnedMaxRows - 1
        const int keys_here = rows_here + (r_last + 1 < n_rows ? 1 : 0);        // + the row the last line may run into
        if (threadIdx.x == 0) n_owned = 0;
        for (int i = threadIdx.x; i < keys_here; i += kThreads) tile_key[i] = source_token<PHASE>(source, r0 + i);
        __syncthreads();
        for (int i = threadIdx.x; i < rows_here; i += kThreads) {
            const int64_t r = r0 + i;
            const int32_t key = tile_key[i];
            if (PHASE == 1 && source.pending(key)) continue;
            if constexpr (PHASE >= 2)
                if (only_late && !source.template in_phase<PHASE>(key)) continue;
            if ((PHASE < 2 || classes > 1) && source.owner(key, r) != cls) continue;
            const int64_t begin = r * row_bytes;
            // lines whose first byte is in row r, and for late rows the one that row r begins in
            const int64_t first = (begin + (only_late ? 0 : 127)) >> 7, next = (begin + row_bytes + 127) >> 7;
            const uint8_t* base = source.address(key, r);
            bool later = false;                                                     // the next row is another phase's
            if (PHASE == 1) later = i + 1 < keys_here && source.pending(tile_key[i + 1]);
            if constexpr (PHASE == 3) later = i + 1 < keys_here && source.after(tile_key[i + 1]);
            const uint8_t* after = i + 1 < keys_here && !later ? source.address(tile_key[i + 1], r + 1) : nullptr;
            const uint32_t at = atomicAdd(&n_owned, 1u);
            own_base[at] = base ? base : zeros;
            own_next[at] = after ? after - row_bytes : (later ? nullptr : zeros);
            own_meta[at] = (uint32_t)(first - line0 + 256) | ((uint32_t)(next - first) << 12) | ((uint32_t)(first * 128 - begin + bias) << 20) |
                           (base ? 0u : 1u << 30) | (after ? 0u : 1u << 31);
        }
        __syncthreads();

        const uint32_t items = n_owned * slots;          // `slots` 16-byte chunks per owned row, some of them beyond its lines
        for (uint32_t round = 0; round < items; round += kTile) {
            const uint8_t* from[kUnroll];
            uint32_t out_off[kUnroll], which[kUnroll], in_off[kUnroll];
            bool whole[kUnroll], cross[kUnroll];
            // (in_off: bytes from the row's start; from PHASE 2 on negative before it)
            // one division per thread: its further chunks lie kThreads = step_rows * slots + step_rest chunks on
            const uint32_t w0 = round + threadIdx.x;
            uint32_t j = __umulhi(w0, chunks.slot_magic), within = w0 - j * slots;   // exact: w0 * slots < 2^32
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const bool live = round + threadIdx.x + u * kThreads < items;
                const uint32_t jj = live ? j : 0u;
                const uint32_t meta = own_meta[jj];
                const uint32_t line = (meta & 4095u) + (within >> 3) - 256u;          // relative to the tile; wraps if before it
                bool mine = live && (within >> 3) < ((meta >> 12) & 255u) && line < lines_here;
                out_off[u] = line * 128u + (within & 7u) * 16u;
                const int32_t off = (int32_t)(((meta >> 20) & 255u) + within * 16u) - bias;
                const bool beyond = off >= (int32_t)row_bytes;                         // the chunk lies in the next output row
                const uint8_t* base = beyond ? own_next[jj] : own_base[jj];
                const bool zero = (meta >> (beyond ? 31 : 30)) & 1u;
                if (PHASE & 1) mine = mine && base != nullptr;
                if (PHASE >= 2) mine = mine && off > -16;                              // wholly the row before's otherwise
                whole[u] = mine && out_off[u] + 16u <= tile_limit && (beyond || off + 16 <= (int32_t)row_bytes) && (PHASE < 2 || off >= 0);
                cross[u] = mine && !whole[u] && out_off[u] < tile_limit;
                from[u] = (whole[u] && !zero) ? base + off : zeros;
                in_off[u] = (uint32_t)off;
                which[u] = jj;
                j += chunks.step_rows;
                within += chunks.step_rest;
                if (within >= slots) {
                    within -= slots;
                    ++j;
                }
            }
            u32x4 vals[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) vals[u] = ((GlobalChunk16Ptr)from[u])->v;
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                if (!cross[u]) continue;
                // dword by dword: the rest of the row, then the start of the next one (or the output's ragged
                // end); what another phase or the row before writes is left out
                const uint32_t meta = own_meta[which[u]];
                const uint8_t *a = own_base[which[u]], *b = own_next[which[u]];
                uint32_t wds[4] = {0u, 0u, 0u, 0u};
                uint32_t* const to = reinterpret_cast<uint32_t*>(out + tile_byte0 + out_off[u]);
                bool all = true;
                bool ours[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int32_t off = (int32_t)in_off[u] + 4 * e;
                    const bool beyond = off >= (int32_t)row_bytes;
                    const bool zero = (meta >> (beyond ? 31 : 30)) & 1u;
                    ours[e] = out_off[u] + 4u * e < tile_limit && (!(PHASE & 1) || !beyond || b) && (PHASE < 2 || off >= 0);
                    all = all && ours[e];
                    if (ours[e] && !zero) wds[e] = *(GlobalU32Ptr)((beyond ? b : a) + off);
                }
                vals[u] = u32x4{wds[0], wds[1], wds[2], wds[3]};
                whole[u] = all;                  // stored below with the others
                if (all) continue;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (ours[e]) to[e] = wds[e];
            }
            uint8_t* tile_out = out + tile_byte0;
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                if (whole[u]) __builtin_nontemporal_store(vals[u], reinterpret_cast<u32x4*>(tile_out + out_off[u]));
            }
        }
        if (PHASE < 2 || (unit += gridDim.x - beside.blocks) >= units) return;
        __syncthreads();   // the lists are made again
    }
}

template <typename V, typename Source>
__global__ __launch_bounds__(kThreads) void gather_elems_kernel(Source source, uint32_t row_elems,
                                                                int64_t total_elems, V* __restrict__ out) {
    const int64_t tile = (int64_t)blockIdx.x * kTile;
    int64_t row0;
    if (tile < ((int64_t)1 << 32)) row0 = (uint32_t)tile / row_elems;
    else row0 = tile / (int64_t)row_elems;
    const uint32_t col0 = (uint32_t)(tile - row0 * row_elems);

    V vals[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
        const uint32_t e = col0 + threadIdx.x + u * kThreads;
        const uint32_t dr = e / row_elems;
        const uint32_t col = e - dr * row_elems;
        const int64_t g = tile + threadIdx.x + u * kThreads;
        vals[u] = zero_of<V>();
        if (g < total_elems) {
            const int64_t row = row0 + dr;
            const uint8_t* base = source.address(source_token<0>(source, row), row);
            if (base) vals[u] = reinterpret_cast<const V*>(base)[col];
        }
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
        const int64_t g = tile + threadIdx.x + u * kThreads;
        if (g < total_elems) __builtin_nontemporal_store(vals[u], out + g);
    }
}

// Largest power-of-two width (16, 8, 4, 2 or 1) dividing everything given.
inline int common_alignment(uint64_t bits) {
    if ((bits & 15) == 0) return 16;
    if ((bits & 7) == 0) return 8;
    if ((bits & 3) == 0) return 4;
    if ((bits & 1) == 0) return 2;
    return 1;
}

template <typename V, typename Source>
inline void launch_elems(const Source& source, int32_t row_bytes, int64_t n, void* out, hipStream_t stream) {
    const uint32_t row_elems = (uint32_t)(row_bytes / (int)sizeof(V));
    const int64_t total = n * (int64_t)row_elems;
    const int64_t blocks = (total + kTile - 1) / kTile;
    hipLaunchKernelGGL((gather_elems_kernel<V, Source>), dim3((unsigned)blocks), dim3(kThreads), 0, stream, source,
                       row_elems, total, reinterpret_cast<V*>(out));
}

// Flat gather in 16-byte chunks of the output; UNIT (4 or 2) divides everything.
template <int UNIT> inline int64_t chunk_blocks(int32_t row_bytes, int64_t n) {
    return (n * (int64_t)(row_bytes / UNIT) + kTile * (16 / UNIT) - 1) / (kTile * (16 / UNIT));
}
template <int UNIT, int PHASE, typename Source, typename Beside = NothingBeside, typename Parts = OnePart>
inline bool launch_chunks(const Source& source, int32_t row_bytes, int64_t n, void* out, const uint8_t* zeros, hipStream_t stream,
                          const Beside& beside = {}, const Parts& parts = {}, int64_t more_blocks = 0) {
    const uint32_t row_units = (uint32_t)row_bytes / UNIT, tile_units = kTile * (16 / UNIT);
    const int64_t total = n * (int64_t)row_units;
    const int64_t blocks = chunk_blocks<UNIT>(row_bytes, n) + beside.blocks + more_blocks;
    if (blocks > 0x7fffffffLL) return false;
    // the in-block offsets stay below row_units + tile_units: exact while that is < 2^32 / row_units
    const bool small = (uint64_t)row_units * ((uint64_t)row_units + tile_units) < ((uint64_t)1 << 32);
    if (small && row_units > 1) {
        const uint32_t magic = (uint32_t)((((uint64_t)1 << 32) + row_units - 1) / row_units);
        hipLaunchKernelGGL((gather_chunks_kernel<Source, true, UNIT, PHASE, Beside, Parts>), dim3((unsigned)blocks), dim3(kThreads), 0, stream,
                           source, row_units, magic, total, n - 1, zeros, static_cast<uint8_t*>(out), beside, parts);
    } else {
        hipLaunchKernelGGL((gather_chunks_kernel<Source, false, UNIT, PHASE, Beside, Parts>), dim3((unsigned)blocks), dim3(kThreads), 0, stream,
                           source, row_units, 0u, total, n - 1, zeros, static_cast<uint8_t*>(out), beside, parts);
    }
    return true;
}

// Device address of 16 zero bytes (defined once, in gather.hip); nullptr on failure.
const uint8_t* zero_chunk();

// Rows that are only 2-byte aligned: whether the chunk kernel is faster than an element of 2 bytes per thread. Its blocks
// write 16 KiB where the other's write 2, so small outputs leave compute units idle; in short rows most pieces cross a
// row end, which costs two loads from rows that are far apart. Time over the other kernel's, table of 20 000 / 1 M rows:
// 66-byte rows 1.27 / 1.24 at 1 MiB of output, 0.97 / 0.97 at 4, 0.75 / 0.74 at 16; 2050-byte rows 1.17 / 1.18, 0.89 /
// 0.89, 0.51 / 0.49; 34-byte rows 1.03 / 0.84 at 7 MB, 0.94 / 1.34 at 34, 0.62 / 1.35 at 136 (the second from 3 M rows, out
// of cache); 48-byte rows, which no piece crosses, 0.98 / 0.99, 0.79 / 0.77, 0.55 / 0.71.
inline bool two_byte_chunks_pay(int32_t row_bytes, int64_t out_bytes, int64_t table_bytes) {
    if (row_bytes >= 32 && row_bytes % 16 == 0) return out_bytes >= (int64_t)1 << 20;
    if (row_bytes >= 56) return out_bytes >= (int64_t)1 << 22;
    return row_bytes >= 16 && out_bytes >= (int64_t)1 << 25 && table_bytes <= (int64_t)1 << 22;   // a table that one L2 holds
}

// `src_align`: power of two dividing the row size, every source pitch and every
// source base address. Returns false if the launch would need more blocks than
// a grid dimension holds.
template <typename Source>
inline bool launch(const Source& source, int src_align, int32_t row_bytes, int64_t n, void* out, hipStream_t stream) {
    if (n == 0) return true;
    const uint8_t* zeros = zero_chunk();
    if (!zeros) return false;
    const uint64_t out_bits = (uint64_t)(uintptr_t)out;
    // the chunk kernel wherever its 16-byte pieces apply (an aligned output, and rows that a piece crosses at most once
    // unless its dword path can follow) and pay
    if ((out_bits & 15) == 0 && src_align >= 4) return launch_chunks<4, 0>(source, row_bytes, n, out, zeros, stream);
    if constexpr (Source::kAlign < 4)
        if ((out_bits & 15) == 0 && two_byte_chunks_pay(row_bytes, n * row_bytes, source.table_bytes()))
            return launch_chunks<2, 0>(source, row_bytes, n, out, zeros, stream);
    const int align = common_alignment((uint64_t)src_align | out_bits);
    const int64_t total = n * (int64_t)(row_bytes / align);
    if ((total + kTile - 1) / kTile > 0x7fffffffLL) return false;
    switch (align) {
        case 8: launch_elems<u32x2>(source, row_bytes, n, out, stream); break;
        case 4: launch_elems<uint32_t>(source, row_bytes, n, out, stream); break;
        default:
            if constexpr (Source::kAlign < 4) launch_elems<uint16_t>(source, row_bytes, n, out, stream);
            break;
    }
    return true;
}

// Whether the line-owner gather applies and pays: long enough rows, enough requests, an aligned output.
inline bool owned_applies(int src_align, int32_t row_bytes, int64_t n, const void* out) {
    return src_align >= 4 && ((uintptr_t)out & 15) == 0 && row_bytes >= kOwnedMinRowBytes && row_bytes <= kOwnedMaxRowBytes && n >= 4096;
}

inline ChunkGrid chunk_grid(uint32_t lines) {
    ChunkGrid g;
    g.slots = lines * 8u;
    // items of a workgroup stay far below 2^32 / slots: the multiply-high division is exact
    g.slot_magic = (uint32_t)((((uint64_t)1 << 32) + g.slots - 1) / g.slots);
    g.step_rows = (uint32_t)kThreads / g.slots;
    g.step_rest = (uint32_t)kThreads % g.slots;
    return g;
}

template <int PHASE, typename Source, typename Beside = NothingBeside>
inline bool launch_owned(const Source& source, int32_t row_bytes, int64_t n, void* out, const uint8_t* zeros, hipStream_t stream,
                         const Beside& beside = {}) {
    OwnedLines g = {};
    g.row_bytes = (uint32_t)row_bytes;
    g.total_bytes = n * (int64_t)row_bytes;
    g.n_rows = n;
    const uint32_t lines = (uint32_t)(row_bytes + 127) / 128;
    g.chunks = chunk_grid(lines);
    const int64_t tiles = ((g.total_bytes + 127) / 128 + kOwnedTileLines - 1) / kOwnedTileLines;
    int64_t blocks = tiles * kOwnerClasses;
    if (blocks > 0x7fffffffLL) return false;
    if (PHASE >= 2) {
        g.late_chunks = chunk_grid(lines + 1);
        g.tiles = (uint32_t)tiles;
        g.late_classes = blocks <= kOwnedLateBlocks ? kOwnerClasses : 1;
        const int64_t whole_from = (int64_t)((double)n * kWholeShare);
        g.whole_from = whole_from < 0xffffffffLL ? (uint32_t)whole_from : 0xffffffffu;
        // several units to a workgroup of a large launch, since few rows leave most of it without any; a multiple of the
        // classes, so that the units of class c are done by workgroups whose number is c modulo the classes
        if (blocks > kOwnedLateBlocks) blocks = blocks / kLateUnits > kOwnedLateBlocks ? blocks / kLateUnits : kOwnedLateBlocks;
        blocks = (blocks + kOwnerClasses - 1) / kOwnerClasses * kOwnerClasses;
    }
    blocks += beside.blocks;
    if (blocks > 0x7fffffffLL) return false;
    hipLaunchKernelGGL((gather_owned_lines_kernel<Source, PHASE, Beside>), dim3((unsigned)blocks), dim3(kThreads), 0, stream, source, g,
                       zeros, static_cast<uint8_t*>(out), beside);
    return true;
}

}  // namespace taser_gather
