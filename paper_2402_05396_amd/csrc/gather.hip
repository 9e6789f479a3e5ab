// taser_gather_features: feature slicing from a table in device memory
// (TASER, arXiv 2402.05396, Sec. 3.4 / Alg. 3: serve the feature row of every
// requested id). A pure byte mover, bounded by HBM bandwidth.
#include "gather_kernel.h"
#include "taser_internal.h"

namespace {

struct TableSource {
    static constexpr int kAlign = 2;
    const uint8_t* table;
    int64_t pitch_bytes;
    const int32_t* ids;
    int64_t rows;
    int64_t table_bytes() const { return rows * pitch_bytes; }
    __device__ __forceinline__ int32_t key(int64_t i) const { return ids[i]; }
    __device__ __forceinline__ int32_t resolve(int32_t id) const { return id; }
    __device__ __forceinline__ bool pending(int32_t) const { return false; }
    __device__ __forceinline__ const uint8_t* address(int32_t id, int64_t) const {
        const bool ok = id >= 0 && id < rows;
        const uint8_t* at = table + (int64_t)(ok ? id : 0) * pitch_bytes;   // computed either way: no branch
        return ok ? at : nullptr;
    }
};

// Up to two gathers after the first: where their blocks begin, their ids and outputs.
struct MoreParts {
    static constexpr bool kMore = true;
    struct Part {
        uint32_t first_block;
        const int32_t* ids;
        int64_t total_units, last_row;
        uint8_t* out;
    } part[2];
    __device__ __forceinline__ uint32_t enter(uint32_t block, TableSource& source, int64_t& total_units, int64_t& last_row,
                                                    uint8_t* __restrict__& out) const {
        const int p = block >= part[1].first_block ? 1 : block >= part[0].first_block ? 0 : -1;   // uniform
        if (p < 0) return block;
        source.ids = part[p].ids;
        total_units = part[p].total_units;
        last_row = part[p].last_row;
        out = part[p].out;
        return block - part[p].first_block;
    }
};

template <int UNIT>
bool launch_parts(const TableSource& source, int32_t row_bytes, const TaserGatherPart* parts, int n_parts, const uint8_t* zeros, hipStream_t stream) {
    using namespace taser_gather;
    int64_t blocks = chunk_blocks<UNIT>(row_bytes, parts[0].n);
    const int64_t first = blocks;
    MoreParts more;
    for (int i = 0; i < 2; ++i) {
        more.part[i] = MoreParts::Part{0xffffffffu, nullptr, 0, 0, nullptr};
        if (i + 1 >= n_parts) continue;
        const TaserGatherPart& p = parts[i + 1];
        if (blocks > 0x7fffffffLL) return false;
        more.part[i] = MoreParts::Part{(uint32_t)blocks, p.ids, p.n * (int64_t)(row_bytes / UNIT), p.n - 1, static_cast<uint8_t*>(p.out)};
        blocks += chunk_blocks<UNIT>(row_bytes, p.n);
    }
    return launch_chunks<UNIT, 0>(source, row_bytes, parts[0].n, parts[0].out, zeros, stream, NothingBeside{}, more, blocks - first);
}

}  // namespace

// 16 zero bytes in device memory. External linkage and "used": a device variable
// that no kernel names is otherwise dropped from the code object, and looking it
// up by symbol then fails inside the runtime.
__device__ __attribute__((used)) uint32_t taser_zero_chunk_storage[4] = {0u, 0u, 0u, 0u};

const uint8_t* taser_gather::zero_chunk() {
    // per device: every GPU holds its own copy of the symbol
    static const uint8_t* cached[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    if (!cached[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(taser_zero_chunk_storage)) != hipSuccess) return nullptr;
        cached[dev] = static_cast<const uint8_t*>(p);
    }
    return cached[dev];
}

void taser_resolve_device_constants() { (void)taser_gather::zero_chunk(); }

int taser_launch_gather(const void* table, int64_t rows, int32_t row_bytes, int64_t pitch_bytes, const int32_t* ids,
                        int64_t n, void* out, hipStream_t stream) {
    taser_clear_stale_hip_error();
    const int align = taser_gather::common_alignment((uint64_t)row_bytes | (uint64_t)pitch_bytes |
                                                     (uint64_t)(uintptr_t)table);
    const TableSource source{static_cast<const uint8_t*>(table), pitch_bytes, ids, rows};
    TaserProfileSpan span(stream, "gather_rows");
    if (!taser_gather::launch(source, align, row_bytes, n, out, stream))
        return taser_fail(TASER_E_RANGE, "gather: %lld rows of %d bytes exceed one launch", (long long)n, row_bytes);
    TASER_HIP_TRY(hipGetLastError());
    return TASER_OK;
}

int taser_launch_gather_parts(const void* table, int64_t rows, int32_t row_bytes, int64_t pitch_bytes, const TaserGatherPart* parts,
                              int n_parts, hipStream_t stream) {
    const int align = taser_gather::common_alignment((uint64_t)row_bytes | (uint64_t)pitch_bytes | (uint64_t)(uintptr_t)table);
    // one launch where every part's output suits the chunk kernel and all blocks fit
    int64_t n = 0;
    for (int i = 0; i < n_parts; ++i) n += parts[i].n;
    bool together = n_parts > 1 && n_parts <= 3 && (align >= 4 || taser_gather::two_byte_chunks_pay(row_bytes, n * row_bytes, rows * pitch_bytes));
    for (int i = 0; i < n_parts; ++i) together = together && parts[i].n > 0 && ((uintptr_t)parts[i].out & 15) == 0;
    if (together) {
        taser_clear_stale_hip_error();
        const uint8_t* zeros = taser_gather::zero_chunk();
        if (!zeros) return taser_fail(TASER_E_HIP, "gather: the zero constant is not available on this device");
        const TableSource source{static_cast<const uint8_t*>(table), pitch_bytes, parts[0].ids, rows};
        TaserProfileSpan span(stream, "gather_rows");
        together = align >= 4 ? launch_parts<4>(source, row_bytes, parts, n_parts, zeros, stream)
                              : launch_parts<2>(source, row_bytes, parts, n_parts, zeros, stream);
        TASER_HIP_TRY(hipGetLastError());
    }
    for (int i = 0; i < n_parts && !together; ++i) {
        const int rc = taser_launch_gather(table, rows, row_bytes, pitch_bytes, parts[i].ids, parts[i].n, parts[i].out, stream);
        if (rc != TASER_OK) return rc;
    }
    return TASER_OK;
}

extern "C" int taser_gather_features(const void* table, int64_t rows, int32_t row_bytes,
                                     int64_t pitch_bytes, const int32_t* ids, int64_t n, void* out,
                                     void* hip_stream) {
    if (n < 0 || rows < 0) return taser_fail(TASER_E_ARG, "gather_features: negative size");
    if (row_bytes <= 0 || (row_bytes & 1)) return taser_fail(TASER_E_ARG, "gather_features: row_bytes = %d must be positive and even", row_bytes);
    if (pitch_bytes < row_bytes || (pitch_bytes & 1)) return taser_fail(TASER_E_ARG, "gather_features: pitch_bytes = %lld must be even and >= row_bytes", (long long)pitch_bytes);
    if (n == 0) return TASER_OK;
    if (!ids || !out) return taser_fail(TASER_E_ARG, "gather_features: null ids or out");
    if (!table && rows > 0) return taser_fail(TASER_E_ARG, "gather_features: null table");
    if (((uintptr_t)out & 1) || ((uintptr_t)table & 1)) return taser_fail(TASER_E_ARG, "gather_features: table and out must be 2-byte aligned");
    return taser_launch_gather(table, rows, row_bytes, pitch_bytes, ids, n, out, (hipStream_t)hip_stream);
}
