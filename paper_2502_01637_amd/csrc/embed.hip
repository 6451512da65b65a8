// Fused lookup + gather: Algorithm 1's inference branch in one pass.
//
// Each workgroup first resolves the longest match for its tile of positions
// (the same tile lookup as scone_lookup, ids kept in LDS), then copies the
// tile's rows into the contiguous output block that those positions own.
// Fusing removes the id round trip through HBM and the separate
// latency-bound lookup launch.  Tiles are small (16 to 32 KiB of rows) so the
// grid holds many generations of short-lived workgroups: some wait on hash
// probes while the others on the same compute unit keep HBM busy with row
// copies.  Measured on MI355X this matches, within a few percent, the two
// separate kernels back to back: the hash probes are random HBM reads that
// cost bandwidth the row stream would otherwise use, so overlapping them
// hides their latency but not their cost.
#include "row_copy.h"
#include "tile_lookup.h"

namespace scone {
namespace {

// How a tile's rows are cut into units: 16-byte units of rows of 2^shift of them,
// 16-byte aligned; 16-byte units of rows of any width and alignment (RowUnits);
// the same with 64-bit indexes, for rows of 2 GiB and more; or single bytes, for
// rows below 16.
enum RowMode { kRowPow2 = 0, kRowAny = 1, kRowWide = 2, kRowBytes = 3 };

template <RowMode kMode>
struct Unit {
    typedef u32x4_any type;
    typedef uint32_t index;
};
template <>
struct Unit<kRowPow2> {
    typedef u32x4 type;
    typedef uint32_t index;
};
template <>
struct Unit<kRowWide> {
    typedef u32x4_any type;
    typedef uint64_t index;
};
template <>
struct Unit<kRowBytes> {
    typedef uint8_t type;
    typedef uint32_t index;
};

// Row copy helpers for one batch of U units per thread (unit i of the tile's
// output block).  A bad id reads row 0 and the unit is zeroed afterwards, so
// the loads of a batch carry no branch and stay in flight together.
template <RowMode kMode, int U>
struct TileCopy {
    typedef typename Unit<kMode>::type V;
    typedef typename Unit<kMode>::index I;
    const int32_t* s_id;
    const uint8_t* __restrict__ rows;
    uint8_t* __restrict__ dst;
    int64_t n_rows;
    const RowUnits& ru;

    __device__ __forceinline__ I per_row() const {
        return kMode == kRowWide ? (I)((ru.row_bytes + 15) / 16) : (I)ru.upr;
    }
    __device__ __forceinline__ void split(I i, I& r, int64_t& off) const {
        if constexpr (kMode == kRowPow2) {
            r = i >> ru.log;
            off = (int64_t)(i & (ru.upr - 1)) * 16;
        } else if constexpr (kMode == kRowBytes) {
            r = ru.div(i);
            off = (int64_t)(i - r * ru.upr);
        } else {
            r = kMode == kRowWide ? i / per_row() : (I)ru.div((uint32_t)i);
            off = ru.offset(i - r * per_row());
        }
    }
    __device__ __forceinline__ V load_one(I i, bool& ok) const {
        I r;
        int64_t off;
        split(i, r, off);
        const int64_t id = s_id[r];
        ok = (id >= 0) & (id < n_rows);
        const int64_t src = ok ? id : 0;
        const int64_t at = kMode == kRowPow2 ? src << (ru.log + 4) : src * ru.row_bytes;
        return *reinterpret_cast<const V*>(rows + at + off);
    }
    __device__ __forceinline__ void store_one(I i, V v, bool ok) const {
        int64_t at;
        if constexpr (kMode == kRowAny || kMode == kRowWide) {
            I r;
            split(i, r, at);
            at += (int64_t)r * ru.row_bytes;
        } else {
            at = (int64_t)i * sizeof(V);
        }
        __builtin_nontemporal_store(ok ? v : V{}, reinterpret_cast<V*>(dst + at));
    }
    __device__ __forceinline__ void load(I base, V (&v)[U], bool (&ok)[U]) const {
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = load_one(base + u * kTileThreads, ok[u]);
    }
    __device__ __forceinline__ bool store(I base, V (&v)[U], const bool (&ok)[U]) const {
        bool bad = false;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            store_one(base + u * kTileThreads, v[u], ok[u]);
            bad |= !ok[u];
        }
        return bad;
    }
};

template <int SB, int G, RowMode kMode, int U>
__global__ __launch_bounds__(kTileThreads) void k_embed(
    const typename SlotOps<SB>::Slot* __restrict__ slots, uint64_t mask,
    const int32_t* __restrict__ X, int64_t T, int P, int max_n, int64_t tiles_per_row,
    const uint8_t* __restrict__ rows, int64_t n_rows, RowUnits ru, uint8_t* __restrict__ out,
    int32_t* __restrict__ ids_out, int8_t* __restrict__ len_out, unsigned* __restrict__ err,
    int64_t block0) {
    __shared__ int32_t s_tok[TileShape<G>::kPositions + kMaxHalo];
    __shared__ int32_t s_id[TileShape<G>::kPositions];

    const int64_t blk = block_index(block0);
    const int64_t b = blk / tiles_per_row;
    const int64_t t0 = (blk - b * tiles_per_row) * (int64_t)P;
    stage_tokens(s_tok, X + b * T, T, t0, P, max_n - 1);
    __syncthreads();
    if (threadIdx.x < ((P * G + 63) & ~63)) {  // whole waves only
        int32_t id;
        int len;
        bool tok_ok;
        tile_lookup<SB, G>(slots, mask, s_tok, T, t0, P, max_n, id, len, tok_ok);
        const int p = threadIdx.x / G;
        const int64_t t = t0 + p;
        if (threadIdx.x % G == 0 && p < P) {
            s_id[p] = id;
            if (t < T) {
                if (!tok_ok) atomicOr(err, err_bit(SCONE_ETOKEN));
                if (ids_out) ids_out[b * T + t] = id;
                if (len_out) len_out[b * T + t] = (int8_t)len;
            }
        }
    }
    __syncthreads();

    // Copy the tile's rows: positions t0 .. t0+npos-1 own one contiguous
    // output block of npos * upr units.  Whole batches are software-pipelined
    // (the next batch's loads are issued before this batch's stores).
    const uint32_t npos = (uint32_t)((T - t0) < P ? (T - t0) : P);
    const TileCopy<kMode, U> cp{s_id, rows, out + (b * T + t0) * ru.row_bytes, n_rows, ru};
    typedef typename Unit<kMode>::type V;
    typedef typename Unit<kMode>::index I;
    const I total = npos * cp.per_row();
    constexpr I kStride = kTileThreads * U;
    const I whole = total / kStride * kStride;
    bool bad = false;
    I base = threadIdx.x;
    if (whole > 0) {
        V a[U];
        bool oka[U];
        cp.load(base, a, oka);
        for (; base + kStride < whole; base += kStride) {
            V nb[U];
            bool okb[U];
            cp.load(base + kStride, nb, okb);
            bad |= cp.store(base, a, oka);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                a[u] = nb[u];
                oka[u] = okb[u];
            }
        }
        bad |= cp.store(base, a, oka);
        base += kStride;
    }
    for (I i = base; i < total; i += kTileThreads) {  // ragged remainder
        bool okk;
        const V v = cp.load_one(i, okk);
        cp.store_one(i, v, okk);
        bad |= !okk;
    }
    if (bad) atomicOr(err, err_bit(SCONE_EROW));
}

struct Call {
    const scone_table* tb;
    const int32_t* X;
    int64_t B, T;
    int max_n;
    const void* rows;
    int64_t n_rows, row_bytes;
    void* out;
    int32_t* ids;
    int8_t* lens;
    unsigned* err;
    hipStream_t st;
};

template <int SB, int G, RowMode kMode, int U>
hipError_t launch(const Call& c, RowUnits ru) {
    using Slot = typename SlotOps<SB>::Slot;
    // Positions per workgroup: up to 16 positions and 32 KiB of rows, at
    // least 4 positions.  Short-lived workgroups let the probes of some
    // overlap the copies of others on the same compute unit (16 to 32 KiB
    // per workgroup measured best for 2 and 4 KiB rows).
    int P = TileShape<G>::kPositions < 16 ? TileShape<G>::kPositions : 16;
    while (P > 4 && (int64_t)P * c.row_bytes > (32 << 10)) P >>= 1;
    const int64_t tiles = (c.T + P - 1) / P;
    return launch_blocks(c.B * tiles, kTileThreads, [&](int64_t b0, dim3 grid) {
        hipLaunchKernelGGL((k_embed<SB, G, kMode, U>), grid, dim3(kTileThreads), 0, c.st,
                           static_cast<const Slot*>(c.tb->slots), (uint64_t)c.tb->capacity - 1,
                           c.X, c.T, P, c.max_n, tiles, static_cast<const uint8_t*>(c.rows),
                           c.n_rows, ru, static_cast<uint8_t*>(c.out), c.ids, c.lens, c.err, b0);
    });
}

template <RowMode kMode, int U = 4>
hipError_t dispatch(const Call& c, const RowUnits& ru) {
    const bool one = tile_lanes_for(c.max_n) == 1;
    if (c.tb->slot_bytes == 16)
        return one ? launch<16, 1, kMode, U>(c, ru) : launch<16, 2, kMode, U>(c, ru);
    return one ? launch<32, 1, kMode, U>(c, ru) : launch<32, 2, kMode, U>(c, ru);
}

}  // namespace
}  // namespace scone

extern "C" int scone_embed(const scone_table_t* table, const int32_t* token_ids, int64_t B,
                           int64_t T, int32_t max_n, const void* rows, int64_t n_rows,
                           int64_t row_bytes, int32_t placement, void* out, int32_t* fgram_ids,
                           int8_t* match_len, void* stream) {
    using namespace scone;
    if (!table || B < 0 || T < 0 || max_n < 1 || n_rows < 0 || row_bytes <= 0)
        return SCONE_EINVAL;
    if (placement != SCONE_PLACE_HBM && placement != SCONE_PLACE_HOST) return SCONE_EINVAL;
    if (B > 0 && T > ((int64_t)1 << 62) / B) return SCONE_EINVAL;
    if (B * T > ((int64_t)1 << 62) / row_bytes) return SCONE_EINVAL;
    if (B * T == 0) return SCONE_OK;
    if (!token_ids || !out || (!rows && n_rows > 0)) return SCONE_EINVAL;
    {
        const int64_t n = B * T, out_b = n * row_bytes;
        const void* outs[3] = {out, fgram_ids, match_len};
        const int64_t outs_b[3] = {out_b, span_bytes(n, 4), n};
        for (int i = 0; i < 3; ++i) {
            if (overlaps(outs[i], outs_b[i], token_ids, span_bytes(n, 4)) ||
                overlaps(outs[i], outs_b[i], rows, span_bytes(n_rows, row_bytes)))
                return SCONE_EINVAL;
            for (int j = i + 1; j < 3; ++j)
                if (overlaps(outs[i], outs_b[i], outs[j], outs_b[j])) return SCONE_EINVAL;
        }
    }
    int dev = 0;
    SCONE_HIP_TRY(hipGetDevice(&dev));
    if (dev != table->device) return SCONE_EINVAL;
    unsigned* err = device_error_word();
    if (!err) return SCONE_EHIP;
    const int eff = max_n < table->max_len ? max_n : table->max_len;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (n_rows == 0) {
        // No row is valid: the ids are still produced, the output is zeroed.
        hipError_t e0 = hipSuccess;
        if (fgram_ids || match_len)
            e0 = launch_lookup(table, token_ids, B, T, eff, fgram_ids, match_len, err, st);
        if (e0 == hipSuccess) e0 = launch_zero_rows(out, B * T * row_bytes, err, st);
        return status_of(e0);
    }
    const Call c{table, token_ids, B, T, eff, rows, n_rows, row_bytes, out, fgram_ids, match_len,
                 err, st};
    if (row_bytes < 16) return status_of(dispatch<kRowBytes>(c, row_units(row_bytes, 1)));
    if (!unit_row_bytes(row_bytes)) {
        RowUnits wide{};
        wide.row_bytes = row_bytes;
        return status_of(dispatch<kRowWide>(c, wide));
    }
    const RowUnits ru = row_units(row_bytes);
    const uintptr_t align = (uintptr_t)rows | (uintptr_t)out | (uintptr_t)row_bytes;
    const bool pow2 = (align & 15) == 0 && (ru.upr & (ru.upr - 1)) == 0;
    if (pow2) return status_of(dispatch<kRowPow2>(c, ru));
    // Over PCIe a batch of one unit per thread in flight is faster than of four from
    // 1 KiB on (rows that repeat are then in the caches more often): 16K rows of
    // 1,536 bytes 348 us against 359, of 4,608 1,062 against 1,078; 999 rows of 4,608
    // bytes 82 against 98.  Rows of 768 bytes took 184 against 178.
    if (placement == SCONE_PLACE_HOST && row_bytes >= 1024)
        return status_of(dispatch<kRowAny, 1>(c, ru));
    return status_of(dispatch<kRowAny>(c, ru));
}
