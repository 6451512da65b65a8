// Row copies shared by the gather, embed and pipelined kernels.
#pragma once

#include "scone_internal.h"

namespace scone {

// One wavefront copies part `part` of W equal parts of the row of ids[r]
// (64*U 16-byte units in all: 1, 2, 4 or 8 KiB) into row r of `out`.  The
// id is wave-uniform, so every load is a scalar row base plus the lane
// offset; all U/W loads are issued before the U/W stores, which are
// non-temporal (the output is not re-read by this path).  An id outside
// [0, n_rows) writes zeros and raises SCONE_EROW.  All 64 lanes call it.
template <int U, int W>
__device__ __forceinline__ void copy_row_part(const int32_t* __restrict__ ids, int64_t r,
                                              int part, const u32x4* __restrict__ rows,
                                              int64_t n_rows, u32x4* __restrict__ out,
                                              unsigned* __restrict__ err) {
    static_assert(W >= 1 && U % W == 0, "W must divide the row's units");
    constexpr int UW = U / W;
    const int lane = threadIdx.x & 63;
    const int64_t id = ids[r];
    const bool ok = (id >= 0) & (id < n_rows);
    const u32x4* src = rows + (ok ? id : 0) * (64 * U) + part * (64 * UW);
    u32x4 v[UW];
#pragma unroll
    for (int u = 0; u < UW; ++u) v[u] = src[u * 64 + lane];
    u32x4* dst = out + r * (64 * U) + part * (64 * UW);
#pragma unroll
    for (int u = 0; u < UW; ++u)
        __builtin_nontemporal_store(ok ? v[u] : u32x4{}, dst + u * 64 + lane);
    if (!ok && lane == 0 && part == 0) atomicOr(err, err_bit(SCONE_EROW));
}

// Wavefronts per row of 64*U units for the standalone gather and for the
// gather half of the pipelined step.  Measured on rows of 4 KiB over a 41 GB
// table: the standalone gather with 1 KiB per wavefront is 2% faster on the
// Zipf workload and 8% faster on uniform random ids than with whole rows;
// inside the pipelined step, next to the lookup workgroups, 2 KiB per
// wavefront is the fastest (whole rows and 1 KiB parts are 3-4% slower).
// Rows of 1 and 2 KiB stay whole: on the 2 KiB-row workload, 1 KiB parts
// cost 15% on its Zipf ids, which mostly hit the caches.
__host__ __device__ constexpr int gather_row_waves(int U) { return U >= 4 ? U : 1; }
__host__ __device__ constexpr int pipelined_row_waves(int U) { return U >= 4 ? U / 2 : 1; }

// Units per row (16 bytes each) that copy_row_part handles, as its U; 0 otherwise.
__host__ __device__ constexpr int wave_row_units(int64_t row_bytes) {
    return row_bytes == 1024 ? 1 : row_bytes == 2048 ? 2 : row_bytes == 4096 ? 4
                                                       : row_bytes == 8192 ? 8 : 0;
}

// ------------------------------------------------------- rows of any width --
// A row of at least 16 bytes is copied as ceil(row_bytes / 16) units of 16 bytes,
// at byte 16 c of the row; where the width is no multiple of 16 the last unit
// lies 16 bytes before the row's end, over part of the one before it (both
// write the same bytes).  Loads and stores are 16 bytes whatever the
// alignment: global memory takes unaligned dwordx4 accesses, and the type below
// says so to the compiler.  A unit's row is its index over the units per row, by
// multiplication.  Before, the gather took 64-bit divisions and units as narrow as
// the alignment, and the fused kernel single bytes: 131K rows of 2002 bytes took
// 166 us to gather (now 84, 6.3 TB/s), of 4100 bytes 198 us (now 162), and 26K
// rows of 3 KiB 95 us in the fused kernel (now 27.5).  Widths that 16 divides moved
// by less than 7%, all of them down; the gather's widths that 8 divides and 16
// doesn't were 5% slower and have units of their own.

typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(1)));

struct RowUnits {
    int64_t row_bytes;
    uint64_t mul64;  // floor(2^64 / upr) + 1 (unused for upr = 1)
    uint32_t upr;    // units per row
    uint32_t mul;    // floor(2^(31 + log) / upr) + 1
    int log;         // the smallest with 2^log >= upr

    // k / upr for k < 2^31: mul * upr exceeds 2^(31 + log) by at most upr <= 2^log,
    // so the quotient is exact (Granlund and Montgomery, 1994).
    __device__ __forceinline__ uint32_t div(uint32_t k) const {
        return (uint32_t)(((uint64_t)k * mul) >> (31 + log));
    }
    // i / upr for 0 <= i < 2^62: the product may round up by one.
    __device__ __forceinline__ int64_t div64(int64_t i) const {
        if (upr == 1) return i;
        int64_t q = (int64_t)__umul64hi((uint64_t)i, mul64);
        if (q * upr > i) --q;
        return q;
    }
    __device__ __forceinline__ int64_t offset(int64_t c) const {  // byte of unaligned unit c
        const int64_t o = c * 16;
        return o <= row_bytes - 16 ? o : row_bytes - 16;
    }
};

// Rows that the unit copies handle: unit indexes inside a workgroup (16 rows at
// most, or a row and 1,024 units) stay below 2^31.
inline bool unit_row_bytes(int64_t row_bytes) {
    return row_bytes >= 16 && row_bytes < ((int64_t)1 << 31);
}

inline RowUnits row_units(int64_t row_bytes, int unit_bytes = 16) {
    RowUnits u;
    u.row_bytes = row_bytes;
    u.upr = (uint32_t)((row_bytes + unit_bytes - 1) / unit_bytes);
    u.log = 0;
    while (((uint64_t)1 << u.log) < u.upr) ++u.log;
    u.mul = (uint32_t)(((uint64_t)1 << (31 + u.log)) / u.upr + 1);
    u.mul64 = u.upr > 1 ? ~0ull / u.upr + 1 : 0;
    return u;
}

// Workgroup `blk` of 256 threads copies units [blk * 256 U, (blk + 1) * 256 U) of
// the n_tok rows of `ids`.  A unit is a V: u32x4_any, or a narrower aligned word
// that divides the row (row_units with its size).  Lanes past the end read the last
// row and store nothing.  An id outside [0, n_rows) (n_rows > 0) writes zeros and
// raises SCONE_EROW.
template <int U, typename V>
__device__ __forceinline__ void copy_units(const int32_t* __restrict__ ids, int64_t n_tok,
                                           int64_t blk, const RowUnits& ru,
                                           const uint8_t* __restrict__ rows, int64_t n_rows,
                                           uint8_t* __restrict__ out,
                                           unsigned* __restrict__ err) {
    const int64_t base = blk * (256 * U);
    const int64_t r0 = ru.div64(base);
    const uint32_t c0 = (uint32_t)(base - r0 * ru.upr);
    int64_t r[U], off[U], id[U];
    V v[U];
    bool in[U], ok[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t k = c0 + u * 256 + threadIdx.x;
        const uint32_t q = ru.div(k);
        r[u] = r0 + q;
        const uint32_t c = k - q * ru.upr;
        off[u] = sizeof(V) == 16 ? ru.offset(c) : (int64_t)c * (int64_t)sizeof(V);
        in[u] = r[u] < n_tok;
        if (!in[u]) r[u] = n_tok - 1;
        id[u] = ids[r[u]];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        ok[u] = (id[u] >= 0) & (id[u] < n_rows);
        v[u] = *reinterpret_cast<const V*>(rows + (ok[u] ? id[u] : 0) * ru.row_bytes + off[u]);
    }
    bool bad = false;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (in[u])
            __builtin_nontemporal_store(
                ok[u] ? v[u] : V{}, reinterpret_cast<V*>(out + r[u] * ru.row_bytes + off[u]));
        bad |= in[u] & !ok[u];
    }
    if (bad) atomicOr(err, err_bit(SCONE_EROW));
}

// Units per thread of copy_units.
constexpr int kUnitsPerThread = 4;

inline int64_t unit_blocks(int64_t n_tok, const RowUnits& u, int per_thread = kUnitsPerThread) {
    return (n_tok * u.upr + 256 * per_thread - 1) / (256 * per_thread);
}

}  // namespace scone
