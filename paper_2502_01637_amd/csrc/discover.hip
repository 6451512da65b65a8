// F-gram discovery on the device: Algorithm 3 with the K-1 linear scans of
// Section 3.1.
//
// Scan n counts the n-grams of every sequence by an exact 64-bit code.  For
// n = 2 the code is (t0 << 16) | t1.  From n = 3 on, an n-gram is counted only
// when both its (n-1)-prefix and its (n-1)-suffix survived scan n-1 (count >=
// the minimum count): an n-gram that reaches the minimum appears inside both
// of them at least as often, so nothing that could survive is skipped.  Every
// survivor of scan n-1 has a dense id, and an n-gram is coded as (dense id of
// its prefix << 16) | last token, which is exact and fits 47 bits at any
// length.  After each scan the survivors get dense ids and every position
// learns the id of the survivor ending there (or -1), which is all the next
// scan reads.
//
// A scan counts without a global counting table.  A random read or atomic
// update reaches about 20 G/s on this card whatever it carries, and a table
// for every distinct n-gram took 28M of them per scan of 16.8M tokens, 75 us to
// clear and 480 us to read back.  Instead the codes are partitioned by hash
// into buckets that a workgroup counts in LDS:
//
//   k_offsets    where each bucket's items start, from the sizes that the
//                previous pass over the positions counted (an upper bound)
//   k_partition  a workgroup merges equal codes of its chunk in LDS and writes
//                one 8-byte item (code, count) per distinct code to its bucket
//   k_sub_*      corpora above kSplitFrom positions: every bucket split once more
//   k_split      by the hash's next bits, so that the parts fit LDS at any size
//   k_bucket     one workgroup per bucket: counts in LDS, then the survivors'
//                dense ids and the candidates, in runs
//   k_surv_*     a hash table of the survivors alone (code -> dense id)
//   k_ids        every position looks its code up there and counts the next
//                scan's bucket sizes on the way
//
// 16.8M tokens (K = 5, 1M f-grams kept), scans 2 to 5: 2,280, 1,760, 1,040 and
// 750 us with the global table, 610, 500, 300 and 130 us now; the whole call
// and the caller's sort of its result 6.76 -> 2.22 ms.
//
// The candidates are all 2-grams and the survivors of scans 3..K; the top S by
// count are found with a threshold search (equal counts at the threshold are
// taken in an unspecified order, as Algorithm 3 allows) and their tokens are
// rebuilt by walking the prefix ids back to scan 2.
#include <algorithm>
#include <cstring>

#include "scone_internal.h"

namespace scone {
namespace {

constexpr int kThreads = 256;
constexpr int kWide = 1024;  // threads of the passes that count in LDS
constexpr uint64_t kEmptyKey = ~0ull;

// An item: code << 14 | count, the count at most a chunk's 8,192 positions.
constexpr int kCountBits = 14;
constexpr uint64_t kCountMask = (1u << kCountBits) - 1;
constexpr int kMaxChunk = 8192;
// Buckets, at most; one per 4,096 positions up to there.  Each has a region per
// group of chunks (chunk index mod 8): consecutive workgroups run on different
// XCDs, so the runs of a few items that chunks append to a region come through
// one L2, which joins them into whole lines.
constexpr int kMaxBuckets = 1024;
constexpr int kGroups = 8;

struct alignas(16) SurvSlot {
    uint64_t key;
    int32_t dense;
    int32_t pad;
};

__device__ __forceinline__ uint64_t count_hash(uint64_t key) {
    return fmix64(key ^ 0x9E3779B97F4A7C15ULL);
}

// The hash's top bits choose the bucket, the next ones the part of a bucket
// that is counted at once, the lowest the slot of a table.
__device__ __forceinline__ uint32_t bucket_of(uint64_t h, int log2_buckets) {
    return (uint32_t)((h >> 1) >> (63 - log2_buckets));
}
__device__ __forceinline__ uint64_t part_of(uint64_t h, int log2_buckets, int bits) {
    return ((h << log2_buckets) >> 1) >> (63 - bits);
}

// __syncthreads after this wavefront's LDS operations have completed.  The
// barrier alone is meant to do that, but in k_ids the compiler (ROCm 7.2)
// leaves the wait out on the paths from the counting adds to it, and a
// wavefront's counts were then missing from the sums now and then.
__device__ __forceinline__ void lds_settled_barrier() {
    __builtin_amdgcn_s_waitcnt(0xF | (7 << 4) | (0 << 8) | (3 << 14));  // lgkmcnt(0)
    __syncthreads();
}

// Code of the 2-gram ending at flat position i, or kEmptyKey.  (Every load of
// the code functions is unconditional, so that a thread's positions are all in
// flight at once.)
__device__ __forceinline__ uint64_t bigram_code(const int32_t* __restrict__ X, uint32_t i,
                                                uint32_t T, bool& bad_token) {
    const int32_t prev = X[i ? i - 1 : 0], tok = X[i];
    const bool ok = tok >= 0 && tok < SCONE_TOKEN_LIMIT;
    bad_token |= !ok;
    // a bad previous token is reported where it is the last one
    const bool whole = ok && prev >= 0 && prev < SCONE_TOKEN_LIMIT && i % T != 0;
    return whole ? ((uint64_t)(uint32_t)prev << 16) | (uint32_t)tok : kEmptyKey;
}

// Code of the n-gram, n >= 3, whose prefix and suffix have the dense ids p
// (ending one earlier) and s (ending here).  Both are -1 at a row's first
// n - 2 positions, so a code never joins two rows.
__device__ __forceinline__ uint64_t ngram_code(int32_t p, int32_t s, int32_t tok) {
    return p < 0 || s < 0 ? kEmptyKey : ((uint64_t)p << 16) | (uint32_t)tok;
}

// The code ending at position i, of scan 2 (kFirst) or of a later one, whose
// previous scan's ids are ids_prev.
template <bool kFirst>
__device__ __forceinline__ uint64_t code_at(const int32_t* __restrict__ X,
                                            const int32_t* __restrict__ ids_prev, uint32_t i,
                                            uint32_t T, bool& bad_token) {
    if constexpr (kFirst) return bigram_code(X, i, T, bad_token);
    const int32_t p = ids_prev[i ? i - 1 : 0], s = ids_prev[i], tok = X[i];
    return ngram_code(i ? p : -1, s, tok);
}

// Bucket sizes of scan 2: sizes[bucket * kGroups + group] += positions.  A
// workgroup takes chunks of one group and adds its LDS counts once.
__global__ __launch_bounds__(kWide) void k_sizes(const int32_t* __restrict__ X, uint32_t BT,
                                                 uint32_t T, uint32_t chunk, uint32_t n_chunks,
                                                 int log2_buckets, unsigned* __restrict__ sizes,
                                                 unsigned* __restrict__ status) {
    __shared__ unsigned s_hist[kMaxBuckets];
    const int buckets = 1 << log2_buckets;
    for (int b = threadIdx.x; b < buckets; b += kWide) s_hist[b] = 0;
    __syncthreads();
    bool bad_token = false;
    for (uint32_t c = blockIdx.x; c < n_chunks; c += gridDim.x) {
        for (uint32_t o = threadIdx.x; o < chunk; o += kWide) {
            const uint32_t i = c * chunk + o;
            if (i >= BT) break;
            const uint64_t key = bigram_code(X, i, T, bad_token);
            if (key != kEmptyKey) atomicAdd(&s_hist[bucket_of(count_hash(key), log2_buckets)], 1u);
        }
    }
    __syncthreads();
    for (int b = threadIdx.x; b < buckets; b += kWide)
        if (s_hist[b]) atomicAdd(sizes + b * kGroups + blockIdx.x % kGroups, s_hist[b]);
    if (bad_token) atomicOr(status, err_bit(SCONE_ETOKEN));
}

// Region starts from the sizes, cursors set to them, the sizes and the survivor
// count cleared for the scan to come.  One workgroup, one bucket per thread.
__global__ __launch_bounds__(kMaxBuckets) void k_offsets(unsigned* __restrict__ sizes, int buckets,
                                                         unsigned* __restrict__ starts,
                                                         unsigned* __restrict__ cursors,
                                                         unsigned* __restrict__ n_surv) {
    __shared__ unsigned s_wave[kMaxBuckets / 64];
    const int b = threadIdx.x, lane = b & 63;
    unsigned v[kGroups], sum = 0;
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
        v[g] = b < buckets ? sizes[b * kGroups + g] : 0;
        sum += v[g];
    }
    unsigned inc = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned y = (unsigned)__shfl_up((int)inc, o);
        if (lane >= o) inc += y;
    }
    if (lane == 63) s_wave[b >> 6] = inc;
    __syncthreads();
    unsigned at = inc - sum;
    for (int w = 0; w < b >> 6; ++w) at += s_wave[w];
    if (b < buckets) {
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            starts[b * kGroups + g] = at;
            cursors[b * kGroups + g] = at;
            sizes[b * kGroups + g] = 0;
            at += v[g];
        }
        if (b == buckets - 1) starts[buckets * kGroups] = at;  // the end mark
    }
    if (b == 0) *n_surv = 0;
}

// The LDS of a workgroup that partitions up to kMaxChunk items.
struct PartLds {
    unsigned long long item[kMaxChunk];
    unsigned hist[kMaxBuckets], region[kMaxBuckets], wave[kWide / 64];
};

// Writes a workgroup's items (0 for none, at most kMaxChunk of them) to the
// regions of their bins (at most kMaxBuckets): bin b's next free place is
// cursors[b * stride].  Every thread calls it, with l.hist zero and l.item free.
template <int N, typename BinOf>
__device__ __forceinline__ void write_by_bin(const uint64_t (&item)[N], int bins, BinOf bin_of,
                                             unsigned* __restrict__ cursors, int stride,
                                             uint64_t* __restrict__ out, PartLds& l) {
    static_assert(kMaxBuckets == kWide, "a thread per bin");
    // Every item's bin and its rank among the workgroup's items there.
    unsigned at[N];
#pragma unroll
    for (int r = 0; r < N; ++r) {
        if (!item[r]) continue;
        const uint32_t b = bin_of(item[r]);
        at[r] = b << 16 | atomicAdd(&l.hist[b], 1u);
    }
    __syncthreads();
    // A thread per bin: where its items start, in LDS and in its region.
    const int b = threadIdx.x, lane = b & 63;
    const unsigned mine = b < bins ? l.hist[b] : 0;
    unsigned inc = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned y = (unsigned)__shfl_up((int)inc, o);
        if (lane >= o) inc += y;
    }
    if (lane == 63) l.wave[b >> 6] = inc;
    const unsigned region = mine ? atomicAdd(cursors + b * stride, mine) : 0;
    __syncthreads();
    unsigned start = inc - mine, total = 0;
    for (int w = 0; w < kWide / 64; ++w) {
        if (w < b >> 6) start += l.wave[w];
        total += l.wave[w];
    }
    l.hist[b] = start;
    l.region[b] = region - start;
    __syncthreads();
    // The items by bin in LDS, so that neighbouring lanes write neighbouring
    // items: one store transaction per run where one per item (8 bytes at 64
    // places per wavefront) ran at the rate of random accesses.
#pragma unroll
    for (int r = 0; r < N; ++r)
        if (item[r]) l.item[l.hist[at[r] >> 16] + (at[r] & 0xFFFF)] = item[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kMaxChunk / kWide; ++r) {
        const unsigned j = r * kWide + threadIdx.x;
        if (j >= total) break;
        const uint64_t w = l.item[j];
        out[l.region[bin_of(w)] + j] = w;
    }
}

// One chunk per workgroup: equal codes are merged in an LDS table (a Zipf
// stream's top bigram is about 1% of all positions, and its bucket would
// otherwise be that much longer than the others), then each code goes to its
// bucket's region.  A code that finds no slot within kProbe steps is written by
// itself: merging is for the frequent codes, which find one early, and the pass
// is bound by its LDS operations.  Whole calls on 16.8M tokens with 1, 2, 4, 8
// and 32 steps took 2.22, 2.31, 2.40, 2.51 and 2.92 ms; with one step a
// frequent code is shut out wherever another took its slot first.
constexpr int kProbe = 2;

template <bool kFirst>
__global__ __launch_bounds__(kWide) void k_partition(const int32_t* __restrict__ X, uint32_t BT,
                                                     uint32_t T,
                                                     const int32_t* __restrict__ ids_prev,
                                                     uint32_t chunk, int log2_buckets,
                                                     unsigned* __restrict__ cursors,
                                                     uint64_t* __restrict__ items) {
    constexpr int R = kMaxChunk / kWide;
    __shared__ PartLds l;
    auto& s_item = l.item;
    const int buckets = 1 << log2_buckets;
#pragma unroll
    for (int r = 0; r < R; ++r) s_item[r * kWide + threadIdx.x] = 0;
    l.hist[threadIdx.x] = 0;
    __syncthreads();
    uint64_t key[R];
    bool bad_token = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t o = r * kWide + threadIdx.x;
        const uint32_t i = blockIdx.x * chunk + o;
        const bool on = o < chunk && i < BT;
        const uint64_t k = code_at<kFirst>(X, ids_prev, on ? i : 0, T, bad_token);
        key[r] = on ? k : kEmptyKey;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (key[r] == kEmptyKey) continue;
        uint32_t s = (uint32_t)count_hash(key[r]) & (kMaxChunk - 1);
        for (int q = 0; q < kProbe; ++q) {
            unsigned long long w = *(volatile unsigned long long*)&s_item[s];
            if (w == 0) {
                w = atomicCAS(&s_item[s], 0ull, (unsigned long long)(key[r] << kCountBits | 1));
                if (w == 0) {
                    key[r] = kEmptyKey;
                    break;
                }
            }
            if (w >> kCountBits == key[r]) {
                atomicAdd(&s_item[s], 1ull);
                key[r] = kEmptyKey;
                break;
            }
            s = (s + 1) & (kMaxChunk - 1);
        }
    }
    __syncthreads();
    // What the table merged and what found no slot in it.
    uint64_t item[2 * R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        item[2 * r] = s_item[r * kWide + threadIdx.x];
        item[2 * r + 1] = key[r] != kEmptyKey ? key[r] << kCountBits | 1 : 0;
    }
    write_by_bin(
        item, buckets,
        [=](uint64_t w) { return bucket_of(count_hash(w >> kCountBits), log2_buckets); },
        cursors + blockIdx.x % kGroups, kGroups, items, l);
}

// --------------------------------------------------------- a second level --
// A bucket of a large corpus has more codes than a table takes by a factor that
// grows with the corpus, and reading it once per part would make the scan's
// cost quadratic (1.07G positions of nearly distinct 2-grams: 587 ms a call).
// Above kSplitFrom positions the hash's next log2_subs bits split every bucket
// once more, for one reading to count, one to write and 8 bytes written per item
// (84 ms).  A bucket's items are taken in slices of kMaxChunk, in turn by the
// workgroups of its row of the grid.

// A bucket's items, from its regions: item j of the bucket is items[j + shift]
// of the region it lies in.  `whole` says that no region has passed the start of
// the next: the pass that counted the regions and the one that filled them agree.
// They are different kernels, and a count that is lost (see lds_settled_barrier)
// would otherwise put one bucket's items over another's with no error.
template <int kRegions>
struct BucketItems {
    unsigned upto[kRegions], shift[kRegions], total;
    bool whole;

    __device__ __forceinline__ BucketItems(const unsigned* __restrict__ begin,
                                           const unsigned* __restrict__ end) {
        total = 0;
        whole = true;
#pragma unroll
        for (int g = 0; g < kRegions; ++g) {
            whole &= end[g] <= begin[g + 1];
            shift[g] = begin[g] - total;
            total += end[g] - begin[g];
            upto[g] = total;
        }
    }
    __device__ __forceinline__ unsigned at(unsigned j) const {
        unsigned sh = shift[0];
#pragma unroll
        for (int g = 1; g < kRegions; ++g) {
            // values, not a choice of addresses, which would keep the arrays in memory
            const unsigned u = upto[g - 1], v = shift[g];
            sh = j >= u ? v : sh;
        }
        return j + sh;
    }
};

// How many of each bucket's items go to each of its sub-buckets.
__global__ __launch_bounds__(kWide) void k_sub_sizes(const uint64_t* __restrict__ items,
                                                     const unsigned* __restrict__ starts,
                                                     const unsigned* __restrict__ cursors,
                                                     int log2_buckets, int log2_subs,
                                                     unsigned* __restrict__ sub_sizes,
                                                     unsigned* __restrict__ status) {
    constexpr int R = kMaxChunk / kWide;
    __shared__ unsigned s_hist[kMaxBuckets];
    const unsigned b = blockIdx.y;
    const BucketItems<kGroups> in(starts + b * kGroups, cursors + b * kGroups);
    if (!in.whole) {
        if (threadIdx.x == 0) atomicOr(status, err_bit(SCONE_EFULL));
        return;
    }
    if (blockIdx.x * kMaxChunk >= in.total) return;
    s_hist[threadIdx.x] = 0;
    __syncthreads();
    for (unsigned j0 = blockIdx.x * kMaxChunk; j0 < in.total; j0 += gridDim.x * kMaxChunk) {
        uint64_t w[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const unsigned j = j0 + r * kWide + threadIdx.x;
            w[r] = j < in.total ? items[in.at(j)] : 0;
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (w[r])
                atomicAdd(&s_hist[part_of(count_hash(w[r] >> kCountBits), log2_buckets,
                                          log2_subs)], 1u);
    }
    lds_settled_barrier();
    if (threadIdx.x < 1u << log2_subs && s_hist[threadIdx.x])
        atomicAdd(sub_sizes + ((size_t)b << log2_subs) + threadIdx.x, s_hist[threadIdx.x]);
}

// Where the sub-buckets of each bucket start: one after another from the
// bucket's own start.  One workgroup per bucket, a thread per sub-bucket.
__global__ __launch_bounds__(kWide) void k_sub_offsets(const unsigned* __restrict__ starts,
                                                       const unsigned* __restrict__ sub_sizes,
                                                       int log2_subs,
                                                       unsigned* __restrict__ sub_starts,
                                                       unsigned* __restrict__ sub_cursors) {
    __shared__ unsigned s_wave[kWide / 64];
    const unsigned s = threadIdx.x, b = blockIdx.x, lane = s & 63;
    const bool on = s < 1u << log2_subs;
    const size_t i = ((size_t)b << log2_subs) + s;
    const unsigned v = on ? sub_sizes[i] : 0;
    unsigned inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned y = (unsigned)__shfl_up((int)inc, o);
        if (lane >= (unsigned)o) inc += y;
    }
    if (lane == 63) s_wave[s >> 6] = inc;
    __syncthreads();
    unsigned at = starts[(size_t)b * kGroups] + inc - v;
    for (unsigned w = 0; w < s >> 6; ++w) at += s_wave[w];
    if (on) sub_starts[i] = sub_cursors[i] = at;
    // the end mark
    if (s == 0 && b == gridDim.x - 1) sub_starts[(size_t)gridDim.x << log2_subs] =
        starts[(size_t)gridDim.x * kGroups];
}

__global__ __launch_bounds__(kWide) void k_split(const uint64_t* __restrict__ items,
                                                 const unsigned* __restrict__ starts,
                                                 const unsigned* __restrict__ cursors,
                                                 int log2_buckets, int log2_subs,
                                                 unsigned* __restrict__ sub_cursors,
                                                 uint64_t* __restrict__ out) {
    constexpr int R = kMaxChunk / kWide;
    __shared__ PartLds l;
    const unsigned b = blockIdx.y;
    const BucketItems<kGroups> in(starts + b * kGroups, cursors + b * kGroups);
    if (!in.whole) return;
    for (unsigned j0 = blockIdx.x * kMaxChunk; j0 < in.total; j0 += gridDim.x * kMaxChunk) {
        uint64_t w[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const unsigned j = j0 + r * kWide + threadIdx.x;
            w[r] = j < in.total ? items[in.at(j)] : 0;
        }
        __syncthreads();  // the last slice has been written out
        l.hist[threadIdx.x] = 0;
        __syncthreads();
        write_by_bin(
            w, 1 << log2_subs,
            [=](uint64_t x) {
                return (uint32_t)part_of(count_hash(x >> kCountBits), log2_buckets, log2_subs);
            },
            sub_cursors + ((size_t)b << log2_subs), 1, out, l);
    }
}

// One workgroup per bucket counts its items in an LDS table, all at once or,
// when they have more distinct codes than the table takes, in 2^bits parts by
// the hash's next bits (the bucket is read again for each; distinct codes have
// distinct hashes, so the parts end up small enough).  Then the survivors
// (count >= min_count) get dense ids and the candidates (with keep_all every
// code, else the survivors) are listed, both in a run that the workgroup
// reserves with one atomic.
constexpr int kBucketSlots = 8192;
constexpr int kBucketProbe = 64;

template <int kRegions>  // regions per bucket: kGroups, or 1 on the second level
__global__ __launch_bounds__(kWide) void k_bucket(
    const uint64_t* __restrict__ items, const unsigned* __restrict__ starts,
    const unsigned* __restrict__ cursors, int log2_buckets, uint32_t min_count, int level,
    int keep_all, unsigned* __restrict__ n_surv, uint64_t* __restrict__ skey,
    unsigned* __restrict__ n_cand, uint64_t* __restrict__ cand_key,
    uint32_t* __restrict__ cand_count, int8_t* __restrict__ cand_level,
    unsigned* __restrict__ max_count, unsigned* __restrict__ status) {
    constexpr int R = kBucketSlots / kWide;
    __shared__ unsigned long long s_key[kBucketSlots];
    __shared__ unsigned s_cnt[kBucketSlots];
    __shared__ unsigned s_full, s_ns, s_nc, s_mx;
    const BucketItems<kRegions> in(starts + (size_t)blockIdx.x * kRegions,
                                   cursors + (size_t)blockIdx.x * kRegions);
    const unsigned total = in.total;
    if (!in.whole) {
        if (threadIdx.x == 0) atomicOr(status, err_bit(SCONE_EFULL));
        return;
    }
    if (total == 0) return;
    // A table of at least twice the items, where they are few, up to kBucketSlots.
    unsigned slots = kWide;
    while (slots < kBucketSlots && slots < 2 * total) slots <<= 1;
    const int lane = threadIdx.x & 63;
    const unsigned long long below = (1ull << lane) - 1ull;
    int bits = 0;
    for (uint64_t part = 0; part < (1ull << bits);) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r * kWide >= slots) break;
            s_key[r * kWide + threadIdx.x] = kEmptyKey;
            s_cnt[r * kWide + threadIdx.x] = 0;
        }
        if (threadIdx.x == 0) s_full = s_ns = s_nc = s_mx = 0;
        __syncthreads();
        for (unsigned j0 = 0; j0 < total; j0 += 4 * kWide) {
            if (*(volatile unsigned*)&s_full) break;
            uint64_t w[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const unsigned j = j0 + r * kWide + threadIdx.x;
                w[r] = j < total ? items[in.at(j)] : 0;
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (!w[r]) continue;
                const unsigned long long key = w[r] >> kCountBits;
                const uint64_t h = count_hash(key);
                if (part_of(h, log2_buckets, bits) != part) continue;
                uint32_t s = (uint32_t)h & (slots - 1);
                int q = 0;
                for (; q < kBucketProbe; ++q) {
                    unsigned long long k = *(volatile unsigned long long*)&s_key[s];
                    if (k == kEmptyKey)
                        k = atomicCAS(&s_key[s], (unsigned long long)kEmptyKey, key);
                    if (k == kEmptyKey || k == key) {
                        atomicAdd(&s_cnt[s], (unsigned)(w[r] & kCountMask));
                        break;
                    }
                    s = (s + 1) & (slots - 1);
                }
                if (q == kBucketProbe) *(volatile unsigned*)&s_full = 1;
            }
        }
        __syncthreads();
        if (s_full) {  // the same for the whole workgroup
            ++bits;
            part <<= 1;
            __syncthreads();
            continue;
        }
        uint64_t k[R];
        uint32_t c[R];
        unsigned ns = 0, nc = 0, mx = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            c[r] = 0;
            if (r * kWide >= slots) continue;
            k[r] = s_key[r * kWide + threadIdx.x];
            c[r] = s_cnt[r * kWide + threadIdx.x];  // 0 where the slot is empty
            const bool survive = c[r] >= min_count, cand = survive || (keep_all && c[r]);
            ns += (unsigned)__popcll(__ballot(survive));
            nc += (unsigned)__popcll(__ballot(cand));
            if (cand) mx = c[r] > mx ? c[r] : mx;
        }
        if (mx) atomicMax(&s_mx, mx);
        unsigned bs = 0, bc = 0;
        if (lane == 0) {
            bs = atomicAdd(&s_ns, ns);
            bc = atomicAdd(&s_nc, nc);
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            s_ns = s_ns ? atomicAdd(n_surv, s_ns) : 0;
            s_nc = s_nc ? atomicAdd(n_cand, s_nc) : 0;
            if (s_mx) atomicMax(max_count, s_mx);
        }
        __syncthreads();
        bs = (unsigned)__shfl((int)bs, 0) + s_ns;
        bc = (unsigned)__shfl((int)bc, 0) + s_nc;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r * kWide >= slots) break;
            const bool survive = c[r] >= min_count, cand = survive || (keep_all && c[r]);
            const unsigned long long ms = __ballot(survive), mc = __ballot(cand);
            if (survive && skey) skey[bs + (unsigned)__popcll(ms & below)] = k[r];
            if (cand) {
                const unsigned at = bc + (unsigned)__popcll(mc & below);
                cand_key[at] = k[r];
                cand_count[at] = c[r];
                cand_level[at] = (int8_t)level;
            }
            bs += (unsigned)__popcll(ms);
            bc += (unsigned)__popcll(mc);
        }
        ++part;
        __syncthreads();
    }
}

// Slots of the survivors' table: a power of two of at least twice as many, so
// that the frequent n-grams' slots stay in the caches.  At most 2 BT rounded
// up, the table's room in the workspace.
__device__ __forceinline__ uint64_t surv_slots(unsigned n_surv) {
    uint64_t cap = 64;
    while (cap < 2ull * n_surv) cap <<= 1;
    return cap;
}

__global__ __launch_bounds__(kThreads) void k_surv_clear(const unsigned* __restrict__ n_surv,
                                                         SurvSlot* __restrict__ t) {
    const uint64_t cap = surv_slots(*n_surv);
    for (uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < cap;
         i += (uint64_t)gridDim.x * kThreads)
        t[i] = SurvSlot{kEmptyKey, -1, 0};
}

__global__ __launch_bounds__(kThreads) void k_surv_insert(const unsigned* __restrict__ n_surv,
                                                          const uint64_t* __restrict__ skey,
                                                          SurvSlot* __restrict__ t) {
    const unsigned n = *n_surv;
    const uint64_t mask = surv_slots(n) - 1;
    for (unsigned id = blockIdx.x * kThreads + threadIdx.x; id < n; id += gridDim.x * kThreads) {
        const unsigned long long key = skey[id];
        uint64_t s = count_hash(key) & mask;
        // half the slots stay empty, so one is found
        while (atomicCAS(reinterpret_cast<unsigned long long*>(&t[s].key),
                         (unsigned long long)kEmptyKey, key) != kEmptyKey)
            s = (s + 1) & mask;
        t[s].dense = (int32_t)id;
    }
}

// Dense id of the survivor of scan n ending at every position, or -1, and the
// bucket sizes of scan n + 1 (as k_sizes).  Bound by the random reads: a
// thread has the home slots of kPer positions in flight.
constexpr int kPer = 4;

template <bool kFirst>
__global__ __launch_bounds__(kWide) void k_ids(const int32_t* __restrict__ X, uint32_t BT,
                                               uint32_t T,
                                               const int32_t* __restrict__ ids_prev,
                                               const unsigned* __restrict__ n_surv,
                                               const SurvSlot* __restrict__ t, uint32_t chunk,
                                               uint32_t n_chunks, int log2_buckets,
                                               int32_t* __restrict__ ids_cur,
                                               unsigned* __restrict__ sizes) {
    __shared__ unsigned s_hist[kMaxBuckets];
    __shared__ int32_t s_id[kPer * kWide + 1];  // s_id[j + 1]: id at the step's position j
    const int buckets = 1 << log2_buckets;
    for (int b = threadIdx.x; b < buckets; b += kWide) s_hist[b] = 0;
    const uint64_t mask = surv_slots(*n_surv) - 1;
    bool bad_token = false;
    for (uint32_t c = blockIdx.x; c < n_chunks; c += gridDim.x) {
        const uint32_t c1 = BT - c * chunk < chunk ? BT : (c + 1) * chunk;
        for (uint32_t i0 = c * chunk; i0 < c1; i0 += kPer * kWide) {
            // the step's positions, and on thread 0 the one before them
            uint64_t key[kPer + 1];
            u32x4 slot[kPer + 1];
            uint64_t s[kPer + 1];
#pragma unroll
            for (int r = 0; r <= kPer; ++r) {
                const uint32_t i = r < kPer ? i0 + r * kWide + threadIdx.x : i0 - 1;
                const bool on = r < kPer ? i < c1 : threadIdx.x == 0 && i0 > 0;
                const uint64_t k = code_at<kFirst>(X, ids_prev, on ? i : 0, T, bad_token);
                key[r] = on ? k : kEmptyKey;
            }
#pragma unroll
            for (int r = 0; r <= kPer; ++r) {
                s[r] = count_hash(key[r]) & mask;
                if (key[r] != kEmptyKey) slot[r] = *reinterpret_cast<const u32x4*>(t + s[r]);
            }
            lds_settled_barrier();  // the last step's ids have been read
#pragma unroll
            for (int r = 0; r <= kPer; ++r) {
                int32_t d = -1;
                if (key[r] != kEmptyKey) {
                    for (;;) {  // half the slots are empty, so it ends
                        const uint64_t k = (uint64_t)slot[r].x | (uint64_t)slot[r].y << 32;
                        if (k == key[r]) {
                            d = (int32_t)slot[r].z;
                            break;
                        }
                        if (k == kEmptyKey) break;
                        s[r] = (s[r] + 1) & mask;
                        slot[r] = *reinterpret_cast<const u32x4*>(t + s[r]);
                    }
                }
                const uint32_t o = r * kWide + threadIdx.x;
                if (r < kPer) {
                    s_id[o + 1] = d;
                    if (i0 + o < c1) ids_cur[i0 + o] = d;
                } else if (threadIdx.x == 0) {
                    s_id[0] = d;
                }
            }
            lds_settled_barrier();
#pragma unroll
            for (int r = 0; r < kPer; ++r) {
                const uint32_t o = r * kWide + threadIdx.x;
                if (i0 + o >= c1) continue;
                const int32_t p = s_id[o], d = s_id[o + 1];
                if (p < 0 || d < 0) continue;
                const uint64_t next = ngram_code(p, d, X[i0 + o]);
                atomicAdd(&s_hist[bucket_of(count_hash(next), log2_buckets)], 1u);
            }
        }
    }
    lds_settled_barrier();
    for (int b = threadIdx.x; b < buckets; b += kWide)
        if (s_hist[b]) atomicAdd(sizes + b * kGroups + blockIdx.x % kGroups, s_hist[b]);
}

// The count threshold: the largest count c that at least S candidates reach.
struct Cut {
    uint32_t thresh;   // c, or 0 when every candidate is taken
    uint32_t wide;     // c is at least kHistBins - 1 and not found yet
    int64_t n_above;   // candidates counting more than c
};

// Histogram of candidate counts, exact below kHistBins - 1 and pooled above:
// a workgroup counts runs of candidates in LDS and adds its non-zero bins.
// Nothing when there are no more candidates than wanted.
constexpr int kHistBins = 4096;
constexpr int kHistRun = 8192;
static_assert(kHistBins * sizeof(unsigned long long) >= kMaxBuckets * kGroups * sizeof(unsigned),
              "the bucket sizes lie in the histogram's place");

__global__ __launch_bounds__(kThreads) void k_count_hist(const uint32_t* __restrict__ cnt,
                                                         const unsigned* __restrict__ n_cand,
                                                         int64_t S,
                                                         unsigned long long* __restrict__ hist) {
    __shared__ unsigned h[kHistBins];
    const int64_t n = *n_cand;
    if (n <= S || (int64_t)blockIdx.x * kHistRun >= n) return;
    for (int i = threadIdx.x; i < kHistBins; i += kThreads) h[i] = 0;
    __syncthreads();
    for (int64_t i0 = (int64_t)blockIdx.x * kHistRun; i0 < n;
         i0 += (int64_t)gridDim.x * kHistRun) {
        const int64_t i1 = i0 + kHistRun < n ? i0 + kHistRun : n;
        for (int64_t i = i0 + threadIdx.x; i < i1; i += kThreads) {
            const uint32_t c = cnt[i];
            atomicAdd(&h[c < kHistBins - 1 ? c : kHistBins - 1], 1u);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kHistBins; i += kThreads)
        if (h[i]) atomicAdd(hist + i, (unsigned long long)h[i]);
}

// Reads the cut off the histogram (one workgroup, four bins per thread).
__global__ __launch_bounds__(kWide) void k_cut(const unsigned long long* __restrict__ hist,
                                               const unsigned* __restrict__ n_cand, int64_t S,
                                               Cut* __restrict__ cut) {
    constexpr int R = kHistBins / kWide;
    __shared__ unsigned long long s_sum[kWide / 64];
    if ((int64_t)*n_cand <= S) {
        if (threadIdx.x == 0) *cut = Cut{0, 0, 0};
        return;
    }
    // bins from the highest count down; s = candidates in this thread's bins
    unsigned long long v[R], s = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        v[r] = hist[kHistBins - 1 - (threadIdx.x * R + r)];
        s += v[r];
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long inc = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long y = __shfl_up(inc, o);
        if (lane >= o) inc += y;
    }
    if (lane == 63) s_sum[wave] = inc;
    __syncthreads();
    unsigned long long above = inc - s;
    for (int w = 0; w < wave; ++w) above += s_sum[w];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int c = kHistBins - 1 - (threadIdx.x * R + r);
        if ((int64_t)above < S && (int64_t)(above + v[r]) >= S)  // exactly one bin
            *cut = Cut{(uint32_t)c, c == kHistBins - 1 ? 1u : 0u, (int64_t)above};
        above += v[r];
    }
}

// Candidates counting at least c.
__global__ __launch_bounds__(kThreads) void k_count_at_least(const uint32_t* __restrict__ cnt,
                                                             int64_t n, uint32_t c,
                                                             unsigned long long* __restrict__ out,
                                                             int64_t block0) {
    const int64_t i = block_index(block0) * kThreads + threadIdx.x;
    const bool hit = i < n && cnt[i] >= c;
    const unsigned long long m = __ballot(hit);
    if ((threadIdx.x & 63) == 0 && m) atomicAdd(out, (unsigned long long)__popcll(m));
}

struct LevelKeys {
    const uint64_t* skey[SCONE_MAX_FGRAM_LEN + 1];  // survivors' codes by scan
};

// Emit the selected candidates with their tokens, unless the cut is still to
// be found or the corpus was rejected (an error leaves the outputs as they were).
// A workgroup takes kSelectPerBlock candidates at a time and reserves its output
// rows with one atomic per counter (one per wavefront on a shared counter
// serialises).
constexpr int kSelectPerBlock = 16 * kThreads;

__global__ __launch_bounds__(kThreads) void k_select(
    const uint64_t* __restrict__ cand_key, const uint32_t* __restrict__ cand_count,
    const int8_t* __restrict__ cand_level, const unsigned* __restrict__ n_cands,
    const unsigned* __restrict__ status, const Cut* __restrict__ cut, int64_t S, LevelKeys lk, int max_len, unsigned* __restrict__ n_gt,
    unsigned* __restrict__ n_eq, int32_t* __restrict__ fgrams, int32_t* __restrict__ lengths,
    int32_t* __restrict__ counts) {
    constexpr int R = kSelectPerBlock / kThreads;
    __shared__ unsigned s_gt, s_eq;
    if (cut->wide || *status) return;
    const uint32_t thresh = cut->thresh;
    const int64_t n_above = cut->n_above, n_cand = *n_cands;
    const int lane = threadIdx.x & 63;
    const unsigned long long below = (1ull << lane) - 1ull;
    for (int64_t b0 = (int64_t)blockIdx.x * kSelectPerBlock; b0 < n_cand;
         b0 += (int64_t)gridDim.x * kSelectPerBlock) {
        const int64_t i0 = b0 + threadIdx.x;
        if (threadIdx.x == 0) s_gt = s_eq = 0;
        uint32_t c[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t i = i0 + r * kThreads;
            c[r] = i < n_cand ? cand_count[i] : 0;  // a candidate counts at least 1
        }
        unsigned ng = 0, ne = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            ng += (unsigned)__popcll(__ballot(c[r] > thresh));
            ne += (unsigned)__popcll(__ballot(c[r] && c[r] == thresh));
        }
        __syncthreads();
        unsigned bg = 0, be = 0;
        if (lane == 0) {
            bg = atomicAdd(&s_gt, ng);
            be = atomicAdd(&s_eq, ne);
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            s_gt = s_gt ? atomicAdd(n_gt, s_gt) : 0;
            s_eq = s_eq ? atomicAdd(n_eq, s_eq) : 0;
        }
        __syncthreads();
        bg = (unsigned)__shfl((int)bg, 0) + s_gt;
        be = (unsigned)__shfl((int)be, 0) + s_eq;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const bool gt = c[r] > thresh, eq = c[r] && c[r] == thresh;
            const unsigned long long mg = __ballot(gt), me = __ballot(eq);
            int64_t pos = -1;
            if (gt) {
                pos = bg + (unsigned)__popcll(mg & below);
            } else if (eq) {
                const int64_t e = (int64_t)be + (unsigned)__popcll(me & below);
                if (n_above + e < S) pos = n_above + e;
            }
            bg += (unsigned)__popcll(mg);
            be += (unsigned)__popcll(me);
            if (pos < 0 || pos >= S) continue;
            const int64_t i = i0 + r * kThreads;
            const int level = cand_level[i];
            int32_t tok[SCONE_MAX_FGRAM_LEN];
            uint64_t key = cand_key[i];
            for (int L = level; L >= 3; --L) {
                tok[L - 1] = (int32_t)(key & 0xFFFF);
                key = lk.skey[L - 1][key >> 16];
            }
            tok[1] = (int32_t)(key & 0xFFFF);
            tok[0] = (int32_t)(key >> 16);
            int32_t* row = fgrams + pos * (int64_t)max_len;
            for (int j = 0; j < max_len; ++j) row[j] = j < level ? tok[j] : -1;
            lengths[pos] = level;
            counts[pos] = (int32_t)c[r];
        }
        __syncthreads();  // the bases have been read
    }
}

}  // namespace
}  // namespace scone

namespace scone {
namespace {

// Scratch of one call, carved from one workspace: the survivors' table, the
// dense ids of two consecutive scans, the candidates, the counters and
// histogram, and the survivors' codes of every scan but the last.  What lives
// at different times shares memory: a scan's items (8 bytes per position) lie
// where its survivors' table (at least 32) is made once they are counted, the
// region starts and cursors where the ids of the scan's end are written
// (k_ids, after their last use; the second level's items behind the first's, its
// starts and cursors behind theirs), the bucket sizes in the histogram's place.
struct DiscLayout {
    uint64_t cap;
    int64_t cand_cap;
    size_t table, ids_a, ids_b, cand_key, cand_count, cand_level, ctr, acc, hist;
    size_t skey[SCONE_MAX_FGRAM_LEN + 1];
    size_t total;
};

DiscLayout disc_layout(int64_t BT, int max_len) {
    DiscLayout l{};
    l.cap = 64;
    while ((int64_t)l.cap < 2 * BT) l.cap <<= 1;
    l.cand_cap = BT * (int64_t)(max_len - 1);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off = (off + bytes + 255) & ~(size_t)255;
        return at;
    };
    l.table = take(l.cap * sizeof(SurvSlot));
    l.ids_a = take(BT * sizeof(int32_t));
    l.ids_b = take(BT * sizeof(int32_t));
    l.cand_key = take(l.cand_cap * sizeof(uint64_t));
    l.cand_count = take(l.cand_cap * sizeof(uint32_t));
    l.cand_level = take(l.cand_cap);
    l.ctr = take(16 * sizeof(unsigned));
    l.acc = take(sizeof(unsigned long long));
    l.hist = take(kHistBins * sizeof(unsigned long long));
    for (int L = 2; L < max_len; ++L) l.skey[L] = take(BT * sizeof(uint64_t));
    l.total = off;
    return l;
}

// How a scan cuts up BT positions: chunks of 1,024 to 8,192 (as long as there
// are 256 of them, one per compute unit, the longer the fewer items) and
// buckets of about 4,096 positions, up to kMaxBuckets.
struct Shape {
    uint32_t chunk, n_chunks;
    int log2_buckets;
    int log2_subs;  // sub-buckets of each bucket, 0 for no second level
};

// Above this many positions buckets are split once more, into sub-buckets of up to
// 8,192 positions each, at most 256 per bucket.  Whole calls without / with the
// second level: Zipf(1.1) tokens, K = 3, 20M positions 1.29 / 1.55 ms, 25M 1.95 /
// 2.20, 33.5M 2.82 / 2.33, 268M 33.3 / 16.8, K = 5, 33.5M 4.3 / 4.5; uniform tokens
// (2-grams nearly distinct), K = 3, 20M 2.20 / 1.32, 268M 59.7 / 24.0, K = 2, 537M
// 175 / 41 ms.  A stream of text is the first kind, and the line lies where it gains.
constexpr int64_t kSplitFrom = 1ll << 25;

Shape scan_shape(int64_t BT) {
    Shape s{kWide, 0, 0, 0};
    while (s.chunk < kMaxChunk && BT / (2 * (int64_t)s.chunk) >= 256) s.chunk *= 2;
    s.n_chunks = (uint32_t)((BT + s.chunk - 1) / s.chunk);
    while ((4096ll << s.log2_buckets) < BT && (1 << s.log2_buckets) < kMaxBuckets)
        ++s.log2_buckets;
    if (BT > kSplitFrom)
        while ((8192ll << (s.log2_buckets + s.log2_subs)) < BT) ++s.log2_subs;
    return s;
}

// SCONE_OK when (B, T, max_len) are sizes the call handles.
int disc_sizes_ok(int64_t B, int64_t T, int32_t max_len) {
    if (B < 0 || T < 0) return SCONE_EINVAL;
    if (max_len < 2 || max_len > SCONE_MAX_FGRAM_LEN) return SCONE_EINVAL;
    if (B > 0 && T > ((int64_t)1 << 40) / B) return SCONE_EINVAL;
    const int64_t BT = B * T;
    if (BT >= ((int64_t)1 << 31)) return SCONE_EINVAL;  // dense ids and counters are 32-bit
    // every candidate of every scan is counted in one 32-bit counter
    if (BT * (int64_t)(max_len - 1) >= ((int64_t)1 << 32)) return SCONE_EINVAL;
    return SCONE_OK;
}

}  // namespace
}  // namespace scone

extern "C" int64_t scone_discover_workspace(int64_t B, int64_t T, int32_t max_len) {
    using namespace scone;
    if (disc_sizes_ok(B, T, max_len) != SCONE_OK) return -1;
    return (int64_t)disc_layout(B * T, max_len).total;
}

extern "C" int scone_discover_fgrams(const int32_t* token_ids, int64_t B, int64_t T,
                                     int32_t max_len, int32_t min_count, int64_t S,
                                     int32_t* fgrams, int32_t* lengths, int32_t* counts,
                                     int64_t* n_found, void* workspace, int64_t workspace_bytes,
                                     void* stream) {
    using namespace scone;
    if (!n_found) return SCONE_EINVAL;
    *n_found = 0;
    if (S < 0 || min_count < 1) return SCONE_EINVAL;
    if (disc_sizes_ok(B, T, max_len) != SCONE_OK) return SCONE_EINVAL;
    const int64_t BT = B * T;
    if (BT == 0 || S == 0) return SCONE_OK;
    if (!token_ids || !fgrams || !lengths || !counts) return SCONE_EINVAL;
    const DiscLayout lay = disc_layout(BT, max_len);
    if (workspace && (workspace_bytes < 0 || (uint64_t)workspace_bytes < lay.total))
        return SCONE_EINVAL;
    if ((uintptr_t)workspace % 256 != 0) return SCONE_EINVAL;
    // The selection writes the outputs while it reads candidates from the
    // workspace, and the scans read the corpus while they write the
    // workspace: no two of these buffers may share memory.
    {
        const void* buf[5] = {token_ids, fgrams, lengths, counts, workspace};
        const int64_t len[5] = {span_bytes(BT, 4), span_bytes(S, 4 * (int64_t)max_len),
                                span_bytes(S, 4), span_bytes(S, 4),
                                workspace ? (int64_t)lay.total : 0};
        for (int i = 0; i < 5; ++i)
            for (int j = i + 1; j < 5; ++j)
                if (overlaps(buf[i], len[i], buf[j], len[j])) return SCONE_EINVAL;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);

    // Without a workspace the call takes its scratch in one allocation and
    // frees it before returning (the call is synchronous).
    void* own = nullptr;
    if (!workspace) {
        if (hipMalloc(&own, lay.total) != hipSuccess) {
            (void)hipGetLastError();
            return SCONE_ENOMEM;
        }
        workspace = own;
    }
    auto release = [&]() {  // false if the stream's work failed
        const bool done = hipStreamSynchronize(st) == hipSuccess;
        if (own) (void)hipFree(own);
        return done;
    };
    uint8_t* ws = static_cast<uint8_t*>(workspace);
    SurvSlot* table = reinterpret_cast<SurvSlot*>(ws + lay.table);
    uint64_t* items = reinterpret_cast<uint64_t*>(ws + lay.table);
    int32_t* ids_a = reinterpret_cast<int32_t*>(ws + lay.ids_a);
    int32_t* ids_b = reinterpret_cast<int32_t*>(ws + lay.ids_b);
    uint64_t* cand_key = reinterpret_cast<uint64_t*>(ws + lay.cand_key);
    uint32_t* cand_count = reinterpret_cast<uint32_t*>(ws + lay.cand_count);
    int8_t* cand_level = reinterpret_cast<int8_t*>(ws + lay.cand_level);
    unsigned* ctr = reinterpret_cast<unsigned*>(ws + lay.ctr);
    unsigned long long* acc = reinterpret_cast<unsigned long long*>(ws + lay.acc);
    unsigned long long* hist = reinterpret_cast<unsigned long long*>(ws + lay.hist);
    unsigned* sizes = reinterpret_cast<unsigned*>(ws + lay.hist);
    LevelKeys lk{};
    uint64_t* skeys[SCONE_MAX_FGRAM_LEN + 1] = {};
    for (int L = 2; L < max_len; ++L) {
        skeys[L] = reinterpret_cast<uint64_t*>(ws + lay.skey[L]);
        lk.skey[L] = skeys[L];
    }
    // ctr: [0] status, [1] survivors, [2] candidates, [3] max count, [4] n_gt, [5] n_eq,
    // [8..11] the cut
    Cut* cut = reinterpret_cast<Cut*>(ctr + 8);
    int rc = SCONE_OK;
    const Shape sh = scan_shape(BT);
    const uint32_t n_tok = (uint32_t)BT, row = (uint32_t)T;
    const dim3 wide(kWide), narrow(kThreads);
    // passes over the positions: two workgroups per compute unit, a multiple
    // of kGroups so that each stays with the chunks of one group
    const unsigned g_pos = sh.n_chunks < 512 ? (sh.n_chunks + kGroups - 1) / kGroups * kGroups
                                             : 512;
    const unsigned g_surv = (unsigned)(BT < (1 << 18) ? (BT + kThreads - 1) / kThreads : 1024);
    if (hipMemsetAsync(ctr, 0, 16 * sizeof(unsigned), st) != hipSuccess ||
        hipMemsetAsync(sizes, 0, (sizeof(unsigned) * kGroups) << sh.log2_buckets, st) !=
            hipSuccess)
        rc = SCONE_EHIP;
    if (rc == SCONE_OK)
        hipLaunchKernelGGL(k_sizes, dim3(g_pos), wide, 0, st, token_ids, n_tok, row, sh.chunk,
                           sh.n_chunks, sh.log2_buckets, sizes, ctr + 0);
    int32_t* ids_prev = ids_a;
    int32_t* ids_cur = ids_b;
    for (int n = 2; n <= max_len && rc == SCONE_OK; ++n) {
        unsigned* starts = reinterpret_cast<unsigned*>(ids_cur);
        unsigned* cursors = starts + ((size_t)kGroups << sh.log2_buckets) + 1;
        const uint64_t* counted = items;  // what k_bucket counts, and its regions
        const unsigned *c_starts = starts, *c_cursors = cursors;
        const int log2_counted = sh.log2_buckets + sh.log2_subs;
        hipLaunchKernelGGL(k_offsets, dim3(1), dim3(kMaxBuckets), 0, st, sizes,
                           1 << sh.log2_buckets, starts, cursors, ctr + 1);
        hipLaunchKernelGGL(n == 2 ? k_partition<true> : k_partition<false>, dim3(sh.n_chunks),
                           wide, 0, st, token_ids, n_tok, row, ids_prev, sh.chunk,
                           sh.log2_buckets, cursors, items);
        if (sh.log2_subs) {
            const size_t subs = (size_t)1 << log2_counted;
            unsigned* sub_starts = cursors + ((size_t)kGroups << sh.log2_buckets);
            unsigned* sub_cursors = sub_starts + subs + 1;
            unsigned* sub_sizes = sub_cursors + subs;
            uint64_t* sub_items = items + BT;
            // as many workgroups per bucket as its share of the positions has slices
            const dim3 grid((unsigned)(((BT >> sh.log2_buckets) + kMaxChunk) / kMaxChunk),
                            1u << sh.log2_buckets);
            if (hipMemsetAsync(sub_sizes, 0, subs * sizeof(unsigned), st) != hipSuccess)
                rc = SCONE_EHIP;
            hipLaunchKernelGGL(k_sub_sizes, grid, wide, 0, st, items, starts, cursors,
                               sh.log2_buckets, sh.log2_subs, sub_sizes, ctr + 0);
            hipLaunchKernelGGL(k_sub_offsets, dim3(1u << sh.log2_buckets), wide, 0, st, starts,
                               sub_sizes, sh.log2_subs, sub_starts, sub_cursors);
            hipLaunchKernelGGL(k_split, grid, wide, 0, st, items, starts, cursors,
                               sh.log2_buckets, sh.log2_subs, sub_cursors, sub_items);
            counted = sub_items;
            c_starts = sub_starts;
            c_cursors = sub_cursors;
        }
        hipLaunchKernelGGL(sh.log2_subs ? k_bucket<1> : k_bucket<kGroups>,
                           dim3(1u << log2_counted), wide, 0, st, counted, c_starts,
                           c_cursors, log2_counted, (uint32_t)min_count, n, n == 2 ? 1 : 0,
                           ctr + 1, n < max_len ? skeys[n] : nullptr, ctr + 2, cand_key,
                           cand_count, cand_level, ctr + 3, ctr + 0);
        if (n < max_len) {
            hipLaunchKernelGGL(k_surv_clear, dim3(g_surv), narrow, 0, st, ctr + 1, table);
            hipLaunchKernelGGL(k_surv_insert, dim3(g_surv), narrow, 0, st, ctr + 1, skeys[n],
                               table);
            hipLaunchKernelGGL(n == 2 ? k_ids<true> : k_ids<false>, dim3(g_pos), wide, 0, st,
                               token_ids, n_tok, row, ids_prev, ctr + 1, table, sh.chunk,
                               sh.n_chunks, sh.log2_buckets, ids_cur, sizes);
            int32_t* tmp = ids_prev;
            ids_prev = ids_cur;
            ids_cur = tmp;
        }
        if (hipGetLastError() != hipSuccess) rc = SCONE_EHIP;
    }
    // The cut and the selection follow without a look at the counters, unless
    // the cut lies in the histogram's pooled bin.
    const dim3 g_sel((unsigned)std::min<int64_t>((BT + kSelectPerBlock - 1) / kSelectPerBlock,
                                                 2048));
    auto select = [&]() {
        hipLaunchKernelGGL(k_select, g_sel, narrow, 0, st, cand_key, cand_count, cand_level,
                           ctr + 2, ctr + 0, cut, S, lk, max_len, ctr + 4, ctr + 5, fgrams, lengths,
                           counts);
        return hipGetLastError() == hipSuccess;
    };
    unsigned h[16] = {};
    static_assert(8 * sizeof(unsigned) + sizeof(Cut) <= sizeof(h), "the cut ends the counters");
    auto read_counters = [&]() {
        return hipMemcpyAsync(h, ctr, sizeof(h), hipMemcpyDeviceToHost, st) == hipSuccess &&
               hipStreamSynchronize(st) == hipSuccess;
    };
    if (rc == SCONE_OK) {
        if (hipMemsetAsync(hist, 0, kHistBins * sizeof(unsigned long long), st) != hipSuccess)
            rc = SCONE_EHIP;
        hipLaunchKernelGGL(k_count_hist,
                           dim3((unsigned)std::min<int64_t>((BT + kHistRun - 1) / kHistRun, 1024)),
                           narrow, 0, st, cand_count, ctr + 2, S, hist);
        hipLaunchKernelGGL(k_cut, dim3(1), wide, 0, st, hist, ctr + 2, S, cut);
        if (!select() || !read_counters()) rc = SCONE_EHIP;
    }
    if (rc == SCONE_OK && h[0]) rc = (h[0] & err_bit(SCONE_ETOKEN)) ? SCONE_ETOKEN : SCONE_EFULL;
    const int64_t n_cand = h[2];
    const uint32_t max_c = h[3];
    Cut found{};
    std::memcpy(&found, h + 8, sizeof(found));
    if (rc == SCONE_OK && found.wide) {
        // at least S candidates count >= kHistBins - 1: search the rest
        auto at_least = [&](uint32_t c, int64_t& out) -> bool {
            unsigned long long v = 0;
            if (hipMemsetAsync(acc, 0, sizeof(v), st) != hipSuccess) return false;
            if (launch_blocks((n_cand + kThreads - 1) / kThreads, kThreads,
                              [&](int64_t b0, dim3 grid) {
                                  hipLaunchKernelGGL(k_count_at_least, grid, dim3(kThreads), 0,
                                                     st, cand_count, n_cand, c, acc, b0);
                              }) != hipSuccess ||
                hipMemcpyAsync(&v, acc, sizeof(v), hipMemcpyDeviceToHost, st) != hipSuccess ||
                hipStreamSynchronize(st) != hipSuccess)
                return false;
            out = (int64_t)v;
            return true;
        };
        uint32_t lo = kHistBins - 1, hi = max_c;  // at_least(lo) >= S
        while (lo < hi && rc == SCONE_OK) {
            const uint32_t mid = lo + (hi - lo + 1) / 2;
            int64_t k = 0;
            if (!at_least(mid, k)) rc = SCONE_EHIP;
            else if (k >= S) lo = mid;
            else hi = mid - 1;
        }
        found = Cut{lo, 0, 0};
        if (rc == SCONE_OK && lo < max_c && !at_least(lo + 1, found.n_above)) rc = SCONE_EHIP;
        if (rc == SCONE_OK &&
            (hipMemcpyAsync(cut, &found, sizeof(found), hipMemcpyHostToDevice, st) != hipSuccess ||
             !select()))
            rc = SCONE_EHIP;
    }
    if (!release() && rc == SCONE_OK) rc = SCONE_EHIP;
    if (rc == SCONE_OK) *n_found = n_cand < S ? n_cand : S;
    return rc;
}
