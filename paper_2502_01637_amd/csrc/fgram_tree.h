// The prefix tree of a list of f-grams, for the precompute of F.
//
// Sorted by their tokens, f-grams that begin alike are neighbours.  An f-gram
// of length L adds to the tree the nodes of the depths that it does not share
// with the f-gram before it: share .. L - 1, where share is the length of
// their common prefix, at most L - 1 so that every f-gram has a last node of
// its own.  Chunks are runs of sorted f-grams of at most kChunkRows nodes; a
// chunk's first f-gram adds its whole path again, so that every path lies
// inside one chunk.
//
//   k_short_list            all of the following up to the chunk limits, for fewer than
//                           256 f-grams
//   k_check                 lengths and tokens in range
//   k_rank + k_place        the sort of a short list: each f-gram's rank is the
//                           number of f-grams below it
//   k_radix_* + scan        the sort of a longer one: stable 8-bit passes over
//                           the tokens but the last, from the last byte to the first
//   k_share + scan          share and the inner nodes added before each f-gram
//   k_chunks                chunk limits, read back by the host
//   k_nodes (per chunk)     one record per node
//   k_last_nodes            instead of all but the check, where the model has no layers:
//                           no state but an f-gram's last is read
//
// The sort leaves out the last of max_len tokens, so full-length f-grams with
// one prefix are in any order; only nodes above the last depth are looked up.
#pragma once

#include <cstring>
#include <vector>

#include "scone_internal.h"

namespace scone {
namespace tree {

constexpr int kThreads = 256;

// Nodes per chunk: 256 tiles of 256 rows, a whole number of rounds of the 256
// compute units for every product whose width is a multiple of 256.  Chunks of
// half and of a quarter this size were 0% and 2% slower.
constexpr int64_t kChunkRows = 65536;

// The sort counts ranks, n * n comparisons in two launches, while those are at most
// this many per radix pass (five launches each, one pass for each byte of max_len
// - 1 tokens).  Whole calls of a model with no layers by ranks and by passes: K = 2
// with one pass, 8,000 f-grams 152, 152 us; K = 3 with four, 24,000 291, 316 us, 32,000
// 423, 364; K = 7 with twelve, 8,000 180, 529 us, 32,000 679, 770, 48,000 1,207, 865.
constexpr int64_t kRankPerPass = 100000000;

// One node: its token, its position in the f-gram and the rows of its
// ancestors, oldest first (up[0 .. pos)).
struct alignas(32) Node {
    int32_t up[SCONE_MAX_FGRAM_LEN - 1];
    int32_t pos;
    int32_t tok;
};

struct Chunk {
    int64_t first;  // its first f-gram in sorted order
    int64_t inner;  // inner nodes that the f-grams before it add
    int64_t n_f;    // its f-grams: rows 0 .. n_f - 1 are their last nodes
    int64_t rows;   // all its nodes: rows n_f .. rows - 1 are the inner ones
    int share;      // depths its first f-gram shares with the one before it
};

// Token i of an f-gram of length len plus one, 0 past its end (so that an
// f-gram sorts before those that it begins).  Tokens outside [0, vocab) count
// as 0.
__device__ __forceinline__ uint32_t key_at(const int32_t* __restrict__ row, int len, int i,
                                           int64_t vocab) {
    if (i >= len) return 0;
    const int32_t t = row[i];
    return (uint32_t)((t < 0 || (int64_t)t >= vocab) ? 0 : t) + 1u;
}

// Lengths outside [2, max_len] are an error found before anything is written;
// until then they count as the nearest bound, so that nothing is read out of
// range.
__device__ __forceinline__ int len_of(const int32_t* __restrict__ lengths, int64_t g,
                                      int max_len) {
    const int32_t len = lengths[g];
    return len < 2 ? 2 : len > max_len ? max_len : len;
}

// err_bit of SCONE_ELEN and SCONE_ETOKEN, as f-gram g has them.
__device__ __forceinline__ unsigned data_errors(const int32_t* __restrict__ fgrams,
                                                const int32_t* __restrict__ lengths, int64_t g,
                                                int max_len, int64_t vocab) {
    const int len = len_of(lengths, g, max_len);
    unsigned bad = lengths[g] != len ? err_bit(SCONE_ELEN) : 0u;
    for (int i = 0; i < len; ++i) {
        const int32_t t = fgrams[g * max_len + i];
        if (t < 0 || (int64_t)t >= vocab) bad |= err_bit(SCONE_ETOKEN);
    }
    return bad;
}

__global__ __launch_bounds__(kThreads) void k_check(const int32_t* __restrict__ fgrams,
                                                    const int32_t* __restrict__ lengths,
                                                    int64_t n, int max_len, int64_t vocab,
                                                    unsigned* __restrict__ status) {
    const int64_t g = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (g >= n) return;
    const unsigned bad = data_errors(fgrams, lengths, g, max_len, vocab);
    if (bad) atomicOr(status, bad);
}

// ------------------------------------------------------------- rank sort ----

// The sort key of f-gram g: max_len - 1 tokens, paired into 64 bits (NK words).
template <int NK>
__device__ __forceinline__ void sort_key(const int32_t* __restrict__ fgrams,
                                         const int32_t* __restrict__ lengths, int64_t g,
                                         int max_len, int64_t vocab, uint64_t (&k)[NK]) {
    const int len = len_of(lengths, g, max_len);
#pragma unroll
    for (int w = 0; w < NK; ++w) {
        const uint64_t hi = 2 * w < max_len - 1 ? key_at(fgrams + g * max_len, len, 2 * w, vocab) : 0;
        const uint64_t lo =
            2 * w + 1 < max_len - 1 ? key_at(fgrams + g * max_len, len, 2 * w + 1, vocab) : 0;
        k[w] = (hi << 32) | lo;
    }
}

// Workgroup (x, y) counts, for each of 256 f-grams, how many of kRankTile others
// come before it (equal keys in input order).
constexpr int kRankTile = 64;

template <int NK>
__global__ __launch_bounds__(kThreads) void k_rank(const int32_t* __restrict__ fgrams,
                                                   const int32_t* __restrict__ lengths, int64_t n,
                                                   int max_len, int64_t vocab,
                                                   unsigned* __restrict__ rank) {
    __shared__ uint64_t s_key[kRankTile][NK];
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int64_t j0 = (int64_t)blockIdx.y * kRankTile;
    uint64_t mine[NK] = {};
    if (i < n) sort_key(fgrams, lengths, i, max_len, vocab, mine);
    if (threadIdx.x < kRankTile && j0 + threadIdx.x < n) {
        uint64_t k[NK];
        sort_key(fgrams, lengths, j0 + threadIdx.x, max_len, vocab, k);
#pragma unroll
        for (int w = 0; w < NK; ++w) s_key[threadIdx.x][w] = k[w];
    }
    __syncthreads();
    const int m = n - j0 < kRankTile ? (int)(n - j0) : kRankTile;
    unsigned before = 0;
    for (int j = 0; j < m; ++j) {
        bool lt = false, eq = true;
#pragma unroll
        for (int w = 0; w < NK; ++w) {
            const uint64_t k = s_key[j][w];
            lt |= eq & (k < mine[w]);
            eq &= k == mine[w];
        }
        before += (lt || (eq && j0 + j < i)) ? 1u : 0u;
    }
    if (i < n && before) atomicAdd(rank + i, before);
}

__global__ __launch_bounds__(kThreads) void k_place(const unsigned* __restrict__ rank, int64_t n,
                                                    int32_t* __restrict__ order) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n) order[rank[i]] = (int32_t)i;
}

// ------------------------------------------------------------ radix sort ----
// A workgroup owns kRadixPer consecutive places of the current order, each of
// its four wavefronts a quarter of them.

constexpr int kRadixPer = 4096;

__device__ __forceinline__ int radix_digit(const int32_t* __restrict__ fgrams,
                                           const int32_t* __restrict__ lengths, int64_t g,
                                           int max_len, int64_t vocab, int tok, int shift) {
    return (int)(key_at(fgrams + g * max_len, len_of(lengths, g, max_len), tok, vocab) >> shift) &
           255;
}

// hist[digit * blocks + block]; `in` null stands for the input order.
__global__ __launch_bounds__(kThreads) void k_radix_count(
    const int32_t* __restrict__ fgrams, const int32_t* __restrict__ lengths, int64_t n,
    int max_len, int64_t vocab, int tok, int shift, const int32_t* __restrict__ in,
    uint32_t* __restrict__ hist) {
    __shared__ unsigned s_cnt[256];
    s_cnt[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kRadixPer;
    for (int k = threadIdx.x; k < kRadixPer && base + k < n; k += kThreads) {
        const int64_t g = in ? in[base + k] : base + k;
        atomicAdd(&s_cnt[radix_digit(fgrams, lengths, g, max_len, vocab, tok, shift)], 1u);
    }
    __syncthreads();
    hist[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = s_cnt[threadIdx.x];
}

// Stable scatter; hist holds the exclusive scan of the counts.
__global__ __launch_bounds__(kThreads) void k_radix_scatter(
    const int32_t* __restrict__ fgrams, const int32_t* __restrict__ lengths, int64_t n,
    int max_len, int64_t vocab, int tok, int shift, const int32_t* __restrict__ in,
    const uint32_t* __restrict__ hist, int32_t* __restrict__ out) {
    constexpr int kWaves = kThreads / 64, kPerWave = kRadixPer / kWaves, kRounds = kPerWave / 64;
    __shared__ unsigned s_at[kWaves][256];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int w = 0; w < kWaves; ++w) s_at[w][threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kRadixPer + wave * kPerWave;
    int32_t g[kRounds];
    int dig[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int64_t s = base + r * 64 + lane;
        g[r] = s < n ? (in ? in[s] : (int32_t)s) : -1;
        dig[r] = 0;
        if (g[r] >= 0) {
            dig[r] = radix_digit(fgrams, lengths, g[r], max_len, vocab, tok, shift);
            atomicAdd(&s_at[wave][dig[r]], 1u);
        }
    }
    __syncthreads();
    unsigned at = hist[(int64_t)threadIdx.x * gridDim.x + blockIdx.x];
    for (int w = 0; w < kWaves; ++w) {
        const unsigned c = s_at[w][threadIdx.x];
        s_at[w][threadIdx.x] = at;
        at += c;
    }
    __syncthreads();
    const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        // the lanes with this lane's digit
        unsigned long long same = __ballot(g[r] >= 0);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const unsigned long long m = __ballot((dig[r] >> b) & 1);
            same &= (dig[r] >> b) & 1 ? m : ~m;
        }
        if (g[r] >= 0) {
            const unsigned p = s_at[wave][dig[r]];
            out[p + (unsigned)__popcll(same & below)] = g[r];
        }
        // every lane has read its place before the first of each digit moves it
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        __builtin_amdgcn_wave_barrier();
        if (g[r] >= 0 && (same & below) == 0)
            s_at[wave][dig[r]] += (unsigned)__popcll(same);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        __builtin_amdgcn_wave_barrier();
    }
}

// ------------------------------------------------------- exclusive scans ----
// Three kernels: the sum of every kScanPer values, the scan of those sums by
// one workgroup, and the scan inside each run.

constexpr int kScanPer = 4096;

template <typename T>
__device__ __forceinline__ T wave_inclusive(T v, int lane) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const T u = __shfl_up(v, o);
        if (lane >= o) v += u;
    }
    return v;
}

// Exclusive scan of v over the workgroup's threads; `total` gets the sum.
template <typename T>
__device__ __forceinline__ T block_exclusive(T v, T* s_wave, T& total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const T inc = wave_inclusive(v, lane);
    __syncthreads();
    if (lane == 63) s_wave[wave] = inc;
    __syncthreads();
    T add = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) {
        if (w < wave) add += s_wave[w];
        total += s_wave[w];
    }
    return inc - v + add;
}

template <typename T, typename In>
__global__ __launch_bounds__(kThreads) void k_scan_sums(const In* __restrict__ in, int64_t n,
                                                        T* __restrict__ sums) {
    __shared__ T s_wave[kThreads / 64];
    const int64_t base = (int64_t)blockIdx.x * kScanPer;
    T v = 0;
    for (int k = threadIdx.x; k < kScanPer && base + k < n; k += kThreads) v += (T)in[base + k];
    T total;
    (void)block_exclusive(v, s_wave, total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

template <typename T>
__global__ __launch_bounds__(kThreads) void k_scan_top(T* __restrict__ sums, int64_t n) {
    __shared__ T s_wave[kThreads / 64];
    T carry = 0;
    for (int64_t b = 0; b < n; b += kThreads) {
        const int64_t i = b + threadIdx.x;
        const T v = i < n ? sums[i] : 0;
        T total;
        const T ex = block_exclusive(v, s_wave, total);
        if (i < n) sums[i] = carry + ex;
        carry += total;
    }
}

// out[i] = the sum of in[0 .. i); in and out may be the same array.
template <typename T, typename In>
__global__ __launch_bounds__(kThreads) void k_scan_runs(const In* in, int64_t n,
                                                        const T* __restrict__ sums, T* out) {
    constexpr int kPer = kScanPer / kThreads;
    __shared__ T s_wave[kThreads / 64];
    const int64_t base = (int64_t)blockIdx.x * kScanPer + (int64_t)threadIdx.x * kPer;
    T v[kPer], sum = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        v[k] = base + k < n ? (T)in[base + k] : 0;
        sum += v[k];
    }
    T total;
    T at = sums[blockIdx.x] + block_exclusive(sum, s_wave, total);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        if (base + k < n) out[base + k] = at;
        at += v[k];
    }
}

template <typename T, typename In>
inline hipError_t scan(const In* in, int64_t n, T* sums, T* out, hipStream_t st) {
    const int64_t runs = (n + kScanPer - 1) / kScanPer;
    hipLaunchKernelGGL((k_scan_sums<T, In>), dim3((unsigned)runs), dim3(kThreads), 0, st, in, n,
                       sums);
    hipLaunchKernelGGL(k_scan_top<T>, dim3(1), dim3(kThreads), 0, st, sums, runs);
    hipLaunchKernelGGL((k_scan_runs<T, In>), dim3((unsigned)runs), dim3(kThreads), 0, st, in, n,
                       sums, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ tree ----

// The depths that f-gram g shares with f-gram p, its neighbour in sorted order.
__device__ __forceinline__ int shared_depths(const int32_t* __restrict__ fgrams,
                                             const int32_t* __restrict__ lengths, int max_len,
                                             int64_t vocab, int64_t g, int64_t p) {
    const int len = len_of(lengths, g, max_len), plen = len_of(lengths, p, max_len);
    int c = 0;
    while (c < len - 1 && c < plen &&
           key_at(fgrams + g * max_len, len, c, vocab) ==
               key_at(fgrams + p * max_len, plen, c, vocab))
        ++c;
    return c;
}

// share[s] and the inner nodes that f-gram s adds, for s <= n (the last one is
// an end mark that adds none, so that its scanned value is the total).
__global__ __launch_bounds__(kThreads) void k_share(const int32_t* __restrict__ fgrams,
                                                    const int32_t* __restrict__ lengths,
                                                    int64_t n, int max_len, int64_t vocab,
                                                    const int32_t* __restrict__ order,
                                                    uint8_t* __restrict__ share,
                                                    uint8_t* __restrict__ adds) {
    const int64_t s = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (s > n) return;
    int c = 0, add = 0;
    if (s < n) {
        const int64_t g = order[s];
        if (s > 0) c = shared_depths(fgrams, lengths, max_len, vocab, g, order[s - 1]);
        add = len_of(lengths, g, max_len) - 1 - c;
    }
    share[s] = (uint8_t)c;
    adds[s] = (uint8_t)add;
}

// Nodes per chunk that the limits aim at: the last f-gram of a chunk may pass
// the aim by up to max_len nodes, and its first one adds up to max_len - 1 again.
__host__ __device__ constexpr int64_t chunk_aim(int max_len) { return kChunkRows - 2 * max_len; }

// One chunk limit: the first f-gram with at least k * chunk_aim nodes before it
// (each f-gram before it adds its own last node), the inner nodes before it and
// the depths that it shares.
struct Limit {
    int64_t first, inner;
    int64_t share;
};

__global__ __launch_bounds__(kThreads) void k_chunks(const int64_t* __restrict__ inner, int64_t n,
                                                     const uint8_t* __restrict__ share,
                                                     int max_len, int64_t n_limits,
                                                     Limit* __restrict__ limits) {
    const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (k >= n_limits) return;
    const int64_t want = k * chunk_aim(max_len);
    int64_t lo = 0, hi = n;  // the answer lies in [lo, hi]
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo) / 2;
        if (mid + inner[mid] >= want) hi = mid;
        else lo = mid + 1;
    }
    limits[k] = Limit{lo, inner[lo], (int64_t)share[lo]};
}

// Everything up to the chunk limits for fewer than kThreads f-grams, in one
// workgroup: such a list is one chunk, and the ten operations that this replaces
// are launches one after another (one f-gram through one layer of d = 512 165-174 us,
// now 119-124).
template <int NK>
__global__ __launch_bounds__(kThreads) void k_short_list(
    const int32_t* __restrict__ fgrams, const int32_t* __restrict__ lengths, int n, int max_len,
    int64_t vocab, int32_t* __restrict__ order, uint8_t* __restrict__ share,
    int64_t* __restrict__ inner, Limit* __restrict__ limits, unsigned* __restrict__ status) {
    __shared__ uint64_t s_key[kThreads][NK];
    __shared__ int s_order[kThreads], s_sum[kThreads / 64];
    __shared__ unsigned s_bad;
    const int t = threadIdx.x;
    if (t == 0) s_bad = 0;
    uint64_t mine[NK] = {};
    unsigned bad = 0;
    if (t < n) {
        sort_key(fgrams, lengths, t, max_len, vocab, mine);
        bad = data_errors(fgrams, lengths, t, max_len, vocab);
    }
#pragma unroll
    for (int w = 0; w < NK; ++w) s_key[t][w] = mine[w];
    __syncthreads();
    if (bad) atomicOr(&s_bad, bad);
    int rank = 0;
    for (int j = 0; j < n; ++j) {
        bool lt = false, eq = true;
#pragma unroll
        for (int w = 0; w < NK; ++w) {
            const uint64_t k = s_key[j][w];
            lt |= eq & (k < mine[w]);
            eq &= k == mine[w];
        }
        rank += lt || (eq && j < t) ? 1 : 0;
    }
    if (t < n) s_order[rank] = t;
    __syncthreads();
    int c = 0, add = 0;
    if (t < n) {
        const int g = s_order[t];
        if (t > 0) c = shared_depths(fgrams, lengths, max_len, vocab, g, s_order[t - 1]);
        add = len_of(lengths, g, max_len) - 1 - c;
        order[t] = g;
    }
    int total;
    const int at = block_exclusive(add, s_sum, total);
    if (t <= n) {
        share[t] = (uint8_t)c;
        inner[t] = at;
    }
    if (t == 0) {
        limits[0] = Limit{0, 0, 0};
        limits[1] = Limit{n, total, 0};
        *status = s_bad;
    }
}

// The nodes of one chunk.  A thread owns one f-gram; the node at depth i of its
// path was added by the last f-gram at or before it that added a node at that
// depth: a maximum over the f-grams of the workgroup up to it, or, where that
// lies before the workgroup, the first f-gram of the chunk with the same i + 1
// tokens (found by bisection, once per depth and workgroup).
__global__ __launch_bounds__(kThreads) void k_nodes(const int32_t* __restrict__ fgrams,
                                                    const int32_t* __restrict__ lengths,
                                                    int max_len, int64_t vocab,
                                                    const int32_t* __restrict__ order,
                                                    const uint8_t* __restrict__ share,
                                                    const int64_t* __restrict__ inner, Chunk c,
                                                    Node* __restrict__ nodes) {
    constexpr int kD = SCONE_MAX_FGRAM_LEN - 1;  // depths above the last
    constexpr int kWaves = kThreads / 64;
    __shared__ int s_carry[kD];
    __shared__ int s_wave[kWaves][kD];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int b0 = blockIdx.x * kThreads;  // f-grams are counted from the chunk's first
    const int f = b0 + threadIdx.x;
    const bool valid = f < c.n_f;
    auto len_at = [&](int q) { return len_of(lengths, order[c.first + q], max_len); };
    auto share_at = [&](int q) { return q == 0 ? 0 : (int)share[c.first + q]; };
    // inner nodes of the chunk before f-gram q's
    auto base_at = [&](int q) {
        return q == 0 ? 0 : (int)(inner[c.first + q] - c.inner) + c.share;
    };
    auto row_at = [&](int q, int i) {  // the row of the node that q added at depth i
        return i == len_at(q) - 1 ? q : (int)c.n_f + base_at(q) + i - share_at(q);
    };
    if (threadIdx.x < kD) {
        const int i = threadIdx.x;
        int found = -1;
        if (b0 > 0 && i < share_at(b0)) {
            const int64_t g = order[c.first + b0];
            const int len = len_of(lengths, g, max_len);
            int lo = 0, hi = b0;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                const int64_t m = order[c.first + mid];
                const int mlen = len_of(lengths, m, max_len);
                bool lt = false;
                for (int j = 0; j <= i; ++j) {
                    const uint32_t a = key_at(fgrams + m * max_len, mlen, j, vocab);
                    const uint32_t b = key_at(fgrams + g * max_len, len, j, vocab);
                    if (a != b) {
                        lt = a < b;
                        break;
                    }
                }
                if (lt) lo = mid + 1;
                else hi = mid;
            }
            found = lo;
        }
        s_carry[i] = found;
    }
    int64_t g = 0;
    int len = 0, sh = 0;
    if (valid) {
        g = order[c.first + f];
        len = len_of(lengths, g, max_len);
        sh = share_at(f);
    }
    int by[kD];  // who added the node at each depth
#pragma unroll
    for (int i = 0; i < kD; ++i) {
        int v = (valid && sh <= i && i < len) ? f : -1;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int u = __shfl_up(v, o);
            if (lane >= o) v = u > v ? u : v;
        }
        if (lane == 63) s_wave[wave][i] = v;
        by[i] = v;
    }
    __syncthreads();
    if (!valid) return;
#pragma unroll
    for (int i = 0; i < kD; ++i) {
        int v = by[i];
        for (int w = 0; w < wave; ++w) v = s_wave[w][i] > v ? s_wave[w][i] : v;
        by[i] = s_carry[i] > v ? s_carry[i] : v;
    }
    const int base = base_at(f);
    Node nd;
#pragma unroll
    for (int i = 0; i < kD; ++i) nd.up[i] = 0;
#pragma unroll
    for (int i = 0; i <= kD; ++i) {
        if (i >= len) break;
        const bool last = i == len - 1;
        if (i >= sh) {  // a node of this f-gram's own
            nd.pos = i;
            nd.tok = (int32_t)(key_at(fgrams + g * max_len, len, i, vocab) - 1u);
            nodes[last ? f : (int)c.n_f + base + i - sh] = nd;
        }
        if (!last && i < kD)
            nd.up[i] = i >= sh ? (int)c.n_f + base + i - sh : row_at(by[i], i);
    }
}

// The last nodes of a chunk's f-grams in input order, which is written to `order`:
// all that a model with no layers reads.
__global__ __launch_bounds__(kThreads) void k_last_nodes(const int32_t* __restrict__ fgrams,
                                                         const int32_t* __restrict__ lengths,
                                                         int max_len, int64_t vocab, Chunk c,
                                                         int32_t* __restrict__ order,
                                                         Node* __restrict__ nodes) {
    const int64_t f = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (f >= c.n_f) return;
    const int64_t g = c.first + f;
    const int len = len_of(lengths, g, max_len);
    Node nd{};
    nd.pos = len - 1;
    nd.tok = (int32_t)(key_at(fgrams + g * max_len, len, len - 1, vocab) - 1u);
    nodes[f] = nd;
    order[g] = (int32_t)g;
}

// ------------------------------------------------------------------ host ----

struct Layout {
    int64_t max_rows;   // nodes of the largest chunk
    int64_t n_limits;   // chunk limits, one past the last chunk's end included
    int64_t n_blocks;   // workgroups of a radix pass
    size_t ctl, limits, order_a, order_b, hist, sums, adds, share, inner, nodes, total;
};

inline Layout layout(int64_t n, int max_len) {
    Layout l{};
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off = (off + bytes + 255) & ~(size_t)255;
        return at;
    };
    l.max_rows = n > kChunkRows / max_len ? kChunkRows : n * max_len;
    l.n_limits = n * max_len / chunk_aim(max_len) + 2;
    l.n_blocks = (n + kRadixPer - 1) / kRadixPer;
    l.ctl = take(256);
    l.limits = take((size_t)l.n_limits * sizeof(Limit));
    l.order_a = take((size_t)n * 4);
    l.order_b = take((size_t)n * 4);  // the rank sort's ranks
    l.hist = take((size_t)l.n_blocks * 256 * 4);
    // sums of either scan: of n + 1 values in 64 bits, of the histograms in 32
    l.sums = take((size_t)((n + kScanPer) / kScanPer + 1) * 8 +
                  (size_t)(l.n_blocks * 256 / kScanPer + 1) * 4);
    l.adds = take((size_t)n + 1);
    l.share = take((size_t)n + 1);
    l.inner = take((size_t)(n + 1) * 8);
    l.nodes = take((size_t)l.max_rows * sizeof(Node));
    l.total = off;
    return l;
}

struct Builder {
    const int32_t* fgrams;
    const int32_t* lengths;
    int64_t n;
    int max_len;
    int64_t vocab;
    uint8_t* ws;
    Layout l;
    bool flat;  // no tree: the f-grams' last nodes alone, in input order
    hipStream_t st;

    template <typename T>
    T* at(size_t off) const {
        return reinterpret_cast<T*>(ws + off);
    }
    unsigned* status() const { return at<unsigned>(l.ctl); }
    const int32_t* order() const {
        return at<int32_t>(!flat && radix_passes() % 2 ? l.order_b : l.order_a);
    }
    Node* nodes() const { return at<Node>(l.nodes); }

    // Bytes of the largest key value, `vocab` (a token plus one).
    int key_bytes() const {
        int b = 1;
        while (b < 4 && vocab >> (8 * b)) ++b;
        return b;
    }
    // Radix passes; 0 where the rank sort is used.  Pass 0 writes order_b.
    int radix_passes() const {
        const int passes = (max_len - 1) * key_bytes();
        return n * n <= kRankPerPass * passes ? 0 : passes;
    }

    hipError_t sort() const {
        const unsigned g_n = (unsigned)((n + kThreads - 1) / kThreads);
        if (radix_passes() == 0) {
            unsigned* rank = at<unsigned>(l.order_b);
            const dim3 grid(g_n, (unsigned)((n + kRankTile - 1) / kRankTile)), block(kThreads);
            const hipError_t e = hipMemsetAsync(rank, 0, (size_t)n * 4, st);
            if (e != hipSuccess) return e;
            switch (max_len / 2) {  // words of max_len - 1 tokens, two to a word
                case 1: hipLaunchKernelGGL(k_rank<1>, grid, block, 0, st, fgrams, lengths, n, max_len, vocab, rank); break;
                case 2: hipLaunchKernelGGL(k_rank<2>, grid, block, 0, st, fgrams, lengths, n, max_len, vocab, rank); break;
                default: hipLaunchKernelGGL(k_rank<3>, grid, block, 0, st, fgrams, lengths, n, max_len, vocab, rank); break;
            }
            hipLaunchKernelGGL(k_place, dim3(g_n), block, 0, st, rank, n, at<int32_t>(l.order_a));
            return hipGetLastError();
        }
        const dim3 grid((unsigned)l.n_blocks), block(kThreads);
        uint32_t* hist = at<uint32_t>(l.hist);
        const int32_t* in = nullptr;
        int pass = 0;
        for (int tok = max_len - 2; tok >= 0; --tok)
            for (int b = 0; b < key_bytes(); ++b, ++pass) {
                int32_t* out = at<int32_t>(pass % 2 ? l.order_a : l.order_b);
                hipLaunchKernelGGL(k_radix_count, grid, block, 0, st, fgrams, lengths, n, max_len,
                                   vocab, tok, 8 * b, in, hist);
                const hipError_t e = scan(hist, l.n_blocks * 256, at<uint32_t>(l.sums), hist, st);
                if (e != hipSuccess) return e;
                hipLaunchKernelGGL(k_radix_scatter, grid, block, 0, st, fgrams, lengths, n,
                                   max_len, vocab, tok, 8 * b, in, hist, out);
                in = out;
            }
        return hipGetLastError();
    }

    // The tree up to the chunk limits, on the device.
    hipError_t find_chunks() const {
        const unsigned g_n = (unsigned)((n + kThreads - 1) / kThreads);
        const unsigned g_n1 = (unsigned)((n + kThreads) / kThreads);
        const dim3 block(kThreads);
        if (!flat && n < kThreads) {
            auto launch = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, dim3(1), block, 0, st, fgrams, lengths, (int)n, max_len,
                                   vocab, at<int32_t>(l.order_a), at<uint8_t>(l.share),
                                   at<int64_t>(l.inner), at<Limit>(l.limits), status());
            };
            switch (max_len / 2) {  // words of max_len - 1 tokens, two to a word
                case 1: launch(k_short_list<1>); break;
                case 2: launch(k_short_list<2>); break;
                default: launch(k_short_list<3>); break;
            }
            return hipGetLastError();
        }
        hipError_t e = hipMemsetAsync(status(), 0, sizeof(unsigned), st);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_check, dim3(g_n), block, 0, st, fgrams, lengths, n, max_len, vocab,
                           status());
        if (flat) return hipGetLastError();
        e = sort();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_share, dim3(g_n1), block, 0, st, fgrams, lengths, n, max_len, vocab,
                           order(), at<uint8_t>(l.share), at<uint8_t>(l.adds));
        e = scan(at<uint8_t>(l.adds), n + 1, at<int64_t>(l.sums), at<int64_t>(l.inner), st);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_chunks, dim3((unsigned)((l.n_limits + kThreads - 1) / kThreads)),
                           block, 0, st, at<int64_t>(l.inner), n, at<uint8_t>(l.share), max_len,
                           l.n_limits, at<Limit>(l.limits));
        return hipGetLastError();
    }

    // Sorts the f-grams (unless flat) and finds the chunks; waits for the stream.
    // `bits` gets the data errors found (err_bit of SCONE_ELEN and SCONE_ETOKEN).
    int build(std::vector<Chunk>& chunks, unsigned& bits) const {
        SCONE_HIP_TRY(find_chunks());
        // the status word and, right behind its 256 bytes, the limits in one copy
        std::vector<Limit> lim(flat ? 0 : (size_t)l.n_limits);
        std::vector<uint8_t> back((l.limits - l.ctl) + lim.size() * sizeof(Limit));
        SCONE_HIP_TRY(hipMemcpyAsync(back.data(), ws + l.ctl, back.size(), hipMemcpyDeviceToHost,
                                     st));
        SCONE_HIP_TRY(hipStreamSynchronize(st));
        std::memcpy(&bits, back.data(), sizeof(bits));
        if (flat) {
            for (int64_t s = 0; s < n; s += l.max_rows) {
                const int64_t n_f = n - s < l.max_rows ? n - s : l.max_rows;
                chunks.push_back(Chunk{s, 0, n_f, n_f, 0});
            }
            return SCONE_OK;
        }
        std::memcpy(lim.data(), back.data() + (l.limits - l.ctl), lim.size() * sizeof(Limit));
        for (size_t k = 0; k + 1 < lim.size() && lim[k].first < n; ++k) {
            Chunk c;
            c.first = lim[k].first;
            c.inner = lim[k].inner;
            c.n_f = lim[k + 1].first - c.first;
            c.share = (int)lim[k].share;
            c.rows = c.n_f + lim[k + 1].inner - c.inner + c.share;
            if (c.rows > l.max_rows) return SCONE_EHIP;  // cannot happen: see chunk_aim
            chunks.push_back(c);
        }
        return SCONE_OK;
    }

    // Writes the nodes of one of build's chunks.
    hipError_t fill_nodes(const Chunk& c) const {
        if (flat) {
            hipLaunchKernelGGL(k_last_nodes, dim3((unsigned)((c.n_f + kThreads - 1) / kThreads)),
                               dim3(kThreads), 0, st, fgrams, lengths, max_len, vocab, c,
                               at<int32_t>(l.order_a), nodes());
            return hipGetLastError();
        }
        hipLaunchKernelGGL(k_nodes, dim3((unsigned)((c.n_f + kThreads - 1) / kThreads)),
                           dim3(kThreads), 0, st, fgrams, lengths, max_len, vocab, order(),
                           at<uint8_t>(l.share), at<int64_t>(l.inner), c, nodes());
        return hipGetLastError();
    }
};

}  // namespace tree
}  // namespace scone
