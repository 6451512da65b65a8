// Building the f-gram dictionary: an open-addressing hash table in HBM.
//
// The paper stores the f-gram layer as a dense row matrix plus a hash
// dictionary from f-grams to row indices (Section 2), built before serving
// (Section 3.2).  Here the dictionary is a power-of-two array of slots with
// linear probing from the start of the key's 64-byte bucket.  Insertion
// claims the first empty slot on the key's probe path with a 64-bit
// compare-and-swap on the slot's first key word, then writes the rest of the
// key and the id.  Two f-grams with one key walk the same path, so the second
// one meets the first one's slot: a compare-and-swap that finds the key's own
// first word makes the key a suspect, and only where there are suspects does a
// second pass read every key's path and report a key that stands in it twice
// (a duplicate f-gram).
//
// A third pass adds the suffix entries that let lookups skip probes: for
// every f-gram of length 4 or more, the entry of its last three tokens gets
// kExtBit, and for every f-gram of length 6 or more, so does the entry of its
// last five; where that suffix is not itself an f-gram, a marker entry
// (id kMarkerId) is inserted for it.  Two threads may insert the same marker
// at once, leaving two identical copies; lookups read whichever comes first
// on the probe path, so that costs a slot and nothing else.  The slot count
// allows for one marker per such suffix.
//
// All of it is random 128-byte lines of the table: 10M f-grams of length 2-5
// (a table of 1 GB) take 807 us to insert and 590 us to mark on MI355X.  The
// passes use read-modify-writes and plain loads only: a marking pass that
// published its slots with agent-scope release and acquire, which write back
// and invalidate the whole L2, took 7.3 ms.
#include <algorithm>
#include <cmath>
#include <new>

#include "scone_internal.h"

namespace scone {
namespace {

constexpr int kBuildThreads = 256;

template <typename Tok>
__device__ __forceinline__ bool tokens_in_range(const Tok* tok, int n) {
    bool ok = true;
    for (int i = 0; i < n; ++i) ok &= (tok[i] >= 0) & (tok[i] < SCONE_TOKEN_LIMIT);
    return ok;
}

template <int SB>
__global__ __launch_bounds__(kBuildThreads) void k_insert(
    const int32_t* __restrict__ fgrams, const int32_t* __restrict__ lengths,
    const int32_t* __restrict__ ids, int64_t n, int max_len,
    typename SlotOps<SB>::Slot* __restrict__ slots, uint64_t mask, unsigned* __restrict__ status,
    unsigned* __restrict__ suspects, int64_t block0) {
    const int64_t k = block_index(block0) * kBuildThreads + threadIdx.x;
    if (k >= n) return;
    const int len = lengths[k];
    const int32_t id = ids[k];
    if (len < 2 || len > max_len) {
        atomicOr(status, err_bit(SCONE_ELEN));
        return;
    }
    if (id < 0 || id == kMarkerId) {
        atomicOr(status, err_bit(SCONE_EID));
        return;
    }
    const int32_t* tok = fgrams + k * (int64_t)max_len;
    if (!tokens_in_range(tok, len)) {
        atomicOr(status, err_bit(SCONE_ETOKEN));
        return;
    }
    const Key key = pack_key(tok, len);
    uint64_t s = home_slot(key, mask, Bucket<SB>::kSlots);
    for (uint64_t step = 0; step <= mask; ++step) {
        unsigned long long* w0 = reinterpret_cast<unsigned long long*>(&slots[s].w0);
        const uint64_t old = atomicCAS(w0, 0ull, (unsigned long long)key.w0);
        if (old == 0) {
            SlotOps<SB>::write_rest(slots, s, key, id);
            return;
        }
        if (old == key.w0) atomicOr(suspects, 1u);
        s = (s + 1) & mask;
    }
    atomicOr(status, err_bit(SCONE_EFULL));
}

// Reports keys that stand twice in their probe path (a path ends at its first
// empty slot).  Runs only where the insertion met a suspect and every input
// was in range (an input error comes first, and leaves keys out of the table).
constexpr int kSweepBlocks = 2048;  // workgroups of the passes that take runs of f-grams
constexpr int kCountBlocks = 512;   // of the count, whose adds to one word are serialised

template <int SB>
__global__ __launch_bounds__(kBuildThreads) void k_verify(
    const int32_t* __restrict__ fgrams, const int32_t* __restrict__ lengths, int64_t n,
    int max_len, const typename SlotOps<SB>::Slot* __restrict__ slots, uint64_t mask,
    unsigned* __restrict__ status, const unsigned* __restrict__ suspects) {
    if (*suspects == 0) return;
    if (__hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) &
        (err_bit(SCONE_ELEN) | err_bit(SCONE_EID) | err_bit(SCONE_ETOKEN) | err_bit(SCONE_EFULL)))
        return;
    for (int64_t k = (int64_t)blockIdx.x * kBuildThreads + threadIdx.x; k < n;
         k += (int64_t)gridDim.x * kBuildThreads) {
        const Key key = pack_key(fgrams + k * (int64_t)max_len, lengths[k]);
        uint64_t s = home_slot(key, mask, Bucket<SB>::kSlots);
        int found = 0;
        for (uint64_t step = 0; step <= mask && found < 2; ++step) {
            uint64_t w0, w1;
            int32_t id;
            SlotOps<SB>::read(slots, s, w0, w1, id);
            if (w0 == 0) break;
            found += w0 == key.w0 && w1 == key.w1 ? 1 : 0;
            s = (s + 1) & mask;
        }
        if (found > 1) atomicOr(status, err_bit(SCONE_EDUP));
    }
}

// Counts the f-grams of length 4..max_len and 6..max_len (the suffix entries
// the third pass may add).  Each workgroup takes a strided run of the lengths
// and adds each count once: with one workgroup per 256 lengths, the adds to
// the two counters were serialised and took 472 us for 10M f-grams instead of
// 17 us.
__global__ __launch_bounds__(kBuildThreads) void k_count_long(
    const int32_t* __restrict__ lengths, int64_t n, int max_len,
    unsigned long long* __restrict__ counts) {
    __shared__ unsigned s_c[2];
    if (threadIdx.x < 2) s_c[threadIdx.x] = 0;
    __syncthreads();
    unsigned c4 = 0, c6 = 0;
    const int64_t stride = (int64_t)gridDim.x * kBuildThreads;
    for (int64_t k = (int64_t)blockIdx.x * kBuildThreads + threadIdx.x; k < n; k += 8 * stride) {
        int len[8];  // eight loads in flight
#pragma unroll
        for (int u = 0; u < 8; ++u) len[u] = k + u * stride < n ? lengths[k + u * stride] : 0;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            c4 += len[u] >= 4 && len[u] <= max_len ? 1u : 0u;
            c6 += len[u] >= 6 && len[u] <= max_len ? 1u : 0u;
        }
    }
    if (c4) atomicAdd(&s_c[0], c4);
    if (c6) atomicAdd(&s_c[1], c6);
    __syncthreads();
    if (threadIdx.x < 2 && s_c[threadIdx.x])
        atomicAdd(counts + threadIdx.x, (unsigned long long)s_c[threadIdx.x]);
}

// Gives the entry of `key` (3 or 5 tokens) kExtBit, inserting a marker when the
// key has no entry; returns whether it inserted one.
//
// A plain look comes first: most suffixes that many f-grams share are found
// with the bit set, from the L2.  Plain loads may be older than other
// workgroups' writes, so what they don't show is settled with
// read-modify-writes.  A length-3 key is whole in its first word (52 bits; the
// second is 0), so one compare-and-swap claims or finds its slot.  A length-5
// key has 20 bits in the second word: the claimer writes that word and then
// `ready`, each with a read-modify-write that has returned before the next, and
// others compare the second word only once they have seen `ready`; a slot that
// is not ready counts as another key (at worst a second, identical marker).
// The id word of a marker is written with an atomic OR of all its bits, since
// another thread may set kExtBit at the same time.
constexpr int kMaxLooks = 256;

template <int SB, int kTokens>
__device__ __forceinline__ bool mark_suffix(typename SlotOps<SB>::Slot* slots, uint64_t mask,
                                            const Key& key, unsigned* status) {
    static_assert(kTokens == 3 || (kTokens == 5 && SB == 32), "suffixes of 3 or 5 tokens");
    constexpr int BW = Bucket<SB>::kSlots;
    const uint64_t home = home_slot(key, mask, BW);
    // an entry's ready word is read before its key words, so that these are whole
#pragma unroll
    for (int i = 0; i < BW; ++i) {
        if (kTokens == 5) {
            const uint32_t ready = SlotOps<SB>::load_ready(slots, home + i);
            if (!ready) continue;
        }
        uint64_t w0, w1;
        int32_t id;
        SlotOps<SB>::read(slots, home + i, w0, w1, id);
        if (w0 == key.w0 && w1 == key.w1 && id < 0) return false;
    }
    uint64_t s = home;
    int looks = 0;
    for (uint64_t step = 0; step <= mask;) {
        const uint64_t old =
            atomicCAS(reinterpret_cast<unsigned long long*>(&slots[s].w0), 0ull,
                      (unsigned long long)key.w0);
        unsigned* idp = reinterpret_cast<unsigned*>(&slots[s].id);
        if (old == 0) {
            if (kTokens == 5) SlotOps<SB>::publish_w1(slots, s, key.w1);
            atomicOr(idp, (unsigned)kMarkerId | kExtBit);
            return true;
        }
        if (old == key.w0) {
            if (kTokens == 5 && !SlotOps<SB>::ready_now(slots, s) && ++looks < kMaxLooks) continue;
            if (kTokens == 3 || SlotOps<SB>::same_w1(slots, s, key.w1)) {
                atomicOr(idp, kExtBit);
                return false;
            }
        }
        s = (s + 1) & mask;
        ++step;
    }
    atomicOr(status, err_bit(SCONE_EFULL));
    return false;
}

// Marks every suffix and counts the markers inserted (one add per workgroup).
// Skipped when an input was rejected: the table is given up then.
template <int SB>
__global__ __launch_bounds__(kBuildThreads) void k_mark(
    const int32_t* __restrict__ fgrams, const int32_t* __restrict__ lengths, int64_t n,
    int max_len, typename SlotOps<SB>::Slot* __restrict__ slots, uint64_t mask, unsigned* status,
    unsigned long long* __restrict__ markers) {
    __shared__ unsigned s_c;
    if (threadIdx.x == 0) s_c = 0;
    __syncthreads();
    unsigned c = 0;
    if (__hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0)
        for (int64_t k = (int64_t)blockIdx.x * kBuildThreads + threadIdx.x; k < n;
             k += (int64_t)gridDim.x * kBuildThreads) {
            const int len = lengths[k];
            const int32_t* tok = fgrams + k * (int64_t)max_len;
            if (len >= 4) c += mark_suffix<SB, 3>(slots, mask, pack_key(tok + len - 3, 3), status);
            if constexpr (SB == 32)
                if (len >= 6)
                    c += mark_suffix<SB, 5>(slots, mask, pack_key(tok + len - 5, 5), status);
        }
    for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off);
    if ((threadIdx.x & 63) == 0 && c) atomicAdd(&s_c, c);
    __syncthreads();
    if (threadIdx.x == 0 && s_c) atomicAdd(markers, (unsigned long long)s_c);
}

// The build's control words, before the slots in a caller's memory.
struct Control {
    unsigned status;             // err_bit of every data error found
    unsigned suspects;           // an insertion met its own first word
    unsigned long long long4;    // f-grams of length 4 or more, and of 6 or more
    unsigned long long long6;
    unsigned long long markers;  // suffix markers inserted
};
constexpr int64_t kControlBytes = 256;

template <int SB>
hipError_t launch_build(const int32_t* fgrams, const int32_t* lengths, const int32_t* ids,
                        int64_t n, int max_len, void* slots, uint64_t mask, Control* ctl,
                        hipStream_t st) {
    using Slot = typename SlotOps<SB>::Slot;
    Slot* sl = static_cast<Slot*>(slots);
    const int64_t blocks = (n + kBuildThreads - 1) / kBuildThreads;
    const dim3 sweep((unsigned)std::min<int64_t>(blocks, kSweepBlocks)), block(kBuildThreads);
    const hipError_t e = launch_blocks(blocks, kBuildThreads, [&](int64_t b0, dim3 grid) {
        hipLaunchKernelGGL(k_insert<SB>, grid, block, 0, st, fgrams, lengths, ids, n, max_len, sl,
                           mask, &ctl->status, &ctl->suspects, b0);
    });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_verify<SB>, sweep, block, 0, st, fgrams, lengths, n, max_len, sl, mask,
                       &ctl->status, &ctl->suspects);
    if (max_len >= 4)
        hipLaunchKernelGGL(k_mark<SB>, sweep, block, 0, st, fgrams, lengths, n, max_len, sl, mask,
                           &ctl->status, &ctl->markers);
    return hipGetLastError();
}

int slot_bytes_for(int max_len) { return max_len <= kMaxLenSlot16 ? 16 : 32; }

int build_sizes_ok(int64_t n, int32_t max_len, double max_load) {
    if (n < 0 || max_len < 2 || max_len > SCONE_MAX_FGRAM_LEN) return SCONE_EINVAL;
    if (!(max_load > 0.0 && max_load <= 0.9)) return SCONE_EINVAL;
    // At most n entries plus one suffix entry per f-gram of length >= 4 and
    // one more per f-gram of length >= 6, so n * 3 bounds them.
    if (std::ceil(3.0 * (double)n / max_load) > (double)(1ull << 40)) return SCONE_EINVAL;
    return SCONE_OK;
}

// Whether there can be lengths of 4 and more, which take suffix entries.
bool has_long(int64_t n, int32_t max_len) { return n > 0 && max_len >= 4; }

// Slots for these lengths: the smallest power of two >= max(64, entries /
// max_load).  Where has_long, the lengths are counted on the device, in `ctl`
// (zeroed here), and the call waits for the stream; else it does nothing there.
int count_slots(const int32_t* lengths, int64_t n, int32_t max_len, double max_load,
                Control* ctl, hipStream_t st, uint64_t& cap) {
    unsigned long long more[2] = {0, 0};
    if (has_long(n, max_len)) {
        SCONE_HIP_TRY(hipMemsetAsync(ctl, 0, sizeof(Control), st));
        const int64_t blocks = (n + kBuildThreads - 1) / kBuildThreads;
        hipLaunchKernelGGL(k_count_long, dim3((unsigned)std::min<int64_t>(blocks, kCountBlocks)),
                           dim3(kBuildThreads), 0, st, lengths, n, (int)max_len, &ctl->long4);
        SCONE_HIP_TRY(hipGetLastError());
        SCONE_HIP_TRY(hipMemcpyAsync(more, &ctl->long4, sizeof(more), hipMemcpyDeviceToHost, st));
        SCONE_HIP_TRY(hipStreamSynchronize(st));
    }
    const double entries = (double)n + (double)more[0] + (double)more[1];
    const double want = std::max(64.0, std::ceil(entries / max_load));
    cap = 64;
    while ((double)cap < want) cap <<= 1;
    return SCONE_OK;
}

// Fills a table of `cap` slots in `slots` and makes its handle; waits for the
// stream.  `cleared`: count_slots has zeroed the control words.
int fill_table(const int32_t* fgrams, const int32_t* lengths, const int32_t* ids, int64_t n,
               int32_t max_len, void* slots, uint64_t cap, Control* ctl, bool cleared, int dev,
               hipStream_t st, scone_table_t** out) {
    const int slot_bytes = slot_bytes_for(max_len);
    if (!cleared) SCONE_HIP_TRY(hipMemsetAsync(ctl, 0, sizeof(Control), st));
    SCONE_HIP_TRY(hipMemsetAsync(slots, 0, cap * (uint64_t)slot_bytes, st));
    if (n > 0) {
        const hipError_t e =
            slot_bytes == 16
                ? launch_build<16>(fgrams, lengths, ids, n, max_len, slots, cap - 1, ctl, st)
                : launch_build<32>(fgrams, lengths, ids, n, max_len, slots, cap - 1, ctl, st);
        if (e != hipSuccess) return SCONE_EHIP;
    }
    Control h{};
    SCONE_HIP_TRY(hipMemcpyAsync(&h, ctl, sizeof(h), hipMemcpyDeviceToHost, st));
    SCONE_HIP_TRY(hipStreamSynchronize(st));
    if (h.status) {
        // Report argument-like data errors before structural ones.
        for (int c : {SCONE_ELEN, SCONE_EID, SCONE_ETOKEN, SCONE_EDUP, SCONE_EFULL})
            if (h.status & err_bit(c)) return c;
        return SCONE_EFULL;
    }
    // More markers than the slots were sized for (the lengths have changed since).
    if ((double)n + (double)h.markers > 0.9 * (double)cap) return SCONE_EFULL;
    scone_table* t = new (std::nothrow) scone_table();
    if (!t) return SCONE_ENOMEM;
    t->device = dev;
    t->max_len = max_len;
    t->slot_bytes = slot_bytes;
    t->n = n;
    t->capacity = (int64_t)cap;
    t->entries = n + (int64_t)h.markers;
    t->slots = slots;
    *out = t;
    return SCONE_OK;
}

}  // namespace
}  // namespace scone

extern "C" int scone_build_fgram_table(const int32_t* fgrams, const int32_t* lengths,
                                       const int32_t* ids, int64_t n, int32_t max_len,
                                       double max_load, void* stream, scone_table_t** out) {
    using namespace scone;
    if (!out) return SCONE_EINVAL;
    *out = nullptr;
    int rc = build_sizes_ok(n, max_len, max_load);
    if (rc != SCONE_OK) return rc;
    if (n > 0 && (!fgrams || !lengths || !ids)) return SCONE_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    int dev = 0;
    SCONE_HIP_TRY(hipGetDevice(&dev));
    void *ctl = nullptr, *slots = nullptr;
    if (hipMalloc(&ctl, kControlBytes) != hipSuccess) {
        (void)hipGetLastError();
        return SCONE_ENOMEM;
    }
    uint64_t cap = 0;
    rc = count_slots(lengths, n, max_len, max_load, static_cast<Control*>(ctl), st, cap);
    if (rc == SCONE_OK &&
        hipMalloc(&slots, cap * (uint64_t)slot_bytes_for(max_len)) != hipSuccess) {
        (void)hipGetLastError();
        slots = nullptr;
        rc = SCONE_ENOMEM;
    }
    if (rc == SCONE_OK)
        rc = fill_table(fgrams, lengths, ids, n, max_len, slots, cap, static_cast<Control*>(ctl),
                        has_long(n, max_len), dev, st, out);
    if (rc == SCONE_OK) (*out)->owned = slots;
    else (void)hipStreamSynchronize(st);
    if (rc != SCONE_OK && slots) (void)hipFree(slots);
    (void)hipFree(ctl);
    return rc;
}

extern "C" int scone_fgram_table_bytes(const int32_t* lengths, int64_t n, int32_t max_len,
                                       double max_load, void* scratch, void* stream,
                                       int64_t* bytes) {
    using namespace scone;
    if (!bytes) return SCONE_EINVAL;
    *bytes = 0;
    int rc = build_sizes_ok(n, max_len, max_load);
    if (rc != SCONE_OK) return rc;
    if (!scratch || (uintptr_t)scratch % 256 != 0 || (n > 0 && !lengths)) return SCONE_EINVAL;
    if (overlaps(scratch, kControlBytes, lengths, span_bytes(n, 4))) return SCONE_EINVAL;
    uint64_t cap = 0;
    rc = count_slots(lengths, n, max_len, max_load, static_cast<Control*>(scratch),
                     static_cast<hipStream_t>(stream), cap);
    if (rc == SCONE_OK)
        *bytes = (int64_t)(cap * (uint64_t)slot_bytes_for(max_len)) + kControlBytes;
    else  // the scratch is the caller's again, whatever was queued there
        (void)hipStreamSynchronize(static_cast<hipStream_t>(stream));
    return rc;
}

namespace scone {
namespace {

// The build in the caller's memory: `sized` takes the slots from memory_bytes, which
// scone_fgram_table_bytes has counted; else they are counted here.
int build_in(const int32_t* fgrams, const int32_t* lengths, const int32_t* ids, int64_t n,
             int32_t max_len, double max_load, void* memory, int64_t memory_bytes, bool sized,
             void* stream, scone_table_t** out) {
    if (!out) return SCONE_EINVAL;
    *out = nullptr;
    int rc = build_sizes_ok(n, max_len, max_load);
    if (rc != SCONE_OK) return rc;
    if (n > 0 && (!fgrams || !lengths || !ids)) return SCONE_EINVAL;
    if (!memory || (uintptr_t)memory % 256 != 0 || memory_bytes < kControlBytes)
        return SCONE_EINVAL;
    if (overlaps(memory, memory_bytes, fgrams, span_bytes(n, 4 * (int64_t)max_len)) ||
        overlaps(memory, memory_bytes, lengths, span_bytes(n, 4)) ||
        overlaps(memory, memory_bytes, ids, span_bytes(n, 4)))
        return SCONE_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    int dev = 0;
    SCONE_HIP_TRY(hipGetDevice(&dev));
    Control* ctl = static_cast<Control*>(memory);
    const int64_t slot = slot_bytes_for(max_len);
    uint64_t cap = 0;
    if (sized) {
        cap = (uint64_t)((memory_bytes - kControlBytes) / slot);
        if (cap < 64 || (cap & (cap - 1)) != 0 ||
            (int64_t)cap * slot + kControlBytes != memory_bytes ||
            (double)cap < std::ceil((double)n / max_load))
            return SCONE_EINVAL;
    } else {
        rc = count_slots(lengths, n, max_len, max_load, ctl, st, cap);
        if (rc == SCONE_OK && memory_bytes < (int64_t)cap * slot + kControlBytes)
            rc = SCONE_EINVAL;
    }
    if (rc == SCONE_OK)
        rc = fill_table(fgrams, lengths, ids, n, max_len,
                        static_cast<uint8_t*>(memory) + kControlBytes, cap, ctl,
                        !sized && has_long(n, max_len), dev, st, out);
    // the memory is the caller's again, whatever was queued there
    if (rc != SCONE_OK) (void)hipStreamSynchronize(st);
    return rc;
}

}  // namespace
}  // namespace scone

extern "C" int scone_build_fgram_table_in(const int32_t* fgrams, const int32_t* lengths,
                                          const int32_t* ids, int64_t n, int32_t max_len,
                                          double max_load, void* memory, int64_t memory_bytes,
                                          void* stream, scone_table_t** out) {
    return scone::build_in(fgrams, lengths, ids, n, max_len, max_load, memory, memory_bytes, false,
                           stream, out);
}

extern "C" int scone_build_fgram_table_sized(const int32_t* fgrams, const int32_t* lengths,
                                             const int32_t* ids, int64_t n, int32_t max_len,
                                             double max_load, void* memory, int64_t memory_bytes,
                                             void* stream, scone_table_t** out) {
    return scone::build_in(fgrams, lengths, ids, n, max_len, max_load, memory, memory_bytes, true,
                           stream, out);
}
