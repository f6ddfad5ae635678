// Internal host-side interface between the C ABI (hg_api.hip) and the kernel
// translation units.  Not installed; not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

#include "hg_device.h"

namespace hg {

#define HG_TRY(expr)                        \
    do {                                    \
        hipError_t e__ = (expr);            \
        if (e__ != hipSuccess) return e__;  \
    } while (0)

// Calls f() the first time it is reached with a given device current and
// then never again for that device (kernel attributes such as the dynamic LDS
// limit are set per device).  Two threads arriving together may both call f,
// which must therefore be idempotent; a failed f is tried again next time.
template <typename F>
hipError_t once_per_device(std::atomic<uint64_t>& done, F&& f) {
    int dev = 0;
    HG_TRY(hipGetDevice(&dev));
    const uint64_t bit = dev >= 0 && dev < 64 ? 1ull << dev : 0;
    if (bit && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
    HG_TRY(f());
    done.fetch_or(bit, std::memory_order_release);
    return hipSuccess;
}

inline uint64_t ceil_div(uint64_t a, uint64_t b) { return (a + b - 1) / b; }
inline uint32_t log2_ceil(uint64_t x) {
    uint32_t r = 0;
    while ((1ull << r) < x) ++r;
    return r;
}
inline uint64_t pow2_ceil(uint64_t x) { return 1ull << log2_ceil(x ? x : 1); }
inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Event-timed launch range (see hg_prof.hip): inactive unless profiling is on.
struct ProfRange {
    const char* name;
    hipStream_t s;
    hipEvent_t e0 = nullptr;
    ProfRange(const char* nm, hipStream_t st);
    ~ProfRange();
    ProfRange(const ProfRange&) = delete;
    ProfRange& operator=(const ProfRange&) = delete;
};
#define HG_PROF_CAT2(a, b) a##b
#define HG_PROF_CAT(a, b) HG_PROF_CAT2(a, b)
#define HG_PROF(name, s) ::hg::ProfRange HG_PROF_CAT(hg_prof_, __LINE__)(name, s)

// The allocator that temporary workspace comes from (hg_set_allocator); both
// functions NULL means ws_alloc / hipFreeAsync.
struct WsHook {
    void* (*alloc)(size_t bytes, hipStream_t s, void* ctx) = nullptr;
    void (*free)(void* p, hipStream_t s, void* ctx) = nullptr;
    void* ctx = nullptr;
};
WsHook ws_hook();  // the hook installed now (hg_api.hip)

// Temporary memory in stream order, given back with hipFreeAsync.  The device's
// own pool unmaps what is free at every synchronisation and maps it anew at the
// next call: for 2^27 64-bit queries 3 to 50 ms a call, against 3 ms of kernels.
// While tables or collections live, blocks therefore come from a pool of the
// library's that keeps up to 1/64 of the device's memory (4.5 GiB of 288; 2^28
// grouped queries take 2.8), and that is emptied when the last of them is freed,
// when an allocation of the library fails and by hg_set_allocator.  Under stream capture, and for a
// stream whose device is unknown, plain hipMallocAsync.
hipError_t ws_alloc(void** p, size_t bytes, hipStream_t s);
// hipMalloc and hipMallocAsync that empty the pools and try again when memory is
// out.
hipError_t dev_malloc(void** p, size_t bytes);
hipError_t dev_malloc_async(void** p, size_t bytes, hipStream_t s);
// Held by every table and collection.
struct PoolUser {
    PoolUser();
    ~PoolUser();
    PoolUser(const PoolUser&) = delete;
    PoolUser& operator=(const PoolUser&) = delete;
};

// Temporary device memory of one call, released at scope exit in stream
// order: work already enqueued on s may still be using it.  The block goes
// back to the allocator that gave it, even if another hook was installed
// meanwhile.
struct Workspace {
    void* p = nullptr;
    hipStream_t s;
    WsHook h{};
    explicit Workspace(hipStream_t st) : s(st) {}
    Workspace(const Workspace&) = delete;
    Workspace& operator=(const Workspace&) = delete;
    hipError_t get(size_t bytes) {
        if (p) return hipErrorInvalidValue;  // one block per object
        if (bytes == 0) bytes = 256;
        h = ws_hook();
        if (!h.alloc) return ws_alloc(&p, bytes, s);
        p = h.alloc(bytes, s, h.ctx);
        if (!p) return hipErrorOutOfMemory;
        if ((uintptr_t)p % 256) {  // the carvers and vector loads assume 256-byte blocks
            h.free(p, s, h.ctx);
            p = nullptr;
            return hipErrorInvalidValue;
        }
        return hipSuccess;
    }
    ~Workspace() {
        if (!p) return;
        if (h.alloc)
            h.free(p, s, h.ctx);
        else
            (void)hipFreeAsync(p, s);
    }
};

// A bump allocator over one workspace buffer (sizes first, then pointers).
struct Carver {
    char* base;
    size_t off = 0;
    explicit Carver(void* b) : base((char*)b) {}
    template <typename T>
    T* take(size_t count) {
        off = align_up(off, 256);
        T* p = base ? (T*)(base + off) : nullptr;
        off += count * sizeof(T);
        return p;
    }
};

// ---- partition geometry shared by the V2 kernels --------------------------
// Entries per partition tile.  Long runs per digit save partial lines beyond the
// L2 and large tiles cost LDS, that is waves in flight: 8192 32-bit keys where
// any order needs one set of counters (2^28 keys, first pass: 639 us, in tiles of
// 4096 1150); 4096 64-bit keys, or 32-bit keys ranked stably with counters per
// wave (2^26 keys, first pass: 216 us, in tiles of 8192 255 to 342).
constexpr uint32_t part_tile(size_t key_size, bool any_order) {
    return key_size == 4 && any_order ? 8192u : 4096u;
}
constexpr int kPartThreads = 256;  // of the batched partition
constexpr int kLocalThreads = 512;
// Keys per thread a bin held in LDS may have, and the bin's capacity: 9 for
// 32-bit keys (4608 keys, bins planned at about 4096); 6 for 64-bit keys
// (3072 keys, bins planned at about 2048, so that a bin's LDS leaves room for
// more workgroups per CU).
template <typename Key>
constexpr int light_items() { return sizeof(Key) == 8 ? 6 : 9; }
template <typename Key>
constexpr uint32_t light_cap() { return kLocalThreads * light_items<Key>(); }
constexpr int kHeavyItems = 8;
constexpr uint32_t kHeavyChunk = kLocalThreads * kHeavyItems;  // chunk of an oversize bin
// Bins above slice_keys(n) keys are split over workgroups, slice by slice.  A
// bin below it is one workgroup's serial work, so slices shrink with n until a
// build has about 2048 of them: with 2^17 keys at any n, the largest such bin
// of 2^26 Zipf(1.2) keys ran 860 us alone.  (Builds of up to 2^17 keys split
// nothing.)
inline uint32_t slice_keys(uint64_t n) {
    if (n <= (1u << 17)) return 1u << 17;
    uint32_t k = 1u << 14;
    while (k < (1u << 17) && (uint64_t)k * 2048 < n) k <<= 1;
    return k;
}
// Most split bins of a build of n keys (n / slice_keys(n)), as a bound that
// grows with n (table_ws_bytes); their slices are at most twice as many.
inline uint32_t split_cap(uint64_t n) {
    const uint64_t a = n <= (1u << 17) ? 0 : n >> 14, b = n >> 17;
    return (uint32_t)((a < 2048 ? a : 2048) > b ? (a < 2048 ? a : 2048) : b) + 1;
}
// Device counters of a build, zeroed by its first kernel: oversize bins, split
// bins, their slices, long buckets of the chunked path, their chunks, whether
// a bin held in LDS listed a long bucket (written by the per-bin kernel only: the
// rare path's first kernel reads it while its own workgroups run, and its waves
// have to agree on it, since barriers follow).
enum : uint32_t { kCtrHeavy, kCtrSplit, kCtrSlices, kCtrLong, kCtrChunks, kCtrListed, kCtrWords };
constexpr uint32_t kMaxLocalBits = 12;                          // buckets per bin <= 4096
constexpr uint32_t kMaxDigitBits = 11;                       // partition fan-out <= 2048
constexpr uint32_t kOneTierBits = 9;                         // single partition pass up to 512 bins

// How a V2 build splits the bucket index h (Alg. 2): the low `k` bits pick the
// bucket inside a final bin, the bits above pick the final bin.  The final bin
// index is split into one or two partition digits of b1 (and b2) bits.
struct V2Plan {
    uint32_t k = 0;        // log2 buckets per final bin
    uint32_t bins = 0;     // final bins B2 = ceil(V / 2^k)
    uint32_t tiers = 1;    // partition passes (1 or 2)
    uint32_t b1 = 0, b2 = 0;
    uint64_t n = 0, V = 0;
    uint32_t tile = 0;     // entries per partition tile
    uint32_t ntiles1 = 0, nchunks1 = 0, ch1 = 1;
    uint32_t ntiles2_ub = 0, nchunks2_ub = 0, ch2 = 1;
};

V2Plan plan_v2(uint64_t n, uint64_t V, int key_bits, uint32_t bins_hint, bool any_order);

// Workspace bytes needed by a build.
size_t build_ws_bytes(int variant, uint64_t n, uint64_t V, int key_bits, uint32_t bins_hint);
// The most that any build of up to n_cap keys and V_cap buckets needs (without a
// bins hint).  That is not always the largest build's: fewer keys over the same
// range take wider bins, whose slice histograms are longer, or one partition pass
// of many digits instead of two of few.
size_t table_ws_bytes(uint64_t n_cap, uint64_t V_cap, int key_bits);

// Scan workspace for `n` inputs.
size_t scan_ws_bytes(uint64_t n);

// Exclusive scan of n uint32 counts into n+1 outputs of OutT.  If `copy` is
// not null it also receives the first n outputs (as uint32).
template <typename OutT>
hipError_t scan_excl(const uint32_t* in, uint64_t n, OutT* out, uint32_t* copy, void* ws,
                     hipStream_t s);

hipError_t fill_u32(uint32_t* p, uint64_t n, uint32_t v, hipStream_t s);
// out[ids[p]] = vals[p] for p < n, where ids holds every index of [0, n)
// once; for large n through the V2 partition passes by id and per-bin LDS
// placement (hg_v2.hip).  ws: scatter_perm_ws_bytes(n) bytes.
size_t scatter_perm_ws_bytes(uint64_t n);
hipError_t scatter_perm(const uint32_t* ids, const uint32_t* vals, uint64_t n, uint32_t* out,
                        void* ws, hipStream_t s);
// *out = the longest bucket (max of offsets[b+1] - offsets[b] over b < V).
hipError_t max_bucket_len(const uint32_t* offsets, uint64_t V, uint32_t* out, hipStream_t s);

// Stable LSD radix sort of n (key, value) uint32 pairs by the low `bits` bits
// of the key (hg_sort.hip): ping-pongs between (k0, v0) and (k1, v1); the
// sorted pairs end in (k1, v1) when *in_alt, else in (k0, v0).  ws:
// sort_pairs_ws_bytes(n).
size_t sort_pairs_ws_bytes(uint64_t n);
hipError_t sort_pairs_u32(uint32_t* k0, uint32_t* v0, uint32_t* k1, uint32_t* v1, uint64_t n,
                          uint32_t bits, void* ws, bool* in_alt, hipStream_t s);

// *out = sum of v[0..n) (out outside v).
hipError_t sum_u64(const unsigned long long* v, uint64_t n, unsigned long long* out,
                   hipStream_t s);

// uint64 slots of a probe / intersection total buffer for m queries (or B
// entries): slot 0 receives the total, the others hold per-workgroup sums.
uint64_t probe_total_slots(uint64_t m);

template <typename Key>
hipError_t run_hash(const Key* keys, uint64_t n, uint64_t V, uint64_t seed, uint32_t* out,
                    hipStream_t s);

template <typename Key>
hipError_t run_histogram(const Key* keys, uint64_t n, uint64_t V, uint64_t seed, uint32_t* counts,
                         uint32_t block, bool plain, hipStream_t s);

template <typename Key>
hipError_t run_build_v1(const Key* keys, uint64_t n, uint64_t V, uint64_t seed, uint32_t* offsets,
                        uint32_t* ids, Key* ekeys, void* ws, uint32_t block, bool plain,
                        hipStream_t s);

// ---- probe index -------------------------------------------------------------
// Buckets holding more entries than this get a key-run summary: their distinct
// keys in ascending order, each with its count and the start of its run in a
// key-grouped copy of the bucket's ids.
constexpr uint32_t kRunBucket = 32;

// Index entries of 32-bit keys.  fmix32 is a bijection, so inside bucket
// h = fmix32(k ^ seed) mod V a key is identified by its quotient
// floor(fmix32(k ^ seed) / V), which takes only `qb` bits: 4 at V = 2^28.  An
// entry of 4 or 8 bytes therefore holds every key of all but the longest
// buckets, exactly: its low 4 bits are a code, the fields above it depend on
// the code.
//   0..13   the bucket's length (at most cap); field i (qb bits, from bit 4)
//           is the quotient of its i-th key, unused fields are 0
//   14      a bucket of cap + 1 .. kRunBucket entries: how many of them equal
//           the first one (8 bits), the first one's quotient (qb bits) and an
//           nf-bit filter over the other keys' quotients (filter_bit)
//   15      a bucket of more than kRunBucket entries: bit 4: they all equal
//           the first one; bit 5: it has no key runs (after an erase) and is
//           scanned; then the first one's quotient and how many equal it (0:
//           more than the remaining bits hold)
// Codes 14 and 15 find the bucket through the offsets when the entry does not
// settle a query.
// (With entries of 16 bytes, {len, key0, key1, key2}, the index of 2^28 buckets is 4
// GiB of the build's writes, and windows of the grouped probe twice an XCD's L2.)
// `one` has bit 0 of every field set, `low` all but the top bit of every
// field and `high` the top bits: they compare all fields with a quotient at
// once (held_matches).
struct HeadFmt {
    uint32_t bytes = 0;  // 4 or 8; 16: wide entries, of keys (index_fmt)
    uint32_t qb = 0, cap = 0, nf = 0;
    uint64_t one = 0, low = 0, high = 0;
};
constexpr uint32_t kCodeMedium = 14, kCodeLong = 15, kMaxHeld = 13;

// Quotient entries: four bytes when they hold the buckets that matter: a query that hits sees
// a bucket of 1 + Poisson(n / V) keys, of which a capacity of 2 + 2n/V leaves
// out at most 2% at loads 0.25 to 8; else eight.
inline HeadFmt head_fmt(uint64_t n, uint64_t V, int key_bits) {
    HeadFmt f;
    if (key_bits == 64) {
        f.bytes = 16;
        return f;
    }
    const uint32_t q = (uint32_t)(0xffffffffull / V);
    while (f.qb < 32 && (q >> f.qb)) ++f.qb;
    if (f.qb == 0) f.qb = 1;
    const uint32_t c4 = 28 / f.qb < kMaxHeld ? 28 / f.qb : kMaxHeld;
    f.bytes = (c4 >= 3 && (uint64_t)(c4 - 2) * V >= 2 * n) ? 4 : 8;
    const uint32_t bits = 8 * f.bytes;
    f.cap = (bits - 4) / f.qb < kMaxHeld ? (bits - 4) / f.qb : kMaxHeld;
    f.nf = bits - 12 - f.qb < 32 ? bits - 12 - f.qb : 32;
    for (uint32_t i = 0; i < f.cap; ++i) {
        const uint64_t field = ((1ull << f.qb) - 1) << (i * f.qb);
        f.one |= 1ull << (i * f.qb);
        f.high |= 1ull << (i * f.qb + f.qb - 1);
        f.low |= field;
    }
    f.low &= ~f.high;
    return f;
}

// Wide entries, 16 bytes {len, y, z, w}, in which buckets longer than the entry holds
// are found without the offsets:
//   32-bit keys, len <= 3           y, z, w = the keys (unused: 0)
//   32-bit keys, len <= kRunBucket  y = start, z = the first key, w = how many equal
//                                   it (8 bits) and a 24-bit filter_bit filter of
//                                   the other keys
//   64-bit keys, len <= kRunBucket  y = start, z and w = the key of a bucket of one,
//                                   or the filter of the keys of more (filter_bits64)
//   longer                          y = start, z = key runs (0: none, after an
//                                   erase), w = the key of a single run (32 bits)
constexpr uint32_t kWideKeys = 3;

// The entries of a table: wide ones for 64-bit keys, and for 32-bit keys where eight
// bytes of quotients leave out too many of the buckets that a hit sees (1 + Poisson(n /
// V) keys), whose offsets and edges then come after the entry.  A quotient takes 32
// bits at V = 1, 21 below 2^12 (two a bucket), 16 at 2^16 and 8 at 2^24, and the larger
// the table, the more half the bytes are worth.  2^24 queries in input order, entries
// of 8 : 16 bytes, at the loads on either side of each line: V = 2^10 load 0.5, 67 : 51
// us; 2^14 load 0.5 and 1, 84 : 85 and 99 : 92; 2^17 load 1.5 and 3, 118 : 120 and 167 :
// 157; 2^21 load 5 and 6, 453 : 457 and 510 : 495; 2^24 load 8, 700 : 735 (its build 1981
// : 1644).  Fewer queries, intersections and builds move with them.
inline bool wide_entries(uint64_t n, uint64_t V) {
    if (V < (1u << 12)) return true;
    const uint64_t halves = V <= (1u << 16) ? 1 : V <= (1u << 18) ? 3 : V <= (1u << 22) ? 10 : 16;
    return 2 * n > halves * V;
}
inline HeadFmt index_fmt(uint64_t n, uint64_t V, int key_bits) {
    if (key_bits == 32 && !wide_entries(n, V)) return head_fmt(n, V, key_bits);
    HeadFmt f;
    f.bytes = 16;
    return f;
}

// The most index memory that a build of up to n_cap keys and V_cap buckets needs: with
// n_cap keys entries are wide up to some range, the smaller n the smaller it is.
inline size_t index_bytes(uint64_t n_cap, uint64_t V_cap, int key_bits) {
    if (key_bits == 64) return V_cap * 16;
    uint64_t a = 1, b = V_cap;  // the last wide range of [1, V_cap]
    while (a < b) {
        const uint64_t m = a + (b - a + 1) / 2;
        if (wide_entries(n_cap, m)) a = m;
        else b = m - 1;
    }
    return a * 16 > V_cap * 8 ? a * 16 : V_cap * 8;
}

// Filter bit (of nf) of a quotient.
__host__ __device__ inline uint32_t filter_bit(uint32_t q, uint32_t nf) {
    return (uint32_t)(((uint64_t)(q * 0x9E3779B1u) * nf) >> 32);
}

// Probe index entry of a 32-bit-key bucket of len <= kRunBucket entries whose
// i-th key has the quotient quot(i) (HeadFmt).
template <typename Quot>
__host__ __device__ __forceinline__ uint64_t short_word(const HeadFmt& f, uint32_t len, Quot quot) {
    if (len <= f.cap) {
        uint64_t w = len;
        for (uint32_t i = 0; i < len; ++i) w |= (uint64_t)quot(i) << (4 + i * f.qb);
        return w;
    }
    const uint32_t q0 = quot(0);
    uint32_t c0 = 1, filt = 0;
    for (uint32_t i = 1; i < len; ++i) {
        const uint32_t q = quot(i);
        if (q == q0) ++c0;
        else filt |= 1u << filter_bit(q, f.nf);
    }
    return (uint64_t)kCodeMedium | (uint64_t)c0 << 4 | (uint64_t)q0 << 12 |
           (uint64_t)filt << (12 + f.qb);
}

// Fields of an entry of c <= cap keys that equal the quotient q, as the top
// bits of those fields: all fields at once -- a field of x is zero exactly
// when neither its low part plus all ones carries into its top bit nor that
// bit is set.
template <typename T>
__host__ __device__ __forceinline__ T held_matches(T e, uint32_t c, uint32_t q, const HeadFmt& f) {
    const T x = (e >> 4) ^ ((T)q * (T)f.one);
    const T nonzero = ((x & (T)f.low) + (T)f.low) | x;
    return ~nonzero & (T)f.high & (((T)1 << (c * f.qb)) - 1);
}

template <typename T>
__host__ __device__ __forceinline__ uint32_t popcount(T x) {
    return (uint32_t)(sizeof(T) == 8 ? __builtin_popcountll(x) : __builtin_popcount((uint32_t)x));
}

// held_matches as a mask over the bucket's keys.
template <typename T>
__host__ __device__ __forceinline__ uint32_t held_mask(T m, uint32_t c, const HeadFmt& f) {
    uint32_t mask = 0;
    for (uint32_t i = 0; i < c; ++i)
        mask |= (uint32_t)((m >> (i * f.qb + f.qb - 1)) & 1) << i;
    return mask;
}

// A 64-bit-key bucket of 2..kRunBucket entries keeps a 64-bit filter of all
// its keys in place of the first key: two bits per key, from the top twelve
// bits of a multiplicative hash.  A query with either bit clear matches none
// of the bucket's keys.
__host__ __device__ inline uint64_t filter_bits64(uint64_t k) {
    const uint64_t x = k * 0x9E3779B97F4A7C15ull;
    return (1ull << (x >> 58)) | (1ull << ((x >> 52) & 63u));
}

// Key-run summary of the long buckets (more than kRunBucket entries): three
// arrays parallel to the edge array.  For a long bucket at edge positions
// [st, st + len) holding R distinct keys, run r < R has the key
// run_key[st + r] (ascending in r) and ends at run_end[st + r] (an offset
// from st: runs are cumulative), and kperm[st .. st + len) lists the bucket's
// ids grouped by key in run order, in bucket order inside each group.  A
// bucket of one repeated key (R = 1) writes no kperm: its ids are the edge
// array's own.  Wide entries hold R, and R = 0 marks a long bucket without runs
// (after an erase), which probes scan.  Quotient entries (HeadFmt): run_end[st +
// len - 1] is R for R > 1 (when R = len that is the last run's end, else the place
// is free).
struct RunsDev {
    void* run_key = nullptr;     // Key[n]
    uint32_t* run_end = nullptr; // [n]
    uint32_t* kperm = nullptr;   // [n]
};

// Long buckets a per-bin kernel leaves to the general pass: bin g lists them
// in gen_list[gen_region(start of bin g, g) ...] and stores their number in
// gen_cnt[g].  A bin of L entries has at most L / (kRunBucket + 1) long
// buckets, so the regions of consecutive bins never overlap and the list
// needs n / (kRunBucket + 1) + bins + 1 entries.
__host__ __device__ inline uint32_t gen_region(uint32_t bin_start, uint32_t g) {
    return bin_start / (kRunBucket + 1) + g;
}
inline uint64_t gen_list_cap(uint64_t n, uint64_t bins) { return n / (kRunBucket + 1) + bins + 1; }

// Where a V2 build writes its probe index (head == null: none) and the
// key-run summary of its long buckets.  fmt, hp and the lists are set by the
// build.
struct IndexOut {
    void* head = nullptr;  // fmt.bytes per bucket
    HeadFmt fmt{};
    HashParams hp{};       // 32-bit keys: for the quotients
    RunsDev runs{};
    uint32_t* gen_list = nullptr;
    uint32_t* gen_cnt = nullptr;  // [bins]
    uint32_t* gen_any = nullptr;  // set when a bin held in LDS lists a bucket
};

// The rare path of a build, after its per-bin kernel: bins too large for LDS
// and the long buckets whose key runs the per-bin kernels left (hg_runs.hip).
// Its work lists live on the device, so nothing waits for the host.  ws:
// runs_ws_bytes(n) bytes; rkeys / rids: the build's reorganised entries, free
// afterwards; ctr: kCtrWords counters.
struct RareArgs {
    const uint32_t* bin_start;
    const uint32_t* heavy_list;
    const uint32_t *huge_list, *huge_s0, *slice_owner;
    uint32_t *slice_hist, *range_sum;
    uint32_t* ctr;
    uint32_t huge_cap, slice_cap, slice;
    uint32_t k, bins, V;
    uint32_t any_order;
};
// A table of one bin that fits in LDS (n <= light_cap, V <= 2^k <= 2^12): the
// whole build in one workgroup.  ANY, W: layout and index entry bytes.
// bin_start: 2 words of workspace.
template <typename Key, bool ANY, int W>
hipError_t run_build_one(const Key* keys, uint64_t n, uint32_t k, uint32_t V, uint32_t* offsets,
                         uint32_t* ids, Key* ekeys, typename KeyTraits<Key>::Params hp,
                         const IndexOut& ix, uint32_t* bin_start, Key* rkeys, uint32_t* rids,
                         void* ws, hipStream_t s);
size_t runs_ws_bytes(uint64_t n);
size_t range_sum_words(uint64_t slices);  // words of RareArgs::range_sum
template <typename Key>
hipError_t run_rare(const RareArgs& a, uint32_t* offsets, uint32_t* ids, Key* ekeys, uint64_t n,
                    typename KeyTraits<Key>::Params hp, const IndexOut& ix, Key* rkeys,
                    uint32_t* rids, void* ws, hipStream_t s);

// ix.head (may be null): V probe index entries (index_fmt(n, V, key width)), one
// per bucket, and the key-run summary of long buckets (IndexOut).  stable: ids ascend inside
// every bucket (otherwise their order there is unspecified).
template <typename Key>
hipError_t run_build_v2(const Key* keys, uint64_t n, uint64_t V, uint64_t seed, uint32_t* offsets,
                        uint32_t* ids, Key* ekeys, IndexOut& ix, void* ws,
                        uint32_t bins_hint, bool stable, hipStream_t s);

// ---- probing ---------------------------------------------------------------
struct TableDev {
    const uint32_t* offsets;
    const uint32_t* ids;
    const void* keys;
    uint64_t n, V, seed;
    const void* head = nullptr;   // per-bucket probe index, when the build wrote one
    HeadFmt fmt{};                // its entries
    RunsDev runs{};               // key-run summary of long buckets (with head)
    const uint32_t* len = nullptr;  // live entries per bucket, after an erase (n = slots)
};

// ---- erasing keys ----------------------------------------------------------
// len[h] = offsets[h+1] - offsets[h]
hipError_t init_lengths(const uint32_t* offsets, uint64_t V, uint32_t* len, hipStream_t s);

// Remove every live entry whose key is one of del[0 .. m); dead and touched
// are zeroed byte arrays of t.n and t.V entries (left zeroed); head is the
// table's probe index; *d_removed (device, zeroed) gets the number removed.
template <typename Key>
hipError_t run_erase(const TableDev& t, uint32_t* len, uint8_t* dead, uint8_t* touched,
                     void* head, const Key* del, uint64_t m, unsigned long long* d_removed,
                     hipStream_t s);

// Compacted ids / keys of the live entries at new_off (the exclusive scan of
// len); either output may be null.
template <typename Key>
hipError_t run_export_live(const TableDev& t, const uint32_t* len, const uint32_t* new_off,
                           uint32_t* out_ids, Key* out_keys, hipStream_t s);

size_t probe_ws_bytes(uint64_t m);

// counts (may be null) and/or the total (may be null: else a buffer of
// probe_total_slots(m) uint64, the total lands in slot 0).  held (may be
// null; 32-bit keys with the probe index): per query, 0x8000 | the mask of the
// matching keys when its bucket is held whole in its index entry, else 0 --
// what the pairs pass needs instead of that entry.
// xcd_order: query tiles are dealt out per XCD (xcd_tile), for queries that
// are grouped by bucket range.  gate (device, may be null): when *gate == 0
// the launch probes q_in into counts_in in input order instead.  bytes (may be
// null): the counts as bytes, with counts written only from 255 on (bytes 255);
// not for queries in input order.
template <typename Key>
hipError_t run_probe_counts(const TableDev& t, const Key* queries, uint64_t m, uint32_t* counts,
                            unsigned long long* d_total, hipStream_t s,
                            uint16_t* held = nullptr, bool xcd_order = false,
                            const uint32_t* gate = nullptr, const Key* q_in = nullptr,
                            uint32_t* counts_in = nullptr, uint8_t* bytes = nullptr);

// The same counts (and total) with the queries first grouped by bucket range
// and the counts put back in input order; ws holds
// probe_grouped_ws_bytes(m, t.V, sizeof(Key)) bytes.  decide: a sample of
// the queries taken on the device first picks input order instead when one
// range would hold more than kGroupSkew times its share of them (skewed
// queries read few index lines, which stay cached anyway); the grouping
// passes then find no tiles and the probe launch reads the queries in place.
size_t probe_grouped_ws_bytes(uint64_t m, uint64_t V, size_t key_size);
template <typename Key>
hipError_t run_probe_grouped(const TableDev& t, const Key* queries, uint64_t m, uint32_t* counts,
                             unsigned long long* d_total, void* ws, hipStream_t s,
                             bool decide = false);

// positions[j] = first pair slot of query j (exclusive scan of counts);
// held: the counting pass's per-query codes, or null.
template <typename Key>
hipError_t run_probe_pairs(const TableDev& t, const Key* queries, uint64_t m,
                           const uint64_t* positions, uint32_t* build_ids, uint32_t* probe_ids,
                           hipStream_t s, const uint16_t* held = nullptr);

// Intersection over b's edges: per-edge counts (edge order) and, optionally,
// counts scattered to b's input order.
template <typename Key>
hipError_t run_intersect_counts(const TableDev& a, const TableDev& b, uint32_t* edge_counts,
                                uint32_t* counts_by_input, unsigned long long* d_total,
                                hipStream_t s);

template <typename Key>
hipError_t run_intersect_pairs(const TableDev& a, const TableDev& b, const uint64_t* positions,
                               uint32_t* a_ids, uint32_t* b_ids, hipStream_t s);

// ---- collections: many small tables built once, intersected many times ----

// Device view of a collection (every pointer device memory).
struct CollDev {
    const uint32_t* set_off;  // S + 1 entry offsets of the sets
    const uint64_t* bb;       // S + 2 bucket bases (bb[S] = bb[S+1] = total buckets)
    const uint32_t* offsets;  // total buckets + 1
    const uint32_t* ids;
    const void* keys;
    uint32_t S;
};

// Sizes decided on the device, read back by coll_plan.
struct CollPlan {
    uint64_t *cw, *cb, *cv;  // S + 2 entries each, in the plan workspace
    uint64_t n, buckets, weight, big_keys, big_buckets;
    bool bad;  // set_off not a valid non-decreasing offset array from 0
};

size_t coll_plan_ws_bytes(uint32_t S);
// bb: S + 2 entries, receives the bucket bases; waits for the device.
hipError_t coll_plan(const uint32_t* set_off, uint32_t S, int shift, void* ws, uint64_t* bb,
                     CollPlan* plan, hipStream_t s);
size_t coll_build_ws_bytes(const CollPlan& p, int key_bits);
template <typename Key>
hipError_t run_coll_build(const Key* keys, const uint32_t* set_off, uint32_t S, uint64_t seed,
                          const uint64_t* bb, const CollPlan& p, void* ws, uint32_t* offsets,
                          uint32_t* ids, Key* ekeys, bool* bad, hipStream_t s);
size_t coll_pairs_ws_bytes(uint64_t Q);
// counts (Q entries) and h_total may be null; *bad when a pair index is out of range.
template <typename Key>
hipError_t run_coll_intersect(const CollDev& a, const CollDev& b, uint64_t seed,
                              const uint32_t* pairs, uint64_t Q, unsigned long long* counts,
                              uint64_t* h_total, void* ws, bool* bad, hipStream_t s);

}  // namespace hg
