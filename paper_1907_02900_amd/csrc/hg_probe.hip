// Probing a HashGraph (Sec. 3.4).
//
// HashGraph-Probe-Standard: each query is hashed with Eq. 1, the bucket's
// segment [offsets[h], offsets[h+1]) of the edge array is scanned, and every
// entry with an equal key is counted (all instances, not the first).  When
// the V2 build wrote the per-bucket probe index, one entry of 4, 8 or 16 bytes
// answers most queries instead (HeadFmt, wide_entries), so they cost one
// random read.  Each thread owns several queries (coalesced, strided by the
// block) and issues all their entry or offset loads before using any, to keep
// many random reads in flight.  Pairs are written in a second pass at
// positions given by an exclusive scan of the counts, so pairs are grouped by
// query id.
//
// HashGraph-Probe-New (Alg. 3): both inputs are built into HashGraphs with the
// same hash and V, and bucket x of A is intersected with bucket x of B for
// every x.  B's edges are walked in edge order, so the buckets of A are read
// in increasing order (streaming, cache-friendly) instead of at random.
#include <type_traits>

#include "hg_internal.h"

namespace hg {

namespace {

constexpr int kProbeThreads = 256;
constexpr int kProbeItems = 8;

// Entries of ekeys[lo, hi) equal to q.  Past the first few keys the scan
// reads 16 bytes at a time (aligned), so a medium bucket costs a few wide
// loads instead of one load per key.
template <typename Key>
__device__ __forceinline__ uint32_t count_in_bucket(const Key* __restrict__ ekeys, uint32_t lo,
                                                    uint32_t hi, Key q) {
    constexpr uint32_t V = 16 / sizeof(Key);  // keys per 16-byte load
    uint32_t c = 0;
    uint32_t p = lo;
    if (hi - lo > 2 * V) {
        for (; p % V; ++p) c += (ekeys[p] == q) ? 1u : 0u;
        for (; p + V <= hi; p += V) {
            const uint4 w = *reinterpret_cast<const uint4*>(ekeys + p);
            if constexpr (sizeof(Key) == 4) {
                c += (w.x == q) + (w.y == q) + (w.z == q) + (w.w == q);
            } else {
                c += ((((uint64_t)w.y << 32) | w.x) == q) + ((((uint64_t)w.w << 32) | w.z) == q);
            }
        }
    }
    for (; p < hi; ++p) c += (ekeys[p] == q) ? 1u : 0u;
    return c;
}

// Key-run summary of the long buckets (see hg_runs.hip and RunsDev): runs
// of a bucket starting at edge position st are at [st, st + R) of key / end.
template <typename Key>
struct Runs {
    const Key* key;         // distinct keys, ascending inside each long bucket
    const uint32_t* end;    // end of each run's group (offset from the bucket start)
    const uint32_t* kperm;  // ids grouped by key (buckets of several keys)
};

// A table as the kernels below read it.
template <typename Key>
struct View {
    const uint32_t* off;
    const uint32_t* len;  // live entries per bucket after an erase, else null
    const void* head;     // probe index, or null
    const Key* keys;
    const uint32_t* ids;
    Runs<Key> runs;
    HeadFmt f;
    typename KeyTraits<Key>::Params hp;

    __device__ __forceinline__ uint32_t bucket_end(uint32_t h, uint32_t lo) const {
        return len ? lo + len[h] : off[h + 1];
    }
};

template <typename Key>
View<Key> view_of(const TableDev& t) {
    return View<Key>{t.offsets, t.len, t.head, (const Key*)t.keys, t.ids,
                     Runs<Key>{(const Key*)t.runs.run_key, t.runs.run_end, t.runs.kperm}, t.fmt,
                     KeyTraits<Key>::make(t.V, t.seed)};
}

// The template parameter W of the kernels: bytes of an index entry (4 or 8:
// quotients of 32-bit keys, 16: wide entries), 0 without the index.
template <int W>
struct EntryOf;
template <>
struct EntryOf<0> { using T = uint2; };  // offsets[h], end
template <>
struct EntryOf<4> { using T = uint32_t; };
template <>
struct EntryOf<8> { using T = uint64_t; };
template <>
struct EntryOf<16> { using T = uint4; };

// Run of q among runs [r0, r0 + d) (keys ascending), or ~0u if q is absent.
template <typename Key>
__device__ __forceinline__ uint32_t find_run(const Key* __restrict__ rk, uint32_t r0, uint32_t d,
                                             Key q) {
    uint32_t lo = r0, hi = r0 + d;  // first run with key >= q
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (rk[mid] < q) lo = mid + 1;
        else hi = mid;
    }
    return (lo < r0 + d && rk[lo] == q) ? lo : ~0u;
}

// A long bucket: `runs` key runs (0: none, the bucket is scanned), of which
// one holds its single key.
struct LongRef {
    uint32_t st, end, runs;
};

// Key runs of a long bucket with the entry e, which ends at edge position `end`.
template <int W>
__device__ __forceinline__ uint32_t runs_in(const typename EntryOf<W>::T& e,
                                            const uint32_t* __restrict__ run_end, uint32_t end) {
    if constexpr (W == 16) return e.z;
    else return (e >> 5) & 1 ? 0u : (e >> 4) & 1 ? 1u : run_end[end - 1];
}

template <typename Key, int W>
__device__ __forceinline__ LongRef long_ref(const View<Key>& t, uint32_t h,
                                            const typename EntryOf<W>::T& e) {
    LongRef r;
    if constexpr (W == 16) {
        r.st = e.y;
        r.end = e.y + e.x;
    } else {
        r.st = t.off[h];
        r.end = t.bucket_end(h, r.st);
    }
    r.runs = runs_in<W>(e, t.runs.end, r.end);
    return r;
}

// Group [*gb, *ge) (offsets from the bucket start) of q in a long bucket with
// key runs; false if q is not in it.
template <typename Key>
__device__ __forceinline__ bool run_group(const LongRef& r, const Runs<Key>& runs, Key q,
                                          uint32_t* gb, uint32_t* ge) {
    if (r.runs == 1) {
        *gb = 0;
        *ge = r.end - r.st;
        return runs.key[r.st] == q;
    }
    const uint32_t i = find_run(runs.key, r.st, r.runs, q);
    if (i == ~0u) return false;
    *gb = i > r.st ? runs.end[i - 1] : 0u;
    *ge = runs.end[i];
    return true;
}

template <typename Key>
__device__ __forceinline__ uint32_t count_long(const View<Key>& t, const LongRef& r, Key q) {
    if (r.runs == 0) return count_in_bucket(t.keys, r.st, r.end, q);
    uint32_t gb, ge;
    return run_group(r, t.runs, q, &gb, &ge) ? ge - gb : 0u;
}

// Bucket (and, 32-bit keys, quotient) of a query.
template <typename Key>
__device__ __forceinline__ uint32_t locate(const View<Key>& t, Key q, uint32_t& quot) {
    if constexpr (sizeof(Key) == 4) {
        uint32_t h;
        quot = KeyTraits<uint32_t>::quotient(q, t.hp, h);
        return h;
    } else {
        quot = 0;
        return KeyTraits<Key>::bucket(q, t.hp);
    }
}

// (Without an index the bucket is [offsets[h], offsets[h + 1]): erasing needs the
// index, so such a table has no lengths, and a test for them between the two loads
// cost every query: 2^28 queries of 2^28 buckets 12.34 ms with it, 11.92 without.)
template <typename Key, int W>
__device__ __forceinline__ typename EntryOf<W>::T entry_at(const View<Key>& t, uint32_t h) {
    if constexpr (W == 0) return make_uint2(t.off[h], t.off[h + 1]);
    else return ((const typename EntryOf<W>::T*)t.head)[h];
}

// Matches of q in the bucket whose entry is e, if the entry settles them;
// else kUnsettled (counts stay below 2^32 - 1: so do the entries).
constexpr uint32_t kUnsettled = 0xffffffffu;

template <typename Key, int W>
__device__ __forceinline__ uint32_t count_settled(const View<Key>& t,
                                                  const typename EntryOf<W>::T& e, Key q,
                                                  uint32_t quot) {
    if constexpr (W == 16 && sizeof(Key) == 4) {
        const uint32_t len = e.x;
        if (len <= kWideKeys)
            return (len >= 1 && e.y == q) + (len >= 2 && e.z == q) + (len >= 3 && e.w == q);
        // {len, start, first key, its count | filter of the others}, or {len,
        // start, runs, the key of a single run}
        if (len > kRunBucket) return e.z != 1 ? kUnsettled : e.w == q ? len : 0u;
        if (e.z == q) return e.w & 0xffu;
        return (e.w >> (8 + filter_bit(q, 24))) & 1u ? kUnsettled : 0u;
    } else if constexpr (W == 16) {
        const uint32_t len = e.x;
        const uint64_t f = (uint64_t)e.z | ((uint64_t)e.w << 32);
        if (len <= 1) return len == 1 && f == (uint64_t)q ? 1u : 0u;
        // {len, start, filter of the bucket's keys}: read the bucket only
        // when both of q's filter bits are set
        const uint64_t b = filter_bits64((uint64_t)q);
        return len <= kRunBucket && (f & b) != b ? 0u : kUnsettled;
    } else {
        const uint32_t code = (uint32_t)e & 15u;
        if (code <= kMaxHeld) return popcount(held_matches(e, code, quot, t.f));
        // the first key's matches are counted in the entry; the rest of the
        // bucket is read only when the query is not the first key and (medium)
        // its filter bit is set, (long) there are other keys
        const bool medium = code == kCodeMedium;
        const uint32_t qmask = (uint32_t)((1ull << t.f.qb) - 1);
        const bool lead = ((uint32_t)(e >> (medium ? 12 : 6)) & qmask) == quot;
        const uint32_t n = medium ? (uint32_t)(e >> 4) & 0xffu : (uint32_t)(e >> (6 + t.f.qb));
        if (lead) return n ? n : kUnsettled;  // (0: not held)
        const bool others = medium ? (uint32_t)(e >> (12 + t.f.qb + filter_bit(quot, t.f.nf))) & 1u
                                   : !((uint32_t)(e >> 4) & 1u);
        return others ? kUnsettled : 0u;
    }
}

// The keys of a wide entry of at most kWideKeys 32-bit keys that equal q, as a mask.
__device__ __forceinline__ uint32_t wide_mask(const uint4& e, uint32_t q) {
    return (e.x >= 1 && e.y == q ? 1u : 0u) | (e.x >= 2 && e.z == q ? 2u : 0u) |
           (e.x >= 3 && e.w == q ? 4u : 0u);
}

// Matches of q in bucket h, whose entry e does not settle them.
template <typename Key, int W>
__device__ __forceinline__ uint32_t count_unsettled(const View<Key>& t,
                                                    const typename EntryOf<W>::T& e, Key q,
                                                    uint32_t h) {
    if constexpr (W == 16) {
        if (e.x > kRunBucket) return count_long(t, long_ref<Key, W>(t, h, e), q);
        // (32-bit keys: the first key is settled)
        return count_in_bucket(t.keys, e.y + (sizeof(Key) == 4 ? 1u : 0u), e.y + e.x, q);
    } else {
        if (((uint32_t)e & 15u) == kCodeLong) return count_long(t, long_ref<Key, W>(t, h, e), q);
        const uint32_t lo = t.off[h];
        return count_in_bucket(t.keys, lo + 1, t.bucket_end(h, lo), q);
    }
}

// Probe-Standard counts.  W: each query reads its bucket's index entry (one
// random access when the entry settles it); W = 0: it reads offsets[h],
// offsets[h+1] and scans the edge array.  xcd_tiles = 0: block b
// takes query tile b; else the grid has 8 * ceil(xcd_tiles / 8) blocks and
// tiles are dealt out by xcd_tile, so that each XCD walks one contiguous run
// of queries (queries grouped by bucket range then read one L2-sized window
// of the index per XCD at a time).  gate (may be null): when *gate == 0 the
// launch probes q_in into counts_in instead, block b taking tile b (the
// grouped probe decides on the device whether its queries were grouped).
// bytes (may be null): counts go there as bytes, and to counts only from 255 on.
// held (32-bit keys): per query 0x8000 | the mask of the bucket's keys equal
// to it when it has matches and its entry holds the bucket whole, else 0.
template <typename Key, int W>
__global__ __launch_bounds__(kProbeThreads) void k_probe_count(
    const Key* __restrict__ q, uint64_t m, View<Key> t, uint32_t* __restrict__ counts,
    unsigned long long* __restrict__ total, uint16_t* __restrict__ held, uint32_t xcd_tiles,
    const uint32_t* __restrict__ gate, const Key* __restrict__ q_in,
    uint32_t* __restrict__ counts_in, uint8_t* __restrict__ bytes) {
    __shared__ uint64_t red[kProbeThreads / kWave + 1];
    uint32_t tile = xcd_tiles ? xcd_tile(blockIdx.x, xcd_tiles) : blockIdx.x;
    if (gate && *gate == 0u) {
        q = q_in;
        counts = counts_in;
        bytes = nullptr;
        tile = blockIdx.x;
    }
    const uint64_t base = (uint64_t)tile * (kProbeThreads * kProbeItems) + threadIdx.x;
    Key qq[kProbeItems];
    uint32_t quot[kProbeItems];
    typename EntryOf<W>::T e[kProbeItems];
#pragma unroll
    for (int r = 0; r < kProbeItems; ++r) {
        const uint64_t j = base + (uint64_t)r * kProbeThreads;
        qq[r] = (j < m) ? q[j] : (Key)0;
    }
#pragma unroll
    for (int r = 0; r < kProbeItems; ++r) {
        const uint64_t j = base + (uint64_t)r * kProbeThreads;
        quot[r] = 0;
        e[r] = typename EntryOf<W>::T{};
        if (j < m) e[r] = entry_at<Key, W>(t, locate(t, qq[r], quot[r]));
    }
    uint64_t sum = 0;
#pragma unroll
    for (int r = 0; r < kProbeItems; ++r) {
        const uint64_t j = base + (uint64_t)r * kProbeThreads;
        uint32_t c;
        if constexpr (W == 0) {
            c = count_in_bucket(t.keys, e[r].x, e[r].y, qq[r]);
        } else {
            c = count_settled<Key, W>(t, e[r], qq[r], quot[r]);
            if (c == kUnsettled)  // (not for j >= m: their entry is empty)
                c = count_unsettled<Key, W>(t, e[r], qq[r], KeyTraits<Key>::bucket(qq[r], t.hp));
        }
        if (j < m && counts) {
            if (bytes) bytes[j] = (uint8_t)(c < 255u ? c : 255u);
            if (!bytes || c >= 255u) counts[j] = c;
        }
        if constexpr (W == 4 || W == 8) {
            if (held && j < m) {
                const uint32_t code = (uint32_t)e[r] & 15u;
                held[j] = (uint16_t)(c && code <= kMaxHeld
                                         ? 0x8000u | held_mask(held_matches(e[r], code, quot[r], t.f),
                                                               code, t.f)
                                         : 0u);
            }
        }
        if constexpr (W == 16 && sizeof(Key) == 4) {
            if (held && j < m)
                held[j] = (uint16_t)(c && e[r].x <= kWideKeys ? 0x8000u | wide_mask(e[r], qq[r]) : 0u);
        }
        sum += c;
    }
    if (total) {
        uint64_t all;
        block_excl_scan64<kProbeThreads>(sum, red, &all);
        if (threadIdx.x == 0) total[1 + blockIdx.x] = all;  // reduced by sum_u64
    }
}

// Writes a query's pairs: its output range [positions[j], positions[j+1]) is
// known from the counting pass, and a query whose range is empty reads
// nothing more.  Each thread first loads what its kProbeItems queries need --
// with the counting pass's codes (held) only the bucket's start -- so that
// their random reads overlap.
template <typename Key, int W>
__global__ __launch_bounds__(kProbeThreads) void k_probe_pairs(
    const Key* __restrict__ q, uint64_t m, View<Key> t, const uint64_t* __restrict__ positions,
    uint32_t* __restrict__ build_ids, uint32_t* __restrict__ probe_ids,
    const uint16_t* __restrict__ held) {
    const uint64_t base = (uint64_t)blockIdx.x * (kProbeThreads * kProbeItems) + threadIdx.x;
    Key qq[kProbeItems];
    uint32_t hh[kProbeItems], st[kProbeItems];
    typename EntryOf<W>::T e[kProbeItems];
    uint64_t pos[kProbeItems], pend[kProbeItems];
    uint32_t mask[kProbeItems];  // the bucket's matching keys, when known from its entry
#pragma unroll
    for (int r = 0; r < kProbeItems; ++r) {
        const uint64_t j = base + (uint64_t)r * kProbeThreads;
        qq[r] = (j < m) ? q[j] : (Key)0;
        pos[r] = (j < m) ? positions[j] : 0ull;
        pend[r] = (j < m) ? positions[j + 1] : 0ull;
        mask[r] = (W && held && j < m) ? held[j] & 0x7fffu : 0u;
    }
#pragma unroll
    for (int r = 0; r < kProbeItems; ++r) {
        uint32_t quot;
        hh[r] = locate(t, qq[r], quot);
        e[r] = typename EntryOf<W>::T{};
        st[r] = 0;
        if (pos[r] == pend[r]) continue;
        if (!mask[r]) e[r] = entry_at<Key, W>(t, hh[r]);
        if (W && sizeof(Key) == 4) st[r] = t.off[hh[r]];
    }
#pragma unroll
    for (int r = 0; r < kProbeItems; ++r) {
        if (pos[r] == pend[r]) continue;
        const uint32_t j = (uint32_t)(base + (uint64_t)r * kProbeThreads);
        const Key k = qq[r];
        uint64_t o = pos[r];
        uint32_t lo = st[r], hi = lo, mk = mask[r];
        if constexpr (W == 0) {
            lo = e[r].x;
            hi = e[r].y;
        } else {
            bool longb;
            if constexpr (W == 16) {
                longb = e[r].x > kRunBucket;
                if constexpr (sizeof(Key) == 4) {
                    if (!mk && e[r].x <= kWideKeys) mk = wide_mask(e[r], k);
                    if (!mk) hi = lo + e[r].x;
                } else {
                    lo = e[r].y;
                    hi = lo + e[r].x;
                }
            } else {
                const uint32_t code = (uint32_t)e[r] & 15u;
                if (!mk && code <= kMaxHeld) {
                    uint32_t quot;
                    locate(t, k, quot);
                    mk = held_mask(held_matches(e[r], code, quot, t.f), code, t.f);
                }
                longb = !mk && code == kCodeLong;
                if (!mk) hi = t.bucket_end(hh[r], lo);
            }
            if (longb) {
                const LongRef ref = long_ref<Key, W>(t, hh[r], e[r]);
                if (ref.runs) {
                    // the ids of q's group, in bucket order: the edge array's own
                    // for a bucket of one key, else its group in kperm
                    uint32_t gb, ge;
                    if (run_group(ref, t.runs, k, &gb, &ge)) {
                        const uint32_t* src = (ref.runs == 1 ? t.ids : t.runs.kperm) + ref.st;
                        for (uint32_t x = gb; x < ge && o < pend[r]; ++x, ++o) {
                            build_ids[o] = src[x];
                            probe_ids[o] = j;
                        }
                    }
                    continue;
                }
            }
        }
        for (; mk && o < pend[r]; mk &= mk - 1, ++o) {
            build_ids[o] = t.ids[lo + __builtin_ctz(mk)];
            probe_ids[o] = j;
        }
        for (uint32_t p = lo; p < hi && o < pend[r]; ++p)
            if (t.keys[p] == k) {
                build_ids[o] = t.ids[p];
                probe_ids[o] = j;
                ++o;
            }
    }
}

// Whether slot p of B, holding key k, is stale (behind its bucket's live
// entries after an erase): such slots get edge count 0 and no count by input.
template <typename Key>
__device__ __forceinline__ bool stale(const View<Key>& b, uint64_t p, Key k) {
    if (!b.len) return false;
    const uint32_t h = KeyTraits<Key>::bucket(k, b.hp);
    return p - b.off[h] >= b.len[h];
}

// Alg. 3 over B's edges p: count the entries of A's bucket h(key_p) equal to
// key_p.  A and B share hash parameters, so h is recomputed from B's key.
//
// With A's quotient entries (W = 4 or 8) or without its index (W = 0).  A's buckets come in
// increasing order, so its index entries are streamed: they are smaller than its
// offsets and keys together.  A thread's counts are stored after the last of its
// loads, since a load waits for the stores before it: 2^23 edges by 2^20 to 2^24
// buckets without the index 27 to 66 us, now 25 to 63 (64-bit keys 34 to 79, now 31 to
// 76).
template <typename Key, int W>
__global__ __launch_bounds__(kProbeThreads) void k_intersect_count(
    View<Key> a, View<Key> b, uint64_t nb, uint32_t* __restrict__ edge_counts,
    uint32_t* __restrict__ counts_by_input, unsigned long long* __restrict__ total) {
    __shared__ uint64_t red[kProbeThreads / kWave + 1];
    uint64_t sum = 0;
    const uint64_t base = (uint64_t)blockIdx.x * (kProbeThreads * kProbeItems) + threadIdx.x;
    Key kk[kProbeItems];
    uint32_t quot[kProbeItems], c[kProbeItems];
    typename EntryOf<W>::T e[kProbeItems];
#pragma unroll
    for (int r = 0; r < kProbeItems; ++r) {
        const uint64_t p = base + (uint64_t)r * kProbeThreads;
        kk[r] = p < nb ? b.keys[p] : (Key)0;
    }
#pragma unroll
    for (int r = 0; r < kProbeItems; ++r) {
        const uint64_t p = base + (uint64_t)r * kProbeThreads;
        quot[r] = 0;
        e[r] = typename EntryOf<W>::T{};
        if (p < nb) e[r] = entry_at<Key, W>(a, locate(a, kk[r], quot[r]));
    }
    uint32_t gone = 0;  // stale slots of B, as bits
#pragma unroll
    for (int r = 0; r < kProbeItems; ++r) {
        const uint64_t p = base + (uint64_t)r * kProbeThreads;
        c[r] = 0;
        if (p >= nb) continue;
        if (stale(b, p, kk[r])) {
            gone |= 1u << r;
        } else if constexpr (W == 0) {
            c[r] = count_in_bucket(a.keys, e[r].x, e[r].y, kk[r]);
        } else {
            c[r] = count_settled<Key, W>(a, e[r], kk[r], quot[r]);
            if (c[r] == kUnsettled)
                c[r] = count_unsettled<Key, W>(a, e[r], kk[r], KeyTraits<Key>::bucket(kk[r], a.hp));
        }
        sum += c[r];
    }
    if (edge_counts) {
#pragma unroll
        for (int r = 0; r < kProbeItems; ++r) {
            const uint64_t p = base + (uint64_t)r * kProbeThreads;
            if (p < nb) edge_counts[p] = c[r];
        }
    }
    if (counts_by_input) {
#pragma unroll
        for (int r = 0; r < kProbeItems; ++r) {
            const uint64_t p = base + (uint64_t)r * kProbeThreads;
            if (p < nb && !(gone >> r & 1u)) counts_by_input[b.ids[p]] = c[r];
        }
    }
    if (total) {
        uint64_t all;
        block_excl_scan64<kProbeThreads>(sum, red, &all);
        if (threadIdx.x == 0) total[1 + blockIdx.x] = all;  // reduced by sum_u64
    }
}

// Matches of k in A's bucket h, by its offsets: a scan, or A's key runs when the
// bucket is long and has them.
template <typename Key, int W>
__device__ __forceinline__ uint32_t count_by_offsets(const uint32_t* __restrict__ a_off,
                                                     const uint32_t* __restrict__ a_len,
                                                     const void* __restrict__ a_head,
                                                     const Runs<Key>& runs,
                                                     const Key* __restrict__ a_keys, uint32_t h,
                                                     Key k) {
    const uint32_t lo = a_off[h], hi = a_len ? lo + a_len[h] : a_off[h + 1];
    if (hi - lo > kRunBucket) {
        const auto e = ((const typename EntryOf<W>::T*)a_head)[h];
        const uint32_t n = runs_in<W>(e, runs.end, hi);
        uint32_t gb, ge;
        if (n != 0) return run_group(LongRef{lo, hi, n}, runs, k, &gb, &ge) ? ge - gb : 0u;
    }
    return count_in_bucket(a_keys, lo, hi, k);
}

// With an index of wide entries, which would cost more to stream than the two
// offsets, or of quotients that settle too few edges (scan_offsets): the entries are
// read for long buckets only.  One edge after the other, each
// loaded and counted before the next: as a batch like the above, with the branch for
// long buckets in it, 2^23 64-bit edges by 2^20 to 2^24 buckets of load 0.25 to 4 took
// 37 to 93 us, so 30 to 79.
template <typename Key, int W>
__global__ __launch_bounds__(kProbeThreads) void k_intersect_scan(
    const uint32_t* __restrict__ a_off, const uint32_t* __restrict__ a_len,
    const void* __restrict__ a_head, Runs<Key> runs, const Key* __restrict__ a_keys,
    const uint32_t* __restrict__ b_off, const uint32_t* __restrict__ b_len,
    const Key* __restrict__ b_keys, const uint32_t* __restrict__ b_ids, uint64_t nb,
    typename KeyTraits<Key>::Params hp, uint32_t* __restrict__ edge_counts,
    uint32_t* __restrict__ counts_by_input, unsigned long long* __restrict__ total) {
    __shared__ uint64_t red[kProbeThreads / kWave + 1];
    uint64_t sum = 0;
    const uint64_t base = (uint64_t)blockIdx.x * (kProbeThreads * kProbeItems) + threadIdx.x;
#pragma unroll
    for (int r = 0; r < kProbeItems; ++r) {
        const uint64_t p = base + (uint64_t)r * kProbeThreads;
        if (p < nb) {
            const Key k = b_keys[p];
            const uint32_t h = KeyTraits<Key>::bucket(k, hp);
            if (b_len && p - b_off[h] >= b_len[h]) {
                if (edge_counts) edge_counts[p] = 0;
                continue;
            }
            const uint32_t c = count_by_offsets<Key, W>(a_off, a_len, a_head, runs, a_keys, h, k);
            if (edge_counts) edge_counts[p] = c;
            if (counts_by_input) counts_by_input[b_ids[p]] = c;
            sum += c;
        }
    }
    if (total) {
        uint64_t all;
        block_excl_scan64<kProbeThreads>(sum, red, &all);
        if (threadIdx.x == 0) total[1 + blockIdx.x] = all;  // reduced by sum_u64
    }
}

template <typename Key, int W>
__global__ __launch_bounds__(kProbeThreads) void k_intersect_pairs(
    View<Key> a, View<Key> b, uint64_t nb, const uint64_t* __restrict__ positions,
    uint32_t* __restrict__ out_a, uint32_t* __restrict__ out_b) {
    uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t st = (uint64_t)gridDim.x * blockDim.x;
    for (; p < nb; p += st) {
        // an edge whose output range is empty (no match, or a stale slot of
        // B, whose count is 0) reads nothing more
        uint64_t pos = positions[p];
        const uint64_t pend = positions[p + 1];
        if (pos == pend) continue;
        const Key k = b.keys[p];
        const uint32_t h = KeyTraits<Key>::bucket(k, a.hp);
        const uint32_t lo = a.off[h], hi = a.bucket_end(h, lo);
        const uint32_t bid = b.ids[p];
        if constexpr (W != 0) {
            if (hi - lo > kRunBucket) {
                const LongRef ref = long_ref<Key, W>(a, h, entry_at<Key, W>(a, h));
                if (ref.runs != 0) {
                    uint32_t gb, ge;
                    if (run_group(ref, a.runs, k, &gb, &ge)) {
                        const uint32_t* src = (ref.runs == 1 ? a.ids : a.runs.kperm) + ref.st;
                        for (uint32_t x = gb; x < ge && pos < pend; ++x) {
                            out_a[pos] = src[x];
                            out_b[pos] = bid;
                            ++pos;
                        }
                    }
                    continue;
                }
            }
        }
        for (uint32_t i = lo; i < hi && pos < pend; ++i)
            if (a.keys[i] == k) {
                out_a[pos] = a.ids[i];
                out_b[pos] = bid;
                ++pos;
            }
    }
}

uint32_t grid_for(uint64_t items, uint32_t per_block) {
    uint64_t g = ceil_div(items, per_block);
    return (uint32_t)(g ? g : 1);
}

}  // namespace

size_t probe_ws_bytes(uint64_t m) {
    // counts (m uint32), positions (m+1 uint64), scan workspace
    return align_up(m * 4, 256) + align_up((m + 1) * 8, 256) + scan_ws_bytes(m) + 512;
}

uint64_t probe_total_slots(uint64_t m) {
    // one per block, the grid rounded up to whole XCD rounds (xcd_order)
    return 1 + (m ? 8 * (((uint64_t)grid_for(m, kProbeThreads * kProbeItems) + 7) / 8) : 0);
}

// Whether A's 8-byte entries are streamed, or its offsets scanned: past some load the
// entries leave too many keys of B to the edge array, whose bucket then takes the
// offsets as well.  Entries : offsets, at the lines: 2^18 and 2^19 buckets of load 1.5
// 11 : 10 us, of load 1 9 : 9; 2^21 and 2^22 of load 4 by 2^22 edges 54 : 36 and 59 : 41,
// of load 3 by half a table 23 : 24 and 31 : 32; 2^24 of load 4 by 2^24 edges 200 : 209.
// (A few edges of B leave most of A's lines unread: 2^22 buckets of load 4 by 2^18 edges
// 24 : 31.)
bool scan_offsets(const TableDev& a, const TableDev& b) {
    if (a.V <= (1u << 19)) return 2 * a.n >= 3 * a.V;
    return a.V <= (1u << 23) && a.n >= 4 * a.V && 4 * b.n >= a.V;
}

// Calls f with the bytes of t's index entries (0: no index) as a constant.
template <typename Key, typename F>
void with_entry(const TableDev& t, F&& f) {
    if (!t.head) f(std::integral_constant<int, 0>{});
    else if constexpr (sizeof(Key) == 8) f(std::integral_constant<int, 16>{});
    else if (t.fmt.bytes == 4) f(std::integral_constant<int, 4>{});
    else if (t.fmt.bytes == 8) f(std::integral_constant<int, 8>{});
    else f(std::integral_constant<int, 16>{});
}

template <typename Key>
hipError_t run_probe_counts(const TableDev& t, const Key* queries, uint64_t m, uint32_t* counts,
                            unsigned long long* d_total, hipStream_t s, uint16_t* held,
                            bool xcd_order, const uint32_t* gate, const Key* q_in,
                            uint32_t* counts_in, uint8_t* bytes) {
    if (m == 0) return d_total ? fill_u32((uint32_t*)d_total, 2, 0u, s) : hipSuccess;
    const uint32_t tiles = grid_for(m, kProbeThreads * kProbeItems);
    const uint32_t xt = xcd_order ? tiles : 0u;
    const dim3 grid(xcd_order ? 8 * ((tiles + 7) / 8) : tiles);
    {
        HG_PROF("probe_count", s);
        with_entry<Key>(t, [&](auto w) {
            hipLaunchKernelGGL((k_probe_count<Key, decltype(w)::value>), grid,
                               dim3(kProbeThreads), 0, s, queries, m, view_of<Key>(t), counts,
                               d_total, held, xt, gate, q_in, counts_in, bytes);
        });
    }
    HG_TRY(hipGetLastError());
    return d_total ? sum_u64(d_total + 1, grid.x, d_total, s) : hipSuccess;
}

template <typename Key>
hipError_t run_probe_pairs(const TableDev& t, const Key* queries, uint64_t m,
                           const uint64_t* positions, uint32_t* build_ids, uint32_t* probe_ids,
                           hipStream_t s, const uint16_t* held) {
    if (m == 0) return hipSuccess;
    const uint32_t g = grid_for(m, kProbeThreads * kProbeItems);
    {
        HG_PROF("probe_pairs", s);
        with_entry<Key>(t, [&](auto w) {
            hipLaunchKernelGGL((k_probe_pairs<Key, decltype(w)::value>), dim3(g),
                               dim3(kProbeThreads), 0, s, queries, m, view_of<Key>(t), positions,
                               build_ids, probe_ids, held);
        });
    }
    return hipGetLastError();
}

template <typename Key>
hipError_t run_intersect_counts(const TableDev& a, const TableDev& b, uint32_t* edge_counts,
                                uint32_t* counts_by_input, unsigned long long* d_total,
                                hipStream_t s) {
    if (b.n == 0) return d_total ? fill_u32((uint32_t*)d_total, 2, 0u, s) : hipSuccess;
    const uint32_t grid = grid_for(b.n, kProbeThreads * kProbeItems);
    {
        HG_PROF("intersect_count", s);
        with_entry<Key>(a, [&](auto w) {
            constexpr int W = decltype(w)::value;
            bool by_entry = W != 16;
            if constexpr (W == 8) by_entry = !scan_offsets(a, b);
            if constexpr (W != 16)
                if (by_entry)
                    hipLaunchKernelGGL((k_intersect_count<Key, W>), dim3(grid),
                                       dim3(kProbeThreads), 0, s, view_of<Key>(a), view_of<Key>(b),
                                       b.n, edge_counts, counts_by_input, d_total);
            if constexpr (W == 8 || W == 16)
                if (!by_entry)
                    hipLaunchKernelGGL((k_intersect_scan<Key, W>), dim3(grid), dim3(kProbeThreads),
                                       0, s, a.offsets, a.len, a.head, view_of<Key>(a).runs,
                                       (const Key*)a.keys, b.offsets, b.len, (const Key*)b.keys,
                                       b.ids, b.n, KeyTraits<Key>::make(a.V, a.seed), edge_counts,
                                       counts_by_input, d_total);
        });
    }
    HG_TRY(hipGetLastError());
    return d_total ? sum_u64(d_total + 1, grid, d_total, s) : hipSuccess;
}

template <typename Key>
hipError_t run_intersect_pairs(const TableDev& a, const TableDev& b, const uint64_t* positions,
                               uint32_t* a_ids, uint32_t* b_ids, hipStream_t s) {
    if (b.n == 0) return hipSuccess;
    uint32_t g = grid_for(b.n, kProbeThreads);
    if (g > 8192) g = 8192;
    {
        HG_PROF("intersect_pairs", s);
        with_entry<Key>(a, [&](auto w) {
            hipLaunchKernelGGL((k_intersect_pairs<Key, decltype(w)::value>), dim3(g),
                               dim3(kProbeThreads), 0, s, view_of<Key>(a), view_of<Key>(b), b.n,
                               positions, a_ids, b_ids);
        });
    }
    return hipGetLastError();
}

#define HG_PINST(Key)                                                                           \
    template hipError_t run_probe_counts<Key>(const TableDev&, const Key*, uint64_t, uint32_t*, \
                                              unsigned long long*, hipStream_t, uint16_t*, bool, \
                                              const uint32_t*, const Key*, uint32_t*, uint8_t*); \
    template hipError_t run_probe_pairs<Key>(const TableDev&, const Key*, uint64_t,             \
                                             const uint64_t*, uint32_t*, uint32_t*,             \
                                             hipStream_t, const uint16_t*);                     \
    template hipError_t run_intersect_counts<Key>(const TableDev&, const TableDev&, uint32_t*,  \
                                                  uint32_t*, unsigned long long*, hipStream_t); \
    template hipError_t run_intersect_pairs<Key>(const TableDev&, const TableDev&,              \
                                                 const uint64_t*, uint32_t*, uint32_t*,         \
                                                 hipStream_t);
HG_PINST(uint32_t)
HG_PINST(uint64_t)

}  // namespace hg
