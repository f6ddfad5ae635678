// Device code shared by the single-table V2 build (hg_v2.hip) and the batched
// build (hg_batch.hip): stable ranking of a tile by a digit, in-LDS sorting of
// a bin by bucket, and the per-bin build bodies.
#pragma once

#include "hg_internal.h"

namespace hg {
namespace v2dev {

constexpr int W_PART = kPartThreads / kWave;
constexpr int W_LOCAL = kLocalThreads / kWave;
constexpr uint32_t kFixMax = 16;  // longest bucket whose ids are ranked by counting

// ------------------------------------------------------------ ranking -----

// Digit-major exclusive scan of the per-wave digit counters wcnt[w][d]
// (W waves, D digits): afterwards wcnt[w][d] holds the position of wave w's
// first item of digit d in the stably sorted tile, and dstart[d] the start
// of digit d.  Barrier on exit.
template <int THREADS>
__device__ __forceinline__ void scan_wave_digit_counts(uint32_t D, uint32_t* wcnt,
                                                       uint32_t* dstart, uint32_t* tmp) {
    constexpr int W = THREADS / kWave;
    const uint32_t per = (D + THREADS - 1) / THREADS;
    const uint32_t d0 = threadIdx.x * per;
    uint32_t mine = 0;
    for (uint32_t j = 0; j < per; ++j) {
        const uint32_t d = d0 + j;
        if (d < D)
#pragma unroll
            for (int w = 0; w < W; ++w) mine += wcnt[w * D + d];
    }
    uint32_t all;
    uint32_t run = block_excl_scan<THREADS>(mine, tmp, &all);
    for (uint32_t j = 0; j < per; ++j) {
        const uint32_t d = d0 + j;
        if (d < D) {
            dstart[d] = run;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const uint32_t v = wcnt[w * D + d];
                wcnt[w * D + d] = run;
                run += v;
            }
        }
    }
    __syncthreads();
}

// Stable rank of up to 64*ITEMS items per wave by a digit of `bits` bits
// (D = 2^bits <= 2048).  Item r of a lane is entry (wave base + r*64 + lane);
// items with dig >= D are ignored.  Per round every lane reads its digit's
// running count in the wave's counter row and the lowest lane of each group
// of equal digits adds the group's size with a non-returning LDS atomic.  LDS
// performs a wave's operations in issue order, so a read sees exactly the
// items of the wave's earlier rounds, and no round waits for the previous
// one.  Every round runs unconditionally (a round without valid items costs
// its ballots and changes nothing), which keeps the code straight-line.  On
// return pos[r] is the item's index in the tile sorted stably by digit
// (undefined for ignored items).  Contains barriers.
template <int THREADS, int ITEMS>
__device__ __forceinline__ void rank_stable(const uint32_t (&dig)[ITEMS], uint32_t bits,
                                            uint32_t* wcnt, uint32_t* dstart, uint32_t* tmp,
                                            uint32_t (&pos)[ITEMS]) {
    constexpr int W = THREADS / kWave;
    const uint32_t D = 1u << bits, mask = D - 1;
    const uint32_t w = threadIdx.x / kWave;
    for (uint32_t i = threadIdx.x; i < W * D; i += THREADS) wcnt[i] = 0;
    __syncthreads();
    uint32_t* my = wcnt + w * D;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t d = dig[r];
        const bool valid = d < D;
        const uint64_t peers = match_digit(d, (int)bits, ballot(valid));
        const uint32_t below = mbcnt(peers);
        pos[r] = my[d & mask] + below;
        if (valid && below == 0)
            __hip_atomic_fetch_add(&my[d], (uint32_t)__popcll(peers), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __syncthreads();
    scan_wave_digit_counts<THREADS>(D, wcnt, dstart, tmp);
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) pos[r] += my[dig[r] & mask];
}

// Rank of up to THREADS*ITEMS items by a digit of `bits` bits with no order
// among equal digits: one returning LDS atomic per item on per-workgroup
// counters, then an exclusive scan of the counts.  pos[r] is the item's index
// in the tile grouped by digit (undefined for items with dig >= D);
// dstart[d] the start of digit d.  `cnt` holds D counters.  Contains
// barriers.
template <int THREADS, int ITEMS>
__device__ __forceinline__ void rank_any(const uint32_t (&dig)[ITEMS], uint32_t bits,
                                         uint32_t* cnt, uint32_t* dstart, uint32_t* tmp,
                                         uint32_t (&pos)[ITEMS]) {
    const uint32_t D = 1u << bits, mask = D - 1;
    for (uint32_t i = threadIdx.x; i < D; i += THREADS) cnt[i] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r)
        if (dig[r] < D) pos[r] = atomicAdd(&cnt[dig[r]], 1u);
    __syncthreads();
    const uint32_t per = (D + THREADS - 1) / THREADS;
    const uint32_t d0 = threadIdx.x * per;
    uint32_t mine = 0;
    for (uint32_t j = 0; j < per; ++j)
        if (d0 + j < D) mine += cnt[d0 + j];
    uint32_t all;
    uint32_t run = block_excl_scan<THREADS>(mine, tmp, &all);
    for (uint32_t j = 0; j < per; ++j)
        if (d0 + j < D) {
            dstart[d0 + j] = run;
            run += cnt[d0 + j];
        }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) pos[r] += dstart[dig[r] & mask];
}

// Exclusive scan of a matrix of counts in (column, row) order, in place: rows [c0,
// c1), D columns, starting at `start`; dbase[d] receives column d's start, and
// with_starts() runs once they are there.  part: [2 * THREADS], dbase: [D], tmp:
// [THREADS / 64 + 1], in LDS.  One workgroup against memory latency: up to 16 row
// groups walk the rows side by side with eight loads in flight each.  Barriers.
template <int THREADS, typename F>
__device__ __forceinline__ void scan_columns(uint32_t* __restrict__ mat, uint32_t c0, uint32_t c1,
                                             uint32_t D, uint32_t start, uint32_t* part,
                                             uint32_t* dbase, uint32_t* tmp, F&& with_starts) {
    static_assert((1u << kMaxDigitBits) <= 2 * THREADS, "at most two digits per thread");
    const uint32_t per = D > (uint32_t)THREADS ? 2u : 1u;
    uint32_t G = (uint32_t)THREADS / D;  // row groups (D is a power of two)
    G = G > 16 ? 16 : (G ? G : 1);
    const uint32_t d0 = per == 2 ? threadIdx.x * 2 : threadIdx.x & (D - 1);
    const uint32_t grp = per == 2 ? 0u : threadIdx.x / D;
    const uint32_t len = (c1 - c0 + G - 1) / G;
    const uint32_t ra = grp < G && c0 + grp * len < c1 ? c0 + grp * len : c1;
    const uint32_t rb = c1 - ra > len ? ra + len : c1;
    for (uint32_t j = 0; j < per; ++j) {
        uint32_t acc = 0;
        for (uint32_t c = ra; c < rb; c += 8) {
            uint32_t v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = c + u < rb ? mat[(size_t)(c + u) * D + d0 + j] : 0u;
#pragma unroll
            for (int u = 0; u < 8; ++u) acc += v[u];
        }
        if (grp < G) part[grp * D + d0 + j] = acc;
    }
    __syncthreads();
    uint32_t tot[2] = {0, 0};
    if (grp == 0)
        for (uint32_t j = 0; j < per; ++j)
            for (uint32_t x = 0; x < G; ++x) tot[j] += part[x * D + d0 + j];
    uint32_t all;
    const uint32_t ex = start + block_excl_scan<THREADS>(tot[0] + tot[1], tmp, &all);
    if (grp == 0) {
        dbase[d0] = ex;
        if (per == 2) dbase[d0 + 1] = ex + tot[0];
    }
    __syncthreads();
    with_starts();
    for (uint32_t j = 0; j < per; ++j) {
        if (ra >= rb) break;
        uint32_t r = dbase[d0 + j];
        for (uint32_t x = 0; x < grp; ++x) r += part[x * D + d0 + j];
        for (uint32_t c = ra; c < rb; c += 8) {
            uint32_t v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = c + u < rb ? mat[(size_t)(c + u) * D + d0 + j] : 0u;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (c + u < rb) mat[(size_t)(c + u) * D + d0 + j] = r;
                r += v[u];
            }
        }
    }
}

// -------------------------------------------------- per-bin LDS build -----

// Place one chunk of <= ITEMS*64*W entries held in registers: two stable LSD
// ranking passes over the local bucket index (lo bits, then hi bits) leave
// the chunk sorted by bucket in skeys/sids/sb.  Items are balanced over the
// waves: wave w owns entries [w*chunk, (w+1)*chunk).
template <typename Key, int ITEMS>
__device__ __forceinline__ void sort_chunk_by_bucket(Key (&kk)[ITEMS], uint32_t (&id)[ITEMS],
                                                     uint32_t (&b)[ITEMS], uint32_t rounds,
                                                     uint32_t cl, uint32_t wchunk, uint32_t k,
                                                     Key* skeys, uint32_t* sids, uint16_t* sb,
                                                     uint32_t* wcnt, uint32_t* dstart,
                                                     uint32_t* tmp) {
    const uint32_t NB = 1u << k;
    const uint32_t lo_bits = (k + 1) / 2, hi_bits = k / 2;
    const uint32_t w = threadIdx.x / kWave, lane = lane_id();
    uint32_t dig[ITEMS], pos[ITEMS];
    if (k == 0) {
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            const uint32_t e = w * wchunk + r * kWave + lane;
            if ((uint32_t)r < rounds && r * kWave + lane < wchunk && e < cl) {
                skeys[e] = kk[r];
                sids[e] = id[r];
                sb[e] = 0;
            }
        }
        return;
    }
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) dig[r] = (b[r] < NB) ? (b[r] & ((1u << lo_bits) - 1)) : 64u;
    rank_stable<kLocalThreads, ITEMS>(dig, lo_bits, wcnt, dstart, tmp, pos);
#pragma unroll
    for (int r = 0; r < ITEMS; ++r)
        if ((uint32_t)r < rounds && b[r] < NB) {
            skeys[pos[r]] = kk[r];
            sids[pos[r]] = id[r];
            sb[pos[r]] = (uint16_t)b[r];
        }
    __syncthreads();
    if (hi_bits == 0) return;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t e = w * wchunk + r * kWave + lane;
        if ((uint32_t)r < rounds && r * kWave + lane < wchunk && e < cl) {
            kk[r] = skeys[e];
            id[r] = sids[e];
            b[r] = sb[e];
            dig[r] = b[r] >> lo_bits;
        } else {
            b[r] = NB;
            dig[r] = 64u;
        }
    }
    // rank_stable synchronises before counting, so every wave has finished
    // reading the buffers before any wave overwrites them below
    rank_stable<kLocalThreads, ITEMS>(dig, hi_bits, wcnt, dstart, tmp, pos);
#pragma unroll
    for (int r = 0; r < ITEMS; ++r)
        if ((uint32_t)r < rounds && b[r] < NB) {
            skeys[pos[r]] = kk[r];
            sids[pos[r]] = id[r];
            sb[pos[r]] = (uint16_t)b[r];
        }
}

// Exclusive scan of cnt[0..NB) in place (NB a power of two); returns via
// cnt; *total gets the sum.  All threads must call it.
__device__ __forceinline__ void scan_counts(uint32_t* cnt, uint32_t NB, uint32_t base,
                                            uint32_t* tmp) {
    const uint32_t per = NB >= (uint32_t)kLocalThreads ? NB / kLocalThreads : 1u;
    const uint32_t i0 = threadIdx.x * per;
    uint32_t v[16];
    uint32_t mine = 0;
    for (uint32_t j = 0; j < per; ++j) {
        v[j] = (i0 + j < NB) ? cnt[i0 + j] : 0u;
        mine += v[j];
    }
    uint32_t all;
    uint32_t run = base + block_excl_scan<kLocalThreads>(mine, tmp, &all);
    for (uint32_t j = 0; j < per; ++j)
        if (i0 + j < NB) {
            cnt[i0 + j] = run;
            run += v[j];
        }
    __syncthreads();
}

// Exclusive scan of cnt[0..NB) in place (base 0); returns the largest count.
// `tmp` needs 2 * (waves per block) words.  All threads must call it.
__device__ __forceinline__ uint32_t scan_counts_max(uint32_t* cnt, uint32_t NB, uint32_t* tmp) {
    const uint32_t per = NB >= (uint32_t)kLocalThreads ? NB / kLocalThreads : 1u;
    const uint32_t i0 = threadIdx.x * per;
    uint32_t v[16];
    uint32_t mine = 0, mx = 0;
    for (uint32_t j = 0; j < per; ++j) {
        v[j] = (i0 + j < NB) ? cnt[i0 + j] : 0u;
        mine += v[j];
        mx = v[j] > mx ? v[j] : mx;
    }
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1) {
        const uint32_t o = __shfl_xor(mx, d, kWave);
        mx = o > mx ? o : mx;
    }
    uint32_t all;
    uint32_t run = block_excl_scan<kLocalThreads>(mine, tmp, &all);
    if (lane_id() == 0) tmp[W_LOCAL + threadIdx.x / kWave] = mx;
    for (uint32_t j = 0; j < per; ++j)
        if (i0 + j < NB) {
            cnt[i0 + j] = run;
            run += v[j];
        }
    __syncthreads();
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < W_LOCAL; ++i) m = tmp[W_LOCAL + i] > m ? tmp[W_LOCAL + i] : m;
    __syncthreads();
    return m;
}

// LDS bytes of light_bin_body / heavy_bin_body for 2^k buckets per bin.
template <typename Key>
__host__ __device__ inline size_t light_smem(uint32_t k) {
    const size_t NB = 1u << k;
    return light_cap<Key>() * (sizeof(Key) + 4 + 2) + NB * 4 + W_LOCAL * 64 * 4 + 64 * 4 +
           (2 * W_LOCAL + 2) * 4 + 64;
}

template <typename Key>
inline size_t heavy_smem(uint32_t k) {
    const size_t NB = 1u << k;
    return kHeavyChunk * (sizeof(Key) + 4 + 2) + 2 * NB * 4 + W_LOCAL * 64 * 4 + 64 * 4 +
           (2 * W_LOCAL + 2) * 4 + 64;
}

__device__ __forceinline__ void store_word(const IndexOut& ix, uint32_t bucket, uint64_t w) {
    if (ix.fmt.bytes == 4) ((uint32_t*)ix.head)[bucket] = (uint32_t)w;
    else ((uint64_t*)ix.head)[bucket] = w;
}

// Wide entry of a bucket (wide_entries); one longer than kRunBucket later gets its
// key-run summary in z and w.  `k` points at the bucket's first key.
__device__ __forceinline__ uint4 wide_entry(uint32_t start, uint32_t end, const uint32_t* k) {
    const uint32_t len = end - start;
    if (len <= kWideKeys)
        return make_uint4(len, len >= 1 ? k[0] : 0u, len >= 2 ? k[1] : 0u, len >= 3 ? k[2] : 0u);
    const uint32_t k0 = k[0];
    uint32_t c0 = 0, filt = 0;
    if (len <= kRunBucket) {
        c0 = 1;
        // four keys per round, so that their loads overlap
#pragma unroll 1
        for (uint32_t i = 1; i < len; i += 4) {
            uint32_t kv[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) kv[j] = i + j < len ? k[i + j] : k0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (i + j >= len) continue;
                if (kv[j] == k0) ++c0;
                else filt |= 1u << filter_bit(kv[j], 24);
            }
        }
    }
    return make_uint4(len, start, k0, c0 | filt << 8);
}

__device__ __forceinline__ uint4 wide_entry(uint32_t start, uint32_t end, const uint64_t* k) {
    const uint32_t len = end - start;
    uint64_t z = len == 1 ? k[0] : 0ull;
    if (len >= 2 && len <= kRunBucket) {
#pragma unroll 1
        for (uint32_t i = 0; i < len; i += 4) {
            uint64_t kv[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) kv[j] = i + j < len ? k[i + j] : k[0];
#pragma unroll
            for (int j = 0; j < 4; ++j) z |= filter_bits64(kv[j]);
        }
    }
    return make_uint4(len, start, (uint32_t)z, (uint32_t)(z >> 32));
}

// Whether a table's entries are wide; W: their bytes where the caller knows them,
// else 0.
template <typename Key, int W>
__device__ __forceinline__ bool is_wide(const IndexOut& ix) {
    return sizeof(Key) == 8 || (W ? W == 16 : ix.fmt.bytes == 16);
}

// Writes the index entry of a bucket of at most kRunBucket entries, edge
// positions [start, end), whose first key is at k (LDS or global).
template <typename Key, int W = 0>
__device__ __forceinline__ void put_short(const IndexOut& ix, uint32_t bucket, uint32_t start,
                                          uint32_t end, const Key* k) {
    if (is_wide<Key, W>(ix)) {
        ((uint4*)ix.head)[bucket] = wide_entry(start, end, k);
    } else if constexpr (sizeof(Key) == 4) {
        store_word(ix, bucket, short_word(ix.fmt, end - start, [&](uint32_t i) {
                       uint32_t h;
                       return KeyTraits<uint32_t>::quotient(k[i], ix.hp, h);
                   }));
    }
}

// Writes the index entry of a long bucket of R key runs (R = 0: none), whose
// first key `lead` clead entries equal, and (quotient entries) R itself behind the
// runs.
template <typename Key, int W = 0>
__device__ __forceinline__ void put_long(const IndexOut& ix, uint32_t bucket, uint32_t len,
                                         uint32_t start, uint32_t R, Key lead, uint32_t clead) {
    if (is_wide<Key, W>(ix)) {
        ((uint4*)ix.head)[bucket] =
            make_uint4(len, start, R, sizeof(Key) == 4 && R == 1 ? (uint32_t)lead : 0u);
    } else if constexpr (sizeof(Key) == 4) {
        uint32_t h;
        const uint32_t room = 8 * ix.fmt.bytes - 6 - ix.fmt.qb;  // at least 17 bits
        uint64_t w = (uint64_t)KeyTraits<uint32_t>::quotient(lead, ix.hp, h) << 6 |
                     (R == 0 ? 32u : R == 1 ? 16u : 0u) | kCodeLong;
        if (R && (room >= 32 || clead >> room == 0)) w |= (uint64_t)clead << (6 + ix.fmt.qb);
        store_word(ix, bucket, w);
        if (R > 1) ix.runs.run_end[start + len - 1] = R;
    }
}

// LDS of the per-bin key runs (after light_smem's layout, 16-byte aligned):
// the bin's long buckets (their range in the bin and bucket id), two counters
// and one 64-entry buffer per wave for the keys that differ from a bucket's
// first key.
template <typename Key>
struct LongLds {
    static constexpr uint32_t cap = light_cap<Key>() / (kRunBucket + 1) + 1;
    uint32_t* cnt;   // [0] long buckets of the bin, [1] of them left to the general pass
    uint32_t* lohi;  // [cap] lo | hi << 16: the bucket's range in the bin
    uint32_t* bkt;   // [cap] bucket id
    Key* wkey;       // [W_LOCAL * 64]
    uint16_t* wpos;  // [W_LOCAL * 64]
    __host__ __device__ static constexpr size_t bytes() {
        return 16 + 8 * cap + (sizeof(Key) + 2) * W_LOCAL * kWave + 32;
    }
    __device__ explicit LongLds(unsigned char* p) {
        cnt = (uint32_t*)p;
        lohi = cnt + 4;
        bkt = lohi + cap;
        wkey = (Key*)(((uintptr_t)(bkt + cap) + 15) & ~(uintptr_t)15);
        wpos = (uint16_t*)(wkey + W_LOCAL * kWave);
    }
};

__host__ __device__ inline size_t align16(size_t x) { return (x + 15) & ~(size_t)15; }

// Most medium buckets a bin can list (lengths above head_lane_max).
template <typename Key>
__host__ __device__ constexpr uint32_t medium_cap() {
    return light_cap<Key>() / (sizeof(Key) == 4 ? 9 : 17) + 1;
}

// LDS bytes of a light bin that also builds its index entries and key runs:
// beside light_smem, the long buckets and, where the bucket sort's scratch
// was, the medium buckets and (32-bit keys) one entry word per bucket.  At 2^12
// buckets 77.6 KB: two workgroups per CU.
template <typename Key>
__host__ __device__ inline size_t light_smem_index(uint32_t k) {
    const size_t scratch = light_cap<Key>() * 2;
    const size_t words = 4 * medium_cap<Key>() + (sizeof(Key) == 4 ? (size_t)4 << k : 0);
    return align16(light_smem<Key>(k) - scratch) + LongLds<Key>::bytes() + 16 +
           (words > scratch ? words : scratch) + 16;
}

// Sort the 64 lanes' (key, position) pairs ascending (bitonic network over
// lane shuffles; positions are distinct, so the order is total).
template <typename Key>
__device__ __forceinline__ void wave_sort_pairs(Key& k, uint32_t& p) {
    const uint32_t lane = lane_id();
#pragma unroll
    for (uint32_t size = 2; size <= (uint32_t)kWave; size <<= 1) {
#pragma unroll
        for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
            const Key ok = __shfl_xor(k, (int)stride, kWave);
            const uint32_t op = __shfl_xor(p, (int)stride, kWave);
            const bool up = (lane & size) == 0;
            const bool lower = (lane & stride) == 0;
            const bool other_less = ok < k || (ok == k && op < p);
            if ((lower == up) ? other_less : !other_less) {
                k = ok;
                p = op;
            }
        }
    }
}

// Buckets whose index entry one lane builds key by key (quotient entries: those
// past the entry's capacity, whose keys it hashes again).  Longer ones up
// to kRunBucket entries -- common only when keys repeat many times -- are
// listed and built by groups of 32 lanes (bin_medium_heads) instead of one
// lane walking them.
template <int W>
__host__ __device__ constexpr uint32_t head_lane_max() { return W == 16 ? 16u : 8u; }

// Lists a bucket whose index entry is not one lane's work: the long buckets
// (more than kRunBucket entries; their entries are written with their key
// runs) and the medium ones (their entries are written by lane groups), med[]
// packing lo | len << 13 | v << 19 (v = local bucket).  False: neither.
template <typename Key, int W>
__device__ __forceinline__ bool list_bucket(const LongLds<Key>& lr, uint32_t* med, uint32_t v0,
                                            uint32_t v, uint32_t lo, uint32_t hi) {
    const uint32_t len = hi - lo;
    if (len > kRunBucket) {
        const uint32_t t = atomicAdd(&lr.cnt[0], 1u);
        lr.lohi[t] = lo | (hi << 16);
        lr.bkt[t] = v0 + v;
        return true;
    }
    if (len > head_lane_max<W>()) {
        med[atomicAdd(&lr.cnt[2], 1u)] = lo | (len << 13) | (v << 19);
        return true;
    }
    return false;
}

// OR over each row of 16 lanes, left in the row's last lane (lanes 15, 31,
// 47, 63): four DPP row shifts (a lane shifted in from outside the row reads
// 0).  Whole wave.
__device__ __forceinline__ uint32_t row_or16(uint32_t f) {
    f |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)f, 0x111, 0xf, 0xf, false);  // row_shr:1
    f |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)f, 0x112, 0xf, 0xf, false);  // row_shr:2
    f |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)f, 0x114, 0xf, 0xf, false);  // row_shr:4
    f |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)f, 0x118, 0xf, 0xf, false);  // row_shr:8
    return f;
}

// The OR of half g's 32 lanes, from the rows' ORs; uniform values, selected per
// lane.
__device__ __forceinline__ uint32_t half_or(uint32_t f, uint32_t g) {
    const uint32_t r = row_or16(f);
    const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)r, 15);
    const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)r, 31);
    const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)r, 47);
    const uint32_t d = (uint32_t)__builtin_amdgcn_readlane((int)r, 63);
    return g == 0 ? (a | b) : (c | d);
}

// Index entries of the bin's medium buckets (more than head_lane_max and at
// most kRunBucket entries): each wave takes two buckets at a time, lane s of half g
// holding key s of its bucket; the first key's count is a ballot and the filter an
// OR over the half -- the same entry put_short builds with one lane.  Called by
// whole waves after a barrier that follows the list's construction.
template <typename Key, int W>
__device__ __forceinline__ void bin_medium_heads(const IndexOut& ix, const LongLds<Key>& lr,
                                                 const uint32_t* list, const Key* skeys,
                                                 uint32_t out, uint32_t v0) {
    constexpr uint32_t G = 32, PER = kWave / G;
    static_assert(kRunBucket <= G, "a medium bucket fits a half wave");
    const uint32_t n = lr.cnt[2];
    const uint32_t w = threadIdx.x / kWave, lane = lane_id();
    const uint32_t g = lane / G, s = lane % G;
    for (uint32_t j0 = w * PER; j0 < n; j0 += W_LOCAL * PER) {  // uniform per wave
        const uint32_t j = j0 + g;
        const bool have = j < n;
        const uint32_t e = have ? list[j] : 0u;
        const uint32_t lo = e & 0x1fffu, len = (e >> 13) & 0x3fu, v = e >> 19;
        const bool in = have && s < len;
        const Key k0 = skeys[lo];
        const Key kx = in ? skeys[lo + s] : k0;
        if constexpr (sizeof(Key) == 4) {
            // (listed buckets are longer than an entry's capacity)
            const uint64_t eq = ballot(in && kx == k0);
            const uint32_t c0 = (uint32_t)__popcll((eq >> (g * G)) & ((1ull << G) - 1ull));
            uint32_t h, q = kx;
            if (W != 16) q = KeyTraits<uint32_t>::quotient(kx, ix.hp, h);
            const uint32_t nf = W == 16 ? 24u : ix.fmt.nf;
            const uint32_t f =
                half_or((in && kx != k0) ? (1u << filter_bit(q, nf)) : 0u, g);
            if (have && s == 0 && W == 16)
                ((uint4*)ix.head)[v0 + v] = make_uint4(len, out + lo, (uint32_t)k0, c0 | f << 8);
            if (have && s == 0 && W != 16)  // lane 0's key is the first one
                store_word(ix, v0 + v,
                           (uint64_t)kCodeMedium | (uint64_t)c0 << 4 | (uint64_t)q << 12 |
                               (uint64_t)f << (12 + ix.fmt.qb));
        } else {
            const uint64_t z = in ? filter_bits64((uint64_t)kx) : 0ull;
            const uint32_t zl = half_or((uint32_t)z, g), zh = half_or((uint32_t)(z >> 32), g);
            if (have && s == 0) ((uint4*)ix.head)[v0 + v] = make_uint4(len, out + lo, zl, zh);
        }
    }
}

// Key runs and index entry of one long bucket, by one wave: its entries are
// keys[lo, hi) with ids ids_[lo, hi) (in LDS or in global memory), its first
// edge is at st, its bucket id b.  The entries equal to the bucket's first
// key (the lead key) form one run; the others, when there are at most 64, are
// sorted across the wave's lanes and cut into runs, and the lead run is
// slotted in among them.  bk / bp: the wave's 64-entry LDS buffers.  Returns
// false, having written nothing, when more than 64 entries differ from the
// lead key (uniform across the wave).
template <typename Key, int W = 0>
__device__ __forceinline__ bool wave_bucket_runs(const IndexOut& ix, const Key* keys,
                                                 const uint32_t* ids_, uint32_t lo, uint32_t hi,
                                                 uint32_t st, uint32_t b, Key* bk, uint16_t* bp) {
    const uint32_t lane = lane_id();
    Key* rkey = (Key*)ix.runs.run_key;
    uint32_t* rend = ix.runs.run_end;
    uint32_t* kperm = ix.runs.kperm;
    const uint32_t len = hi - lo;
    const Key lead = keys[lo];
    uint32_t no = 0;  // entries whose key differs from the lead key
    for (uint32_t c = lo; c < hi; c += kWave) {
        const uint32_t p = c + lane;
        const Key x = p < hi ? keys[p] : lead;
        const bool o = x != lead;
        const uint64_t bal = ballot(o);
        const uint32_t slot = no + mbcnt(bal);
        if (o && slot < (uint32_t)kWave) {
            bk[slot] = x;
            bp[slot] = (uint16_t)(p - lo);
        }
        no += (uint32_t)__popcll(bal);
        if (no > (uint32_t)kWave) return false;  // too many others: stop reading
    }
    if (no == 0) {  // one key: its ids are the edge array's own
        if (lane == 0) {
            rkey[st] = lead;
            rend[st] = len;
            put_long<Key, W>(ix, b, len, st, 1u, lead, len);
        }
        return true;
    }
    // the buffer written above is read by other lanes of the same wave:
    // LDS executes a wave's operations in order; keep the compiler's too
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const bool valid = lane < no;
    Key k = valid ? bk[lane] : (Key)~(Key)0;
    uint32_t p = valid ? (uint32_t)bp[lane] : 0xffffffffu;
    wave_sort_pairs<Key>(k, p);
    const Key kprev = __shfl_up(k, 1, kWave);
    const Key knext = __shfl_down(k, 1, kWave);
    const bool first = valid && (lane == 0 || kprev != k);
    const bool last = valid && (lane + 1 == no || knext != k);
    const bool below = valid && k < lead;
    const uint64_t fb = ballot(first), lb = ballot(below);
    const uint32_t nless = (uint32_t)__popcll(lb);       // others below the lead key
    const uint32_t rl = (uint32_t)__popcll(fb & lb);     // runs below the lead key
    const uint32_t clead = len - no;
    const uint32_t r = mbcnt(fb) + (first ? 1u : 0u) - 1u + (below ? 0u : 1u);
    if (valid) kperm[st + lane + (below ? 0u : clead)] = ids_[lo + p];
    if (first) rkey[st + r] = k;
    if (last) rend[st + r] = lane + 1 + (below ? 0u : clead);
    if (lane == 0) {
        rkey[st + rl] = lead;
        rend[st + rl] = nless + clead;
        put_long<Key, W>(ix, b, len, st, (uint32_t)__popcll(fb) + 1u, lead, clead);
    }
    // the lead key's ids, in bucket order, after the smaller keys' runs
    uint32_t done = 0;
    for (uint32_t c = lo; c < hi; c += kWave) {
        const uint32_t q = c + lane;
        const bool isl = q < hi && keys[q] == lead;
        const uint64_t bal = ballot(isl);
        if (isl) kperm[st + nless + done + mbcnt(bal)] = ids_[q];
        done += (uint32_t)__popcll(bal);
    }
    return true;
}

// Key runs of the long buckets of a bin held in LDS (skeys / sids in bucket
// order, the bin's first edge at `out`), one wave per bucket.  The entries
// equal to the bucket's first key (the lead key) form one run; the others,
// when there are at most 64, are sorted across the wave's lanes and cut into
// runs, and the lead run is slotted in among them.  A bucket with more other
// keys is listed for the general pass.  Whole workgroup; barriers.
template <typename Key, int W>
__device__ __forceinline__ void bin_long_runs(const IndexOut& ix, const LongLds<Key>& lr,
                                              const uint32_t* med, const Key* skeys,
                                              const uint32_t* sids, uint32_t out, uint32_t g,
                                              uint32_t v0) {
    __syncthreads();
    bin_medium_heads<Key, W>(ix, lr, med, skeys, out, v0);
    const uint32_t nl = lr.cnt[0];
    const uint32_t w = threadIdx.x / kWave, lane = lane_id();
    Key* bk = lr.wkey + w * kWave;
    uint16_t* bp = lr.wpos + w * kWave;
    for (uint32_t j = w; j < nl; j += W_LOCAL) {
        const uint32_t lh = lr.lohi[j], lo = lh & 0xffffu, hi = lh >> 16;
        const uint32_t b = lr.bkt[j];
        if (!wave_bucket_runs<Key, W>(ix, skeys, sids, lo, hi, out + lo, b, bk, bp) && lane == 0)
            ix.gen_list[gen_region(out, g) + atomicAdd(&lr.cnt[1], 1u)] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        ix.gen_cnt[g] = lr.cnt[1];
        if (lr.cnt[1]) *ix.gen_any = 1u;
    }
}

// Index entries of a bin's buckets (32-bit keys).  Entry words are put together
// key by key, not bucket by bucket: each ORs its quotient into its bucket's
// word in LDS (`or_part(f, high)`: the lower or upper 32 bits of every key),
// one atomic a key and no divergence, then each thread adds the code and
// stores the word.  A lane walking its bucket's keys would run as long as the
// longest bucket of its wave, about five rounds at load 1.  Entries of eight
// bytes take a second round for their upper halves, so that the words need 4
// bytes of LDS per bucket either way.  words[] is zero on entry; cnt[v] = start
// of bucket v in the bin, cnt[NB] = its end.  Whole workgroup; barriers.
template <int W, typename OrPart>
__device__ __forceinline__ void words_of_bin(OrPart or_part, uint32_t* words, const uint32_t* skeys,
                                             uint32_t out, uint32_t v0, uint32_t nb,
                                             const uint32_t* cnt, uint32_t* __restrict__ offsets,
                                             const IndexOut& ix, const LongLds<uint32_t>& lr,
                                             uint32_t* med) {
    constexpr uint32_t PER = (1u << kMaxLocalBits) / kLocalThreads;
    const HeadFmt& f = ix.fmt;
    or_part(words, false);
    __syncthreads();
    uint32_t lo32[PER];
    if constexpr (W == 8) {
#pragma unroll
        for (uint32_t j = 0; j < PER; ++j) {
            const uint32_t v = threadIdx.x + j * kLocalThreads;
            if (v < nb) {
                lo32[j] = words[v];
                words[v] = 0;
            }
        }
        __syncthreads();
        or_part(words, true);
        __syncthreads();
    }
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j) {
        const uint32_t v = threadIdx.x + j * kLocalThreads;
        if (v >= nb) continue;
        const uint32_t lo = cnt[v], hi = cnt[v + 1], len = hi - lo;
        offsets[v0 + v] = out + lo;
        if (len <= f.cap) {
            if constexpr (W == 8)
                ((uint64_t*)ix.head)[v0 + v] = (uint64_t)words[v] << 32 | lo32[j] | len;
            else
                ((uint32_t*)ix.head)[v0 + v] = words[v] | len;
        } else if (!list_bucket<uint32_t, W>(lr, med, v0, v, lo, hi)) {
            put_short<uint32_t, W>(ix, v0 + v, out + lo, out + hi, skeys + lo);
        }
    }
}

// The part (lower or upper 32 bits) of an entry that the i-th key of its
// bucket, with quotient q, fills.
__device__ __forceinline__ void or_field(uint32_t* word, const HeadFmt& f, uint32_t i, uint32_t q,
                                         bool high) {
    const uint32_t sh = 4 + i * f.qb;
    if (i >= f.cap) return;
    if (!high) {
        if (sh < 32) atomicOr(word, q << sh);
    } else if (sh + f.qb > 32) {
        atomicOr(word, sh < 32 ? q >> (32 - sh) : q << (sh - 32));
    }
}

// Build one bin of L <= light_cap<Key>() keys whose buckets are [v0, v0 + nb) with
// nb <= 2^k.  Entry e (e < L) of the bin is src_keys[e], with id src_ids[e]
// (or id_base + e when src_ids is null).  The bin's keys and ids go to
// ekeys/ids[out + p] for p < L, sorted by bucket with ids ascending inside a
// bucket, and offsets[v0 + v] = out + (start of bucket v in the bin).
// Usual case (every bucket of the bin holds at most kFixMax keys, or any order
// is allowed): an LDS counting sort -- the counting atomic returns each key's
// arrival rank in its bucket, so that placing it takes no second one -- and, in
// the stable layout, its rank by id counted over the bucket.  Otherwise the bin (in id order) is stably ranked by local
// bucket.
// With W > 0, ix.head also receives each bucket's probe index entry.
// `bucket_of(key, e, q)` gives the local bucket (< nb) of entry e and, where an
// index is written, sets q to its quotient (32-bit keys).
// Called by a whole workgroup of kLocalThreads threads.
// ANY: any order inside a bucket; W: bytes of an index entry (0: no index).
template <typename Key, bool ANY, int W, typename BucketOf>
__device__ __forceinline__ void light_bin_body_by(const Key* __restrict__ src_keys,
                                                  const uint32_t* __restrict__ src_ids,
                                                  uint32_t id_base, uint32_t L, uint32_t out,
                                                  uint32_t v0, uint32_t k, uint32_t nb,
                                                  BucketOf bucket_of,
                                                  uint32_t* __restrict__ offsets,
                                                  const IndexOut& ix, uint32_t* __restrict__ ids,
                                                  Key* __restrict__ ekeys, unsigned char* smem) {
    constexpr int IT = light_items<Key>();
    constexpr uint32_t kLightCap = light_cap<Key>();
    const uint32_t NB = 1u << k;
    Key* skeys = (Key*)smem;
    uint32_t* sids = (uint32_t*)(skeys + kLightCap);
    uint32_t* cnt = sids + kLightCap;              // NB + 1 (in light_smem's padding)
    uint32_t* wcnt = cnt + NB + 1;                 // W * 64
    uint32_t* dstart = wcnt + W_LOCAL * 64;        // 64
    uint32_t* tmp = dstart + 64;                   // 2 * W + 2
    // the bin's long buckets, when the probe index is written, then the
    // bucket sort's scratch, whose place the lists of medium buckets and the
    // entry words take (stable layout: afterwards)
    const size_t front = align16(light_smem<Key>(k) - 2 * kLightCap);
    const LongLds<Key> lr(smem + front);
    uint16_t* sb = W ? (uint16_t*)(smem + align16(front + LongLds<Key>::bytes()))
                     : (uint16_t*)(tmp + 2 * W_LOCAL + 2);
    static_assert(kLightCap <= 8192u, "a medium-list entry holds lo in 13 bits");
    uint32_t* med = (uint32_t*)sb;
    uint32_t* words = med + medium_cap<Key>();
    constexpr bool by_key = W == 4 || W == 8;  // entry words put together key by key
    const uint32_t w = threadIdx.x / kWave, lane = lane_id();
    // balance the bin over the waves in whole rounds of 64
    const uint32_t wchunk = (((L + W_LOCAL - 1) / W_LOCAL) + kWave - 1) & ~(uint32_t)(kWave - 1);
    const uint32_t wb = w * wchunk;
    const uint32_t mylen = L > wb ? ((L - wb < wchunk) ? L - wb : wchunk) : 0u;
    const uint32_t rounds = (mylen + kWave - 1) / kWave;

    Key kk[IT];
    // br: the local bucket, and above it the rank in the bucket
    uint32_t id[IT], br[IT], qt[IT];
    constexpr uint32_t kNone = ~0u, kBktMask = (1u << (kMaxLocalBits + 1)) - 1;
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const uint32_t e = wb + r * kWave + lane;
        if ((uint32_t)r < rounds && r * kWave + lane < mylen) {
            kk[r] = src_keys[e];
            id[r] = src_ids ? src_ids[e] : id_base + e;
        } else {
            kk[r] = 0;
            id[r] = 0;
        }
    }
    for (uint32_t i = threadIdx.x; i < NB; i += kLocalThreads) cnt[i] = 0;
    if (by_key)
        for (uint32_t i = threadIdx.x; i < NB; i += kLocalThreads) words[i] = 0;
    if (W && threadIdx.x < 3) lr.cnt[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        br[r] = kNone;
        qt[r] = 0;
        if ((uint32_t)r < rounds && r * kWave + lane < mylen) {
            const uint32_t b = bucket_of(kk[r], wb + r * kWave + lane, qt[r]);
            br[r] = b | atomicAdd(&cnt[b], 1u) << (kMaxLocalBits + 1);
        }
    }
    __syncthreads();
    // bucket starts (in place) and the largest bucket of the bin
    const uint32_t maxc = scan_counts_max(cnt, NB, tmp);
    if (threadIdx.x == 0) cnt[NB] = L;
    // whether br holds every key's place in its bucket
    const bool ranked = ANY || maxc <= kFixMax;
    if (ranked) {
        if constexpr (!ANY) {
            // a key's place in its bucket is the number of the bucket's ids
            // below its own, counted by every key over the ids placed in the
            // order of arrival.  (One lane per bucket sorting it in registers
            // took 122 VGPRs and a list of the buckets to sort.)
#pragma unroll
            for (int r = 0; r < IT; ++r)
                if (br[r] != kNone)
                    sids[cnt[br[r] & kBktMask] + (br[r] >> (kMaxLocalBits + 1))] = id[r];
            __syncthreads();
#pragma unroll
            for (int r = 0; r < IT; ++r) {
                if (br[r] == kNone) continue;
                const uint32_t v = br[r] & kBktMask;
                const uint32_t lo = cnt[v], hi = cnt[v + 1];
                uint32_t below = 0;
                if (hi - lo > 1)
                    for (uint32_t i = lo; i < hi; ++i) below += sids[i] < id[r] ? 1u : 0u;
                br[r] = v | below << (kMaxLocalBits + 1);
            }
            __syncthreads();
        }
#pragma unroll
        for (int r = 0; r < IT; ++r) {
            if (br[r] != kNone) {
                const uint32_t slot = cnt[br[r] & kBktMask] + (br[r] >> (kMaxLocalBits + 1));
                skeys[slot] = kk[r];
                sids[slot] = id[r];
            }
        }
        __syncthreads();
    } else {
        if constexpr (!ANY) {
            uint32_t b[IT];
#pragma unroll
            for (int r = 0; r < IT; ++r) {
                b[r] = br[r] == kNone ? NB : br[r] & kBktMask;
                br[r] = kNone;  // (not kept in registers over the sort)
                qt[r] = 0;
            }
            sort_chunk_by_bucket<Key, IT>(kk, id, b, rounds, L, wchunk, k, skeys, sids, sb, wcnt,
                                          dstart, tmp);
            __syncthreads();
        }
    }
    if constexpr (by_key) {
        if (!ranked) {  // the words' place held the bucket sort's scratch
            for (uint32_t i = threadIdx.x; i < NB; i += kLocalThreads) words[i] = 0;
            __syncthreads();
        }
        words_of_bin<W>(
            [&](uint32_t* wd, bool high) {
                if (ranked) {  // from registers
#pragma unroll
                    for (int r = 0; r < IT; ++r)
                        if (br[r] != kNone)
                            or_field(&wd[br[r] & kBktMask], ix.fmt, br[r] >> (kMaxLocalBits + 1),
                                     qt[r], high);
                } else if constexpr (!ANY) {  // from the sorted bin
                    for (uint32_t p = threadIdx.x; p < L; p += kLocalThreads) {
                        uint32_t q;
                        const uint32_t v = bucket_of(skeys[p], p, q);
                        or_field(&wd[v], ix.fmt, p - cnt[v], q, high);
                    }
                }
            },
            words, skeys, out, v0, nb, cnt, offsets, ix, lr, med);
    } else {
        for (uint32_t v = threadIdx.x; v < nb; v += kLocalThreads) {
            const uint32_t lo = cnt[v], hi = cnt[v + 1];
            offsets[v0 + v] = out + lo;
            if (W && !list_bucket<Key, W>(lr, med, v0, v, lo, hi))
                put_short<Key, W>(ix, v0 + v, out + lo, out + hi, skeys + lo);
        }
    }
    for (uint32_t p = threadIdx.x; p < L; p += kLocalThreads) {
        ekeys[out + p] = skeys[p];
        ids[out + p] = sids[p];
    }
    if constexpr (W != 0) bin_long_runs<Key, W>(ix, lr, med, skeys, sids, out, v0 >> k, v0);
}

// The usual bin: buckets [v0, v0 + nb) of the table's hash function.
template <typename Key, bool ANY, int W>
__device__ __forceinline__ void light_bin_body(const Key* __restrict__ src_keys,
                                               const uint32_t* __restrict__ src_ids,
                                               uint32_t id_base, uint32_t L, uint32_t out,
                                               uint32_t v0, uint32_t k, uint32_t nb,
                                               const typename KeyTraits<Key>::Params& hp,
                                               uint32_t* __restrict__ offsets,
                                               const IndexOut& ix,
                                               uint32_t* __restrict__ ids, Key* __restrict__ ekeys,
                                               unsigned char* smem) {
    light_bin_body_by<Key, ANY, W>(
        src_keys, src_ids, id_base, L, out, v0, k, nb,
        [&](Key key, uint32_t, uint32_t& q) {
            if constexpr (sizeof(Key) == 4) {
                uint32_t h;
                q = KeyTraits<Key>::quotient(key, hp, h);
                return h - v0;
            } else {
                return KeyTraits<Key>::bucket(key, hp) - v0;
            }
        },
        offsets, ix, ids, ekeys, smem);
}

// Pointers into the heavy_smem layout.
template <typename Key>
struct HeavyLds {
    Key* skeys;
    uint32_t* sids;
    uint16_t* sb;
    uint32_t *cur, *tcnt, *wcnt, *dstart, *tmp;
    __device__ HeavyLds(unsigned char* smem, uint32_t NB) {
        skeys = (Key*)smem;
        sids = (uint32_t*)(skeys + kHeavyChunk);
        sb = (uint16_t*)(sids + kHeavyChunk);
        cur = (uint32_t*)(sb + kHeavyChunk);  // NB: running cursors
        tcnt = cur + NB;                      // NB: chunk-local bucket starts
        wcnt = tcnt + NB;
        dstart = wcnt + W_LOCAL * 64;
        tmp = dstart + 64;
    }
};

// Place L entries (arriving in id order) of one bin, chunk by chunk, in
// order: each chunk is sorted by bucket in LDS and written at the running
// per-bucket cursors cur[0 .. 2^k), which hold absolute edge positions on
// entry and are advanced past the placed entries on return.  Writes outside
// [lo, hi) are dropped (they cannot happen for consistent counts).  With
// any_order a chunk is grouped by bucket with one returning LDS atomic per
// key (the lanes sharing the wave's first lane's bucket take one for the
// group) instead of two stable ranking passes.  Uses the heavy_smem layout;
// whole workgroup.
template <typename Key>
__device__ __forceinline__ void place_in_chunks(const Key* __restrict__ src_keys,
                                                const uint32_t* __restrict__ src_ids,
                                                uint32_t id_base, uint32_t L, uint32_t lo,
                                                uint32_t hi, uint32_t v0, uint32_t k,
                                                const typename KeyTraits<Key>::Params& hp,
                                                uint32_t* __restrict__ ids,
                                                Key* __restrict__ ekeys, unsigned char* smem,
                                                bool any_order = false) {
    constexpr int IT = kHeavyItems;
    constexpr uint32_t CAP = kHeavyChunk;
    const uint32_t NB = 1u << k;
    const HeavyLds<Key> m(smem, NB);
    Key* skeys = m.skeys;
    uint32_t* sids = m.sids;
    uint16_t* sb = m.sb;
    uint32_t *cur = m.cur, *tcnt = m.tcnt, *wcnt = m.wcnt, *dstart = m.dstart, *tmp = m.tmp;
    const uint32_t w = threadIdx.x / kWave, lane = lane_id();
    const uint32_t nchunk = (uint32_t)(((uint64_t)L + CAP - 1) / CAP);
    for (uint32_t ci = 0; ci < nchunk; ++ci) {
        const uint32_t c0 = ci * CAP;
        const uint32_t cl = (L - c0 < CAP) ? L - c0 : CAP;
        const uint32_t wchunk =
            (((cl + W_LOCAL - 1) / W_LOCAL) + kWave - 1) & ~(uint32_t)(kWave - 1);
        const uint32_t wb = w * wchunk;
        const uint32_t mylen = cl > wb ? ((cl - wb < wchunk) ? cl - wb : wchunk) : 0u;
        const uint32_t rounds = (mylen + kWave - 1) / kWave;
        Key kk[IT];
        uint32_t id[IT], b[IT];
#pragma unroll
        for (int r = 0; r < IT; ++r) {
            const uint32_t e = c0 + wb + r * kWave + lane;
            if ((uint32_t)r < rounds && r * kWave + lane < mylen) {
                kk[r] = src_keys[e];
                id[r] = src_ids ? src_ids[e] : id_base + e;
            } else {
                kk[r] = 0;
                id[r] = 0;
            }
        }
        for (uint32_t i = threadIdx.x; i < NB; i += kLocalThreads) tcnt[i] = 0;
        __syncthreads();
        // bins this large usually hold a hot key: the lanes whose bucket
        // equals the wave's first lane's add their count with one atomic (a
        // single LDS address hit by every lane would serialise 64 ways), the
        // others add one each
#pragma unroll
        for (int r = 0; r < IT; ++r) {
            const bool valid = (uint32_t)r < rounds && r * kWave + lane < mylen;
            b[r] = valid ? KeyTraits<Key>::bucket(kk[r], hp) - v0 : NB;
            const uint32_t b0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)b[r]);
            const bool first = valid && b[r] == b0;
            const uint64_t same = ballot(first);
            if (first) {
                if (mbcnt(same) == 0) atomicAdd(&tcnt[b0], (uint32_t)__popcll(same));
            } else if (valid) {
                atomicAdd(&tcnt[b[r]], 1u);
            }
        }
        if (any_order) {
            __syncthreads();
            // chunk-local bucket starts; the slots taken below turn them into
            // bucket ends, and a bucket starts where the one before it ends
            scan_counts(tcnt, NB, 0u, tmp);
#pragma unroll
            for (int r = 0; r < IT; ++r) {
                const bool valid = b[r] < NB;
                const uint32_t b0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)b[r]);
                const bool first = valid && b[r] == b0;
                const uint64_t same = ballot(first);
                uint32_t slot = 0;
                if (first) {
                    uint32_t base = 0;
                    if (mbcnt(same) == 0) base = atomicAdd(&tcnt[b0], (uint32_t)__popcll(same));
                    slot = (uint32_t)__shfl((int)base, (int)__builtin_ctzll(same), kWave) +
                           mbcnt(same);
                } else if (valid) {
                    slot = atomicAdd(&tcnt[b[r]], 1u);
                }
                if (valid) {
                    skeys[slot] = kk[r];
                    sids[slot] = id[r];
                    sb[slot] = (uint16_t)b[r];
                }
            }
            __syncthreads();
            for (uint32_t p = threadIdx.x; p < cl; p += kLocalThreads) {
                const uint32_t bb = sb[p];
                const uint32_t st = bb ? tcnt[bb - 1] : 0u;
                const uint32_t o = cur[bb] + (p - st);
                if (o - lo < hi - lo) {
                    ekeys[o] = skeys[p];
                    ids[o] = sids[p];
                }
            }
            __syncthreads();
            for (uint32_t i = threadIdx.x; i < NB; i += kLocalThreads)
                cur[i] += tcnt[i] - (i ? tcnt[i - 1] : 0u);
            __syncthreads();
            continue;
        }
        sort_chunk_by_bucket<Key, IT>(kk, id, b, rounds, cl, wchunk, k, skeys, sids, sb, wcnt,
                                      dstart, tmp);
        __syncthreads();
        // chunk-local bucket starts (exclusive scan of tcnt)
        scan_counts(tcnt, NB, 0u, tmp);
        for (uint32_t p = threadIdx.x; p < cl; p += kLocalThreads) {
            const uint32_t bb = sb[p];
            const uint32_t o = cur[bb] + (p - tcnt[bb]);
            if (o - lo < hi - lo) {
                ekeys[o] = skeys[p];
                ids[o] = sids[p];
            }
        }
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < NB; i += kLocalThreads) {
            const uint32_t nxt = (i + 1 < NB) ? tcnt[i + 1] : cl;
            cur[i] += nxt - tcnt[i];
        }
        __syncthreads();
    }
}

// Adds the keys' buckets (from v0 on) to cnt, for keys among which one is hot:
// lanes sharing the first active lane's bucket count with one LDS atomic, the
// others one each.  U loads in flight per thread.  Whole workgroup; no barrier.
template <typename Key, int U>
__device__ __forceinline__ void count_hot_buckets(const Key* __restrict__ keys, uint32_t L,
                                                  uint32_t v0,
                                                  const typename KeyTraits<Key>::Params& hp,
                                                  uint32_t* cnt) {
    for (uint32_t i0 = threadIdx.x; i0 < L; i0 += U * kLocalThreads) {
        Key k[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            k[u] = i0 + u * kLocalThreads < L ? keys[i0 + u * kLocalThreads] : (Key)0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i0 + u * kLocalThreads >= L) continue;
            const uint32_t b = KeyTraits<Key>::bucket(k[u], hp) - v0;
            const uint32_t b0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)b);
            const uint64_t same = ballot(b == b0);
            if (b != b0) atomicAdd(&cnt[b], 1u);
            else if (mbcnt(same) == 0) atomicAdd(&cnt[b0], (uint32_t)__popcll(same));
        }
    }
}

// The same for a bin of any size (arriving in id order) in one workgroup:
// keys counted per bucket first, then placed with place_in_chunks, so
// placement stays stable.
template <typename Key, int U = 8>
__device__ __forceinline__ void heavy_bin_body(const Key* __restrict__ src_keys,
                                               const uint32_t* __restrict__ src_ids,
                                               uint32_t id_base, uint32_t L, uint32_t out,
                                               uint32_t v0, uint32_t k, uint32_t nb,
                                               const typename KeyTraits<Key>::Params& hp,
                                               uint32_t* __restrict__ offsets,
                                               const IndexOut& ix,
                                               uint32_t* __restrict__ ids, Key* __restrict__ ekeys,
                                               unsigned char* smem, bool any_order = false) {
    const uint32_t NB = 1u << k;
    const HeavyLds<Key> m(smem, NB);
    uint32_t *cur = m.cur, *tmp = m.tmp;

    for (uint32_t i = threadIdx.x; i < NB; i += kLocalThreads) cur[i] = 0;
    __syncthreads();
    count_hot_buckets<Key, U>(src_keys, L, v0, hp, cur);
    __syncthreads();
    scan_counts(cur, NB, out, tmp);
    for (uint32_t i = threadIdx.x; i < nb; i += kLocalThreads) offsets[v0 + i] = cur[i];
    place_in_chunks<Key>(src_keys, src_ids, id_base, L, out, out + L, v0, k, hp, ids, ekeys,
                         smem, any_order);
    // cur[v] is now the end of bucket v; the bin's edges are in ekeys.  Long
    // buckets are listed for the general pass, which builds their key runs.
    if (ix.head) {
        uint32_t* nlisted = tmp + 2 * W_LOCAL + 2;  // inside heavy_smem's padding
        if (threadIdx.x == 0) *nlisted = 0;
        __syncthreads();
        for (uint32_t v = threadIdx.x; v < nb; v += kLocalThreads) {
            const uint32_t lo = v ? cur[v - 1] : out;
            if (cur[v] - lo > kRunBucket)
                ix.gen_list[gen_region(out, v0 >> k) + atomicAdd(nlisted, 1u)] = v0 + v;
            else
                put_short<Key>(ix, v0 + v, lo, cur[v], ekeys + lo);
        }
        __syncthreads();
        if (threadIdx.x == 0) ix.gen_cnt[v0 >> k] = *nlisted;
    }
}

}  // namespace v2dev
}  // namespace hg
