// HashGraph-V2 (Alg. 2) on gfx950.
//
// The paper's idea -- first move keys into bins of contiguous bucket ranges so
// that the final placement is cache-local -- mapped onto CDNA4 without any
// global atomics:
//   * a final bin is a power-of-two range of 2^k buckets holding about 4096
//     32-bit keys (2048 64-bit keys) on average, so that its keys, ids and
//     bucket counters fit in the LDS of one 512-thread workgroup;
//   * keys reach their final bin by one or two stable partition passes over a
//     digit (a bit-field) of the bucket index.  Each pass is: per-tile digit
//     histograms (LDS), a segmented column scan of the tile x digit matrix
//     (giving every tile an exact base per digit: deterministic, no atomics),
//     and a partition kernel that ranks a tile's keys by digit with wave64
//     ballots and writes digit-contiguous runs;
//   * one workgroup per final bin counts, scans and stably places the bin's
//     keys in LDS and
//     writes the bin's edge segment and offsets with coalesced stores.  Bins
//     larger than LDS (heavy skew only) are listed on the device and handled
//     by the rare path's kernel (hg_runs.hip).
// Every pass keeps input order among equal digits, so ids come out ascending
// inside each bucket: the result is the stable layout, entry for entry.
//
// Stable ranking (rank_stable) finds equal digits in a round of 64 items with
// one ballot per digit bit and keeps per-wave running counts in LDS, updated
// with non-returning atomics so that rounds do not wait on each other.
#include <type_traits>

#include "hg_v2_device.h"

namespace hg {

namespace {

using namespace v2dev;

// Segments of the source array, each cut into tiles of `tile` entries, and
// the tiles grouped into chunks of `ch` consecutive tiles for the column scan.
// One segment known to the host (seg_start null): n entries, ntiles, nchunks.
struct Segs {
    uint32_t* seg_start;     // [S+1]
    uint32_t* tile_prefix;   // [S+1]
    uint32_t* chunk_prefix;  // [S+1]
    uint32_t S;
    uint32_t ch;
    uint32_t n, ntiles, nchunks, tile;

    __device__ __forceinline__ uint32_t start(uint32_t s) const {
        return seg_start ? seg_start[s] : (s ? n : 0u);
    }
    __device__ __forceinline__ uint32_t tile0(uint32_t s) const {
        return seg_start ? tile_prefix[s] : (s ? ntiles : 0u);
    }
    __device__ __forceinline__ uint32_t chunk0(uint32_t s) const {
        return seg_start ? chunk_prefix[s] : (s ? nchunks : 0u);
    }
};

Segs one_segment(uint64_t n, uint32_t ntiles, uint32_t nchunks, uint32_t ch, uint32_t tile) {
    return Segs{nullptr, nullptr, nullptr, 1, ch, (uint32_t)n, ntiles, nchunks, tile};
}

// largest s in [0, S) with pre[s] <= x (pre non-decreasing, pre[0] = 0)
__device__ __forceinline__ uint32_t find_seg(const uint32_t* __restrict__ pre, uint32_t S,
                                             uint32_t x) {
    uint32_t lo = 0, hi = S;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (pre[mid] <= x) lo = mid;
        else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ bool locate_tile(const Segs& g, uint32_t t, uint32_t& seg,
                                            uint32_t& begin, uint32_t& end) {
    if (t >= g.tile0(g.S)) return false;
    seg = g.S > 1 ? find_seg(g.tile_prefix, g.S, t) : 0u;
    begin = g.start(seg) + (t - g.tile0(seg)) * g.tile;
    const uint32_t se = g.start(seg + 1);
    end = (se - begin > g.tile) ? begin + g.tile : se;
    return true;
}

// (xcd_tile: the runs that neighbouring tiles write for a digit meet in
// one XCD's L2)

// ---------------------------------------------------- tile histograms -----

// ID_DIGIT: the digit is a bit-field of the entry's id (ids[i] >> shift)
// instead of the bucket of its key (the scatter by a permutation below).
// QUERIES: the same code, instantiated apart for grouping a probe's queries
// so that kernel traces tell it from the build's passes (also below).
// HBM-bound on uniform keys (2^28: 226 us, 4.8 TB/s read).  A hot digit would
// serialise a wave's lanes on one counter, so each digit has four, side by side,
// of which a lane takes lane % 4: 2^26 Zipf(1.2) keys 147 -> 65 us a pass, the
// uniform ones unchanged.
constexpr int kHistThreads = 512;

template <typename Key, bool ID_DIGIT, bool QUERIES, uint32_t TILE>
__global__ __launch_bounds__(kHistThreads) void k_tile_hist(
    const Key* __restrict__ keys, Segs g, typename KeyTraits<Key>::Params hp, uint32_t shift,
    uint32_t bits, uint32_t* __restrict__ mat, uint32_t tiles_ub,
    const uint32_t* __restrict__ ids = nullptr) {
    extern __shared__ __align__(16) uint32_t cnt[];
    const uint32_t D = 1u << bits;
    const uint32_t t = xcd_tile(blockIdx.x, tiles_ub);
    uint32_t seg, begin, end;
    if (!locate_tile(g, t, seg, begin, end)) return;
    for (uint32_t d = threadIdx.x; d < D; d += kHistThreads)
        ((uint4*)cnt)[d] = make_uint4(0u, 0u, 0u, 0u);
    constexpr int IT = TILE / kHistThreads;
    Key k[IT];
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const uint32_t i = begin + r * kHistThreads + threadIdx.x;
        if (ID_DIGIT) k[r] = (i < end) ? (Key)ids[i] : (Key)0;
        else k[r] = (i < end) ? keys[i] : (Key)0;
    }
    __syncthreads();
    const uint32_t mask = D - 1;
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const uint32_t i = begin + r * kHistThreads + threadIdx.x;
        const uint32_t v = ID_DIGIT ? (uint32_t)k[r] : KeyTraits<Key>::bucket(k[r], hp);
        if (i < end) atomicAdd(&cnt[((v >> shift) & mask) * 4 + (threadIdx.x & 3u)], 1u);
    }
    __syncthreads();
    uint32_t* row = mat + (size_t)t * D;
    for (uint32_t d = threadIdx.x; d < D; d += kHistThreads) {
        const uint4 c = ((const uint4*)cnt)[d];
        row[d] = c.x + c.y + c.z + c.w;
    }
}

// ------------------------------------- segmented column scan of [tile][digit]
// base(t, d) = seg_start[s] + sum_{d' < d} total_s(d') + sum_{t' < t in s} M[t'][d]
// i.e. the exclusive prefix in (segment, digit, tile) order: where tile t's
// keys of digit d go in the stably partitioned output.

__device__ __forceinline__ bool locate_chunk(const Segs& g, uint32_t c, uint32_t& seg,
                                             uint32_t& t0, uint32_t& t1) {
    if (c >= g.chunk0(g.S)) return false;
    seg = g.S > 1 ? find_seg(g.chunk_prefix, g.S, c) : 0u;
    t0 = g.tile0(seg) + (c - g.chunk0(seg)) * g.ch;
    const uint32_t te = g.tile0(seg + 1);
    t1 = (te - t0 > g.ch) ? t0 + g.ch : te;
    return true;
}

__global__ __launch_bounds__(256) void k_colscan_reduce(const uint32_t* __restrict__ mat, Segs g,
                                                        uint32_t D, uint32_t* __restrict__ csum) {
    uint32_t seg, t0, t1;
    if (!locate_chunk(g, blockIdx.x, seg, t0, t1)) return;
    for (uint32_t d = threadIdx.x; d < D; d += 256) {
        uint32_t s = 0;
        uint32_t t = t0;
        for (; t + 8 <= t1; t += 8) {
            uint32_t v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = mat[(size_t)(t + u) * D + d];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; t < t1; ++t) s += mat[(size_t)t * D + d];
        csum[(size_t)blockIdx.x * D + d] = s;
    }
}

// One workgroup per segment: digit totals, their exclusive scan, then chunk
// sums become chunk bases.  It is one workgroup against memory latency (256
// rows of 256 digits at 2^28 keys), so up to 16 row groups walk the chunks side
// by side with eight loads in flight each: 78 -> 14 us at 2^28, 25 -> 6 us at
// 300 007 keys, against one thread per digit walking all rows.
// It knows where every digit of its segment starts, so the starts that the next
// kernels need come from here as well, not from launches of their own.
constexpr int kSegThreads = 1024;

// What a segment scan derives from its digits' starts (all null: nothing).
struct SegsOut {
    uint32_t* zero = nullptr;  // [kCtrWords], cleared (one segment)
    Segs next{};               // the segments of the second pass, one per digit (seg_start set)
    // final bins (bin = segment * digits + digit): their starts, and the lists
    // of those too large for the LDS kernel
    uint32_t* bin_start = nullptr;  // [bins + 1]
    uint32_t bins = 0, n = 0, V = 0, light_keys = 0, slice = 0;
    uint32_t* offsets = nullptr;    // offsets[V] = n
    uint32_t *heavy_list = nullptr, *ctr = nullptr;
    uint32_t *huge_list = nullptr, *huge_s0 = nullptr, *slice_owner = nullptr;
    uint32_t huge_cap = 0, slice_cap = 0;
};

__device__ void next_segments(const Segs& g, const uint32_t* dbase, uint32_t n, uint32_t* tmp);
__device__ void note_bin(const SegsOut& o, uint32_t b, uint32_t st, uint32_t nx);

__global__ __launch_bounds__(kSegThreads) void k_colscan_seg(Segs g, uint32_t D,
                                                             uint32_t* __restrict__ csum,
                                                             SegsOut out) {
    __shared__ uint32_t tmp[kSegThreads / kWave + 1];
    __shared__ uint32_t part[2 * kSegThreads];   // [row group][digit] sums
    __shared__ uint32_t dbase[1u << kMaxDigitBits];
    const uint32_t s = blockIdx.x;
    const uint32_t c0 = g.chunk0(s), c1 = g.chunk0(s + 1);
    if (out.zero && threadIdx.x < kCtrWords) {
        out.zero[threadIdx.x] = 0;
        __threadfence();  // before the atomics below
    }
    if (c0 == c1 && !out.bin_start) return;
    scan_columns<kSegThreads>(csum, c0, c1, D, g.start(s), part, dbase, tmp, [&] {
        if (out.bin_start)
            for (uint32_t d = threadIdx.x; d < D; d += kSegThreads)
                note_bin(out, s * D + d, dbase[d], d + 1 < D ? dbase[d + 1] : g.start(s + 1));
        if (out.next.seg_start) next_segments(out.next, dbase, g.start(1), tmp);
    });
}

__global__ __launch_bounds__(256) void k_colscan_down(uint32_t* __restrict__ mat, Segs g, uint32_t D,
                                                      const uint32_t* __restrict__ csum) {
    uint32_t seg, t0, t1;
    if (!locate_chunk(g, blockIdx.x, seg, t0, t1)) return;
    for (uint32_t d = threadIdx.x; d < D; d += 256) {
        uint32_t r = csum[(size_t)blockIdx.x * D + d];
        uint32_t t = t0;
        for (; t + 8 <= t1; t += 8) {
            uint32_t v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = mat[(size_t)(t + u) * D + d];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                mat[(size_t)(t + u) * D + d] = r;
                r += v[u];
            }
        }
        for (; t < t1; ++t) {
            const uint32_t v = mat[(size_t)t * D + d];
            mat[(size_t)t * D + d] = r;
            r += v;
        }
    }
}

// ------------------------------------------------------------ partition ---

// Consecutive queries that one workgroup of k_ungroup_by_pos puts back in order:
// whole tiles, and a query's place among them fits 16 bits.
constexpr uint32_t kUngroupSpan = 16384;

// How a workgroup takes a tile: 8 items per thread, so that 64 VGPRs and the LDS
// leave 24 to 32 waves a CU.  With 256 threads of 16 items (12 waves a CU) 2^27
// 64-bit keys took 952 and 912 us a stable pass, now 723 and 709; 2^28 any-order
// 32-bit keys in 8192-key tiles 856 us the first pass and 1061 the second, now
// 640 and 1028.
template <typename Key, bool STABLE>
struct PartGeo {
    static constexpr uint32_t kTile = part_tile(sizeof(Key), !STABLE);
    static constexpr int kItems = 8;
    static constexpr int kThreads = kTile / kItems;
};

// LDS of a partition tile, in this order: keys, ids (32 bits where the entries
// carry ids, else their 16-bit place in the tile), digits of 64-bit keys (32-bit
// keys are hashed again instead: their hash costs less than the LDS), the ranking
// counters (per wave where it is stable), digit starts, output bases.  What a
// tile takes sets how many share a CU: a 512-digit any-order tile of 8192 32-bit
// keys 70 KB with ids and 54 without, two workgroups a CU either way.
template <typename Key, bool HAS_IDS, bool STABLE>
struct PartLds {
    using Geo = PartGeo<Key, STABLE>;
    static constexpr uint32_t kTile = Geo::kTile, kWaves = Geo::kThreads / kWave;
    static constexpr bool kDigits = sizeof(Key) == 8;
    using Id = typename std::conditional<HAS_IDS, uint32_t, uint16_t>::type;
    Key* keys;
    Id* ids;
    uint16_t* dig;
    uint32_t *wcnt, *dstart, *tbase, *tmp;
    static constexpr size_t entry() { return sizeof(Key) + sizeof(Id) + (kDigits ? 2 : 0); }
    static size_t bytes(uint32_t bits) {
        const size_t D = (size_t)1 << bits;
        return kTile * entry() + (STABLE ? kWaves : 1) * D * 4 + 2 * D * 4 + (kWaves + 1) * 4 + 64;
    }
    __device__ PartLds(unsigned char* p, uint32_t D) {
        keys = (Key*)p;
        ids = (Id*)(keys + kTile);
        dig = (uint16_t*)(ids + kTile);
        wcnt = (uint32_t*)(dig + (kDigits ? kTile : 0));
        dstart = wcnt + (STABLE ? kWaves : 1) * D;
        tbase = dstart + D;
        tmp = tbase + D;
    }
};

// Stable partition of one tile by a digit of the bucket index.  Writes every
// entry to base(tile, digit) + its rank among the tile's entries of that
// digit.
// STABLE: entries of equal digit keep their order (rank_stable); otherwise
// their order inside a run is unspecified (rank_any, no ballots).
// QUERIES: instead of ids, dst_ids (may be null) receives 16-bit places in
// the kUngroupSpan queries that k_ungroup_by_pos puts back together.
template <typename Key, bool HAS_IDS, bool STABLE, bool ID_DIGIT = false, bool QUERIES = false>
__global__ __launch_bounds__((PartGeo<Key, STABLE>::kThreads)) void k_tile_partition(
    const Key* __restrict__ src_keys, const uint32_t* __restrict__ src_ids,
    Key* __restrict__ dst_keys, uint32_t* __restrict__ dst_ids, Segs g,
    typename KeyTraits<Key>::Params hp, uint32_t shift, uint32_t bits,
    const uint32_t* __restrict__ base, uint32_t tiles_ub) {
    using Geo = PartGeo<Key, STABLE>;
    constexpr int IT = Geo::kItems, kThreads = Geo::kThreads;
    using Lds = PartLds<Key, HAS_IDS, STABLE>;
    const uint32_t D = 1u << bits;
    extern __shared__ __align__(16) unsigned char smem[];
    const Lds m(smem, D);

    const uint32_t t = xcd_tile(blockIdx.x, tiles_ub);
    uint32_t seg, begin, end;
    if (!locate_tile(g, t, seg, begin, end)) return;
    const uint32_t cnt = end - begin;
    const uint32_t w = threadIdx.x / kWave, lane = lane_id();
    const uint32_t mask = D - 1;
    const uint32_t wbase = w * (kWave * IT);

    Key k[IT];
    uint32_t id[IT], dig[IT], pos[IT];
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const uint32_t e = wbase + r * kWave + lane;
        k[r] = e < cnt ? src_keys[begin + e] : (Key)0;
        id[r] = HAS_IDS && e < cnt ? src_ids[begin + e] : 0u;
    }
    // the tile's digit bases, loaded now so that their latency overlaps the
    // ranking (D <= 2048: at most kRowPer per thread)
    constexpr int kRowPer = (1 << kMaxDigitBits) / kThreads;
    const uint32_t* row = base + (size_t)t * D;
    uint32_t rowv[kRowPer];
#pragma unroll
    for (int j = 0; j < kRowPer; ++j) {
        const uint32_t d = threadIdx.x + j * kThreads;
        rowv[j] = d < D ? row[d] : 0u;
    }
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const uint32_t e = wbase + r * kWave + lane;
        const uint32_t v = ID_DIGIT ? id[r] : KeyTraits<Key>::bucket(k[r], hp);
        dig[r] = (e < cnt) ? ((v >> shift) & mask) : D;
    }
    if (STABLE) rank_stable<kThreads, IT>(dig, bits, m.wcnt, m.dstart, m.tmp, pos);
    else rank_any<kThreads, IT>(dig, bits, m.wcnt, m.dstart, m.tmp, pos);
#pragma unroll
    for (int j = 0; j < kRowPer; ++j) {
        const uint32_t d = threadIdx.x + j * kThreads;
        if (d < D) m.tbase[d] = rowv[j] - m.dstart[d];
    }
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        if (dig[r] < D) {
            m.keys[pos[r]] = k[r];
            m.ids[pos[r]] = HAS_IDS ? (typename Lds::Id)id[r]
                                    : (typename Lds::Id)(wbase + r * kWave + lane);
            if (Lds::kDigits) m.dig[pos[r]] = (uint16_t)dig[r];
        }
    }
    __syncthreads();
    // every output lies inside this segment's range; the guard keeps a
    // corrupted base from turning into a stray store
    const uint32_t seg_lo = g.start(seg), seg_len = g.start(seg + 1) - seg_lo;
    uint16_t* dst_place = (uint16_t*)dst_ids;
    const uint32_t place0 = QUERIES ? (t % (kUngroupSpan / Geo::kTile)) * Geo::kTile : 0u;
    for (uint32_t p = threadIdx.x; p < cnt; p += kThreads) {
        const Key key = m.keys[p];
        const uint32_t x = m.ids[p];
        const uint32_t d = Lds::kDigits ? m.dig[p]
                                        : ((ID_DIGIT ? x : KeyTraits<Key>::bucket(key, hp)) >> shift) & mask;
        const uint32_t o = m.tbase[d] + p;
        if (o - seg_lo < seg_len) {
            dst_keys[o] = key;
            if (QUERIES) {
                if (dst_ids) dst_place[o] = (uint16_t)(place0 + x);
            } else {
                dst_ids[o] = HAS_IDS ? x : begin + x;
            }
        }
    }
}

// ------------------------------------------------------ grouped probing ---

// Puts counts found in grouped order back in input order.  Entry e of
// partition tile t was written to base(t, d) + its rank inside the tile's run
// of digit d, with its place among kUngroupSpan queries in `place`.  The runs of
// consecutive tiles are adjacent in grouped order, so one workgroup takes the
// tiles [t0, t1) of kUngroupSpan queries: its run of digit d is
// [base(t0, d), next(t1, d)), next being base(t1, d), or past the last tile the
// start of digit d + 1 (m after the last digit).  A wave takes the runs of up to
// 64 consecutive digits, one lane finds each run's start and length, and each
// run's first 64 entries are one load of places and one of counts, eight runs in
// flight; what is longer (32 entries are usual, skew lengthens runs) is listed and
// taken by the whole workgroup.  Counts go to LDS by place and from there in
// input order; they come as bytes, and 255 stands for the 32-bit one in `wide`,
// which the thread that meets it writes itself.  One segment (S = 1).
// Bound by HBM and by latency: 3 bytes read and 4 written per query.  2^28
// queries: 943 us with 32-bit positions and counts and a binary search over the
// runs' starts per entry, 725 with these bytes and a walk along the starts, 503
// by runs.
constexpr uint32_t kUngroupThreads = 1024;
constexpr uint32_t kUngroupLong = kUngroupSpan / (kWave + 1);  // runs above 64 entries, at most
static_assert((1u << 9) <= kUngroupThreads, "a wave's digits fit its lanes");

__global__ __launch_bounds__(kUngroupThreads, 8) void k_ungroup_by_pos(
    uint64_t m, uint32_t ntiles, uint32_t tile, uint32_t bits, const uint32_t* __restrict__ base,
    uint32_t groups, const uint16_t* __restrict__ place, const uint8_t* __restrict__ src,
    const uint32_t* __restrict__ wide, uint32_t* __restrict__ dst,
    const uint32_t* __restrict__ gate) {
    if (gate && *gate != 1u) return;  // the probe kept input order
    __shared__ uint32_t sval32[kUngroupSpan / 4];
    __shared__ uint32_t lstart[kUngroupLong], llen[kUngroupLong];
    __shared__ uint32_t nlong;
    uint8_t* sval = (uint8_t*)sval32;
    const uint32_t D = 1u << bits;
    const uint32_t gi = xcd_tile(blockIdx.x, groups);
    if (gi >= groups) return;
    if (threadIdx.x == 0) nlong = 0;
    __syncthreads();
    const uint32_t tiles = kUngroupSpan / tile;
    const uint32_t t0 = gi * tiles;
    const uint32_t t1 = t0 + tiles < ntiles ? t0 + tiles : ntiles;
    const uint64_t begin = (uint64_t)t0 * tile;
    const uint64_t end64 = (uint64_t)t1 * tile;
    const uint32_t cnt = (uint32_t)((end64 < m ? end64 : m) - begin);
    const uint32_t lane = lane_id();
    constexpr uint32_t W = kUngroupThreads / kWave;
    const uint32_t per = (D + W - 1) / W;  // digits per wave, at most 64
    const uint32_t d = threadIdx.x / kWave * per + lane;
    uint32_t b = 0, c = 0;
    if (lane < per && d < D) {
        b = base[(size_t)t0 * D + d];
        const uint32_t nx = t1 < ntiles ? base[(size_t)t1 * D + d]
                                        : (d + 1 < D ? base[d + 1] : (uint32_t)m);
        c = nx - b;
        if (c > kWave) {
            const uint32_t i = atomicAdd(&nlong, 1u);
            if (i < kUngroupLong) {
                lstart[i] = b;
                llen[i] = c;
            }
        }
    }
    // entry o of the grouped order, with its place and count loaded
    auto put = [&](uint32_t o, uint32_t p, uint32_t v) {
        if (p < cnt) {
            sval[p] = (uint8_t)v;
            if (v == 255u) dst[begin + p] = wide[o];
        }
    };
    constexpr uint32_t U = 8;
    for (uint32_t i0 = 0; i0 < per; i0 += U) {  // (lanes past the wave's digits hold c = 0)
        uint32_t o[U], p[U], v[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t st = __builtin_amdgcn_readlane(b, i0 + u);
            const uint32_t len = __builtin_amdgcn_readlane(c, i0 + u);
            o[u] = st + lane;
            const bool in = lane < len && o[u] < m;
            p[u] = in ? place[o[u]] : ~0u;
            v[u] = in ? src[o[u]] : 0u;
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) put(o[u], p[u], v[u]);
    }
    __syncthreads();
    const uint32_t nl = nlong < kUngroupLong ? nlong : kUngroupLong;
    for (uint32_t l = 0; l < nl; ++l)
        for (uint32_t i = kWave + threadIdx.x; i < llen[l]; i += kUngroupThreads) {
            const uint32_t o = lstart[l] + i;
            if (o < m) put(o, place[o], src[o]);
        }
    __syncthreads();
    for (uint32_t p = threadIdx.x; p < cnt; p += kUngroupThreads)
        if (sval[p] != 255u) dst[begin + p] = sval[p];
}

constexpr uint32_t kGroupBits = 9;  // ranges of a grouped probe: 2^kGroupBits at most

// A range holding more than kGroupSkew times an even share of the sampled
// queries keeps a probe in input order.
constexpr uint32_t kGroupSkew = 8;

// So does a share of more than this many eighths of sampled neighbours in one range:
// such queries come in runs or already by bucket, and share the index lines that
// grouping would bring together.  Of queries that repeat the one before with
// probability f, input order was the faster from f = 0.3 at 2^23 buckets (load 4), 0.4
// at 2^25, 0.46 at 2^26 and 0.63 at 2^28: 2^26 queries of 2^26 buckets in bucket order
// take 0.24 ms in input order and 0.91 grouped, in runs of eight 0.24 and 0.85.
uint32_t group_local_eighths(uint64_t V) {
    return V < (1ull << 26) ? 3u : V < (1ull << 27) ? 4u : 5u;
}

// Whether grouping pays for these queries, from a sample: up to kGroupSample
// queries, 16 neighbours (a line of them, one page) at each of 1024 places spread
// evenly over the input, are hashed into the ranges, and when
// one range holds more than kGroupSkew times an even share of them the probe
// keeps input order (skewed queries read few index lines, which stay cached
// anyway); also when more than local / 8 of the neighbours share a range (not asked
// below 2^kGroupBits ranges, where neighbours meet by chance).  Neighbours that equal
// each other make the sample one of 1024 places: an even spread over 512 ranges then
// leaves a range with 2 on average, and 17 of them, the line of kGroupSkew, has a
// chance of 10^-10.  Writes the one segment of the grouping passes -- with no tiles
// at all for input order, so that every grouping kernel returns at once --
// and gate[0] = 1 (grouped) or 0 (input order).  One workgroup, bound by the
// latency of its loads: 35 us at 2^28 queries with each sample on a page of its
// own, now below 11.
constexpr uint32_t kGroupSample = 1u << 14;  // 16 per thread, loaded together
constexpr uint32_t kSampleRun = 16;

template <typename Key>
__global__ __launch_bounds__(1024) void k_group_sample(const Key* __restrict__ q, uint64_t m,
                                                       typename KeyTraits<Key>::Params hp,
                                                       uint32_t shift, uint32_t bits, Segs g,
                                                       uint32_t ntiles, uint32_t nchunks,
                                                       uint32_t local,
                                                       uint32_t* __restrict__ gate) {
    __shared__ uint32_t cnt[1u << kMaxDigitBits];
    __shared__ uint32_t wmax[1024 / kWave];
    __shared__ uint32_t near;  // neighbours in one range
    const uint32_t D = 1u << bits;
    for (uint32_t d = threadIdx.x; d < D; d += 1024) cnt[d] = 0;
    if (threadIdx.x == 0) near = 0;
    __syncthreads();
    const uint32_t S = m < kGroupSample ? (uint32_t)m : kGroupSample;
    constexpr int IT = kGroupSample / 1024;
    const uint64_t step = m > kGroupSample ? m / (kGroupSample / kSampleRun) : kSampleRun;
    Key k[IT];
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const uint32_t i = r * 1024 + threadIdx.x;
        k[r] = i < S ? q[(uint64_t)(i / kSampleRun) * step + i % kSampleRun] : (Key)0;
    }
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const uint32_t i = r * 1024 + threadIdx.x;
        const uint32_t d = (KeyTraits<Key>::bucket(k[r], hp) >> shift) & (D - 1);
        if (i < S) atomicAdd(&cnt[d], 1u);
        const uint32_t next = (uint32_t)__shfl_down((int)d, 1, kWave);
        const uint64_t same = ballot(i + 1 < S && i % kSampleRun != kSampleRun - 1 && next == d);
        if (lane_id() == 0 && same) atomicAdd(&near, (uint32_t)__popcll(same));
    }
    __syncthreads();
    uint32_t mx = 0;
    for (uint32_t d = threadIdx.x; d < D; d += 1024) mx = cnt[d] > mx ? cnt[d] : mx;
    for (int o = kWave / 2; o > 0; o >>= 1) {
        const uint32_t x = (uint32_t)__shfl_xor((int)mx, o, kWave);
        mx = x > mx ? x : mx;
    }
    if (lane_id() == 0) wmax[threadIdx.x / kWave] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 1024 / kWave; ++w) mx = wmax[w] > mx ? wmax[w] : mx;
        const uint32_t pairs = S - 1 - (S - 1) / kSampleRun;
        const bool apart = D < (1u << kGroupBits) || 8 * near <= local * pairs;
        const bool grouped = apart && (uint64_t)mx * D <= (uint64_t)kGroupSkew * S;
        gate[0] = grouped ? 1u : 0u;
        g.seg_start[0] = 0;
        g.seg_start[1] = (uint32_t)m;
        g.tile_prefix[0] = 0;
        g.tile_prefix[1] = grouped ? ntiles : 0u;
        g.chunk_prefix[0] = 0;
        g.chunk_prefix[1] = grouped ? nchunks : 0u;
    }
}

// ------------------------------------------------- from digits' starts ---

// Tier-2 segments, one per tier-1 digit, from the digits' starts (in LDS).
// One workgroup; S <= 2048.
__device__ void next_segments(const Segs& g, const uint32_t* dbase, uint32_t n, uint32_t* tmp) {
    const uint32_t S = g.S;
    const uint32_t per = (S + kSegThreads - 1) / kSegThreads;  // <= 2
    uint32_t nt[2] = {0, 0}, nc[2] = {0, 0}, st[2] = {0, 0};
    uint32_t mt = 0, mc = 0;
    for (uint32_t j = 0; j < per; ++j) {
        const uint32_t a = threadIdx.x * per + j;
        if (a < S) {
            const uint32_t s0 = dbase[a];
            const uint32_t s1 = a + 1 < S ? dbase[a + 1] : n;
            st[j] = s0;
            nt[j] = (s1 - s0 + g.tile - 1) / g.tile;
            nc[j] = (nt[j] + g.ch - 1) / g.ch;
            mt += nt[j];
            mc += nc[j];
        }
    }
    uint32_t tt, tc;
    uint32_t rt = block_excl_scan<kSegThreads>(mt, tmp, &tt);
    uint32_t rc = block_excl_scan<kSegThreads>(mc, tmp, &tc);
    for (uint32_t j = 0; j < per; ++j) {
        const uint32_t a = threadIdx.x * per + j;
        if (a < S) {
            g.seg_start[a] = st[j];
            g.tile_prefix[a] = rt;
            g.chunk_prefix[a] = rc;
            rt += nt[j];
            rc += nc[j];
        }
    }
    if (threadIdx.x == 0) {
        g.seg_start[S] = n;
        g.tile_prefix[S] = tt;
        g.chunk_prefix[S] = tc;
    }
}

// Final bin b = [st, nx) of the partitioned array (b past the last bin: empty):
// its start, and its place in a list when it is too large for the LDS kernel.
// Bins above `slice` keys are split into slices of that many for several
// workgroups: they are listed in huge_list with their first slice in huge_s0,
// and slice_owner maps every slice back to its entry.
__device__ void note_bin(const SegsOut& o, uint32_t b, uint32_t st, uint32_t nx) {
    if (b >= o.bins) return;
    o.bin_start[b] = st;
    if (b + 1 == o.bins) {
        o.bin_start[o.bins] = o.n;
        o.offsets[o.V] = o.n;
    }
    const uint32_t L = nx - st;
    if (L <= o.light_keys) return;
    if (L <= o.slice) {
        o.heavy_list[atomicAdd(&o.ctr[kCtrHeavy], 1u)] = b;
        return;
    }
    // capacities hold: a split bin has > slice keys, so there are at most
    // n / slice of them and fewer than 2n / slice slices
    const uint32_t ns = (L + o.slice - 1) / o.slice;
    const uint32_t idx = atomicAdd(&o.ctr[kCtrSplit], 1u);
    const uint32_t s0 = atomicAdd(&o.ctr[kCtrSlices], ns);
    if (idx < o.huge_cap && s0 + ns <= o.slice_cap) {
        o.huge_list[idx] = b;
        o.huge_s0[idx] = s0;
        for (uint32_t j = 0; j < ns; ++j) o.slice_owner[s0 + j] = idx;
    }
}

// One workgroup per final bin g (buckets [g*2^k, min((g+1)*2^k, V))) that
// holds at most light_cap<Key>() keys.
// ANY: any order inside a bucket; W: bytes of an index entry (0: none).
// Both are constants so that a bin carries the code of its own layout only: 57 to 80
// VGPRs in any order, 101 to 128 stable (whose bins with a bucket of more than kFixMax
// keys are sorted in registers), and two workgroups per CU need 128.
template <typename Key, bool ANY, int W>
__global__ __launch_bounds__(kLocalThreads, 4) void k_local_light(
    const Key* __restrict__ src_keys, const uint32_t* __restrict__ src_ids,
    const uint32_t* __restrict__ bin_start, typename KeyTraits<Key>::Params hp, uint32_t k,
    uint32_t* __restrict__ offsets, IndexOut ix, uint32_t* __restrict__ ids,
    Key* __restrict__ ekeys) {
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t g = blockIdx.x;
    const uint32_t start = bin_start[g], end = bin_start[g + 1];
    const uint32_t L = end - start;
    if (L > light_cap<Key>()) return;  // oversize bins are left to the rare path
    const uint32_t NB = 1u << k, v0 = g << k, V = hp.range;
    const uint32_t nb = (V - v0 < NB) ? V - v0 : NB;
    light_bin_body<Key, ANY, W>(src_keys + start, src_ids + start, 0u, L, start, v0, k, nb, hp,
                                offsets, ix, ids, ekeys, smem);
}

// Calls f with any_order and the index entry's bytes as constants.
template <typename Key, typename F>
void with_layout(bool any_order, const IndexOut& ix, F&& f) {
    auto by_width = [&](auto any) {
        if (!ix.head) f(any, std::integral_constant<int, 0>{});
        else if constexpr (sizeof(Key) == 8) f(any, std::integral_constant<int, 16>{});
        else if (ix.fmt.bytes == 4) f(any, std::integral_constant<int, 4>{});
        else if (ix.fmt.bytes == 8) f(any, std::integral_constant<int, 8>{});
        else f(any, std::integral_constant<int, 16>{});
    };
    if (any_order) by_width(std::true_type{});
    else by_width(std::false_type{});
}

// Final step of the scatter by a permutation: bin g holds the entries whose
// ids are [g << k, (g << k) + 2^k) (every id occurs once, so the bin starts at
// g << k after the partition passes); they are placed in LDS by id and
// written out with coalesced stores.  HBM-bound once a thread's eight entries are
// loaded together: 2^25 entries 108 -> 83 us (12 bytes each, 4.8 TB/s).
__global__ __launch_bounds__(512) void k_perm_place(const uint32_t* __restrict__ vals,
                                                    const uint32_t* __restrict__ ids, uint64_t n,
                                                    uint32_t k, uint32_t* __restrict__ out) {
    __shared__ uint32_t buf[1u << kMaxLocalBits];
    const uint64_t start = (uint64_t)blockIdx.x << k;
    const uint32_t len = (uint32_t)(n - start < (1ull << k) ? n - start : (1ull << k));
    constexpr int IT = (1 << kMaxLocalBits) / 512;
    uint32_t off[IT], v[IT];
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const uint32_t i = r * 512 + threadIdx.x;
        off[r] = i < len ? (uint32_t)(ids[start + i] - start) : ~0u;
        v[r] = i < len ? vals[start + i] : 0u;
    }
#pragma unroll
    for (int r = 0; r < IT; ++r)
        if (off[r] < len) buf[off[r]] = v[r];
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < len; i += 512) out[start + i] = buf[i];
}

__global__ void k_perm_direct(const uint32_t* __restrict__ ids, const uint32_t* __restrict__ vals,
                              uint64_t n, uint32_t* __restrict__ out) {
    uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t st = (uint64_t)gridDim.x * blockDim.x;
    for (; p < n; p += st) {
        const uint32_t id = ids[p];
        if (id < n) out[id] = vals[p];
    }
}

constexpr uint64_t kPermDirectMax = 1ull << 20;  // below this the output stays in L2

V2Plan perm_plan(uint64_t n);

}  // namespace

// ------------------------------------------------------------------ plan --

namespace {

// About 4096 keys per final bin for 32-bit keys (2^k * n / V ~ 4096), 2048 for
// 64-bit keys, whose LDS bin then still leaves room for two workgroups per CU.
uint64_t bin_keys(int key_bits) { return key_bits == 64 ? 2048 : 4096; }

// The passes of a plan whose n, V, tile and k are set.
void plan_passes(V2Plan& p) {
    p.bins = (uint32_t)ceil_div(p.V, 1ull << p.k);
    const uint32_t bits = log2_ceil(p.bins);
    if (bits <= kOneTierBits) {
        p.tiers = 1;
        p.b1 = bits;
        p.b2 = 0;
    } else {
        p.tiers = 2;
        p.b1 = bits / 2;
        p.b2 = bits - p.b1;
    }
    p.ntiles1 = (uint32_t)ceil_div(p.n, p.tile);
    p.ch1 = (uint32_t)pow2_ceil(ceil_div(p.ntiles1 ? p.ntiles1 : 1, 256));
    p.nchunks1 = (uint32_t)ceil_div(p.ntiles1, p.ch1);
    if (p.tiers == 2) {
        const uint32_t S = 1u << p.b1;
        p.ntiles2_ub = p.ntiles1 + S;
        p.ch2 = (uint32_t)pow2_ceil(ceil_div(p.ntiles1 ? p.ntiles1 : 1, (uint64_t)S * 4));
        p.nchunks2_ub = (uint32_t)ceil_div(p.ntiles2_ub, p.ch2) + S;
    }
}

}  // namespace

V2Plan plan_v2(uint64_t n, uint64_t V, int key_bits, uint32_t bins_hint, bool any_order) {
    V2Plan p;
    p.tile = part_tile(key_bits / 8, any_order);
    p.n = n;
    p.V = V;
    uint32_t k;
    if (bins_hint) {
        k = log2_ceil(ceil_div(V, bins_hint));
    } else if (n == 0) {
        k = kMaxLocalBits;
    } else {
        const double r = (double)bin_keys(key_bits) * (double)V / (double)n;
        k = 0;
        while (k < kMaxLocalBits && (double)(1ull << (k + 1)) <= r) ++k;
    }
    if (k > kMaxLocalBits) k = kMaxLocalBits;
    const uint32_t kv = log2_ceil(V);
    if (k > kv) k = kv;
    p.k = k;
    plan_passes(p);
    return p;
}

namespace {

struct V2Ws {
    void* rkeys;
    uint32_t* rids;
    uint32_t *m1, *c1, *m2, *c2, *bin_start, *heavy_list;
    uint32_t* ctr;  // [kCtrWords]
    uint32_t *huge_list, *huge_s0, *slice_owner, *slice_hist, *range_sum;
    uint32_t huge_cap, slice_cap;
    uint32_t *gen_list, *gen_cnt;  // long buckets left to the general key-run pass
    void* runs_ws;
    Segs s1, s2;
};

// What the partition passes need: the reorganised entries, the [tile][digit] matrices
// and their chunk sums, the segments.
void layout_passes(Carver& c, const V2Plan& p, size_t key_size, V2Ws& w) {
    w.rkeys = c.take<char>(p.n * key_size);
    w.rids = c.take<uint32_t>(p.n);
    const uint32_t D1 = 1u << p.b1, D2 = 1u << p.b2;
    w.m1 = c.take<uint32_t>((size_t)p.ntiles1 * D1);
    w.c1 = c.take<uint32_t>((size_t)p.nchunks1 * D1);
    w.s1 = one_segment(p.n, p.ntiles1, p.nchunks1, p.ch1, p.tile);
    if (p.tiers == 2) {
        w.m2 = c.take<uint32_t>((size_t)p.ntiles2_ub * D2);
        w.c2 = c.take<uint32_t>((size_t)p.nchunks2_ub * D2);
        w.s2.seg_start = c.take<uint32_t>(D1 + 1);
        w.s2.tile_prefix = c.take<uint32_t>(D1 + 1);
        w.s2.chunk_prefix = c.take<uint32_t>(D1 + 1);
        w.s2.S = D1;
        w.s2.ch = p.ch2;
        w.s2.tile = p.tile;
    }
}

// One layout used both to size a build's workspace (base == nullptr) and to carve it.
size_t layout_v2(void* ws, const V2Plan& p, size_t key_size, V2Ws* out) {
    Carver c(ws);
    V2Ws w{};
    layout_passes(c, p, key_size, w);
    w.bin_start = c.take<uint32_t>((size_t)p.bins + 1);
    w.heavy_list = c.take<uint32_t>((size_t)p.bins);
    w.ctr = c.take<uint32_t>(kCtrWords);
    w.huge_cap = split_cap(p.n);
    w.slice_cap = 2 * w.huge_cap;
    w.huge_list = c.take<uint32_t>(w.huge_cap);
    w.huge_s0 = c.take<uint32_t>(w.huge_cap);
    w.slice_owner = c.take<uint32_t>(w.slice_cap);
    w.slice_hist = c.take<uint32_t>((size_t)w.slice_cap << p.k);
    w.range_sum = c.take<uint32_t>(range_sum_words(w.slice_cap));
    w.gen_list = c.take<uint32_t>(gen_list_cap(p.n, p.bins));
    w.gen_cnt = c.take<uint32_t>((size_t)p.bins + 1);
    w.runs_ws = c.take<char>(runs_ws_bytes(p.n));
    if (out) *out = w;
    return c.off + 256;
}

// for_probe: profiled under the grouped probe's names
hipError_t colscan(uint32_t* mat, const Segs& g, uint32_t D, uint32_t* csum, uint32_t nchunks_ub,
                   hipStream_t s, bool for_probe, const SegsOut& out) {
    if (g.ch == 1) {  // chunks of one tile: the matrix is its own chunk sums
        HG_PROF(for_probe ? "probe_group_scan_seg" : "v2_colscan_seg", s);
        hipLaunchKernelGGL(k_colscan_seg, dim3(g.S), dim3(kSegThreads), 0, s, g, D, mat, out);
        return hipGetLastError();
    }
    {
        HG_PROF(for_probe ? "probe_group_scan_reduce" : "v2_colscan_reduce", s);
        hipLaunchKernelGGL(k_colscan_reduce, dim3(nchunks_ub), dim3(256), 0, s,
                           (const uint32_t*)mat, g, D, csum);
    }
    HG_TRY(hipGetLastError());
    {
        HG_PROF(for_probe ? "probe_group_scan_seg" : "v2_colscan_seg", s);
        hipLaunchKernelGGL(k_colscan_seg, dim3(g.S), dim3(kSegThreads), 0, s, g, D, csum, out);
    }
    HG_TRY(hipGetLastError());
    {
        HG_PROF(for_probe ? "probe_group_scan_down" : "v2_colscan_down", s);
        hipLaunchKernelGGL(k_colscan_down, dim3(nchunks_ub), dim3(256), 0, s, mat, g, D,
                           (const uint32_t*)csum);
    }
    return hipGetLastError();
}

template <typename Key, bool ID_DIGIT, bool QUERIES, bool STABLE>
void launch_hist(dim3 grid, hipStream_t s, const Key* keys, const uint32_t* ids, const Segs& g,
                 typename KeyTraits<Key>::Params hp, uint32_t shift, uint32_t bits, uint32_t* mat,
                 uint32_t tiles_ub) {
    hipLaunchKernelGGL((k_tile_hist<Key, ID_DIGIT, QUERIES, PartGeo<Key, STABLE>::kTile>), grid,
                       dim3(kHistThreads), 16u << bits, s, keys, g, hp, shift, bits, mat, tiles_ub,
                       ids);
}

template <typename Key, bool HAS_IDS, bool STABLE, bool ID_DIGIT = false, bool QUERIES = false>
void launch_partition(dim3 grid, hipStream_t s, const Key* src_keys, const uint32_t* src_ids,
                      Key* dst_keys, uint32_t* dst_ids, const Segs& g,
                      typename KeyTraits<Key>::Params hp, uint32_t shift, uint32_t bits,
                      const uint32_t* mat, uint32_t tiles_ub) {
    hipLaunchKernelGGL((k_tile_partition<Key, HAS_IDS, STABLE, ID_DIGIT, QUERIES>), grid,
                       dim3(PartGeo<Key, STABLE>::kThreads),
                       (PartLds<Key, HAS_IDS, STABLE>::bytes(bits)), s,
                       src_keys, src_ids, dst_keys, dst_ids, g, hp, shift, bits, mat, tiles_ub);
}

// One stable (or any-order) partition pass over the tiles of segments g.
// id_digit (32-bit entries with ids only): the digit comes from the id.
// tier: 1 or 2 for the build's passes, 3 for grouping the queries of a probe
// (profiled under its own names), where dst_ids may be null and receives the
// places that k_ungroup_by_pos reads.
template <typename Key>
hipError_t partition_pass(const Key* src_keys, const uint32_t* src_ids, Key* dst_keys,
                          uint32_t* dst_ids, const Segs& g, typename KeyTraits<Key>::Params hp,
                          uint32_t shift, uint32_t bits, uint32_t* mat, uint32_t* csum,
                          uint32_t tiles_ub, uint32_t nchunks_ub, int tier, bool stable,
                          hipStream_t s, bool id_digit = false, const SegsOut& out = SegsOut{}) {
    const uint32_t D = 1u << bits;
    const uint32_t grid = (uint32_t)(8 * ceil_div(tiles_ub, 8));
    if (id_digit && (sizeof(Key) != 4 || !src_ids || stable)) return hipErrorInvalidValue;
    if (tier == 3 && (src_ids || stable)) return hipErrorInvalidValue;
    if (bits > kMaxDigitBits) return hipErrorInvalidValue;  // the kernels hold at most 2048 digits
    {
        HG_PROF(tier == 1 ? "v2_tile_hist_t1" : tier == 2 ? "v2_tile_hist_t2" : "probe_group_hist", s);
        const auto launch = id_digit    ? launch_hist<Key, true, false, false>
                            : tier == 3 ? launch_hist<Key, false, true, false>
                            : stable    ? launch_hist<Key, false, false, true>
                                        : launch_hist<Key, false, false, false>;
        launch(dim3(grid), s, src_keys, src_ids, g, hp, shift, bits, mat, tiles_ub);
    }
    HG_TRY(hipGetLastError());
    HG_TRY(colscan(mat, g, D, csum, nchunks_ub, s, tier == 3, out));
    {
        HG_PROF(tier == 1 ? "v2_partition_t1" : tier == 2 ? "v2_partition_t2" : "probe_group", s);
        const auto launch = id_digit        ? launch_partition<Key, true, false, true>
                            : tier == 3     ? launch_partition<Key, false, false, false, true>
                            : src_ids       ? (stable ? launch_partition<Key, true, true>
                                                      : launch_partition<Key, true, false>)
                            : stable        ? launch_partition<Key, false, true>
                                            : launch_partition<Key, false, false>;
        launch(dim3(grid), s, src_keys, src_ids, dst_keys, dst_ids, g, hp, shift, bits, mat,
               tiles_ub);
    }
    return hipGetLastError();
}

template <typename Key>
hipError_t set_smem_limits() {
    static std::atomic<uint64_t> done{0};
    return once_per_device(done, [] {
        const int lim = 160 * 1024;
        HG_TRY(hipFuncSetAttribute((const void*)k_tile_partition<Key, true, true>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, lim));
        HG_TRY(hipFuncSetAttribute((const void*)k_tile_partition<Key, false, true>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, lim));
        HG_TRY(hipFuncSetAttribute((const void*)k_tile_partition<Key, true, false>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, lim));
        HG_TRY(hipFuncSetAttribute((const void*)k_tile_partition<Key, true, false, true>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, lim));
        HG_TRY(hipFuncSetAttribute((const void*)k_tile_partition<Key, false, false>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, lim));
        HG_TRY(hipFuncSetAttribute((const void*)k_tile_partition<Key, false, false, false, true>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize, lim));
        hipError_t le = hipSuccess;
        IndexOut ix{};
        for (int i = 0; i < 8; ++i) {  // every layout and entry width
            ix.head = i / 2 ? &le : nullptr;
            ix.fmt.bytes = 2u << (i / 2);
            with_layout<Key>(i & 1, ix, [&](auto any, auto width) {
                const hipError_t e = hipFuncSetAttribute(
                    (const void*)k_local_light<Key, decltype(any)::value, decltype(width)::value>,
                    hipFuncAttributeMaxDynamicSharedMemorySize, lim);
                if (e != hipSuccess) le = e;
            });
        }
        HG_TRY(le);
        return hipSuccess;
    });
}

}  // namespace

size_t build_ws_bytes(int variant, uint64_t n, uint64_t V, int key_bits, uint32_t bins_hint) {
    const size_t ks = key_bits == 64 ? 8 : 4;
    if (variant == 1) {
        Carver c(nullptr);
        c.take<uint32_t>(V);
        c.take<char>(scan_ws_bytes(V));
        return c.off + 256;
    }
    const size_t st = layout_v2(nullptr, plan_v2(n, V, key_bits, bins_hint, false), ks, nullptr);
    const size_t any = layout_v2(nullptr, plan_v2(n, V, key_bits, bins_hint, true), ks, nullptr);
    return st > any ? st : any;
}

size_t table_ws_bytes(uint64_t n_cap, uint64_t V_cap, int key_bits) {
    size_t most = build_ws_bytes(1, n_cap, V_cap, key_bits, 0);
    const uint32_t kv_max = log2_ceil(V_cap);
    for (uint32_t kv = 0; kv <= kv_max; ++kv) {
        // the ranges with ceil(log2 V) = kv
        const uint64_t lo = kv ? (1ull << (kv - 1)) + 1 : 1;
        const uint64_t hi = (1ull << kv) < V_cap ? 1ull << kv : V_cap;
        const uint32_t k_top = kv < kMaxLocalBits ? kv : kMaxLocalBits;
        for (uint32_t k = 0; k <= k_top; ++k) {
            // plan_v2 takes bins of 2^k buckets for bin_keys * V / 2^(k + 1) < n <=
            // bin_keys * V / 2^k, the smallest k also for more keys and the largest
            // for fewer; with them the layout grows with n
            const uint64_t at = bin_keys(key_bits) * hi >> k;
            const uint64_t n = k == 0 || at > n_cap ? n_cap : at;
            if (k < k_top && n <= bin_keys(key_bits) * lo >> (k + 1)) continue;
            for (bool any : {false, true}) {
                V2Plan p;
                p.tile = part_tile(key_bits / 8, any);
                p.n = n;
                p.V = hi;
                p.k = k;
                plan_passes(p);
                // (the numbers of chunks, whose lengths are powers of two, do not
                // grow with n: their bounds)
                const uint32_t S = 1u << p.b1;
                p.nchunks1 = p.ntiles1 < 256 ? p.ntiles1 : 256;
                if (p.tiers == 2)
                    p.nchunks2_ub = (p.ntiles2_ub < 5 * S ? p.ntiles2_ub : 5 * S) + S;
                const size_t b = layout_v2(nullptr, p, key_bits / 8, nullptr);
                most = b > most ? b : most;
            }
        }
    }
    return most;
}

template <typename Key>
hipError_t run_build_v2(const Key* keys, uint64_t n, uint64_t V, uint64_t seed, uint32_t* offsets,
                        uint32_t* ids, Key* ekeys, IndexOut& ix, void* ws,
                        uint32_t bins_hint, bool stable, hipStream_t s) {
    HG_TRY(set_smem_limits<Key>());
    if (n == 0) {
        ix.fmt = index_fmt(0, V, sizeof(Key) * 8);
        if (ix.head) HG_TRY(fill_u32((uint32_t*)ix.head, ix.fmt.bytes / 4 * V, 0u, s));
        return fill_u32(offsets, V + 1, 0u, s);
    }
    const V2Plan p = plan_v2(n, V, sizeof(Key) * 8, bins_hint, !stable);
    ix.fmt = index_fmt(n, V, sizeof(Key) * 8);
    ix.hp = make_hash_params(V, seed);
    V2Ws w;
    layout_v2(ws, p, sizeof(Key), &w);
    ix.gen_list = w.gen_list;
    ix.gen_cnt = w.gen_cnt;
    ix.gen_any = w.ctr + kCtrListed;
    auto hp = KeyTraits<Key>::make(V, seed);
    Key* rkeys = (Key*)w.rkeys;
    hipError_t e = hipSuccess;
    if (p.bins == 1 && n <= light_cap<Key>()) {
        // the whole table is one bin: one workgroup builds it from the input
        with_layout<Key>(!stable, ix, [&](auto any, auto width) {
            e = run_build_one<Key, decltype(any)::value, decltype(width)::value>(
                keys, n, p.k, (uint32_t)V, offsets, ids, ekeys, hp, ix, w.bin_start, rkeys, w.rids,
                w.runs_ws, s);
        });
        return e;
    }
    // the last pass's scan also leaves the final bins' starts and the lists of
    // the oversize ones, the first of two passes the second's segments
    SegsOut bins;
    bins.bin_start = w.bin_start;
    bins.bins = p.bins;
    bins.n = (uint32_t)n;
    bins.V = (uint32_t)V;
    bins.light_keys = light_cap<Key>();
    bins.slice = slice_keys(n);
    bins.offsets = offsets;
    bins.heavy_list = w.heavy_list;
    bins.ctr = w.ctr;
    bins.huge_list = w.huge_list;
    bins.huge_s0 = w.huge_s0;
    bins.slice_owner = w.slice_owner;
    bins.huge_cap = w.huge_cap;
    bins.slice_cap = w.slice_cap;
    if (p.tiers == 1) {
        bins.zero = w.ctr;
        HG_TRY(partition_pass<Key>(keys, nullptr, rkeys, w.rids, w.s1, hp, p.k, p.b1, w.m1, w.c1,
                                   p.ntiles1, p.nchunks1, 1, stable, s, false, bins));
    } else {
        // tier 1 into the table's own arrays, tier 2 into the workspace
        SegsOut first;
        first.zero = w.ctr;
        first.next = w.s2;
        HG_TRY(partition_pass<Key>(keys, nullptr, ekeys, ids, w.s1, hp, p.k + p.b2, p.b1, w.m1,
                                   w.c1, p.ntiles1, p.nchunks1, 1, stable, s, false, first));
        HG_TRY(partition_pass<Key>(ekeys, ids, rkeys, w.rids, w.s2, hp, p.k, p.b2, w.m2, w.c2,
                                   p.ntiles2_ub, p.nchunks2_ub, 2, stable, s, false, bins));
    }
    {
        HG_PROF("v2_local_build", s);
        with_layout<Key>(!stable, ix, [&](auto any, auto width) {
            hipLaunchKernelGGL((k_local_light<Key, decltype(any)::value, decltype(width)::value>),
                               dim3(p.bins), dim3(kLocalThreads),
                               ix.head ? light_smem_index<Key>(p.k) : light_smem<Key>(p.k), s,
                               (const Key*)rkeys, (const uint32_t*)w.rids,
                               (const uint32_t*)w.bin_start, hp, p.k, offsets, ix, ids, ekeys);
        });
    }
    HG_TRY(hipGetLastError());
    const RareArgs a{w.bin_start, w.heavy_list, w.huge_list, w.huge_s0, w.slice_owner,
                     w.slice_hist, w.range_sum, w.ctr, w.huge_cap, w.slice_cap, slice_keys(n),
                     p.k, p.bins, (uint32_t)V, stable ? 0u : 1u};
    return run_rare<Key>(a, offsets, ids, ekeys, n, hp, ix, rkeys, w.rids, w.runs_ws, s);
}

// ------------------------------------------------ scatter by a permutation --
//
// out[ids[p]] = vals[p] for p < n, where ids holds every index of [0, n)
// once (a table's edge ids): Alg. 3's counts, found in B's edge order, put
// back in B's input order.  One random 4-byte store per entry would leave
// partial lines beyond the L2; instead the (value, id) pairs go through the
// same stable partition passes as a V2 build, with the digits taken from the
// id instead of a key's bucket, down to bins of 4096 consecutive ids, and
// each bin is placed in LDS and written out with coalesced stores.

namespace {

V2Plan perm_plan(uint64_t n) {
    // the ids are the "buckets": V = n, bins of 2^12 ids
    return plan_v2(n, n, 32, (uint32_t)ceil_div(n, 1ull << kMaxLocalBits), true);
}

size_t perm_layout(void* ws, const V2Plan& p, V2Ws* w, uint32_t** xv, uint32_t** xi) {
    Carver c(ws);
    layout_passes(c, p, 4, *w);
    *xv = c.take<uint32_t>(p.n);
    *xi = c.take<uint32_t>(p.n);
    return c.off + 256;
}

}  // namespace

size_t scatter_perm_ws_bytes(uint64_t n) {
    if (n <= kPermDirectMax) return 256;
    V2Ws w{};
    uint32_t *xv, *xi;
    return perm_layout(nullptr, perm_plan(n), &w, &xv, &xi);
}

hipError_t scatter_perm(const uint32_t* ids, const uint32_t* vals, uint64_t n, uint32_t* out,
                        void* ws, hipStream_t s) {
    if (n == 0) return hipSuccess;
    if (n <= kPermDirectMax) {
        HG_PROF("scatter_direct", s);
        const uint64_t g = ceil_div(n, 256 * 4);
        hipLaunchKernelGGL(k_perm_direct, dim3((uint32_t)(g > 4096 ? 4096 : g)), dim3(256), 0, s,
                           ids, vals, n, out);
        return hipGetLastError();
    }
    HG_TRY(set_smem_limits<uint32_t>());
    const V2Plan p = perm_plan(n);
    V2Ws w{};
    uint32_t *xv, *xi;
    perm_layout(ws, p, &w, &xv, &xi);
    const auto hp = KeyTraits<uint32_t>::make(1, 0);  // unused: digits come from the ids
    uint32_t* rv = (uint32_t*)w.rkeys;
    if (p.tiers == 1) {
        HG_TRY(partition_pass<uint32_t>(vals, ids, rv, w.rids, w.s1, hp, p.k, p.b1, w.m1, w.c1,
                                        p.ntiles1, p.nchunks1, 1, false, s, true));
    } else {
        SegsOut first;
        first.next = w.s2;
        HG_TRY(partition_pass<uint32_t>(vals, ids, xv, xi, w.s1, hp, p.k + p.b2, p.b1, w.m1,
                                        w.c1, p.ntiles1, p.nchunks1, 1, false, s, true, first));
        HG_TRY(partition_pass<uint32_t>(xv, xi, rv, w.rids, w.s2, hp, p.k, p.b2, w.m2, w.c2,
                                        p.ntiles2_ub, p.nchunks2_ub, 2, false, s, true));
    }
    {
        HG_PROF("scatter_place", s);
        hipLaunchKernelGGL(k_perm_place, dim3(p.bins), dim3(512), 0, s, (const uint32_t*)rv,
                           (const uint32_t*)w.rids, n, p.k, out);
    }
    return hipGetLastError();
}

// --------------------------------------------- grouped Probe-Standard ---
// The queries are first partitioned into up to 2^kGroupBits ranges of
// buckets with their input places (one tile-histogram, column-scan and
// partition pass, as in the build), probed in that order with the tiles
// dealt out per XCD -- each XCD then reads one window of the index at a time
// (2 MiB at 2^28 buckets of 4-byte entries), which its L2 holds, instead of random lines of
// the whole index -- and the counts are put back in input order by
// k_ungroup_by_pos.

namespace {

struct GroupPlan {
    uint32_t bits, shift, tile, ntiles, ch, nchunks;
};

GroupPlan group_plan(uint64_t m, uint64_t V, size_t key_size) {
    GroupPlan p;
    p.tile = part_tile(key_size, true);
    const uint32_t kv = log2_ceil(V);
    p.bits = kv < kGroupBits ? (kv ? kv : 1u) : kGroupBits;  // at least two ranges
    p.shift = kv > p.bits ? kv - p.bits : 0u;
    p.ntiles = (uint32_t)ceil_div(m, p.tile);
    p.ch = (uint32_t)pow2_ceil(ceil_div(p.ntiles ? p.ntiles : 1, 256));
    p.nchunks = (uint32_t)ceil_div(p.ntiles, p.ch);
    return p;
}

struct GroupWs {
    void* gq;        // the queries in grouped order
    uint16_t* place; // their places among kUngroupSpan queries of the input
    uint8_t* gc;     // their counts in grouped order; 255: see wide
    uint32_t* wide;  // the counts from 255 on
    uint32_t *mat, *csum, *ctr;
    Segs seg;
};

size_t layout_group(void* ws, const GroupPlan& p, uint64_t m, size_t key_size, GroupWs* out) {
    Carver c(ws);
    GroupWs w{};
    const uint32_t D = 1u << p.bits;
    w.gq = c.take<char>(m * key_size);
    w.place = c.take<uint16_t>(m);
    w.gc = c.take<uint8_t>(m);
    w.wide = c.take<uint32_t>(m);
    w.mat = c.take<uint32_t>((size_t)p.ntiles * D);
    w.csum = c.take<uint32_t>((size_t)p.nchunks * D);
    w.ctr = c.take<uint32_t>(kCtrWords);
    w.seg.seg_start = c.take<uint32_t>(2);
    w.seg.tile_prefix = c.take<uint32_t>(2);
    w.seg.chunk_prefix = c.take<uint32_t>(2);
    w.seg.S = 1;
    w.seg.ch = p.ch;
    w.seg.tile = p.tile;
    if (out) *out = w;
    return c.off + 256;
}

}  // namespace

size_t probe_grouped_ws_bytes(uint64_t m, uint64_t V, size_t key_size) {
    return layout_group(nullptr, group_plan(m, V, key_size), m, key_size, nullptr);
}

template <typename Key>
hipError_t run_probe_grouped(const TableDev& t, const Key* queries, uint64_t m, uint32_t* counts,
                             unsigned long long* d_total, void* ws, hipStream_t s, bool decide) {
    if (m == 0) return run_probe_counts<Key>(t, queries, m, counts, d_total, s);
    HG_TRY(set_smem_limits<Key>());
    const GroupPlan p = group_plan(m, t.V, sizeof(Key));
    GroupWs w;
    layout_group(ws, p, m, sizeof(Key), &w);
    const auto hp = KeyTraits<Key>::make(t.V, t.seed);
    const uint32_t* gate = decide ? w.ctr : nullptr;  // ctr[0]: 1 grouped, 0 input order
    if (decide) {
        hipLaunchKernelGGL(k_group_sample<Key>, dim3(1), dim3(1024), 0, s, queries, m, hp,
                           p.shift, p.bits, w.seg, p.ntiles, p.nchunks,
                           group_local_eighths(t.V), w.ctr);
        HG_TRY(hipGetLastError());
    } else {
        w.seg = one_segment(m, p.ntiles, p.nchunks, p.ch, p.tile);
    }
    Key* gq = (Key*)w.gq;
    // places only when the counts go back to input order
    HG_TRY(partition_pass<Key>(queries, nullptr, gq, counts ? (uint32_t*)w.place : nullptr, w.seg, hp,
                               p.shift, p.bits, w.mat, w.csum, p.ntiles, p.nchunks, 3, false, s));
    // one probe launch: the grouped queries, or (gate 0) the queries in input
    // order straight into counts
    HG_TRY(run_probe_counts<Key>(t, gq, m, counts ? w.wide : nullptr, d_total, s, nullptr, true,
                                 gate, queries, counts, w.gc));
    if (!counts) return hipSuccess;
    {
        HG_PROF("probe_ungroup", s);
        const uint32_t groups = (uint32_t)ceil_div(p.ntiles, kUngroupSpan / p.tile);
        const uint32_t grid = (uint32_t)(8 * ceil_div(groups, 8));
        hipLaunchKernelGGL(k_ungroup_by_pos, dim3(grid), dim3(kUngroupThreads), 0, s, m, p.ntiles,
                           p.tile, p.bits, (const uint32_t*)w.mat, groups, (const uint16_t*)w.place, (const uint8_t*)w.gc,
                           (const uint32_t*)w.wide, counts, gate);
    }
    return hipGetLastError();
}

template hipError_t run_probe_grouped<uint32_t>(const TableDev&, const uint32_t*, uint64_t,
                                                uint32_t*, unsigned long long*, void*,
                                                hipStream_t, bool);
template hipError_t run_probe_grouped<uint64_t>(const TableDev&, const uint64_t*, uint64_t,
                                                uint32_t*, unsigned long long*, void*,
                                                hipStream_t, bool);

template hipError_t run_build_v2<uint32_t>(const uint32_t*, uint64_t, uint64_t, uint64_t,
                                           uint32_t*, uint32_t*, uint32_t*, IndexOut&, void*,
                                           uint32_t, bool, hipStream_t);
template hipError_t run_build_v2<uint64_t>(const uint64_t*, uint64_t, uint64_t, uint64_t,
                                           uint32_t*, uint32_t*, uint64_t*, IndexOut&, void*,
                                           uint32_t, bool, hipStream_t);

}  // namespace hg
