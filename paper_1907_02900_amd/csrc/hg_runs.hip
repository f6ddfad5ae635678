// The rare path of a V2 build: bins too large for LDS, and the key-run
// summaries of the long buckets that the per-bin kernel left.
//
// Oversize bins.  A bin of at most `slice` keys is one workgroup's work
// (heavy_bin_body).  Larger ones (a hot key) are cut into slices: per-slice
// bucket histograms, their scan over the slices, and a placement per slice.
//
// Key runs.  Probe-Standard (Sec. 3.4) scans a query's whole bucket.  When many
// entries share a bucket -- heavy duplication, or Zipf keys where one key holds
// a large share of the input -- every probe of that bucket pays its full
// length, so a skewed join costs as much as the number of matching pairs.
// For each bucket longer than kRunBucket the table therefore also keeps the
// bucket's distinct keys in ascending order (its runs), each with the end of
// its group in `kperm`, a copy of the bucket's ids grouped by key (bucket
// order inside each group).  A probe of a long bucket binary-searches the
// runs; its pairs are the ids of one group.  Counts and pairs are exactly
// those of a scan.  The arrays are parallel to the edge array (see RunsDev),
// so every bucket's summary has a fixed place and nothing is sized on the
// host: a build with the index never waits for the device.
// Most long buckets are built inside the per-bin kernel, from LDS
// (bin_long_runs): a long bucket is usually one key repeated (duplicates) or
// dominated by one key (skew), so the entries equal to the bucket's first key
// (the lead key) form one run and the few others are sorted across a wave.
// The rest, which the per-bin kernels list per bin:
//   * buckets of up to light_cap keys (k_listed_runs, in LDS): the
//     others are gathered, sorted (bitonic network in LDS) and cut into runs;
//   * longer buckets (from bins too large for LDS), in chunks of kChunk
//     entries spread over the grid: per chunk the others and those below the
//     lead key are counted, a per-bucket scan turns the counts into chunk
//     bases, each chunk then writes its others contiguously to scratch and its
//     lead ids to kperm, and one workgroup per bucket sorts the others (LDS,
//     or a workgroup-wide radix sort through global memory when they exceed
//     LDS) and writes their runs.
//
// Uniform keys need none of it, but every build pays for the launches (2 to 4 us
// each): one kernel for builds of up to 2^17 keys, which split no bin (their
// rare workgroups see each long bucket through alone), eight or, from 2^24 keys,
// nine for larger ones; they were six and twelve.
#include "hg_v2_device.h"

namespace hg {

namespace {

using namespace v2dev;

constexpr int kRT = kLocalThreads;      // threads of the per-bucket kernels (512)
constexpr int kCItems = 8;              // entries per thread of a chunk
constexpr uint32_t kChunk = kRT * kCItems;  // 4096
constexpr uint32_t kRareGrid = 512;     // two workgroups per CU (LDS)
constexpr uint32_t kListedGrid = 2048;
constexpr uint32_t kRangeBits = 8;      // buckets of one workgroup of the slice scan
constexpr uint32_t kRanges = 1u << (kMaxLocalBits - kRangeBits);  // at most, per bin

// Entries the LDS sort of a bucket's other keys holds: light_cap rounded up
// to a power of two (8192 for 32-bit keys, 4096 for 64-bit keys).
template <typename Key>
constexpr uint32_t lds_sort_cap() {
    return sizeof(Key) == 8 ? 4096u : 8192u;
}

// Buckets longer than light_cap go through the chunked path.
template <typename Key>
constexpr uint32_t small_cap() {
    return light_cap<Key>();
}

// LDS of the per-bucket kernels: sort buffer, radix counters, scan temporaries.
template <typename Key>
struct BucketLds {
    Key* sk;          // [lds_sort_cap]
    uint32_t* sp;     // [lds_sort_cap]
    uint32_t* wcnt;   // [W_LOCAL * 256]
    uint32_t* dstart; // [256]
    uint32_t* base;   // [256]
    uint32_t* tmp;    // [2 * W_LOCAL + 2]
    uint32_t* sh;     // [8] broadcast words
    __host__ __device__ static constexpr size_t bytes() {
        return (size_t)lds_sort_cap<Key>() * (sizeof(Key) + 4) + 4 * (W_LOCAL * 256 + 256 + 256 +
                                                                     2 * W_LOCAL + 2 + 8) + 64;
    }
    __device__ explicit BucketLds(unsigned char* p) {
        sk = (Key*)p;
        sp = (uint32_t*)(sk + lds_sort_cap<Key>());
        wcnt = sp + lds_sort_cap<Key>();
        dstart = wcnt + W_LOCAL * 256;
        base = dstart + 256;
        tmp = base + 256;
        sh = tmp + 2 * W_LOCAL + 2;
    }
};

// Bitonic sort of n2 (a power of two) (key, position) pairs in LDS,
// ascending; positions are distinct, so the order is total.  Barriers.
template <typename Key>
__device__ void lds_bitonic(Key* k, uint32_t* p, uint32_t n2) {
    for (uint32_t size = 2; size <= n2; size <<= 1)
        for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
            for (uint32_t i = threadIdx.x; i < n2 / 2; i += kRT) {
                const uint32_t lo = 2 * stride * (i / stride) + (i % stride), hi = lo + stride;
                const bool up = (lo & size) == 0;
                const Key ka = k[lo], kb = k[hi];
                const uint32_t pa = p[lo], pb = p[hi];
                const bool b_less = kb < ka || (kb == ka && pb < pa);
                if (b_less == up) {
                    k[lo] = kb;
                    k[hi] = ka;
                    p[lo] = pb;
                    p[hi] = pa;
                }
            }
            __syncthreads();
        }
}

// Stable LSD radix sort (8-bit digits, every bit of the key) of O pairs
// through global memory by one workgroup: (ka, pa) -> (kb, pb) -> ... The
// number of passes is even, so the result ends in (ka, pa).  Barriers.
template <typename Key>
__device__ void wg_radix_sort(Key* ka, uint32_t* pa, Key* kb, uint32_t* pb, uint32_t O,
                              const BucketLds<Key>& m) {
    constexpr int IT = 8;
    constexpr uint32_t tile = kRT * IT;
    const uint32_t w = threadIdx.x / kWave, lane = lane_id();
    for (uint32_t shift = 0; shift < sizeof(Key) * 8; shift += 8) {
        for (uint32_t d = threadIdx.x; d < 256; d += kRT) m.base[d] = 0;
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < O; i += kRT)
            atomicAdd(&m.base[(uint32_t)(ka[i] >> shift) & 255u], 1u);
        __syncthreads();
        uint32_t all;
        const uint32_t v = threadIdx.x < 256 ? m.base[threadIdx.x] : 0u;
        const uint32_t ex = block_excl_scan<kRT>(v, m.tmp, &all);
        if (threadIdx.x < 256) m.base[threadIdx.x] = ex;
        __syncthreads();
        for (uint32_t t0 = 0; t0 < O; t0 += tile) {
            const uint32_t cnt = O - t0 < tile ? O - t0 : tile;
            Key k[IT];
            uint32_t p[IT], dig[IT], pos[IT];
#pragma unroll
            for (int r = 0; r < IT; ++r) {
                const uint32_t e = w * (kWave * IT) + r * kWave + lane;
                if (e < cnt) {
                    k[r] = ka[t0 + e];
                    p[r] = pa[t0 + e];
                    dig[r] = (uint32_t)(k[r] >> shift) & 255u;
                } else {
                    k[r] = 0;
                    p[r] = 0;
                    dig[r] = 256u;  // ignored by the ranking
                }
            }
            rank_stable<kRT, IT>(dig, 8, m.wcnt, m.dstart, m.tmp, pos);
#pragma unroll
            for (int r = 0; r < IT; ++r)
                if (dig[r] < 256u) {
                    const uint32_t o = m.base[dig[r]] + pos[r] - m.dstart[dig[r]];
                    kb[o] = k[r];
                    pb[o] = p[r];
                }
            __syncthreads();
            for (uint32_t d = threadIdx.x; d < 256; d += kRT)
                m.base[d] += (d + 1 < 256 ? m.dstart[d + 1] : cnt) - m.dstart[d];
            __syncthreads();
        }
        Key* tk = ka;
        ka = kb;
        kb = tk;
        uint32_t* tp = pa;
        pa = pb;
        pb = tp;
    }
}

// Runs of a long bucket (edge positions [st, st + len), lead key `lead`) from
// its O > 0 other entries sorted by (key, position in the bucket) in sk / sp:
// every other entry's id goes to kperm (before the lead key's group when its
// key is smaller, after it otherwise), every run gets its key and end, the
// lead run is slotted in, and the bucket's index entry points at the runs.
// The lead key's ids are written by the caller.  Returns (via m.sh[0]) the
// number of others below the lead key.  Whole workgroup; barriers.
template <typename Key>
__device__ __forceinline__ void emit_runs(const Key* sk, const uint32_t* sp, uint32_t O, Key lead, uint32_t len,
                          uint32_t st, uint32_t b, const uint32_t* ids,
                          const IndexOut& ix, const BucketLds<Key>& m) {
    Key* rkey = (Key*)ix.runs.run_key;
    uint32_t* rend = ix.runs.run_end;
    uint32_t* kperm = ix.runs.kperm;
    if (threadIdx.x == 0) {
        uint32_t lo = 0, hi = O;  // others below the lead key
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (sk[mid] < lead) lo = mid + 1;
            else hi = mid;
        }
        m.sh[0] = lo;
        m.sh[1] = 0;  // runs below the lead key
    }
    __syncthreads();
    const uint32_t nless = m.sh[0], clead = len - O;
    uint32_t runs = 0;  // other runs before this tile
    for (uint32_t t0 = 0; t0 < O; t0 += kRT) {
        const uint32_t i = t0 + threadIdx.x;
        const bool valid = i < O;
        const Key k = valid ? sk[i] : (Key)0;
        const bool first = valid && (i == 0 || sk[i - 1] != k);
        const bool last = valid && (i + 1 == O || sk[i + 1] != k);
        uint32_t all;
        const uint32_t ex = block_excl_scan<kRT>(first ? 1u : 0u, m.tmp, &all);
        if (valid) {
            const bool below = i < nless;
            const uint32_t ro = runs + ex + (first ? 1u : 0u) - 1u;  // run among the others
            const uint32_t r = ro + (below ? 0u : 1u);
            kperm[st + i + (below ? 0u : clead)] = ids[st + sp[i]];
            if (first) rkey[st + r] = k;
            if (last) rend[st + r] = i + 1 + (below ? 0u : clead);
            if (i + 1 == nless) m.sh[1] = ro + 1;
        }
        runs += all;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t rl = m.sh[1];
        rkey[st + rl] = lead;
        rend[st + rl] = nless + clead;
        put_long<Key>(ix, b, len, st, runs + 1, lead, clead);
    }
    __syncthreads();
}

// A bucket of one key: a single run, no kperm (its ids are the edge array's).
template <typename Key>
__device__ __forceinline__ void single_run(const IndexOut& ix, uint32_t b, uint32_t st,
                                           uint32_t len, Key lead) {
    ((Key*)ix.runs.run_key)[st] = lead;
    ix.runs.run_end[st] = len;
    put_long<Key>(ix, b, len, st, 1u, lead, len);
}

struct G2 {
    uint32_t* list;    // [cap] bucket ids
    uint32_t* c0;      // [cap] first chunk
    uint32_t* info;    // [2 * cap] others, others below the lead key
    uint32_t* owner;   // [chunks] bucket (index in list) of each chunk
    uint32_t* oth;     // [chunks] others, then their exclusive prefix in the bucket
    uint32_t* less;    // [chunks] others below the lead key, then their prefix
    uint32_t cap, chunk_cap;
};

struct G2Layout {
    G2 g;
    size_t bytes;
};

G2Layout layout_g2(void* ws, uint64_t n) {
    Carver c(ws);
    G2 g{};
    g.cap = (uint32_t)(n / (light_cap<uint64_t>() + 1) + 1);
    g.chunk_cap = (uint32_t)(n / kChunk + g.cap + 1);
    g.list = c.take<uint32_t>(g.cap);
    g.c0 = c.take<uint32_t>(g.cap);
    g.info = c.take<uint32_t>(2 * (size_t)g.cap);
    g.owner = c.take<uint32_t>(g.chunk_cap);
    g.oth = c.take<uint32_t>(g.chunk_cap);
    g.less = c.take<uint32_t>(g.chunk_cap);
    return G2Layout{g, c.off + 256};
}

// Everything the kernels read and write.
template <typename Key>
struct Rare {
    RareArgs a;
    uint32_t* offsets;
    uint32_t* ids;
    Key* ekeys;
    typename KeyTraits<Key>::Params hp;
    IndexOut ix;
    const Key* src_keys;  // the reorganised entries
    const uint32_t* src_ids;
    Key* skey;            // the same arrays as scratch, once all bins are placed
    uint32_t* spos;
    G2 g2;
};

// End of bucket b of bin g.  (While another workgroup may still be writing the
// next bin's offsets, the bin's own end stands for them.)
template <typename Key>
__device__ __forceinline__ uint32_t bucket_end(const Rare<Key>& x, uint32_t g, uint32_t b) {
    const bool last = ((b + 1) & ((1u << x.a.k) - 1u)) == 0 || b + 1 == x.a.V;
    return last ? x.a.bin_start[g + 1] : x.offsets[b + 1];
}

// Slice `item` of a split bin: its bin and key range.
struct SliceRef {
    uint32_t b, begin, end;
};

__device__ __forceinline__ SliceRef slice_at(const RareArgs& a, uint32_t item) {
    SliceRef r;
    const uint32_t idx = a.slice_owner[item];
    r.b = a.huge_list[idx];
    const uint32_t bs = a.bin_start[r.b], be = a.bin_start[r.b + 1];
    r.begin = bs + (item - a.huge_s0[idx]) * a.slice;
    r.end = (be - r.begin > a.slice) ? r.begin + a.slice : be;
    return r;
}

// Slices of split bin idx.
__device__ __forceinline__ uint32_t slices_of(const RareArgs& a, uint32_t idx) {
    const uint32_t b = a.huge_list[idx];
    return (a.bin_start[b + 1] - a.bin_start[b] + a.slice - 1) / a.slice;
}

// What the first kernel of the rare path does: the oversize bins of a build
// without split ones (whose only kernel it is), or also the split bins' slices, or
// not (k_slice_hist).
enum RareMode : int { kSolo, kBinsAndSlices, kBins };

// An oversize bin, one workgroup.  U: loads in flight (count_hot_buckets).
template <typename Key, bool ANY, int U>
__device__ __forceinline__ void heavy_bin(const Rare<Key>& x, uint32_t i, unsigned char* smem) {
    const RareArgs& a = x.a;
    const uint32_t g = a.heavy_list[i];
    const uint32_t start = a.bin_start[g], end = a.bin_start[g + 1];
    const uint32_t NB = 1u << a.k, v0 = g << a.k;
    const uint32_t nb = (a.V - v0 < NB) ? a.V - v0 : NB;
    heavy_bin_body<Key, U>(x.src_keys + start, x.src_ids + start, 0u, end - start, start, v0, a.k,
                           nb, x.hp, x.offsets, x.ix, x.ids, x.ekeys, smem, ANY);
}

// Bucket histogram of a slice of a split bin: hist[item][0 .. 2^k).
template <typename Key, int U>
__device__ __forceinline__ void slice_hist(const Rare<Key>& x, uint32_t item, unsigned char* smem) {
    const RareArgs& a = x.a;
    uint32_t* cnt = (uint32_t*)smem;
    const uint32_t NB = 1u << a.k;
    const SliceRef r = slice_at(a, item);
    const uint32_t v0 = r.b << a.k;
    for (uint32_t i = threadIdx.x; i < NB; i += kRT) cnt[i] = 0;
    __syncthreads();
    count_hot_buckets<Key, U>(x.src_keys + r.begin, r.end - r.begin, v0, x.hp, cnt);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < NB; i += kRT)
        a.slice_hist[(size_t)item * NB + i] = cnt[i];
    // its sums over ranges of 2^kRangeBits buckets, a wave per range
    const uint32_t lane = lane_id();
    for (uint32_t q = threadIdx.x / kWave; q << kRangeBits < NB; q += W_LOCAL) {
        uint32_t sum = 0;
#pragma unroll
        for (uint32_t j = 0; j < (1u << kRangeBits) / kWave; ++j) {
            const uint32_t v = (q << kRangeBits) + j * kWave + lane;
            sum += v < NB ? cnt[v] : 0u;
        }
        sum = wave_sum(sum);
        if (lane == 0) a.range_sum[(size_t)item * kRanges + q] = sum;
    }
}

// Placement of a slice from its cursors.
template <typename Key, bool ANY>
__device__ __forceinline__ void place_slice(const Rare<Key>& x, uint32_t item,
                                            unsigned char* smem) {
    const RareArgs& a = x.a;
    const uint32_t NB = 1u << a.k;
    const HeavyLds<Key> m(smem, NB);
    const SliceRef r = slice_at(a, item);
    for (uint32_t i = threadIdx.x; i < NB; i += kRT)
        m.cur[i] = a.slice_hist[(size_t)item * NB + i];
    __syncthreads();
    place_in_chunks<Key>(x.src_keys + r.begin, x.src_ids + r.begin, 0u, r.end - r.begin,
                         a.bin_start[r.b], a.bin_start[r.b + 1], r.b << a.k, a.k, x.hp, x.ids,
                         x.ekeys, smem, ANY);
}

// Probe index entries of a split bin's buckets (after their placement); the
// long ones are listed.
template <typename Key>
__device__ __forceinline__ void split_index(const Rare<Key>& x, uint32_t idx,
                                            unsigned char* smem) {
    const RareArgs& a = x.a;
    uint32_t* nlisted = (uint32_t*)smem;
    const uint32_t NB = 1u << a.k;
    const uint32_t b = a.huge_list[idx];
    const uint32_t v0 = b << a.k, nb = (a.V - v0 < NB) ? a.V - v0 : NB;
    const uint32_t bs = a.bin_start[b], be = a.bin_start[b + 1];
    if (threadIdx.x == 0) *nlisted = 0;
    __syncthreads();
    for (uint32_t v = threadIdx.x; v < nb; v += kRT) {
        const uint32_t lo = x.offsets[v0 + v];
        const uint32_t hi = (v + 1 < nb) ? x.offsets[v0 + v + 1] : be;
        if (hi - lo > kRunBucket)
            x.ix.gen_list[gen_region(bs, b) + atomicAdd(nlisted, 1u)] = v0 + v;
        else
            put_short<Key>(x.ix, v0 + v, lo, hi, x.ekeys + lo);
    }
    __syncthreads();
    if (threadIdx.x == 0) x.ix.gen_cnt[b] = *nlisted;
    __syncthreads();
}

// Chunk c of a long bucket: wave w holds entries [w*512, w*512 + 512) of it,
// lane l those at w*512 + j*64 + l, j < kCItems.
struct ChunkRef {
    uint32_t i, b, st, base, cl;
};

__device__ __forceinline__ ChunkRef chunk_at(uint32_t c, const G2& g2, const uint32_t* offsets) {
    ChunkRef r;
    r.i = g2.owner[c];
    r.b = g2.list[r.i];
    r.st = offsets[r.b];
    const uint32_t len = offsets[r.b + 1] - r.st;
    r.base = (c - g2.c0[r.i]) * kChunk;
    r.cl = len - r.base < kChunk ? len - r.base : kChunk;
    return r;
}

template <typename Key>
__device__ __forceinline__ void load_chunk(const ChunkRef& r, const Key* ekeys, Key lead,
                                           Key (&k)[kCItems]) {
    const uint32_t e0 = (threadIdx.x / kWave) * (kCItems * kWave) + lane_id();
#pragma unroll
    for (int j = 0; j < kCItems; ++j)
        k[j] = e0 + j * kWave < r.cl ? ekeys[r.st + r.base + e0 + j * kWave] : lead;
}

// Entries of a chunk that differ from the lead key (o) and of them those below
// it (l): the workgroup's sums, to every thread.  red: 2 * W_LOCAL words of LDS.
// Barriers.
template <typename Key>
__device__ __forceinline__ void count_chunk(const Key (&k)[kCItems], Key lead, uint32_t* red,
                                            uint32_t& o, uint32_t& l) {
    o = l = 0;
#pragma unroll
    for (int j = 0; j < kCItems; ++j) {
        o += k[j] != lead;
        l += k[j] < lead;
    }
    o = wave_sum(o);
    l = wave_sum(l);
    __syncthreads();
    if (lane_id() == 0) {
        red[threadIdx.x / kWave] = o;
        red[W_LOCAL + threadIdx.x / kWave] = l;
    }
    __syncthreads();
    o = l = 0;
    for (int q = 0; q < W_LOCAL; ++q) {
        o += red[q];
        l += red[W_LOCAL + q];
    }
}

// Writes a chunk's others contiguously to the scratch arrays (key, position in
// the bucket) from obase on, and the lead key's ids to kperm after the nless
// smaller keys' ids.  red: W_LOCAL words of LDS.  Barriers.
template <typename Key>
__device__ __forceinline__ void scatter_chunk(const Rare<Key>& x, const ChunkRef& r,
                                              const Key (&k)[kCItems], Key lead, uint32_t obase,
                                              uint32_t nless, uint32_t* red) {
    const uint32_t w = threadIdx.x / kWave;
    const uint32_t e0 = w * (kCItems * kWave) + lane_id();
    uint32_t mine = 0;
#pragma unroll
    for (int j = 0; j < kCItems; ++j) mine += (uint32_t)__popcll(ballot(k[j] != lead));
    __syncthreads();
    if (lane_id() == 0) red[w] = mine;
    __syncthreads();
    uint32_t o = obase;  // others before the wave's next round
    for (uint32_t q = 0; q < w; ++q) o += red[q];
    uint32_t l = r.base + w * (kCItems * kWave) - o;  // lead entries before it
#pragma unroll
    for (int j = 0; j < kCItems; ++j) {
        const uint32_t e = e0 + j * kWave;
        const uint64_t ob = ballot(k[j] != lead), lb = ballot(e < r.cl && k[j] == lead);
        if (k[j] != lead) {
            x.skey[r.st + o + mbcnt(ob)] = k[j];
            x.spos[r.st + o + mbcnt(ob)] = r.base + e;
        } else if (e < r.cl) {
            x.ix.runs.kperm[r.st + nless + l + mbcnt(lb)] = x.ids[r.st + r.base + e];
        }
        o += (uint32_t)__popcll(ob);
        l += (uint32_t)__popcll(lb);
    }
}

// Sorts a long bucket's O > 0 others in the scratch arrays (LDS when they fit,
// else a workgroup radix sort through global memory) and writes its runs.
template <typename Key>
__device__ __forceinline__ void sort_others(const Rare<Key>& x, uint32_t b, uint32_t st,
                                            uint32_t len, uint32_t O, const BucketLds<Key>& m) {
    const Key lead = x.ekeys[st];
    if (O <= lds_sort_cap<Key>()) {
        uint32_t n2 = 1;
        while (n2 < O) n2 <<= 1;
        for (uint32_t t = threadIdx.x; t < n2; t += kRT) {
            m.sk[t] = t < O ? x.skey[st + t] : (Key)~(Key)0;
            m.sp[t] = t < O ? x.spos[st + t] : 0xffffffffu;
        }
        __syncthreads();
        lds_bitonic<Key>(m.sk, m.sp, n2);
        emit_runs<Key>(m.sk, m.sp, O, lead, len, st, b, x.ids, x.ix, m);
    } else {
        // the run arrays of [st, st + O) serve as the second buffer; the
        // sorted pairs end back in the scratch arrays
        wg_radix_sort<Key>(x.skey + st, x.spos + st, (Key*)x.ix.runs.run_key + st,
                           x.ix.runs.run_end + st, O, m);
        emit_runs<Key>(x.skey + st, x.spos + st, O, lead, len, st, b, x.ids, x.ix, m);
    }
}

// The runs of a bucket of any length by one workgroup (builds without split
// bins: at most 2^17 entries).  The scratch arrays' places of the bucket are
// its own bin's reorganised entries, placed by this workgroup before.
template <typename Key>
__device__ __forceinline__ void long_bucket(const Rare<Key>& x, uint32_t b, uint32_t st,
                                            uint32_t len, const BucketLds<Key>& m) {
    ChunkRef r{0, b, st, 0, 0};
    const Key lead = x.ekeys[r.st];
    Key k[kCItems];
    uint32_t O = 0, nless = 0;
    for (r.base = 0; r.base < len; r.base += kChunk) {
        r.cl = len - r.base < kChunk ? len - r.base : kChunk;
        load_chunk<Key>(r, x.ekeys, lead, k);
        uint32_t o, l;
        count_chunk<Key>(k, lead, m.tmp, o, l);
        O += o;
        nless += l;
    }
    if (O == 0) {
        if (threadIdx.x == 0) single_run<Key>(x.ix, b, r.st, len, lead);
        __syncthreads();
        return;
    }
    uint32_t before = 0;
    for (r.base = 0; r.base < len; r.base += kChunk) {
        r.cl = len - r.base < kChunk ? len - r.base : kChunk;
        load_chunk<Key>(r, x.ekeys, lead, k);
        uint32_t o, l;
        count_chunk<Key>(k, lead, m.tmp, o, l);
        scatter_chunk<Key>(x, r, k, lead, before, nless, m.tmp);
        before += o;
    }
    __syncthreads();
    sort_others<Key>(x, b, st, len, O, m);
    __syncthreads();
}

// The listed long buckets of one bin: first each wave finishes the buckets
// whose entries other than the lead key fit its lanes (marking them done in
// the list), then the workgroup sorts the other small ones in LDS; longer ones
// are handed to the chunked path (ctr[kCtrLong] buckets, ctr[kCtrChunks] chunks)
// or, SOLO, seen through by this workgroup.
template <typename Key, bool SOLO>
__device__ __forceinline__ void listed_of_bin(const Rare<Key>& x, uint32_t g, uint32_t listed,
                                              const BucketLds<Key>& m) {
    const IndexOut& ix = x.ix;
    const uint32_t* offsets = x.offsets;
    const uint32_t* ids = x.ids;
    const Key* ekeys = x.ekeys;
    uint32_t* ctr = x.a.ctr;
    const G2& g2 = x.g2;
    uint32_t* list = ix.gen_list + gen_region(x.a.bin_start[g], g);
    {
        // a wave per bucket, its 64-entry buffers in the sort buffers
        const uint32_t w = threadIdx.x / kWave, lane = lane_id();
        Key* bk = m.sk + w * kWave;
        uint16_t* bp = (uint16_t*)m.sp + w * kWave;
        for (uint32_t t = w; t < listed; t += W_LOCAL) {
            const uint32_t b = list[t];
            const uint32_t st = offsets[b], len = bucket_end(x, g, b) - st;
            // (a bucket much longer than a wave rarely has its other
            // keys fit one; it goes to the workgroup below directly)
            if (len > 4u * kWave) continue;
            if (wave_bucket_runs<Key>(ix, ekeys, ids, st, st + len, st, b, bk, bp) && lane == 0)
                list[t] = ~0u;  // done
        }
    }
    __syncthreads();
    for (uint32_t t = 0; t < listed; ++t) {
        const uint32_t b = list[t];
        if (b == ~0u) continue;  // uniform: finished by a wave above
        const uint32_t st = offsets[b], len = bucket_end(x, g, b) - st;
        const Key lead = ekeys[st];
        if (SOLO && len > small_cap<Key>()) {
            long_bucket<Key>(x, b, st, len, m);
            continue;
        }
        if (len > small_cap<Key>()) {
            const uint32_t nch = (len + kChunk - 1) / kChunk;
            if (threadIdx.x == 0) {
                const uint32_t i = atomicAdd(&ctr[kCtrLong], 1u);
                const uint32_t c0 = atomicAdd(&ctr[kCtrChunks], nch);
                m.sh[2] = i;
                m.sh[3] = c0;
                if (i < g2.cap && c0 + nch <= g2.chunk_cap) {
                    g2.list[i] = b;
                    g2.c0[i] = c0;
                }
            }
            __syncthreads();
            const uint32_t i = m.sh[2], c0 = m.sh[3];
            if (i < g2.cap && c0 + nch <= g2.chunk_cap)
                for (uint32_t j = threadIdx.x; j < nch; j += kRT) g2.owner[c0 + j] = i;
            __syncthreads();
            continue;
        }
        // gather the entries that differ from the lead key, in bucket order
        uint32_t O = 0;
        for (uint32_t c = 0; c < len; c += kRT) {
            const uint32_t i = c + threadIdx.x;
            const Key k = i < len ? ekeys[st + i] : lead;
            const bool o = k != lead;
            uint32_t all;
            const uint32_t ex = block_excl_scan<kRT>(o ? 1u : 0u, m.tmp, &all);
            if (o) {
                m.sk[O + ex] = k;
                m.sp[O + ex] = i;
            }
            O += all;
        }
        if (O == 0) {
            if (threadIdx.x == 0) single_run<Key>(ix, b, st, len, lead);
            __syncthreads();
            continue;
        }
        uint32_t n2 = 1;
        while (n2 < O) n2 <<= 1;
        for (uint32_t i = O + threadIdx.x; i < n2; i += kRT) {
            m.sk[i] = (Key)~(Key)0;
            m.sp[i] = 0xffffffffu;
        }
        __syncthreads();
        lds_bitonic<Key>(m.sk, m.sp, n2);
        emit_runs<Key>(m.sk, m.sp, O, lead, len, st, b, ids, ix, m);
        // the lead key's ids, in bucket order, after the smaller keys
        const uint32_t nless = m.sh[0];
        uint32_t done = 0;
        for (uint32_t c = 0; c < len; c += kRT) {
            const uint32_t i = c + threadIdx.x;
            const bool isl = i < len && ekeys[st + i] == lead;
            uint32_t all;
            const uint32_t ex = block_excl_scan<kRT>(isl ? 1u : 0u, m.tmp, &all);
            if (isl) ix.runs.kperm[st + nless + done + ex] = ids[st + i];
            done += all;
        }
        __syncthreads();
    }
}

// First kernel of the rare path: every oversize bin and, as MODE says, the split
// bins' slices or (SOLO) every bin's listed long buckets; nothing here depends on
// another workgroup.
// Bound by its longest oversize bin, one workgroup's chunks one after the other:
// 295 us at 2^26 Zipf(1.2) keys (bins of up to 2^15).  Slices of half that length
// took it to 202, but their histograms' scan and placement cost as much more.
template <typename Key, int MODE, bool ANY>
__global__ __launch_bounds__(kRT) void k_rare_bins(Rare<Key> x) {
    extern __shared__ __align__(16) unsigned char smem[];
    const RareArgs& a = x.a;
    const uint32_t nheavy = a.ctr[kCtrHeavy];
    uint32_t nsl = 0;
    if (MODE == kBinsAndSlices)
        nsl = a.ctr[kCtrSlices] < a.slice_cap ? a.ctr[kCtrSlices] : a.slice_cap;
    // (one load in flight keeps the kernel with the slices within 128 VGPRs)
    constexpr int U = MODE == kBinsAndSlices ? 1 : 8;
    for (uint32_t i = blockIdx.x; i < nheavy + nsl; i += gridDim.x) {
        if (i < nheavy) heavy_bin<Key, ANY, U>(x, i, smem);
        else slice_hist<Key, U>(x, i - nheavy, smem);
        __syncthreads();
    }
    if (MODE != kSolo || !x.ix.head) return;
    // the long buckets of this workgroup's oversize bins, and of the bins held
    // in LDS when one of them listed any (kCtrListed, which no workgroup of this
    // launch writes)
    const BucketLds<Key> m(smem);
    const uint32_t nlight = a.ctr[kCtrListed] ? a.bins : 0u;
    for (uint32_t i = blockIdx.x; i < nheavy + nlight; i += gridDim.x) {
        const uint32_t g = i < nheavy ? a.heavy_list[i] : i - nheavy;
        if (i >= nheavy && a.bin_start[g + 1] - a.bin_start[g] > light_cap<Key>()) continue;
        const uint32_t listed = x.ix.gen_cnt[g];
        if (listed) listed_of_bin<Key, true>(x, g, listed, m);
        __syncthreads();
    }
}

// The scan over the split bins' slice histograms: a workgroup takes 256 buckets
// of a bin, four groups of slices side by side.  Buckets start after the bin's
// lower ranges, whose sums per slice the histogram pass left; every count turns
// into the position of its slice's first entry of the bucket.
constexpr int kScanThreads = 1024;

// The histograms of the split bins' slices in a kernel of their own, so that four
// workgroups share a CU: with the oversize bins, which take 128 VGPRs and 50 KB of
// LDS, the two ran 449 us at 2^26 Zipf(1.2) keys, apart 295 and 71.  Builds below
// kSliceHistMin keys keep them in one kernel, where the launch costs more: whole builds
// of Zipf(1.2) keys in one : in two, 2^22 372 : 376 us, 2^23 465 : 470, 2^24 737 : 724,
// 2^26 2399 : 2289 (uniform keys 2^22 132 : 135, 2^24 335 : 336).
constexpr uint64_t kSliceHistMin = 1ull << 24;

template <typename Key>
__global__ __launch_bounds__(kRT) void k_slice_hist(Rare<Key> x) {
    extern __shared__ __align__(16) unsigned char smem[];
    const RareArgs& a = x.a;
    const uint32_t nsl = a.ctr[kCtrSlices] < a.slice_cap ? a.ctr[kCtrSlices] : a.slice_cap;
    for (uint32_t i = blockIdx.x; i < nsl; i += gridDim.x) {
        slice_hist<Key, 8>(x, i, smem);
        __syncthreads();
    }
}

__global__ __launch_bounds__(kScanThreads) void k_slice_scan(RareArgs a, uint32_t* offsets) {
    constexpr uint32_t B = 1u << kRangeBits, G = kScanThreads / B;
    __shared__ uint32_t tmp[kScanThreads / kWave + 1];
    __shared__ uint32_t part[G][B];
    __shared__ uint32_t start[B];
    const uint32_t NB = 1u << a.k;
    const uint32_t ranges = a.k > kRangeBits ? NB >> kRangeBits : 1u;
    const uint32_t nh = a.ctr[kCtrSplit] < a.huge_cap ? a.ctr[kCtrSplit] : a.huge_cap;
    const uint32_t t = threadIdx.x & (B - 1), grp = threadIdx.x / B;
    for (uint32_t w = blockIdx.x; w < nh * ranges; w += gridDim.x) {
        const uint32_t idx = w / ranges, q = w % ranges;
        const uint32_t b = a.huge_list[idx], s0 = a.huge_s0[idx], ns = slices_of(a, idx);
        const uint32_t v0 = b << a.k, nb = (a.V - v0 < NB) ? a.V - v0 : NB;
        const uint32_t v = (q << kRangeBits) + t;
        uint32_t low = 0;  // entries of the bin in lower ranges
        for (uint32_t i = threadIdx.x; i < ns * q; i += kScanThreads)
            low += a.range_sum[(size_t)(s0 + i / q) * kRanges + i % q];
        uint32_t below;
        (void)block_excl_scan<kScanThreads>(low, tmp, &below);
        const uint32_t len = (ns + G - 1) / G;
        const uint32_t sa = grp * len < ns ? grp * len : ns;
        const uint32_t sb = ns - sa > len ? sa + len : ns;
        uint32_t* h = a.slice_hist + (size_t)s0 * NB + v;
        uint32_t acc = 0;
        if (v < NB)
            for (uint32_t s = sa; s < sb; s += 8) {
                uint32_t c[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) c[u] = s + u < sb ? h[(size_t)(s + u) * NB] : 0u;
#pragma unroll
                for (int u = 0; u < 8; ++u) acc += c[u];
            }
        part[grp][t] = acc;
        __syncthreads();
        uint32_t tot = 0;
        if (grp == 0)
            for (uint32_t g = 0; g < G; ++g) tot += part[g][t];
        uint32_t all;
        const uint32_t ex = a.bin_start[b] + below + block_excl_scan<kScanThreads>(tot, tmp, &all);
        if (grp == 0) {
            start[t] = ex;
            if (v < nb) offsets[v0 + v] = ex;
        }
        __syncthreads();
        uint32_t r = start[t];
        for (uint32_t g = 0; g < grp; ++g) r += part[g][t];
        if (v < NB)
            for (uint32_t s = sa; s < sb; s += 8) {
                uint32_t c[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) c[u] = s + u < sb ? h[(size_t)(s + u) * NB] : 0u;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (s + u < sb) h[(size_t)(s + u) * NB] = r;
                    r += c[u];
                }
            }
        __syncthreads();
    }
}

// Places every slice of every split bin: key and id read once, one LDS counter
// atomic each and two scattered writes, bound by the counters and the writes.
// The order is a template argument: with both orders in one kernel it took 129
// VGPRs, one past what two workgroups per CU leave, and 781 us at 2^26 Zipf(1.2)
// keys, now 472.
template <typename Key, bool ANY>
__global__ __launch_bounds__(kRT) void k_slice_place(Rare<Key> x) {
    extern __shared__ __align__(16) unsigned char smem[];
    const RareArgs& a = x.a;
    const uint32_t nsl = a.ctr[kCtrSlices] < a.slice_cap ? a.ctr[kCtrSlices] : a.slice_cap;
    for (uint32_t i = blockIdx.x; i < nsl; i += gridDim.x) {
        place_slice<Key, ANY>(x, i, smem);
        __syncthreads();
    }
}

// Probe index entries of the split bins, and the listed long buckets of every bin:
// split, oversize, and held in LDS.  Apart from k_rare_bins because the stable
// placement takes 124 to 144 VGPRs there, one workgroup per CU for 64-bit keys, and a
// long bucket's sort is a chain of LDS steps that lives on the second one: 2^24
// 64-bit keys in 2^18 buckets, every bucket listed, stable: the build took 4841 us with
// both in one kernel, now 2928.  The grid gives a build of up to 1024 bins a workgroup
// per bin: with 512 workgroups of up to three bins each, 2^22 32-bit keys in 2^16
// buckets, eight of a key, took 880 us, now 692.
template <typename Key>
__global__ __launch_bounds__(kRT) void k_listed_runs(Rare<Key> x) {
    extern __shared__ __align__(16) unsigned char smem[];
    const RareArgs& a = x.a;
    const uint32_t nh = a.ctr[kCtrSplit] < a.huge_cap ? a.ctr[kCtrSplit] : a.huge_cap;
    const uint32_t nheavy = a.ctr[kCtrHeavy];
    const uint32_t nlight = a.ctr[kCtrListed] ? a.bins : 0u;
    const BucketLds<Key> m(smem);
    for (uint32_t i = blockIdx.x; i < nh + nheavy + nlight; i += gridDim.x) {
        uint32_t g;
        if (i < nh) {
            g = a.huge_list[i];
            split_index<Key>(x, i, smem);
        } else if (i < nh + nheavy) {
            g = a.heavy_list[i - nh];
        } else {
            g = i - nh - nheavy;
            if (a.bin_start[g + 1] - a.bin_start[g] > light_cap<Key>()) continue;
        }
        const uint32_t listed = x.ix.gen_cnt[g];
        if (listed) listed_of_bin<Key, false>(x, g, listed, m);
        __syncthreads();
    }
}

template <typename Key>
__global__ __launch_bounds__(kRT) void k_runs_chunk_count(Rare<Key> x) {
    __shared__ uint32_t red[2 * W_LOCAL];
    const uint32_t c1 = x.a.ctr[kCtrChunks], nc = c1 < x.g2.chunk_cap ? c1 : x.g2.chunk_cap;
    for (uint32_t c = blockIdx.x; c < nc; c += gridDim.x) {
        const ChunkRef r = chunk_at(c, x.g2, x.offsets);
        const Key lead = x.ekeys[r.st];
        Key k[kCItems];
        load_chunk<Key>(r, x.ekeys, lead, k);
        uint32_t o, l;
        count_chunk<Key>(k, lead, red, o, l);
        if (threadIdx.x == 0) {
            x.g2.oth[c] = o;
            x.g2.less[c] = l;
        }
    }
}

// Per long bucket: exclusive prefixes of its chunks' counts (in place), the
// totals, and a bucket of one key finished outright.
template <typename Key>
__global__ __launch_bounds__(kRT) void k_runs_chunk_scan(Rare<Key> x) {
    __shared__ uint32_t tmp[W_LOCAL + 1];
    const G2& g2 = x.g2;
    const uint32_t c1 = x.a.ctr[kCtrLong], nl = c1 < g2.cap ? c1 : g2.cap;
    for (uint32_t i = blockIdx.x; i < nl; i += gridDim.x) {
        const uint32_t b = g2.list[i], c0 = g2.c0[i];
        const uint32_t st = x.offsets[b], len = x.offsets[b + 1] - st;
        const uint32_t nch = (len + kChunk - 1) / kChunk;
        uint32_t co = 0, cl = 0;
        for (uint32_t t0 = 0; t0 < nch; t0 += kRT) {
            const uint32_t j = t0 + threadIdx.x;
            const uint32_t vo = j < nch ? g2.oth[c0 + j] : 0u;
            const uint32_t vl = j < nch ? g2.less[c0 + j] : 0u;
            uint32_t ao, al;
            const uint32_t eo = block_excl_scan<kRT>(vo, tmp, &ao);
            const uint32_t el = block_excl_scan<kRT>(vl, tmp, &al);
            if (j < nch) {
                g2.oth[c0 + j] = co + eo;
                g2.less[c0 + j] = cl + el;
            }
            co += ao;
            cl += al;
        }
        if (threadIdx.x == 0) {
            g2.info[2 * i] = co;
            g2.info[2 * i + 1] = cl;
            if (co == 0) single_run<Key>(x.ix, b, st, len, x.ekeys[st]);
        }
    }
}

template <typename Key>
__global__ __launch_bounds__(kRT) void k_runs_chunk_scatter(Rare<Key> x) {
    __shared__ uint32_t red[W_LOCAL];
    const G2& g2 = x.g2;
    const uint32_t c1 = x.a.ctr[kCtrChunks], nc = c1 < g2.chunk_cap ? c1 : g2.chunk_cap;
    for (uint32_t c = blockIdx.x; c < nc; c += gridDim.x) {
        const ChunkRef r = chunk_at(c, g2, x.offsets);
        if (g2.info[2 * r.i] == 0) continue;  // uniform: a single run, no kperm
        const Key lead = x.ekeys[r.st];
        Key k[kCItems];
        load_chunk<Key>(r, x.ekeys, lead, k);
        scatter_chunk<Key>(x, r, k, lead, g2.oth[c], g2.info[2 * r.i + 1], red);
    }
}

template <typename Key>
__global__ __launch_bounds__(kRT) void k_runs_chunk_sort(Rare<Key> x) {
    extern __shared__ __align__(16) unsigned char smem[];
    const G2& g2 = x.g2;
    const uint32_t c1 = x.a.ctr[kCtrLong], nl = c1 < g2.cap ? c1 : g2.cap;
    const BucketLds<Key> m(smem);
    for (uint32_t i = blockIdx.x; i < nl; i += gridDim.x) {
        const uint32_t b = g2.list[i], O = g2.info[2 * i];
        const uint32_t st = x.offsets[b], len = x.offsets[b + 1] - st;
        if (O) sort_others<Key>(x, b, st, len, O, m);
        __syncthreads();
    }
}

// A table that is one bin held in LDS, from the caller's keys: the per-bin build
// and its long buckets.  (A build of 1500 keys as partition, scan and per-bin
// kernels took 12 launches and 47 us, of which the kernels ran 36.)
template <typename Key, bool ANY, int W>
__global__ __launch_bounds__(kRT) void k_build_one(Rare<Key> x, const Key* __restrict__ keys,
                                                   uint32_t n, uint32_t* bin_start) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (threadIdx.x == 0) {
        bin_start[0] = 0;
        bin_start[1] = n;
        x.offsets[x.a.V] = n;
    }
    light_bin_body<Key, ANY, W>(keys, nullptr, 0u, n, 0u, 0u, x.a.k, x.a.V, x.hp, x.offsets, x.ix,
                                x.ids, x.ekeys, smem);
    if constexpr (W != 0) {
        __syncthreads();
        const uint32_t listed = x.ix.gen_cnt[0];
        if (listed) listed_of_bin<Key, true>(x, 0u, listed, BucketLds<Key>(smem));
    }
}

template <typename Key>
size_t rare_smem(uint32_t k) {
    const size_t h = heavy_smem<Key>(k), b = BucketLds<Key>::bytes();
    return h > b ? h : b;
}

template <typename Key>
hipError_t set_rare_smem() {
    static std::atomic<uint64_t> done{0};
    return once_per_device(done, [] {
        const int lim = (int)rare_smem<Key>(kMaxLocalBits);
        const hipFuncAttribute at = hipFuncAttributeMaxDynamicSharedMemorySize;
        HG_TRY(hipFuncSetAttribute((const void*)k_rare_bins<Key, kSolo, true>, at, lim));
        HG_TRY(hipFuncSetAttribute((const void*)k_rare_bins<Key, kSolo, false>, at, lim));
        HG_TRY(hipFuncSetAttribute((const void*)k_rare_bins<Key, kBins, true>, at, lim));
        HG_TRY(hipFuncSetAttribute((const void*)k_rare_bins<Key, kBinsAndSlices, true>, at, lim));
        HG_TRY(hipFuncSetAttribute((const void*)k_rare_bins<Key, kBins, false>, at, lim));
        HG_TRY(hipFuncSetAttribute((const void*)k_rare_bins<Key, kBinsAndSlices, false>, at, lim));
        HG_TRY(hipFuncSetAttribute((const void*)k_slice_place<Key, true>, at, lim));
        HG_TRY(hipFuncSetAttribute((const void*)k_slice_place<Key, false>, at, lim));
        HG_TRY(hipFuncSetAttribute((const void*)k_listed_runs<Key>, at, lim));
        return hipFuncSetAttribute((const void*)k_runs_chunk_sort<Key>, at, lim);
    });
}

}  // namespace

size_t runs_ws_bytes(uint64_t n) { return layout_g2(nullptr, n).bytes; }
size_t range_sum_words(uint64_t slices) { return slices * kRanges; }

template <typename Key>
hipError_t run_rare(const RareArgs& a, uint32_t* offsets, uint32_t* ids, Key* ekeys, uint64_t n,
                    typename KeyTraits<Key>::Params hp, const IndexOut& ix, Key* rkeys,
                    uint32_t* rids, void* ws, hipStream_t s) {
    HG_TRY(set_rare_smem<Key>());
    const Rare<Key> x{a, offsets, ids, ekeys, hp, ix, rkeys, rids, rkeys, rids,
                      layout_g2(ws, n).g};
    const bool solo = n <= a.slice;  // no bin is split
    const size_t blds = BucketLds<Key>::bytes();
    const size_t lds = solo ? rare_smem<Key>(a.k) : heavy_smem<Key>(a.k);
    const dim3 gb(a.bins < kRareGrid ? a.bins : kRareGrid), th(kRT);
    {
        HG_PROF("v2_rare_bins", s);
        if (solo) {
            const auto f =
                a.any_order ? k_rare_bins<Key, kSolo, true> : k_rare_bins<Key, kSolo, false>;
            hipLaunchKernelGGL(f, gb, th, lds, s, x);
            return hipGetLastError();
        }
        // (slices may outnumber the bins)
        const auto both =
            a.any_order ? k_rare_bins<Key, kBinsAndSlices, true> : k_rare_bins<Key, kBinsAndSlices, false>;
        const auto alone = a.any_order ? k_rare_bins<Key, kBins, true> : k_rare_bins<Key, kBins, false>;
        hipLaunchKernelGGL(n < kSliceHistMin ? both : alone, dim3(kRareGrid), th, lds, s, x);
    }
    HG_TRY(hipGetLastError());
    HG_PROF("v2_split_bins", s);
    if (n >= kSliceHistMin) {
        hipLaunchKernelGGL(k_slice_hist<Key>, dim3(1024), th, (size_t)4 << a.k, s, x);
        HG_TRY(hipGetLastError());
    }
    hipLaunchKernelGGL(k_slice_scan, dim3(256), dim3(kScanThreads), 0, s, a, offsets);
    HG_TRY(hipGetLastError());
    const auto place = a.any_order ? k_slice_place<Key, true> : k_slice_place<Key, false>;
    hipLaunchKernelGGL(place, dim3(kRareGrid), th, heavy_smem<Key>(a.k), s, x);
    HG_TRY(hipGetLastError());
    if (!ix.head) return hipSuccess;
    hipLaunchKernelGGL(k_listed_runs<Key>, dim3(a.bins < kListedGrid / 2 ? 2 * a.bins : kListedGrid),
                       th, blds, s, x);
    HG_TRY(hipGetLastError());
    // long buckets in chunks: grids sized for the most work there can be,
    // strided over what the counters hold
    const dim3 cg(x.g2.chunk_cap < 1024 ? x.g2.chunk_cap : 1024);
    const dim3 bg(x.g2.cap < kRareGrid ? x.g2.cap : kRareGrid);
    hipLaunchKernelGGL(k_runs_chunk_count<Key>, cg, th, 0, s, x);
    HG_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_runs_chunk_scan<Key>, bg, th, 0, s, x);
    HG_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_runs_chunk_scatter<Key>, cg, th, 0, s, x);
    HG_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_runs_chunk_sort<Key>, bg, th, blds, s, x);
    return hipGetLastError();
}

template <typename Key, bool ANY, int W>
hipError_t run_build_one(const Key* keys, uint64_t n, uint32_t k, uint32_t V, uint32_t* offsets,
                         uint32_t* ids, Key* ekeys, typename KeyTraits<Key>::Params hp,
                         const IndexOut& ix, uint32_t* bin_start, Key* rkeys, uint32_t* rids,
                         void* ws, hipStream_t s) {
    static std::atomic<uint64_t> done{0};
    auto smem = [](uint32_t kk) {
        const size_t l = W ? light_smem_index<Key>(kk) : light_smem<Key>(kk);
        return W && BucketLds<Key>::bytes() > l ? BucketLds<Key>::bytes() : l;
    };
    HG_TRY(once_per_device(done, [&] {
        return hipFuncSetAttribute((const void*)k_build_one<Key, ANY, W>,
                                   hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)smem(kMaxLocalBits));
    }));
    RareArgs a{};
    a.bin_start = bin_start;
    a.k = k;
    a.bins = 1;
    a.V = V;
    const Rare<Key> x{a, offsets, ids, ekeys, hp, ix, rkeys, rids, rkeys, rids,
                      layout_g2(ws, n).g};
    HG_PROF("v2_build_one", s);
    hipLaunchKernelGGL((k_build_one<Key, ANY, W>), dim3(1), dim3(kRT), smem(k), s, x, keys,
                       (uint32_t)n, bin_start);
    return hipGetLastError();
}

#define HG_ONE_INST(Key, ANY, W)                                                               \
    template hipError_t run_build_one<Key, ANY, W>(                                            \
        const Key*, uint64_t, uint32_t, uint32_t, uint32_t*, uint32_t*, Key*,                  \
        KeyTraits<Key>::Params, const IndexOut&, uint32_t*, Key*, uint32_t*, void*, hipStream_t);
HG_ONE_INST(uint32_t, false, 0)
HG_ONE_INST(uint32_t, false, 4)
HG_ONE_INST(uint32_t, false, 8)
HG_ONE_INST(uint32_t, false, 16)
HG_ONE_INST(uint32_t, true, 0)
HG_ONE_INST(uint32_t, true, 4)
HG_ONE_INST(uint32_t, true, 8)
HG_ONE_INST(uint32_t, true, 16)
HG_ONE_INST(uint64_t, false, 0)
HG_ONE_INST(uint64_t, false, 16)
HG_ONE_INST(uint64_t, true, 0)
HG_ONE_INST(uint64_t, true, 16)
#undef HG_ONE_INST

template hipError_t run_rare<uint32_t>(const RareArgs&, uint32_t*, uint32_t*, uint32_t*, uint64_t,
                                       HashParams, const IndexOut&, uint32_t*, uint32_t*, void*,
                                       hipStream_t);
template hipError_t run_rare<uint64_t>(const RareArgs&, uint32_t*, uint32_t*, uint64_t*, uint64_t,
                                       HashParams64, const IndexOut&, uint64_t*, uint32_t*, void*,
                                       hipStream_t);

}  // namespace hg
