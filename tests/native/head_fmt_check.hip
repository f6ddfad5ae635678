// Host-side check of the probe index entries of 32-bit keys (hg_internal.h):
// entries of random buckets, over hash ranges and loads that give every
// field width, answer every quotient as counting the bucket does.  Built and
// run by tests/test_head_fmt.py; exits non-zero on the first mismatch.
#include <cstdio>
#include <random>
#include <vector>

#include "hg_internal.h"

using namespace hg;

template <typename T>
static bool check(const HeadFmt& f, const std::vector<uint32_t>& qs, uint32_t q) {
    const uint32_t len = (uint32_t)qs.size();
    const uint64_t w = short_word(f, len, [&](uint32_t i) { return qs[i]; });
    if (sizeof(T) == 4 && (w >> 32)) return false;
    const T e = (T)w;
    uint32_t want = 0, mask = 0;
    for (uint32_t i = 0; i < len; ++i)
        if (qs[i] == q) {
            ++want;
            if (i < 32) mask |= 1u << i;
        }
    const uint32_t code = (uint32_t)e & 15u;
    if (len <= f.cap) {
        if (code != len) return false;
        const T m = held_matches(e, code, q, f);
        return popcount(m) == want && held_mask(m, code, f) == mask;
    }
    if (code != kCodeMedium) return false;
    const uint32_t q0 = (uint32_t)(e >> 12) & (uint32_t)((1ull << f.qb) - 1);
    if (q0 != qs[0]) return false;
    if (q == q0) return ((uint32_t)(e >> 4) & 0xffu) == want;
    // a clear filter bit must mean no match
    return (uint32_t)(e >> (12 + f.qb + filter_bit(q, f.nf))) & 1u || want == 0;
}

int main() {
    std::mt19937_64 rng(7);
    std::vector<uint64_t> ranges = {1, 2, 3, 5, 7, 1000, 0xffffffffull, 0x80000000ull, 0x80000001ull};
    for (int b = 2; b < 32; ++b)
        for (int d = -1; d <= 1; ++d) ranges.push_back((1ull << b) + d);
    int widths[9] = {};
    for (uint64_t V : ranges)
        for (double load : {0.0, 0.25, 0.5, 1.0, 2.0, 4.0, 32.0}) {
            const HeadFmt f = head_fmt((uint64_t)(load * (double)V), V, 32);
            const uint64_t qmax = 0xffffffffull / V;
            if ((f.bytes != 4 && f.bytes != 8) || f.cap < 1 || f.cap > kMaxHeld || f.nf < 1 ||
                f.nf > 32 || (qmax >> f.qb) || 4 + f.cap * f.qb > 8 * f.bytes ||
                12 + f.qb + f.nf > 8 * f.bytes || 6 + f.qb >= 8 * f.bytes) {
                printf("bad format: V %llu load %g\n", (unsigned long long)V, load);
                return 1;
            }
            ++widths[f.bytes];
            for (int it = 0; it < 200; ++it) {
                const uint32_t len = (uint32_t)(rng() % (kRunBucket + 1));
                const uint64_t span = it % 3 == 0 ? qmax + 1 : std::min<uint64_t>(qmax + 1, 1 + rng() % 4);
                std::vector<uint32_t> qs(len);
                for (auto& q : qs) q = (uint32_t)(it % 2 ? rng() % span : qmax - rng() % span);
                for (int t = 0; t < 24; ++t) {
                    const uint32_t q = len && t % 2 ? qs[rng() % len] : (uint32_t)(rng() % (qmax + 1));
                    if (f.bytes == 4 ? !check<uint32_t>(f, qs, q) : !check<uint64_t>(f, qs, q)) {
                        printf("mismatch: V %llu load %g len %u q %u\n", (unsigned long long)V,
                               load, len, q);
                        return 1;
                    }
                }
            }
            // quotient and bucket identify the hash
            const HashParams hp = make_hash_params(V, 0);
            for (int it = 0; it < 1000; ++it) {
                const uint32_t a = it == 0 ? 0xffffffffu : (uint32_t)rng();
                uint32_t r;
                const uint32_t q = divmod_u32(a, hp, r);
                if (q != a / V || r != a % V) {
                    printf("quotient: V %llu a %u\n", (unsigned long long)V, a);
                    return 1;
                }
            }
        }
    if (!widths[4] || !widths[8]) return 1;
    printf("OK\n");
    return 0;
}
