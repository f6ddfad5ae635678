// Host-side check of the choice of index entries (hg_internal.h): quotient entries
// always hold a key's field whole, and the memory set aside for a table's capacities
// covers the entries of every build within them.  Built and run by
// tests/test_index_fmt.py.
#include <cstdio>
#include <random>
#include <vector>

#include "hg_internal.h"

using namespace hg;

int main() {
    std::mt19937_64 rng(5);
    std::vector<uint64_t> Vs = {1, 2, 3, 100, 4095, 4096, 4097, 0xffffffffull};
    for (int b = 2; b < 32; ++b)
        for (int d = -1; d <= 1; ++d) Vs.push_back((1ull << b) + d);
    int widths[17] = {};
    for (uint64_t vc : Vs)
        for (double load : {0.0, 0.1, 0.5, 0.51, 1.0, 1.5, 1.6, 3.0, 5.0, 5.1, 8.0, 8.1, 40.0}) {
            const uint64_t nc = (uint64_t)(load * (double)vc);
            const size_t most = index_bytes(nc, vc, 32);
            if (most > vc * 16 || most < vc * 8 || index_bytes(nc, vc, 64) != vc * 16) {
                printf("bound: n %llu V %llu\n", (unsigned long long)nc, (unsigned long long)vc);
                return 1;
            }
            std::vector<uint64_t> vs = Vs;
            for (int i = 0; i < 30; ++i) vs.push_back(1 + rng() % vc);
            for (uint64_t V : vs) {
                if (V > vc) continue;
                for (uint64_t n : {nc, nc / 2, nc ? nc - 1 : 0, V / 2, V / 2 + 1, V + V / 2, 5 * V, 8 * V, rng() % (nc + 1)}) {
                    if (n > nc) continue;
                    const HeadFmt f = index_fmt(n, V, 32);
                    ++widths[f.bytes];
                    if (V * f.bytes > most || (f.bytes != 16 && (f.cap < 3 || f.bytes != head_fmt(n, V, 32).bytes))) {
                        printf("entries: capacity %llu %llu: n %llu V %llu: %u bytes\n", (unsigned long long)nc,
                               (unsigned long long)vc, (unsigned long long)n, (unsigned long long)V, f.bytes);
                        return 1;
                    }
                }
            }
        }
    if (!widths[4] || !widths[8] || !widths[16]) return 1;
    printf("OK\n");
    return 0;
}
