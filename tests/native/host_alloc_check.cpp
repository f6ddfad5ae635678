// Host paths of the library's memory handling, over fake_hip.h.  One check per
// argument; exits non-zero at the first thing that is wrong.
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <random>
#include <string>
#include <vector>

#include "fake_hip.h"
#include "hashgraph.h"

using fake::st;

static void* const kKeys = (void*)(uintptr_t)0x1000;

#define CHECK(cond, ...)                              \
    do {                                              \
        if (!(cond)) {                                \
            printf("%s:%d: %s: ", __FILE__, __LINE__, #cond); \
            printf(__VA_ARGS__);                      \
            printf("\n");                             \
            exit(1);                                  \
        }                                             \
    } while (0)

// Builds of any size up to a table's capacity allocate nothing.
static void rebuilds_allocate_nothing() {
    std::mt19937_64 rng(3);
    std::vector<std::pair<uint64_t, uint64_t>> caps = {
        {17616076, 1ull << 24}, {17616076, 1ull << 25}, {1ull << 28, 1ull << 28},
        {1ull << 24, 1ull << 24}, {300007, 300007}, {(1 << 17) + 1, 1 << 17},
        {(1 << 21) + 5000, 1 << 21}, {4608, 4096}, {1, 1}, {0, 7}, {1 << 20, 3},
        {5000, 1ull << 28}, {1ull << 30, 1ull << 30}, {0xffffffffull, 0xffffffffull}};
    for (int i = 0; i < 40; ++i) {
        const uint64_t n = 1 + (rng() >> (36 + rng() % 24));
        caps.push_back({n, std::max<uint64_t>(1, i % 2 ? n >> (rng() % 6) : n << (rng() % 4)) &
                               0xffffffffull});
        if (!caps.back().second) caps.back().second = 1;
    }
    for (int kb : {32, 64})
        for (auto [nc, vc] : caps) {
            hg_table* t = nullptr;
            CHECK(hg_table_create(nc, vc, kb, &t) == HG_OK, "%llu %llu", (unsigned long long)nc,
                  (unsigned long long)vc);
            const long before = st.allocs;
            std::vector<uint64_t> Vs = {vc, vc - 1, vc / 2, vc / 2 + 1, vc / 3, vc / 64, 1, 4096};
            for (int b = 1; b < 32; ++b)
                for (int d : {0, 1}) Vs.push_back((1ull << b) + d);
            for (uint64_t V : Vs) {
                if (V < 1 || V > vc) continue;
                // where the bins' width and the number of passes step, and between
                std::vector<uint64_t> ns = {nc, nc - 1, nc / 2, 0, 1, 1 << 17, (1 << 17) + 1,
                                            nc - nc / 20};
                for (int k = 0; k <= 13; ++k)
                    for (int d = -1; d <= 1; ++d) ns.push_back((((kb == 64 ? 2048 : 4096) * V) >> k) + d);
                for (int b = 14; b < 30; ++b) ns.push_back(1ull << b);
                for (uint64_t n : ns) {
                    if (n > nc) continue;
                    for (int form = 0; form < 4; ++form) {
                        hg_build_opts o{};
                        o.any_order = form & 1;
                        o.no_index = form >> 1;
                        CHECK(hg_table_build(t, kKeys, n, V, 1, &o, nullptr) == HG_OK, "build");
                        CHECK(st.allocs == before,
                              "capacity %llu keys %llu buckets, %d bits: %llu keys, %llu buckets, "
                              "any order %d", (unsigned long long)nc, (unsigned long long)vc, kb,
                              (unsigned long long)n, (unsigned long long)V, form & 1);
                    }
                }
            }
            hg_build_opts o{};
            o.variant = HG_VARIANT_V1;
            CHECK(hg_table_build(t, kKeys, nc, vc, 1, &o, nullptr) == HG_OK, "V1");
            CHECK(st.allocs == before, "V1");
            hg_table_free(t);
            CHECK(st.live.empty(), "left over");
        }
}

static uint64_t bytes_of(hg_table* t) {
    hg_table_info i{};
    CHECK(hg_table_view(t, &i) == HG_OK, "view");
    return i.device_bytes;
}

// A call that runs out of memory half-way leaves the table as it was: the next one
// allocates everything it needs.
static void failed_allocations_leave_nothing_half_done() {
    for (int kb : {32, 64}) {
        hg_build_opts plain{};
        plain.no_index = 1;
        for (long at = 0; at < 4; ++at) {
            hg_table* t = nullptr;
            CHECK(hg_build(kKeys, 100000, kb, 1 << 16, 1, &plain, nullptr, &t) == HG_OK, "build");
            CHECK(bytes_of(t) == st.used, "plain table");
            const size_t before = st.used;
            // (the build's workspace comes first)
            st.fail_in = at + 1;
            st.fail_times = 2;
            CHECK(hg_table_build(t, kKeys, 90000, 1 << 16, 1, nullptr, nullptr) == HG_ERR_OOM,
                  "index array %ld", at);
            CHECK(st.used == before, "index array %ld: %zu bytes kept", at, st.used - before);
            st.fail_in = -1;
            CHECK(hg_table_build(t, kKeys, 90000, 1 << 16, 1, nullptr, nullptr) == HG_OK, "retry");
            CHECK(bytes_of(t) == st.used && st.used > before, "index after array %ld failed", at);
            hg_table_free(t);
            CHECK(st.live.empty(), "left over");
        }
        for (int at = 0; at < 5; ++at) {  // three arrays, two fills
            hg_table* t = nullptr;
            CHECK(hg_build(kKeys, 100000, kb, 1 << 16, 1, nullptr, nullptr, &t) == HG_OK, "build");
            const size_t before = st.used;
            st.fail_times = 2;
            if (at < 3) st.fail_in = at;
            else st.memset_fail_in = at - 3;
            CHECK(hg_table_erase(t, kKeys, 10, nullptr, nullptr) != HG_OK, "erase, failure %d", at);
            CHECK(st.used == before, "failure %d: %zu bytes kept", at, st.used - before);
            st.fail_in = st.memset_fail_in = -1;
            st.memsets = 0;
            CHECK(hg_table_erase(t, kKeys, 10, nullptr, nullptr) == HG_OK, "retry");
            CHECK(bytes_of(t) == st.used && st.used > before && st.memsets == 2,
                  "erase after failure %d", at);
            hg_table_free(t);
            CHECK(st.live.empty(), "left over");
        }
    }
}

// The pool: used while tables live, emptied by hg_set_allocator, by an allocation that
// fails, and with the last table; not used under capture.
static void the_pool_is_given_back() {
    uint64_t total = 0;
    hg_table *a = nullptr, *b = nullptr;
    CHECK(hg_build(kKeys, 1 << 20, 32, 1 << 20, 1, nullptr, nullptr, &a) == HG_OK, "build");
    CHECK(st.kept > (8u << 20) && st.pools == 1, "the build's workspace: %zu kept", st.kept);
    CHECK(hg_set_allocator(nullptr, nullptr, nullptr) == HG_OK, "set_allocator");
    CHECK(st.kept == 0 && st.trims == 1, "%zu kept by hg_set_allocator", st.kept);
    CHECK(hg_set_allocator([](size_t, hipStream_t, void*) -> void* { return nullptr; }, nullptr,
                           nullptr) == HG_ERR_INVALID_ARG && st.trims == 1, "half an allocator");
    // a call that needs what the pool holds
    const uint64_t m = 1 << 21;
    CHECK(hg_probe_ordered(a, kKeys, m, (uint32_t*)kKeys, &total, HG_PROBE_GROUPED, nullptr) == HG_OK,
          "probe");
    CHECK(st.kept > m * 11, "%zu kept by the probe", st.kept);
    const size_t held = st.kept;
    st.capacity = st.used + st.kept + (1 << 20);
    CHECK(hg_table_create(1 << 18, 1 << 18, 32, &b) == HG_OK, "a table beside a full pool");
    CHECK(st.kept == 0 && st.used + st.kept <= st.capacity, "%zu kept", st.kept);
    CHECK(hg_table_create(held, 1 << 18, 32, &b) == HG_ERR_OOM, "a table too large");
    st.capacity = ~(size_t)0;
    // a call whose own pool block does not fit beside what the pool holds
    CHECK(hg_probe_ordered(a, kKeys, m, (uint32_t*)kKeys, nullptr, HG_PROBE_GROUPED, nullptr) == HG_OK,
          "probe");
    st.fail_in = 0;
    st.fail_times = 1;
    CHECK(hg_probe_ordered(a, kKeys, 2 * m, (uint32_t*)kKeys, nullptr, HG_PROBE_GROUPED, nullptr) ==
              HG_OK, "probe, second try");
    st.fail_in = -1;
    // under capture: no block of the pool
    const size_t before = st.kept;
    st.capturing = true;
    CHECK(hg_probe_ordered(a, kKeys, 4 * m, (uint32_t*)kKeys, nullptr, HG_PROBE_GROUPED, nullptr) ==
              HG_OK, "captured probe");
    CHECK(st.kept == before, "captured probe took the pool");
    st.capturing = false;
    hg_table_free(a);
    CHECK(st.kept == before, "a table is left");
    hg_table_free(b);
    CHECK(st.kept == 0 && st.live.empty(), "the last table");
}

// Counts by input index (scattered by B's ids) take the entries twice and the passes'
// matrices, not a build's workspace.
static void intersections_take_no_builds_workspace() {
    for (uint64_t n : {1ull << 21, 1ull << 25, (1ull << 25) + 12345, 1ull << 28}) {
        hg_table *a = nullptr, *b = nullptr;
        CHECK(hg_build(kKeys, n, 32, n, 1, nullptr, nullptr, &a) == HG_OK, "build");
        CHECK(hg_build(kKeys, n, 32, n, 1, nullptr, nullptr, &b) == HG_OK, "build");
        static size_t bytes;
        CHECK(hg_set_allocator([](size_t nb, hipStream_t, void*) { bytes = nb; return (void*)4096; },
                               [](void*, hipStream_t, void*) {}, nullptr) == HG_OK, "hook");
        CHECK(hg_intersect(a, b, (uint32_t*)kKeys, nullptr, nullptr, 0, nullptr, nullptr) == HG_OK,
              "intersect");
        // edge counts, positions, two copies of (value, id); 1/8 of a byte to one byte an
        // entry of matrices and scans
        CHECK(bytes >= n * 28 && bytes < n * 29 + (4u << 20), "%llu edges: %zu bytes, %.2f an edge",
              (unsigned long long)n, bytes, (double)bytes / (double)n);
        CHECK(hg_set_allocator(nullptr, nullptr, nullptr) == HG_OK, "hook");
        hg_table_free(a);
        hg_table_free(b);
    }
}

int main(int argc, char** argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "rebuilds") rebuilds_allocate_nothing();
    else if (what == "failures") failed_allocations_leave_nothing_half_done();
    else if (what == "pool") the_pool_is_given_back();
    else if (what == "scatter") intersections_take_no_builds_workspace();
    else return 2;
    printf("OK\n");
    return 0;
}
