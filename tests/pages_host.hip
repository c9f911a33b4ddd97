// Offspring of many tiles put into pages as k_walk's thread 0 takes them, on the
// host: whatever the tiles' shares, the pages and their tables fit where the
// particles and all offspring just fit, and no two offspring get one slot.
#include "../paper_1709_02121_amd/csrc/wbrw_dev.hpp"
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>
using namespace wbrw;

static int one(std::mt19937_64 &g, int64_t N, double scale, int &tables)
{
    const int wt = 1 << (g() % 12), wr = kRangeMin * (1 + (int)(g() % 128));
    const int64_t R = walk_range(N, wt, wr), T = (N + R - 1) / R;
    const int sh = page_bits(R, T);
    std::vector<int64_t> m(T), nl(T, 0);      // offspring of each tile, in all and so far
    int64_t M = 0;
    for (auto &x : m) M += x = g() % 3 ? (int64_t)(scale * 64.0 * ((double)(g() % 1000) / 500.0)) : 0;
    const int64_t cap = N + M;
    if (cap >= (1ll << 25)) return 0;
    std::vector<uint32_t> ptx((cap + kRangeMin - 1) / kRangeMin * kTableShare, ~0u);
    std::vector<std::vector<uint32_t>> page(T, std::vector<uint32_t>(kPages, ~0u));
    std::vector<int> np(T, 1);
    std::vector<uint8_t> taken(cap, 0);
    uint64_t pool = sh < 31 ? (uint64_t)T << sh : 0, entries = 0;
    for (int64_t t = 0; t < T; ++t) page[t][0] = (uint32_t)(t << (sh & 31));
    for (bool left = true; left;) {
        left = false;
        for (int64_t t = 0; t < T; ++t) {
            const int64_t agg = std::min<int64_t>(m[t] - nl[t], 1 + (int64_t)(g() % 2000));
            const int want = sh < 31 ? (int)((nl[t] + agg + ((int64_t)1 << sh) - 1) >> sh) : 1;
            if (want > np[t]) {
                const uint64_t from = pool;
                pool += (uint64_t)(want - np[t]) << sh;
                if (pool > (uint64_t)cap) return std::printf("refused: %ld particles, %ld offspring\n", (long)N, (long)M), 1;
                uint32_t table = page[t][kDirect];
                if (page_table(want) != page_table(np[t])) {
                    const uint32_t old = table;
                    table = (uint32_t)entries;
                    entries += page_table(want);
                    ++tables;
                    if (entries > ptx.size()) return std::printf("tables: %ld particles, %ld offspring\n", (long)N, (long)M), 1;
                    for (int j = 0; j < np[t] - kDirect; ++j) ptx[table + j] = ptx[old + j];
                    page[t][kDirect] = table;
                }
                for (int q = np[t]; q < want; ++q) {
                    const uint32_t first = (uint32_t)from + ((uint32_t)(q - np[t]) << sh);
                    if (q < kDirect) page[t][q] = first; else ptx[table + (q - kDirect)] = first;
                }
                np[t] = want;
            }
            for (int64_t l = nl[t]; l < nl[t] + agg; ++l) {
                const int64_t s = page_slot(page[t].data(), sh, (uint32_t)l, [&] { return ptx.data(); });
                if (s < 0 || s >= cap || taken[s]++) return std::printf("slot %ld of %ld\n", (long)s, (long)cap), 1;
            }
            nl[t] += agg;
            left = left || nl[t] < m[t];
        }
    }
    return 0;
}

int main()
{
    std::mt19937_64 g(1);
    int tables = 0;
    for (int it = 0; it < 1500; ++it) {
        const int64_t N = 1 + (int64_t)std::exp(9.0 * (double)(g() % 10000) / 10000.0);
        if (one(g, N, std::exp(-2.0 + 9.0 * (double)(g() % 10000) / 10000.0), tables)) return 1;
    }
    std::printf("%d tables\n", tables);
    return tables > 5000 ? 0 : 1;
}
