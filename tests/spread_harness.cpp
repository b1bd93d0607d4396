// CPU harness for the order of a batch's work list (spread_items in
// paper_2602_23067_amd/csrc/gcm_plan.h), built with the sanitizers: the items
// stay the same ones, no workgroup's sum of costs ends above what any order must
// reach by more than the largest item, and a list of one round is left alone.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "gcm_plan.h"

using namespace gcm;

#define CHECK(c)                                                                 \
    do {                                                                         \
        if (!(c)) {                                                              \
            std::fprintf(stderr, "check failed line %d: %s\n", __LINE__, #c);    \
            std::exit(1);                                                        \
        }                                                                        \
    } while (0)

int main()
{
    std::mt19937_64 r(23067);
    const uint8_t iv[12] = {};
    for (int it = 0; it < 3000; ++it) {
        const uint32_t waves = (const uint32_t[]){8, 12, 16}[r() % 3], n = 1 + (uint32_t)(r() % 60);
        std::vector<MsgDesc> d(n);
        std::vector<WorkItem> before;
        for (uint32_t i = 0; i < n; ++i) {
            fill_desc(&d[i], 0, iv, 0, r() % 300, 0, 0, r() % 5 ? r() % 3000000 : r() % 20, 0, 0, 0,
                      10 + 2 * (uint32_t)(r() % 3), 6 + (uint32_t)(r() % 7), waves, 0);
            set_groups(&d[i], waves, true);
            for (uint64_t t = 0; t < d[i].n_tiles; t += waves)
                before.push_back(WorkItem{i, (uint32_t)t});
        }
        const uint32_t grid = it % 7 == 0 ? (uint32_t)before.size() + (uint32_t)(r() % 2) : 1 + (uint32_t)(r() % 300);
        std::vector<WorkItem> after = before;
        spread_items(d, waves, grid, &after);
        CHECK(after.size() == before.size());
        std::vector<std::vector<uint8_t>> seen(n);
        for (uint32_t i = 0; i < n; ++i)
            seen[i].assign(d[i].groups, 0);
        std::vector<uint64_t> load(grid, 0);
        uint64_t sum = 0, largest = 0, most = 0;
        for (size_t k = 0; k < after.size(); ++k) {
            CHECK(after[k].msg < n && after[k].first_tile % waves == 0 && after[k].first_tile / waves < d[after[k].msg].groups);
            CHECK(!seen[after[k].msg][after[k].first_tile / waves]++);
            const uint64_t c = item_cost(d[after[k].msg], after[k].first_tile, waves);
            load[k % grid] += c;
            sum += c;
            largest = c > largest ? c : largest;
        }
        for (uint64_t l : load)
            most = l > most ? l : most;
        CHECK(after.size() <= grid || grid < 2 || most <= sum / grid + largest);
        if (after.size() <= grid)
            for (size_t k = 0; k < after.size(); ++k)
                CHECK(after[k].msg == before[k].msg && after[k].first_tile == before[k].first_tile);
    }
    std::printf("spread harness: OK\n");
    return 0;
}
