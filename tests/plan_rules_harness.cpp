// CPU harness for rules of the launch planner (paper_2602_23067_amd/csrc/gcm_plan.h),
// built with the sanitizers.
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

static const uint8_t iv[12] = {};

// Every workgroup of a verdict reads the expected tag and the first writes the
// accept flag: a flag that lies in the tag allows one workgroup only.
static void flag_in_tag()
{
    for (uint32_t tl : {4u, 8u, 12u, 13u, 16u})
        for (int64_t off = -8; off <= 24; ++off) {
            MsgDesc d;
            const uint64_t tag = 1ull << 40;
            fill_desc(&d, 1, iv, 0, 0, 0, 0, 5 << 20, tag, tag + off, 0, 14, 6, 16, 0);
            d.tag_len = tl;
            const bool overlap = off > -4 && off < (int64_t)tl;
            CHECK(overlap ? verdict_groups(d) == 1 : verdict_groups(d) > 1);
            d.op = 0;
            CHECK(verdict_groups(d) == 1);
        }
}

// The cap on a batch's tile sizes.  Where tiles of 2^8 blocks make no more items
// than there are workgroups, the largest item decides: of messages that fill one
// with 2^9 too, it costs 46048 with 2^8 and 80096 with 2^9, and the mean of the
// items adds less than an eighth to the former.  Where there is work for many
// rounds, the start of the items decides: 2^11 halves the 112000 cycles that
// 1.2 GiB spend on it with 2^10, and adds 35000 by its largest item.
static void batch_cap()
{
    std::mt19937_64 r(23067);
    const uint32_t nr[3] = {10, 12, 14};
    const uint8_t used[3] = {1, 1, 1};
    SlotView sv;
    sv.n_slots = 3, sv.used = used, sv.nr = nr;
    for (int it = 0; it < 300; ++it) {
        std::vector<PlanMsg> msgs;
        uint64_t items = 0;
        for (;;) {
            PlanMsg m;
            m.len = (128 << 10) + r() % (1 << 20);
            m.aad_len = r() % 3000;
            m.key_slot = (uint32_t)(r() % 3);
            items += (ghash_blocks(m.aad_len, m.len) + 4095) / 4096;
            if (items > 256)
                break;
            msgs.push_back(m);
            if (r() % 30 == 0)
                break;
        }
        CHECK(batch_cap_log2B(msgs.data(), (uint32_t)msgs.size(), sv, 16, 256) == 8);
    }
    for (int it = 0; it < 20; ++it) {
        std::vector<PlanMsg> msgs(64 + r() % 1200);
        for (auto &m : msgs) {
            m.len = (1300ull << 20) / msgs.size() + r() % 100000;
            m.key_slot = (uint32_t)(r() % 3);
        }
        CHECK(batch_cap_log2B(msgs.data(), (uint32_t)msgs.size(), sv, 16, 256) >= 11);
    }
}

// Every workgroup of a batch comes to a key slot once, and to a message once.
static void key_order()
{
    std::mt19937_64 r(23067);
    for (int it = 0; it < 500; ++it) {
        const uint32_t waves = (const uint32_t[]){8, 12, 16}[r() % 3], n = 1 + (uint32_t)(r() % 60), keys = 1 + (uint32_t)(r() % 6);
        const std::vector<uint8_t> used(keys, 1);
        std::vector<uint32_t> nr(keys);
        for (auto &x : nr)
            x = 10 + 2 * (uint32_t)(r() % 3);
        SlotView sv;
        sv.n_slots = keys, sv.used = used.data(), sv.nr = nr.data();
        std::vector<PlanMsg> msgs(n);
        for (auto &m : msgs) {
            m.len = r() % 3000000;
            m.key_slot = (uint32_t)(r() % keys);
        }
        BatchPlan p;
        plan_batch(msgs.data(), n, sv, waves, 6 + (uint32_t)(r() % 6), &p);
        const uint32_t grid = 1 + (uint32_t)(r() % 300);
        spread_items(p.descs, waves, grid, &p.items);
        for (size_t g = 0; g < grid; ++g) {
            std::vector<uint8_t> key_seen(keys, 0), msg_seen(n, 0);
            for (size_t k = g; k < p.items.size(); k += grid) {
                const uint32_t i = p.items[k].msg, prev = k > g ? p.items[k - grid].msg : n;
                if (k == g || msgs[i].key_slot != msgs[prev].key_slot)
                    CHECK(!key_seen[msgs[i].key_slot]++);
                if (i != prev)
                    CHECK(!msg_seen[i]++);
            }
        }
    }
}

// One wave of the tile kernel clears what it rejects: it finishes a decrypt by
// itself only up to 1 MiB, and any encrypt of one group.
static void finish_bound()
{
    for (uint32_t waves : {8u, 12u, 16u})
        for (uint32_t log2B : {6u, 12u, 16u, 20u})
            for (uint64_t len : {0ull, 1000ull, 1ull << 20, (1ull << 20) + 1, 10ull << 20, 200ull << 20})
                for (uint32_t op : {0u, 1u}) {
                    MsgDesc d;
                    fill_desc(&d, op, iv, 0, 0, 0, 0, len, 0, 0, 0, 14, log2B, waves, 0);
                    set_groups(&d, waves, true);
                    const bool one = d.n_tiles <= (waves == 16 ? 16u : waves == 8 ? 8u : 4u);
                    CHECK(((d.flags & kFinish) != 0) == (one && (op == 0 || len <= 1ull << 20)));
                }
}

// Items of the row kernel: more rows cost more, and so does a larger key, but a
// full item less than half as much again as one row (8.4 us to 6.9 measured).
static void row_items()
{
    for (uint32_t waves : {8u, 12u, 16u})
        for (uint32_t nr : {10u, 12u, 14u}) {
            uint64_t before = 0, one = 0;
            for (uint32_t rows = 1; rows <= (waves == 12 ? 4 : waves); ++rows) {
                MsgDesc d;
                fill_desc(&d, 0, iv, 0, 0, 0, 0, 1024 * rows - 16, 0, 0, 0, nr, 6, waves, 0);
                set_groups(&d, waves, true);
                d.flags |= kRows;
                const uint64_t c = item_cost(d, 0, waves);
                CHECK(c > before);
                one = rows == 1 ? c : one;
                CHECK(2 * c < 3 * one);
                before = c;
                MsgDesc e = d;
                e.nr = nr + 2;
                CHECK(item_cost(e, 0, waves) > c);
            }
        }
}

int main()
{
    flag_in_tag();
    batch_cap();
    key_order();
    finish_bound();
    row_items();
    std::printf("plan rules harness: OK\n");
    return 0;
}
