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

int main()
{
    flag_in_tag();
    std::printf("plan rules harness: OK\n");
    return 0;
}
