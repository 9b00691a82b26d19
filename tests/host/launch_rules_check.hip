// Host-only check of the rules by which launches are shaped (csrc/common.hpp), on either side of each line.  Built with
// `hipcc --cuda-host-only` by tests/test_launch_rules_cpu.py.
#include <cstdio>
#include "common.hpp"
using namespace bagua;

static long checked = 0;
static bool failed = false;
#define EXPECT(cond)                                                            \
    do {                                                                        \
        ++checked;                                                              \
        if (!(cond)) { std::printf("line %d: %s\n", __LINE__, #cond); failed = true; } \
    } while (0)

static void topk_rows()
{
    // 8192 elements: 16 waves of two rows, two workgroups on a CU; 6144: 12, two; 4608: 9, three
    EXPECT(pick_rpw_topk(32, 512) == 2 && pick_rpw_topk(32, 513) == 4 && pick_rpw_topk(32, 1024) == 4 && pick_rpw_topk(32, 1025) == 2);
    EXPECT(pick_rpw_topk(24, 512) == 2 && pick_rpw_topk(24, 513) == 4 && pick_rpw_topk(24, 1024) == 4 && pick_rpw_topk(24, 1302) == 2);
    EXPECT(pick_rpw_topk(18, 768) == 2 && pick_rpw_topk(18, 769) == 4 && pick_rpw_topk(18, 1025) == 2);
    EXPECT(pick_rpw_topk(16, 600) == 2 && pick_rpw_topk(1, 1024) == 2);          // 4096 elements and below: two
    EXPECT(pick_rpw_topk(33, 1) == 4 && pick_rpw_topk(64, 100000) == 4);         // above 32 rows only four fit 16 waves
}

int main()
{
    topk_rows();
    if (failed) return 1;
    std::printf("OK %ld\n", checked);
    return 0;
}
