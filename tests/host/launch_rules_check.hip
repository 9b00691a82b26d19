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

static void ring_fp()
{
    const size_t line = static_cast<size_t>(1) << 29;
    for (int k = 1; k <= 16; ++k) {
        const size_t n = (line + 8 * k - 1) / (8 * k);
        EXPECT(ring_fp_long(k, n) && !ring_fp_long(k, n - 1));
        EXPECT(ring_fp_rows(k, n) == 1 && ring_fp_rows(k, n - 1) == (k < 15 ? 8 : 1));
        // the LDS asked for lets that many workgroups on a CU and no more, and the runtime need not be asked for it
        const size_t lds = lds_for_residency(ring_fp_waves(k));
        EXPECT(lds <= 64 * 1024 && kLdsPerCu / lds == static_cast<size_t>(ring_fp_waves(k)));
        // what replicas far apart in HBM want: 45 KB in flight and more up to 8 peers, 54 KB and more above
        EXPECT(k == 1 || ring_fp_waves(k) * k >= (k <= 8 ? k <= 4 ? 32 : 45 : 54));
    }
    EXPECT(ring_fp_rows(17, 1) == kRowWaves && ring_fp_rows(17, line) == kRowWaves);
}

static void gossip()
{
    const size_t line = static_cast<size_t>(5) << 23;
    EXPECT(gossip_pairs_lds(4096, line) == kLdsForTwo && gossip_pairs_lds(4096, line - 1) == 0 && gossip_pairs_lds(2816, line) == kLdsForTwo);
    EXPECT(gossip_pairs_lds(2560, 4 * line) == 0 && gossip_pairs_lds(4352, 4 * line) == 0);
    EXPECT(kLdsPerCu / kLdsForTwo == 2 && kLdsForTwo + 4 * kMaxWaves * sizeof(float) <= 64 * 1024);
}

int main()
{
    gossip();
    ring_fp();
    topk_rows();
    if (failed) return 1;
    std::printf("OK %ld\n", checked);
    return 0;
}
