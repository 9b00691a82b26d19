// Host-only check of the rules by which launches are shaped (csrc/common.hpp), on either side of each line.  Built with
// `hipcc --cuda-host-only` by tests/test_launch_rules_cpu.py.
#include <cstdio>
#include <vector>
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
    const size_t line = static_cast<size_t>(1) << 27;
    for (int k = 1; k <= 16; ++k) {
        const size_t n = (line + 8 * k - 1) / (8 * k);
        EXPECT(ring_fp_long(k, n) && !ring_fp_long(k, n - 1));
        EXPECT(ring_fp_rows(k) == 1);
        // the LDS asked for lets that many workgroups on a CU and no more, and the runtime need not be asked for it
        const size_t lds = lds_for_residency(ring_fp_waves(k));
        EXPECT(lds <= 64 * 1024 && kLdsPerCu / lds == static_cast<size_t>(ring_fp_waves(k)));
        // what replicas far apart in HBM want: 45 KB in flight and more up to 8 peers, 54 KB and more above
        EXPECT(k == 1 || ring_fp_waves(k) * k >= (k <= 8 ? k <= 4 ? 32 : 45 : 54));
    }
    EXPECT(ring_fp_rows(17) == kRowWaves);
}

static void gossip()
{
    const size_t line = static_cast<size_t>(5) << 23;
    EXPECT(gossip_pairs_lds(4096, line) == kLdsForTwo && gossip_pairs_lds(4096, line - 1) == 0 && gossip_pairs_lds(2816, line) == kLdsForTwo);
    EXPECT(gossip_pairs_lds(2560, 4 * line) == 0 && gossip_pairs_lds(4352, 4 * line) == 0);
    EXPECT(kLdsPerCu / kLdsForTwo == 2 && kLdsForTwo + 4 * kMaxWaves * sizeof(float) <= 64 * 1024);
}

// The order as the kernels apply it, on the host.
static bool permutes(const ChunkOrder o, size_t groups)
{
    std::vector<bool> seen(groups, false);
    for (size_t b = 0; b < groups; ++b) {
        const uint32_t i = static_cast<uint32_t>(b), r = i & ((8u << o.lg) - 1u);
        const uint32_t c = i < o.end ? i - r + ((r & 7u) << o.lg) + (r >> 3) : i;
        if (c >= groups || seen[c]) return false;
        seen[c] = true;
    }
    return true;
}

static void orders()
{
    for (const size_t chunk : {256, 1024, 1280, 4096, 4352, 16384})
        for (const size_t chunks : {1, 7, 2047, 2048, 2049, 2055, 3071, 3072, 5000, 65537}) {
            const ChunkOrder o = chunk_order(chunks, chunk);
            EXPECT((o.lg == 0) == (chunks < 2048) && o.end <= chunks && permutes(o, chunks) && permutes(chunk_order(chunks, chunk, false), chunks));
        }
    for (const unsigned rows : {1, 2, 3, 4, 6, 8, 16, 48, 64})
        for (const unsigned groups : {1, 31, 32, 33, 256, 1000, 4097}) EXPECT(permutes(row_order(groups, rows), groups));
    EXPECT(chunk_order(size_t{1} << 20, 512, false).end == 0 && row_order(4096, 3).end == 0 && row_order(4096, 1).end == 0);

    const size_t line = static_cast<size_t>(1) << 28, line_average = static_cast<size_t>(1) << 25, line_gather = static_cast<size_t>(1) << 26;
    EXPECT(order_pays(line, 1024) && !order_pays(line + 1, 1024));
    for (const size_t chunk : {256, 512, 768, 1280, 16384}) EXPECT(order_pays(8 * line, chunk));
    for (const size_t chunk : {256, 512}) {
        EXPECT(order_pays_average(line_average, chunk, 3) && !order_pays_average(line_average + 1, chunk, 3) && order_pays_average(line, chunk, 2));
        EXPECT(order_pays_gather_minmax(line_gather, chunk) && !order_pays_gather_minmax(line_gather + 1, chunk));
    }
    EXPECT(order_pays_average(line, 768, 8) && order_pays_gather_minmax(line, 768));
}

static void batched()
{
    const size_t low = static_cast<size_t>(1) << 26, high = static_cast<size_t>(1) << 29;
    for (const size_t chunk : {1024, 1536, 2048}) {
        const unsigned threads = static_cast<unsigned>(chunk / (2 * kRow)) * kWave;
        const size_t top = chunk == 1024 ? high / 2 : high;
        EXPECT(batched_groups(low - 1, chunk, threads) == 0 && batched_groups(top + chunk, chunk, threads) == 0);
        const int groups = batched_groups(low, chunk, threads);
        EXPECT(groups * static_cast<int>(threads / kWave) <= 16 && (groups + 1) * static_cast<int>(threads / kWave) > 16 && batched_groups(top, chunk, threads) == groups);
        // with what the MinMax kernel uses of it anyway, that many workgroups fit a CU and no more
        const size_t own = 2 * kMaxWaves * sizeof(float), lds = lds_for_residency(groups, own);
        const size_t granules = (lds + own + kLdsGranule - 1) / kLdsGranule;
        EXPECT(lds + own <= 64 * 1024 && kLdsPerCu / kLdsGranule / granules == static_cast<size_t>(groups));
    }
    for (const size_t chunk : {512, 768, 1280, 1792, 2304, 4096}) EXPECT(batched_groups(2 * low, chunk, 128) == 0);
}

static void momentum()
{
    const size_t line = static_cast<size_t>(7) << 24;
    EXPECT(mom_streams(line + 1, 1, 8) && !mom_streams(line, 1, 8) && !mom_streams(2 * line, 1, 6) && !mom_streams(2 * line, 2, 8));
    EXPECT(pick_rpw_worker(8, BAGUA_RPW_SIGN) == 1);
}

int main()
{
    momentum();
    batched();
    orders();
    gossip();
    ring_fp();
    topk_rows();
    if (failed) return 1;
    std::printf("OK %ld\n", checked);
    return 0;
}
