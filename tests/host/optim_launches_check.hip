// Host-only check of the launches of the optimizer steps after a top-K round: whatever the size, the workgroups cover every chunk, within
// what a grid and a workgroup hold.
#include "fake_runtime.hpp"
#include "optim.hip"

template <bool A, bool B, int MOST>
static bool step(const void* kernel)
{
    return kernel == stub(k_decompress_sgd_topk<A, B, MOST, false, false>) || kernel == stub(k_decompress_adam_topk<A, B, MOST, false, false>) ||
           (MOST == kTopkPart && (kernel == stub(k_decompress_sgd_topk<A, B, kTopkPart, true, false>) || kernel == stub(k_decompress_adam_topk<A, B, kTopkPart, true, false>) ||
                                  kernel == stub(k_decompress_sgd_topk<A, B, kTopkPart, false, true>) || kernel == stub(k_decompress_adam_topk<A, B, kTopkPart, false, true>) ||
                                  kernel == stub(k_decompress_sgd_topk<A, B, kTopkPart, true, true>) || kernel == stub(k_decompress_adam_topk<A, B, kTopkPart, true, true>)));
}
template <int MOST>
static bool takes(const void* kernel)
{
    return step<false, false, MOST>(kernel) || step<false, true, MOST>(kernel) || step<true, false, MOST>(kernel) || step<true, true, MOST>(kernel);
}

// Of the last launch: it covers `chunks` chunks.
static void covers(size_t chunks, size_t chunk, int status, const char* what)
{
    EXPECT(status == BAGUA_OK && g_launches.size() == 1, "%s chunk %zu chunks %zu: status %d", what, chunk, chunks, status);
    if (g_launches.size() != 1) return;
    const Launch& l = g_launches[0];
    const size_t groups = l.grid.x, parts = groups / chunks, rows = chunk / kRow, waves = l.block.x / kWave;
    const size_t rpw = takes<kTopkPart>(l.kernel) || takes<kTopkWhole>(l.kernel) ? 2 : takes<kTopkWholeLong>(l.kernel) ? 4 : 0;
    EXPECT(groups <= kMaxGrid && parts >= 1 && groups == parts * chunks, "%s chunk %zu chunks %zu: %zu workgroups", what, chunk, chunks, groups);
    EXPECT(waves <= kMaxWaves && waves * rpw * parts >= rows && l.lds >= (rows + parts - 1) / parts * kRow * sizeof(float) && l.lds <= 64 * 1024,
           "%s chunk %zu chunks %zu: %zu parts of %zu waves of %zu rows, %zu bytes", what, chunk, chunks, parts, waves, rpw, l.lds);
    EXPECT(waves <= static_cast<size_t>(takes<kTopkPart>(l.kernel) ? topk_step_threads(kTopkPart) : 1024) / kWave, "%s chunk %zu chunks %zu", what, chunk, chunks);
}

// Chunks whole or in parts, on either side of each line (a launch of chunks up to 8192 elements that has a CU for every chunk and late entries; one go
// of longer chunks where the parts need two).
static void whole()
{
    EXPECT(topk_step_whole(256, 8192, 1) && !topk_step_whole(257, 8192, 1) && topk_step_whole(129, 8192, 1) && !topk_step_whole(128, 8192, 1), "8192");
    EXPECT(topk_step_whole(256, 4352, 4352) && !topk_step_whole(240, 4352, 1), "4352");
    for (const size_t chunk : {8448, 9216}) EXPECT(!topk_step_whole(426, chunk, 1) && topk_step_whole(427, chunk, 1) && topk_step_whole(768, chunk, 1) && !topk_step_whole(769, chunk, 1), "three on a CU");
    for (const size_t chunk : {9472, 12288}) EXPECT(!topk_step_whole(341, chunk, 1) && topk_step_whole(342, chunk, chunk) && topk_step_whole(512, chunk, 1) && !topk_step_whole(513, chunk, 1), "two on a CU");
    for (const size_t chunk : {12544, 16384}) {
        EXPECT(!topk_step_whole(352, chunk, chunk / 4) && topk_step_whole(353, chunk, chunk / 4) && topk_step_whole(512, chunk, 1) && !topk_step_whole(513, chunk, 1), "two on a CU");
        EXPECT(!topk_step_whole(288, chunk, chunk / 4 + 1) && topk_step_whole(289, chunk, chunk / 4 + 1), "long lists");
    }
}

int main()
{
    whole();
    for (size_t chunk = 256; chunk <= 16384; chunk += 256) {
        std::vector<size_t> counts = {1, 100, 400, 600, 1000, 3000, size_t{1} << 20, kMaxGrid};
        for (const size_t parts : {2, 3, 4}) counts.insert(counts.end(), {kMaxGrid / parts, kMaxGrid / parts + 1});
        for (const size_t chunks : counts)
            for (const size_t keep : {size_t{1}, chunk / 8, chunk}) {
                if (chunks > (size_t{1} << 24) && keep > 1) continue;
                const size_t n = chunks * chunk - 1;
                auto *idx = far_apart<uint16_t>(1);
                auto *val = far_apart<float>(2), *p = far_apart<float>(3), *m = far_apart<float>(4), *v = far_apart<float>(5);
                g_launches.clear();
                covers(chunks, chunk, bagua_decompress_sgd_step_topk(idx, val, n, chunk, keep, p, m, 0.1f, 0.9f, 0.0f, nullptr), "sgd");
                g_launches.clear();
                covers(chunks, chunk, bagua_decompress_adam_step_topk(idx, val, n, chunk, keep, p, m, v, 0.1f, 0.9f, 0.99f, 1e-8f, 0.0f, 0, nullptr), "adam");
            }
    }
    return finish();
}
