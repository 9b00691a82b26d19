// Host-only check of the launches of the top-K compression: every row of a chunk has a wave that takes it, whatever the rows per wave.
#include "fake_runtime.hpp"
#include "topk.hip"

template <int RPW>
static bool is_compression(const void* kernel)
{
    return kernel == stub(k_compress_topk<RPW, true, true>) || kernel == stub(k_compress_topk<RPW, true, false>) ||
           kernel == stub(k_compress_topk<RPW, false, true>) || kernel == stub(k_compress_topk<RPW, false, false>);
}

int main()
{
    for (size_t chunk = 256; chunk <= 16384; chunk += 256)
        for (const size_t n : {size_t{1}, size_t{4096}, size_t{1} << 20, size_t{1} << 23, (size_t{1} << 23) + 1, size_t{1} << 27})
            for (float* residual : {far_apart<float>(2), static_cast<float*>(nullptr)}) {
                g_launches.clear();
                const int status = bagua_compress_topk_ef(far_apart<float>(1), residual, n, chunk, 1, far_apart<uint16_t>(3), far_apart<float>(4), nullptr);
                EXPECT(status == BAGUA_OK && g_launches.size() == 1, "chunk %zu n %zu", chunk, n);
                if (g_launches.size() != 1) continue;
                const Launch& l = g_launches[0];
                const size_t rows = chunk / kRow, waves = l.block.x / kWave, rpw = is_compression<2>(l.kernel) ? 2 : is_compression<4>(l.kernel) ? 4 : 0;
                EXPECT(l.grid.x == num_chunks(n, chunk) && waves <= kMaxWaves && waves * rpw >= rows && (waves - 1) * rpw < rows,
                       "chunk %zu n %zu: %zu waves of %zu rows", chunk, n, waves, rpw);
            }
    const size_t line = size_t{1} << 23;
    for (const size_t chunk : {512, 1024, 1536}) EXPECT(topk_stores_joint(line + 1, chunk, 2) && !topk_stores_joint(line, chunk, 2) && !topk_stores_joint(line + 1, chunk, 4), "chunk %zu", chunk);
    for (const size_t chunk : {256, 1792, 4096}) EXPECT(!topk_stores_joint(8 * line, chunk, 2), "chunk %zu", chunk);
    return finish();
}
