// Host-only check of the launches of the intra-node averages and the gathers: every row of a chunk has a wave that takes it, and a build that
// prefers four rows per wave gets them.
#include "fake_runtime.hpp"
#include "fused.hip"

template <int RPW, bool EF>
static bool is_average(const void* k)
{
    return k == stub(k_reduce_compress_minmax<RPW, EF, false>) || k == stub(k_reduce_compress_minmax<RPW, EF, true>) ||
           k == stub(k_reduce_compress_sign<RPW, EF, false>) || k == stub(k_reduce_compress_sign<RPW, EF, true>);
}
template <int RPW, bool EF>
static bool is_gather(const void* k)
{
    return k == stub(k_flatten_compress_minmax<RPW, EF, false>) || k == stub(k_flatten_compress_minmax<RPW, EF, true>) ||
           k == stub(k_flatten_sign_compress<RPW, EF, false>) || k == stub(k_flatten_sign_compress<RPW, EF, true>);
}
template <int RPW>
static bool takes(const void* k)
{
    return is_average<RPW, false>(k) || is_average<RPW, true>(k) || is_gather<RPW, false>(k) || is_gather<RPW, true>(k);
}

static void covers(size_t n, size_t chunk, int preferred, int status, const char* what)
{
    EXPECT(status == BAGUA_OK && g_launches.size() == 1, "%s chunk %zu n %zu: status %d", what, chunk, n, status);
    if (g_launches.size() != 1) return;
    const Launch& l = g_launches[0];
    const size_t rows = chunk / kRow, waves = l.block.x / kWave;
    const size_t rpw = takes<1>(l.kernel) ? 1 : takes<2>(l.kernel) ? 2 : takes<4>(l.kernel) ? 4 : 0;
    EXPECT(l.grid.x == num_chunks(n, chunk) && waves <= kMaxWaves && waves * rpw >= rows && (waves - 1) * rpw < rows, "%s chunk %zu n %zu: %zu waves of %zu rows", what,
           chunk, n, waves, rpw);
    EXPECT(preferred == 2 || rpw == 4, "%s chunk %zu n %zu: %zu rows per wave", what, chunk, n, rpw);
}

int main()
{
    const float* xs[3] = {far_apart<const float>(11), far_apart<const float>(12), far_apart<const float>(13)};
    for (size_t chunk = 256; chunk <= 16384; chunk += 256)
        for (const size_t n : {size_t{1}, size_t{4}, size_t{70001}, size_t{1} << 20, (size_t{1} << 20) + 1, size_t{1} << 21, (size_t{1} << 21) + 1, size_t{1} << 25})
            for (float* res : {far_apart<float>(2), static_cast<float*>(nullptr)}) {
                auto* codes = far_apart<uint8_t>(3);
                auto* bits = far_apart<uint32_t>(3);
                auto* meta = far_apart<float>(4);
                void* plan = far_apart<void>(5);
                g_launches.clear();
                covers(n, chunk, BAGUA_RPW_COMPRESS, bagua_reduce_compress_minmax_u8(xs, 3, res, n, chunk, codes, meta, nullptr), "average, MinMax");
                g_launches.clear();
                covers(n, chunk, BAGUA_RPW_SIGN, bagua_reduce_compress_sign_ef(xs, 3, res, n, chunk, bits, meta, nullptr), "average, sign");
                g_launches.clear();
                covers(n, chunk, BAGUA_RPW_COMPRESS, bagua_flatten_compress_minmax_u8(plan, 3, res, n, chunk, codes, meta, nullptr, nullptr), "gather, MinMax");
                g_launches.clear();
                covers(n, chunk, BAGUA_RPW_SIGN, bagua_flatten_sign_compress_ef(plan, 3, res, n, chunk, bits, meta, nullptr, nullptr), "gather, sign");
            }
    return finish();
}
