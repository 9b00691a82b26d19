// Host-only check of the rules by which the low-precision rounds choose their kernels.
#include "fake_runtime.hpp"
#include "ring.hip"

static bool encodes(const void* kernel, bool again, bool is_short)
{
    if (again && is_short) return kernel == stub(k_lp_encode<2, true, true>) || kernel == stub(k_lp_encode<4, true, true>);
    if (again) return kernel == stub(k_lp_encode<2, true, false>) || kernel == stub(k_lp_encode<4, true, false>);
    return !is_short && (kernel == stub(k_lp_encode<2, false, false>) || kernel == stub(k_lp_encode<4, false, false>));
}

// Workers that all choose one way: each is encoded before the first mix, which reads the copies again as long as they are 2^27 elements in all.
static void one_way()
{
    const size_t line = size_t{1} << 27, line_short = size_t{1} << 23;
    const float* x[BAGUA_MAX_WORKERS];
    float *out[BAGUA_MAX_WORKERS], *hat[BAGUA_MAX_WORKERS], *minmax[BAGUA_MAX_WORKERS];
    uint8_t* codes[BAGUA_MAX_WORKERS];
    int peer[BAGUA_MAX_WORKERS];
    for (int i = 0; i < BAGUA_MAX_WORKERS; ++i) {
        x[i] = far_apart<const float>(1 + i);
        out[i] = far_apart<float>(101 + i);
        hat[i] = far_apart<float>(201 + i);
        codes[i] = far_apart<uint8_t>(301 + i);
        minmax[i] = far_apart<float>(401 + i);
    }
    for (const int k : {3, 16, 17, 32})
        for (const size_t n : {size_t{3}, size_t{4}, line / 32, line / 32 + 1, line_short, line_short + 1, line / 3 + 1})
            for (const size_t chunk : {1024, 4096, 16384}) {
                for (int i = 0; i < k; ++i) peer[i] = (i + 1) % k;
                g_launches.clear();
                const int status = bagua_decentralized_avg_peers_lp(x, out, hat, codes, minmax, peer, k, n, chunk, nullptr);
                EXPECT(status == BAGUA_OK && g_launches.size() == static_cast<size_t>(k) + 1, "k %d n %zu", k, n);
                const bool again = k * n <= line, is_short = n >= 4 && n <= line_short;
                for (int i = 0; i < k && i < static_cast<int>(g_launches.size()); ++i)
                    EXPECT(encodes(g_launches[i].kernel, again, again && is_short), "k %d n %zu chunk %zu", k, n, chunk);
            }
}

// Where a ring goes through its peers in one launch again: a peer more costs that launch 2 to 3.5 us whatever the size, the two launches its bytes.
static void two_launches()
{
    const size_t quarter = 24 * 1024;
    for (const size_t chunk : {256, 1024, 2048, 2304, 4096}) {
        const size_t line = (chunk > 2048 ? 24 : 16) * quarter;
        EXPECT(!ring_lp_two_launches(4, 4, chunk) && ring_lp_two_launches(5, 5 * quarter, chunk) && !ring_lp_two_launches(5, 5 * quarter + 1, chunk), "chunk %zu", chunk);
        for (const int k : {24, 25, 32}) EXPECT(ring_lp_two_launches(k, line, chunk) && !ring_lp_two_launches(k, line + 1, chunk), "k %d chunk %zu", k, chunk);
    }
    EXPECT(ring_lp_two_launches(25, 5 << 17, 4352) && !ring_lp_two_launches(32, (5 << 17) + 1, 5888) && ring_lp_two_launches(32, 3 << 18, 6144), "chunks above 4096");
    EXPECT(ring_lp_two_launches(24, 3 << 18, 4352) && !ring_lp_two_launches(24, (3 << 18) + 1, 4352) && ring_lp_two_launches(32, 5 << 18, 16384), "chunks above 4096");
    for (const size_t chunk : {1024, 8192, 16384}) EXPECT(!ring_lp_two_launches(32, 3, chunk) && ring_lp_two_launches(32, 4, chunk), "chunk %zu", chunk);
}

// The one kernel for chunks of more than 32 rows: without tail tests where that pays.
static void folded()
{
    const float* x[3];
    float *out[3], *hat[3], *minmax[3];
    uint8_t* codes[3];
    for (int i = 0; i < 3; ++i) {
        x[i] = far_apart<const float>(1 + i);
        out[i] = far_apart<float>(11 + i);
        hat[i] = far_apart<float>(21 + i);
        codes[i] = far_apart<uint8_t>(31 + i);
        minmax[i] = far_apart<float>(41 + i);
    }
    const size_t line = size_t{1} << 18, long_line = size_t{5} << 24;
    for (const int k : {1, 2, 3})
        for (const size_t n : {size_t{3}, size_t{4}, line, line + 1, 5 * line, 5 * line + 1, long_line / 3, long_line / 3 + 1, long_line}) {
            g_launches.clear();
            const int status = bagua_decentralized_avg(BAGUA_AVG_LP_MINMAX_U8, x, out, hat, codes, minmax, k, n, 16384, nullptr);
            const bool two = k > 1 && n >= 4 && n <= 5 * line;
            EXPECT(status == BAGUA_OK && g_launches.size() == (two ? 2u : 1u), "k %d n %zu", k, n);
            if (two || g_launches.empty()) continue;
            const bool fold = (k == 1 && n <= line) || k * n >= long_line;
            EXPECT(g_launches[0].kernel == (fold ? stub(k_ring_avg_lp_any<4, true>) : stub(k_ring_avg_lp_any<4, false>)), "k %d n %zu", k, n);
        }
}

int main()
{
    folded();
    two_launches();
    one_way();
    return finish();
}
