// Host-only check of the order in which the sign codec's server step goes through the workers (csrc/sign_device.hpp): each once, in
// ascending order, the first one marked, whatever the size of a group.  Built by tests/test_launches_cpu.py.
#include <cstdio>
#include "sign_device.hpp"
using namespace bagua;

static bool g_failed = false;
static long g_checked = 0;

template <int NJ, int REST>
static void groups(int k)
{
    int next = 0;
    for_worker_groups<NJ, REST>(k, [&](auto count, int j, bool first) {
        ++g_checked;
        if (j != next || first != (j == 0)) g_failed = true;
        next = j + decltype(count)::value;
    });
    if (next != k) {
        std::printf("groups of %d, rest %d: %d of %d workers\n", NJ, REST, next, k);
        g_failed = true;
    }
}
template <int NJ>
static void groups()
{
    for (int k = 1; k <= 32; ++k) {
        groups<NJ, kRestOneByOne>(k);
        if (k % NJ == 0) groups<NJ, kRestNone>(k);
        if constexpr (NJ <= 8) groups<NJ, kRestTogether>(k);
    }
}

int main()
{
    groups<1>();
    groups<2>();
    groups<3>();
    groups<4>();
    groups<8>();
    groups<9>();
    groups<12>();
    groups<16>();
    groups<32>();
    if (g_failed) return 1;
    std::printf("OK %ld\n", g_checked);
    return 0;
}
