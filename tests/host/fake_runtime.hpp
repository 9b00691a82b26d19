// The part of the HIP runtime that an entry point's host code calls, recording launches instead of making them, for checks of
// the launches on the CPU.  The sources under test are included into the check and compiled for the host only, so that a kernel is
// known by the address of its stub.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdio>
#include <vector>

struct Launch {
    const void* kernel;
    dim3 grid, block;
    size_t lds;
};
static std::vector<Launch> g_launches;

extern "C" {
hipError_t hipLaunchKernel(const void* kernel, dim3 grid, dim3 block, void**, size_t lds, hipStream_t)
{
    g_launches.push_back(Launch{kernel, grid, block, lds});
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
char __hip_fatbin[64];
}

template <typename... P>
const void* stub(void (*kernel)(P...))
{
    return reinterpret_cast<const void*>(kernel);
}
// An address that is never read; far from those of other numbers, so that tensors of any size lie apart.
template <typename T>
T* far_apart(int number)
{
    return reinterpret_cast<T*>(static_cast<uintptr_t>(number) << 48);
}

static long g_checked = 0;
static bool g_failed = false;
#define EXPECT(cond, ...)                                                                        \
    do {                                                                                         \
        ++g_checked;                                                                             \
        if (!(cond)) {                                                                           \
            std::printf("line %d: %s  ", __LINE__, #cond);                                       \
            std::printf(__VA_ARGS__);                                                            \
            std::printf("\n");                                                                   \
            g_failed = true;                                                                     \
        }                                                                                        \
    } while (0)
static int finish()
{
    if (g_failed) return 1;
    std::printf("OK %ld\n", g_checked);
    return 0;
}
