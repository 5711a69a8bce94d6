/* A device of a few bytes on the host: what csrc/pool.hpp needs of the runtime, for tests/abi/pool_check.cpp. */
#pragma once
#include <cstddef>
#include <cstdlib>
#include <map>

enum hipError_t { hipSuccess = 0, hipErrorOutOfMemory = 2 };

struct FakeDevice {
    size_t room = 1000000, used = 0;
    int mallocs = 0, frees = 0, current = 0;
    std::map<void *, size_t> live;
};
inline FakeDevice &fake() { static FakeDevice d; return d; }

inline hipError_t hipMalloc(void **p, size_t bytes)
{
    FakeDevice &d = fake();
    if (d.used + bytes > d.room) return hipErrorOutOfMemory;
    *p = std::malloc(1);
    d.live[*p] = bytes;
    d.used += bytes;
    ++d.mallocs;
    return hipSuccess;
}
inline hipError_t hipFree(void *p)
{
    FakeDevice &d = fake();
    if (!d.live.count(p)) std::abort();
    d.used -= d.live[p];
    d.live.erase(p);
    ++d.frees;
    std::free(p);
    return hipSuccess;
}
inline hipError_t hipGetDevice(int *dev) { *dev = fake().current; return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
