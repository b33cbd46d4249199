// Stand-in for the HIP allocation calls that lv_arena.h makes: host memory
// under a limit, so that its bookkeeping can be tested without a GPU.
#pragma once
#include <cstddef>
#include <cstdlib>
#include <map>

typedef int hipError_t;
constexpr hipError_t hipSuccess = 0, hipErrorOutOfMemory = 2;

struct FakeDevice {
    std::map<void*, std::size_t> live;
    std::size_t used = 0, limit = ~(std::size_t)0;
    int fail_new = -1;    // host allocations left until one fails (tests)
    bool inside = false;  // the allocations of these functions do not count
};
inline FakeDevice& device()
{
    static FakeDevice d;
    return d;
}
inline hipError_t hipMalloc(void** p, std::size_t n)
{
    FakeDevice& d = device();
    if (d.used + n > d.limit) { *p = nullptr; return hipErrorOutOfMemory; }
    *p = std::malloc(n);
    d.inside = true;
    d.live[*p] = n;
    d.inside = false;
    d.used += n;
    return hipSuccess;
}
inline hipError_t hipFree(void* p)
{
    FakeDevice& d = device();
    auto it = d.live.find(p);
    if (it == d.live.end()) std::abort();  // freed twice, or never allocated
    d.used -= it->second;
    d.live.erase(it);
    std::free(p);
    return hipSuccess;
}
inline hipError_t hipGetLastError() { return hipSuccess; }
