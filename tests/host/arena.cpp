// Device memory bookkeeping of lv_arena.h on a device of limited size.
#include "lv_arena.h"

#include <cstdio>

using namespace lv;

// the fail_new-th allocation from now on fails
void* operator new(std::size_t n)
{
    if (device().fail_new >= 0 && !device().inside && device().fail_new-- == 0) throw std::bad_alloc();
    if (void* p = std::malloc(n)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

#define CHECK(c)                                                         \
    do {                                                                 \
        if (!(c)) {                                                      \
            std::printf("%s:%d: %s\n", __FILE__, __LINE__, #c);          \
            return 1;                                                    \
        }                                                                \
    } while (0)

constexpr size_t MiB = (size_t)1 << 20;

// A worker's arena (not sharing the cache's slabs) gets the memory that the
// cache keeps when the device has no other.
int worker_empties_the_cache()
{
    device().limit = 100 * MiB;
    auto cache = std::make_shared<SlabCache>(80 * MiB);
    {
        auto job = std::make_shared<Arena>(cache);
        DevBuf b(job);
        CHECK(b.ensure(60 * MiB) == hipSuccess);
    }
    CHECK(cache->held() == 60 * MiB && device().used == 60 * MiB);
    {
        auto worker = std::make_shared<Arena>(cache, false);
        DevBuf b(worker);
        CHECK(b.ensure(70 * MiB) == hipSuccess);
        CHECK(cache->held() == 0);
    }
    CHECK(cache->held() == 0 && device().used == 0);  // a worker's slabs do not go to the cache
    return 0;
}

// Jobs take kept slabs; what a slab has beyond the request is reported.
int surplus_is_reported()
{
    device().limit = 100 * MiB;
    auto cache = std::make_shared<SlabCache>(80 * MiB);
    for (size_t first : {40 * MiB, 12 * MiB}) {
        auto job = std::make_shared<Arena>(cache);
        job->reserve(first);
        CHECK(job->surplus() == (first == 40 * MiB ? 0 : 28 * MiB));
    }
    auto small = std::make_shared<Arena>(cache);
    small->reserve(9 * MiB);  // a slab of more than four times the request stays where it is
    CHECK(small->surplus() == 0 && cache->held() == 40 * MiB);
    auto alone = std::make_shared<Arena>();
    alone->reserve(5 * MiB);
    CHECK(alone->surplus() == 0);
    return 0;
}

// The cache gives up its largest slabs until it holds no more than asked.
int shrink_to_the_budget()
{
    device().limit = 100 * MiB;
    auto cache = std::make_shared<SlabCache>(90 * MiB);
    {
        auto a = std::make_shared<Arena>(cache), b = std::make_shared<Arena>(cache), c = std::make_shared<Arena>(cache);
        a->reserve(10 * MiB);
        b->reserve(30 * MiB);
        c->reserve(20 * MiB);
    }
    CHECK(cache->held() == 60 * MiB);
    cache->shrink(60 * MiB);
    CHECK(cache->held() == 60 * MiB);
    cache->shrink(35 * MiB);
    CHECK(cache->held() == 30 * MiB && device().used == 30 * MiB);
    cache->shrink(0);
    CHECK(cache->held() == 0 && device().used == 0);
    return 0;
}

// Host memory that runs out in the middle of any of these is an error code or
// nothing at all, never an exception, and no device memory is lost.
int host_memory_runs_out()
{
    device().limit = 100 * MiB;
    for (int k = 0; k < 12; ++k) {
        auto cache = std::make_shared<SlabCache>(80 * MiB);
        {
            auto arena = std::make_shared<Arena>(cache);
            DevBuf a(arena), b(arena, true), c(arena), d(arena);
            device().fail_new = k;
            const hipError_t e = a.ensure(2 * MiB);
            CHECK(e == hipSuccess || e == hipErrorOutOfMemory);
            arena->reserve(8 * MiB);
            for (DevBuf* q : {&b, &c, &d}) (void)q->ensure(MiB);
            c.release();
            b.release();
            device().fail_new = -1;
            CHECK(a.ensure(2 * MiB) == hipSuccess && c.ensure(MiB) == hipSuccess);
            device().fail_new = k > 6 ? 0 : -1;  // while the slabs go to the cache
        }
        device().fail_new = -1;
    }
    CHECK(device().used == 0);
    return 0;
}

int main()
{
    const int r = worker_empties_the_cache() + surplus_is_reported() + shrink_to_the_budget() +
                  host_memory_runs_out();
    if (r == 0 && device().used == 0) std::printf("ok\n");
    return r == 0 && device().used == 0 ? 0 : 1;
}
