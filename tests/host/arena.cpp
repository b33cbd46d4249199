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
        job->reserve(0, first);
        CHECK(job->surplus() == (first == 40 * MiB ? 0 : 28 * MiB));
    }
    auto small = std::make_shared<Arena>(cache);
    small->reserve(0, 9 * MiB);  // a slab of more than four times the request stays where it is
    CHECK(small->surplus() == 0 && cache->held() == 40 * MiB);
    auto alone = std::make_shared<Arena>();
    alone->reserve(0, 5 * MiB);
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
        a->reserve(0, 10 * MiB);
        b->reserve(0, 30 * MiB);
        c->reserve(0, 20 * MiB);
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

// Buffers that are kept and those that are not lie in slabs of their own as far
// as these have room; trimming frees the slabs that are empty then.
int scratch_is_trimmed()
{
    device().limit = 100 * MiB;
    auto arena = std::make_shared<Arena>();
    DevBuf kept(arena, true), given(arena), over(arena, true), more(arena);
    arena->reserve(8 * MiB, 20 * MiB);
    CHECK(device().live.size() == 2 && arena->held() == 28 * MiB);
    CHECK(given.ensure(8 * MiB) == hipSuccess && over.ensure(8 * MiB) == hipSuccess);
    CHECK(more.ensure(12 * MiB) == hipSuccess && device().live.size() == 2);
    over.release();  // the kept buffer takes its place
    CHECK(kept.ensure(8 * MiB) == hipSuccess && device().live.size() == 2);
    arena->trim();
    CHECK(arena->held() == 28 * MiB);
    more.release();
    given.release();
    arena->trim();
    CHECK(arena->held() == 8 * MiB && device().used == 8 * MiB);
    CHECK(given.ensure(3 * MiB) == hipSuccess);  // of a new slab
    given.release();
    arena->trim();  // too little to be worth a call
    CHECK(device().live.size() == 2);
    auto small = std::make_shared<Arena>();
    small->reserve(3 * MiB, 5 * MiB);
    CHECK(device().live.size() == 3);
    auto job = std::make_shared<Arena>(std::make_shared<SlabCache>(MiB));
    job->reserve(10 * MiB, 10 * MiB);  // a server's job: one slab, nothing trimmed
    job->trim();
    CHECK(device().live.size() == 4 && job->held() == 20 * MiB);
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
            arena->reserve(0, 8 * MiB);
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
    const int r = worker_empties_the_cache() + surplus_is_reported() + shrink_to_the_budget() + scratch_is_trimmed() +
                  host_memory_runs_out();
    if (r == 0 && device().used == 0) std::printf("ok\n");
    return r == 0 && device().used == 0 ? 0 : 1;
}
