// Device memory of handles and servers: fault injection, slabs that finished
// jobs leave to the next ones, arenas and the buffers cut from them.
#pragma once

#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <vector>

namespace lv {

// Allocation with optional fault injection for tests of the out-of-memory
// paths: with LV_FAULT_ALLOC_AT=k in the environment, the k-th device or
// pinned-host allocation made by one entry-point call on the calling thread
// fails with out-of-memory.  The variable is read at the start of every
// graph-creation, louvain, lpa and modularity call (FaultScope), so a test may
// change it between calls.
inline thread_local long t_alloc_count = 0;
inline thread_local long t_fail_at = 0;
struct FaultScope {
    FaultScope()
    {
        t_alloc_count = 0;
        const char* v = std::getenv("LV_FAULT_ALLOC_AT");
        t_fail_at = v ? std::atol(v) : 0L;
    }
};
inline bool fault_now()
{
    ++t_alloc_count;
    return t_fail_at > 0 && t_alloc_count == t_fail_at;
}
inline hipError_t dev_alloc(void** p, size_t bytes)
{
    if (fault_now()) { *p = nullptr; return hipErrorOutOfMemory; }
    return hipMalloc(p, bytes ? bytes : 1);
}

// Device memory that arenas take from and give back to.  Owned by a server
// (its jobs' graphs come and go): keeps at most `bound` bytes of slabs for the
// next job and frees them when it is destroyed, when the server's budget needs
// them (shrink) and when any of the server's allocations finds no memory.
struct Slab {
    char* p = nullptr;
    size_t size = 0;
};
class SlabCache {
public:
    explicit SlabCache(size_t bound) : bound_(bound) {}
    ~SlabCache() { flush(); }
    SlabCache(const SlabCache&) = delete;
    SlabCache& operator=(const SlabCache&) = delete;
    // the smallest kept slab of at least `bytes` (and at most four times that)
    bool take(size_t bytes, Slab& out)
    {
        std::lock_guard<std::mutex> lk(mu_);
        int best = -1;
        for (int t = 0; t < (int)kept_.size(); ++t)
            if (kept_[t].size >= bytes && kept_[t].size / 4 <= bytes && (best < 0 || kept_[t].size < kept_[best].size))
                best = t;
        if (best < 0) return false;
        out = kept_[best];
        held_ -= out.size;
        kept_.erase(kept_.begin() + best);
        return true;
    }
    void put(const Slab& sl)
    {
        {
            std::lock_guard<std::mutex> lk(mu_);
            try {
                if (held_ + sl.size <= bound_) {
                    kept_.push_back(sl);
                    held_ += sl.size;
                    return;
                }
            } catch (const std::bad_alloc&) {  // no host memory to keep it by
            }
        }
        (void)hipFree(sl.p);
    }
    void flush() { shrink(0); }
    // free slabs until at most `bytes` are kept, the largest first
    void shrink(size_t bytes)
    {
        std::lock_guard<std::mutex> lk(mu_);
        while (held_ > bytes) {
            const auto big = std::max_element(kept_.begin(), kept_.end(),
                                              [](const Slab& a, const Slab& b) { return a.size < b.size; });
            (void)hipFree(big->p);
            held_ -= big->size;
            kept_.erase(big);
        }
    }
    size_t held()
    {
        std::lock_guard<std::mutex> lk(mu_);
        return held_;
    }

private:
    std::mutex mu_;
    std::vector<Slab> kept_;
    size_t held_ = 0;
    const size_t bound_;
};

// The device memory of one handle: a few large slabs that its buffers are cut
// from (best fit, neighbours joined when freed), given back when the
// handle goes.  A run on a fresh handle made some 85 allocations, and freeing
// a block of 4 MiB or more costs 0.2-0.9 ms each (the device is drained and
// the block unmapped): of the 38 ms that a job of 16 M entries took from host
// arrays to host labels, 18 were spent there.  Every buffer of an arena is used on the
// handle's stream (a freed block's next user is ordered after its last) or
// after the host has waited for that stream.  Running out of host memory is
// out-of-memory like any other: nothing here throws.
// cache: slabs come from there and go back there (share), or it is only emptied
// when there is no memory (not share: a server's worker, which keeps its slabs).
class Arena {
public:
    explicit Arena(std::shared_ptr<SlabCache> cache = nullptr, bool share = true)
        : cache_(std::move(cache)), share_(share && cache_)
    {
    }
    ~Arena()
    {
        for (auto& r : slabs_) {
            if (share_) cache_->put(r.slab);
            else (void)hipFree(r.slab.p);
        }
    }
    Arena(const Arena&) = delete;
    Arena& operator=(const Arena&) = delete;
    // `keep`: a buffer that the handle keeps between calls, or one that is gone
    // before those come.  They and the others (scratch) come from slabs of
    // their own as far as those have room, and from the end of a free block, so
    // that trim() finds the scratch slabs empty.  bytes: a multiple of 256.
    hipError_t alloc(size_t bytes, bool keep, void** out)
    {
        std::lock_guard<std::mutex> lk(mu_);
        if (carve(bytes, keep, out)) return hipSuccess;
        // scratch grows by half of what is held, at least 1 MiB and at most 256 MiB at a time
        // (by an eighth: a job of 16 M entries 15.3 ms, 14.4 so)
        const size_t extra = keep ? 0 : std::min<size_t>(std::max<size_t>(held_ / 2, MIN_SLAB), (size_t)256 << 20);
        hipError_t e = grow(std::max(bytes, extra), keep);
        if (e == hipErrorOutOfMemory) e = grow(bytes, keep);
        if (e != hipSuccess) return e;
        return carve(bytes, keep, out) ? hipSuccess : hipErrorOutOfMemory;
    }
    void free(void* p, size_t bytes)
    {
        std::lock_guard<std::mutex> lk(mu_);
        for (auto& r : slabs_) {
            if ((char*)p < r.slab.p || (char*)p >= r.slab.p + r.slab.size) continue;
            size_t at = (size_t)((char*)p - r.slab.p);
            auto nx = r.free.lower_bound(at);
            if (nx != r.free.end() && at + bytes == nx->first) {
                bytes += nx->second;
                nx = r.free.erase(nx);
            }
            if (nx != r.free.begin()) {
                auto pv = std::prev(nx);
                if (pv->first + pv->second == at) {
                    pv->second += bytes;
                    return;
                }
            }
            try {
                r.free.emplace(at, bytes);
            } catch (const std::bad_alloc&) {  // unused until the arena goes
            }
            return;
        }
    }
    // Make sure that about `keep` and `scratch` bytes are free for either kind,
    // in one more slab each if they are not (a hint: a failure is left to the
    // allocations that follow).  Little memory, and that of a server's job,
    // comes as one slab: there is nothing to trim.
    void reserve(size_t keep, size_t scratch)
    {
        std::lock_guard<std::mutex> lk(mu_);
        size_t have[2] = {0, 0};
        for (auto& r : slabs_)
            for (auto& f : r.free) have[r.keep] += f.second;
        if (share_ || keep + scratch <= TRIM_MIN) {
            have[0] += have[1];
            scratch += keep;
            keep = 0;
        }
        if (have[1] < keep) (void)grow(keep - have[1], true);
        if (have[0] < scratch) (void)grow(scratch - have[0], false);
    }
    // Give slabs without a buffer in them back to the device, if that is more
    // than TRIM_MIN bytes.  Everything queued on the handle's stream is done.
    void trim()
    {
        std::lock_guard<std::mutex> lk(mu_);
        const auto empty = [](const Region& r) { return r.free.size() == 1 && r.free.begin()->second == r.slab.size; };
        size_t unused = 0;
        for (auto& r : slabs_)
            if (empty(r)) unused += r.slab.size;
        if (share_ || unused <= TRIM_MIN) return;
        for (auto it = slabs_.begin(); it != slabs_.end();) {
            if (empty(*it)) {
                (void)hipFree(it->slab.p);
                held_ -= it->slab.size;
                it = slabs_.erase(it);
            } else {
                ++it;
            }
        }
    }
    // bytes of its slabs, used and free
    size_t held()
    {
        std::lock_guard<std::mutex> lk(mu_);
        return held_;
    }
    // bytes of slabs taken from the cache beyond what was asked for
    size_t surplus()
    {
        std::lock_guard<std::mutex> lk(mu_);
        return surplus_;
    }

private:
    static constexpr size_t MIN_SLAB = (size_t)1 << 20;
    static constexpr size_t TRIM_MIN = (size_t)8 << 20;
    struct Region {
        Slab slab;
        bool keep = false;
        std::map<size_t, size_t> free;  // offset -> length, no two adjacent
    };
    // the smallest free block that fits, of a slab of the same kind if there is one
    bool carve(size_t bytes, bool keep, void** out)
    {
        Region* br = nullptr;
        std::map<size_t, size_t>::iterator best;
        for (auto& r : slabs_)
            for (auto it = r.free.begin(); it != r.free.end(); ++it) {
                if (it->second < bytes) continue;
                const bool kind = r.keep == keep, best_kind = br && br->keep == keep;
                if (!br || (kind && !best_kind) || (kind == best_kind && it->second < best->second)) {
                    br = &r;
                    best = it;
                }
            }
        if (!br) return false;
        const size_t at = best->first, len = best->second;
        if (keep) {
            *out = br->slab.p + at + (len - bytes);
            if (len == bytes) br->free.erase(best);
            else best->second = len - bytes;
        } else {
            *out = br->slab.p + at;
            auto node = br->free.extract(best);
            if (len > bytes) {
                node.key() = at + bytes;
                node.mapped() = len - bytes;
                br->free.insert(std::move(node));
            }
        }
        return true;
    }
    hipError_t grow(size_t bytes, bool keep)
    {
        bytes = (std::max(bytes, MIN_SLAB) + 0xFFFFF) & ~(size_t)0xFFFFF;
        Region r;
        try {  // all the host memory it takes, before the device's
            slabs_.reserve(slabs_.size() + 1);
            r.free.emplace(0, 0);
        } catch (const std::bad_alloc&) {
            return hipErrorOutOfMemory;
        }
        if (share_ && cache_->take(bytes, r.slab)) {
            surplus_ += r.slab.size - bytes;
        } else {
            void* p = nullptr;
            hipError_t e = hipMalloc(&p, bytes);
            if (e == hipErrorOutOfMemory && cache_) {
                cache_->flush();
                (void)hipGetLastError();
                e = hipMalloc(&p, bytes);
            }
            if (e != hipSuccess) {
                (void)hipGetLastError();
                return e;
            }
            r.slab.p = (char*)p;
            r.slab.size = bytes;
        }
        held_ += r.slab.size;
        r.free.begin()->second = r.slab.size;
        r.keep = keep;
        slabs_.push_back(std::move(r));
        return hipSuccess;
    }
    std::mutex mu_;
    std::vector<Region> slabs_;
    size_t held_ = 0;
    size_t surplus_ = 0;
    std::shared_ptr<SlabCache> cache_;
    const bool share_;
};

// Grow-only device buffer, of an arena or (without one) an allocation of its own.
struct DevBuf {
    void* p = nullptr;
    size_t cap = 0;
    std::shared_ptr<Arena> arena;  // where the next allocation comes from
    bool keep = false;             // see Arena::alloc
    std::shared_ptr<Arena> from;   // where p came from
    DevBuf() = default;
    explicit DevBuf(std::shared_ptr<Arena> a, bool keep_ = false) : arena(std::move(a)), keep(keep_) {}
    DevBuf(const DevBuf&) = delete;
    DevBuf& operator=(const DevBuf&) = delete;
    ~DevBuf() { release(); }
    void release()
    {
        if (p) {
            if (from) from->free(p, cap);
            else (void)hipFree(p);
        }
        p = nullptr;
        cap = 0;
        from.reset();
    }
    hipError_t ensure(size_t bytes)
    {
        bytes = (bytes + 255) & ~(size_t)255;
        if (bytes == 0) bytes = 256;
        if (cap >= bytes) return hipSuccess;
        release();
        hipError_t e;
        if (arena) {
            e = fault_now() ? hipErrorOutOfMemory : arena->alloc(bytes, keep, &p);
            if (e == hipSuccess) from = arena;
        } else {
            e = dev_alloc(&p, bytes);
        }
        if (e == hipSuccess) cap = bytes; else p = nullptr;
        return e;
    }
    template <typename T> T* as() const { return (T*)p; }
    void swap(DevBuf& o)
    {
        std::swap(p, o.p);
        std::swap(cap, o.cap);
        std::swap(from, o.from);
    }
};

}  // namespace lv
