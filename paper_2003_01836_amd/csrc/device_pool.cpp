// device_pool.cpp -- idle device blocks kept for the next plan.
//
// A one-shot evaluation allocates and frees some 75 arrays (trees, lists, pairs, the
// plan's own): hipMalloc and hipFree took 3.8 ms of it at 10^6 points and 0.22 ms at
// 10^4, and a kernel that writes newly mapped memory pays for its first touch (the
// mutual pairs of 10^6 points in FP32-mixed: 11.5 ms against 9.7).  One-shot
// evaluations with the pool: 10^6 points FP32-mixed 26.6 to 21.1 ms, 10^4 points FP64
// 0.81 to 0.67 ms, and 0.50 ms with the small tables in one copy each (Pack).
//
// The pool holds at most kPoolBytes of idle blocks (least recently used ones are
// freed first).  It gives back blocks that stayed idle for kPoolIdle when the next
// object is released, and all of them when an allocation of this library finds the
// device out of memory or when the caller asks for it (bltc_release_memory); other
// allocators of the process have no way to reclaim them.  Blocks
// enter it only after a wait for the device (DeviceBlocks::release), so any thread
// and any stream may take them.  Its memory is not cleared: like hipMalloc's, a
// block's contents are undefined.
#include "device_pool.hpp"

#include <algorithm>
#include <chrono>
#include <list>
#include <map>
#include <mutex>
#include <utility>

namespace bltc {
namespace {

using Clock = std::chrono::steady_clock;
constexpr size_t kPoolBytes = size_t(2) << 30;   // 0.7% of the device's memory
constexpr std::chrono::seconds kPoolIdle(10);

class Pool {
public:
    // an idle block of at least `size` bytes, at most a quarter (and 4 KiB) larger
    bool take(int device, size_t size, void** p, size_t* got)
    {
        std::lock_guard<std::mutex> lock(mutex_);
        auto it = by_size_.lower_bound({device, size});
        if (it == by_size_.end() || it->first.first != device ||
            it->first.second > size + size / 4 + 4096)
            return false;
        *p = it->second->p;
        *got = it->first.second;
        idle_ -= it->first.second;
        lru_.erase(it->second);
        by_size_.erase(it);
        return true;
    }

    // keeps the block unless that takes memory that cannot be had
    bool put(int device, size_t size, void* p)
    {
        try {
            std::lock_guard<std::mutex> lock(mutex_);
            auto e = lru_.insert(lru_.end(), Entry{p, Clock::now(), {}});
            try {
                e->at = by_size_.emplace(std::make_pair(device, size), e);
            } catch (...) {
                lru_.erase(e);
                throw;
            }
            idle_ += size;
            return true;
        } catch (...) {
            return false;
        }
    }

    // frees the blocks beyond `limit` bytes and those put before `since`
    bool trim(size_t limit, Clock::time_point since)
    {
        bool any = false;
        for (;;) {
            void* p;
            {
                std::lock_guard<std::mutex> lock(mutex_);
                if (lru_.empty() || (idle_ <= limit && lru_.front().put >= since))
                    return any;
                p = lru_.front().p;
                idle_ -= lru_.front().at->first.second;
                by_size_.erase(lru_.front().at);
                lru_.pop_front();
            }
            (void)hipFree(p);
            any = true;
        }
    }

private:
    struct Entry;
    using Lru = std::list<Entry>;
    using BySize = std::multimap<std::pair<int, size_t>, Lru::iterator>;
    struct Entry {
        void* p;
        Clock::time_point put;
        BySize::iterator at;
    };
    std::mutex mutex_;
    Lru lru_;
    BySize by_size_;
    size_t idle_ = 0;
};

// never destroyed: plans may be destroyed while the process exits
Pool& pool()
{
    static Pool* const p = new Pool;
    return *p;
}

}  // namespace

// steps of 1/16 of the power of two below: sizes that differ a little (another set
// of points) fit each other's blocks; blocks that never enter the pool as they are
size_t block_bytes(size_t n)
{
    if (n > kPoolBytes)
        return n;
    size_t step = 512;
    while (step * 32 <= n)
        step *= 2;
    return (n + step - 1) / step * step;
}

bool release_idle_blocks()
{
    return pool().trim(0, Clock::time_point::max());
}

namespace {

template <class F>
hipError_t with_retry(F&& allocate)
{
    hipError_t e = allocate();
    if (e == hipErrorOutOfMemory && release_idle_blocks())
        e = allocate();
    // the error is the caller's to report, not for the next launch's check to find
    if (e != hipSuccess || hipPeekAtLastError() == hipErrorOutOfMemory)
        (void)hipGetLastError();
    return e;
}

}  // namespace

hipError_t device_malloc(void** p, size_t bytes)
{
    return with_retry([&] { return hipMalloc(p, bytes); });
}

hipError_t device_malloc_async(void** p, size_t bytes, hipStream_t s)
{
    return with_retry([&] { return hipMallocAsync(p, bytes, s); });
}

hipError_t DeviceBlocks::get(void** p, size_t bytes)
{
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess)
        return e;
    held_.emplace_back();   // may throw: before there is a block to lose
    size_t size = block_bytes(std::max<size_t>(bytes, 1));
    if (!pool().take(device, size, p, &size)) {
        e = hipMalloc(p, size);
        if (e == hipErrorOutOfMemory) {
            (void)hipGetLastError();
            size = std::max<size_t>(bytes, 1);
            e = device_malloc(p, size);
        }
    }
    if (e == hipSuccess)
        held_.back() = {*p, size, device};
    else
        held_.pop_back();
    return e;
}

void DeviceBlocks::release()
{
    if (held_.empty())
        return;
    // the smallest block is the one that is freed, and waited with
    size_t least = 0;
    int device = -1;
    bool same = hipGetDevice(&device) == hipSuccess;
    for (size_t i = 0; i < held_.size(); ++i) {
        same = same && held_[i].device == device;
        if (held_[i].size < held_[least].size)
            least = i;
    }
    std::swap(held_[least], held_.back());
    const bool idle = hipFree(held_.back().p) == hipSuccess && same;
    held_.pop_back();
    for (const Block& b : held_)
        if (!idle || b.size > kPoolBytes || !pool().put(b.device, b.size, b.p))
            (void)hipFree(b.p);
    held_.clear();
    (void)pool().trim(kPoolBytes, Clock::now() - kPoolIdle);
}

}  // namespace bltc
