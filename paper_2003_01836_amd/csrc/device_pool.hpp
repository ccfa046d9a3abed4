// device_pool.hpp -- device memory of plans and of the setup phase, reused from
// one object to the next (device_pool.cpp).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstring>
#include <utility>
#include <vector>

namespace bltc {

// hipMalloc; when the device is out of memory the pool's idle blocks are given
// back and the allocation is tried once more.
hipError_t device_malloc(void** p, size_t bytes);
// the same for hipMallocAsync
hipError_t device_malloc_async(void** p, size_t bytes, hipStream_t s);
// Frees the pool's idle blocks on every device; whether there were any.
bool release_idle_blocks();
// Size of the block taken for `n` bytes.
size_t block_bytes(size_t n);

// The device memory of one object, taken piece by piece and released together by
// the destructor.  One hipFree there waits for the device, as freeing every block
// would; then nothing enqueued on any stream uses the other blocks, and they go to
// the pool.  Not for memory that another process or library may still read.
class DeviceBlocks {
public:
    DeviceBlocks() = default;
    DeviceBlocks(const DeviceBlocks&) = delete;
    DeviceBlocks& operator=(const DeviceBlocks&) = delete;
    ~DeviceBlocks() { release(); }

    // at least max(1, bytes) bytes on the current device, contents undefined
    hipError_t get(void** p, size_t bytes);
    void release();

private:
    struct Block {
        void* p;
        size_t size;
        int device;
    };
    std::vector<Block> held_;
};

// Small host tables that go to the device in one copy (a copy costs the host some
// 6 us however small).  Every table starts on a 256-byte boundary of the block;
// tables larger than kMost are left to a copy of their own (add returns false).
// Must outlive the copy.
class Pack {
public:
    static constexpr size_t kMost = 1 << 16;

    template <class T>
    bool add(T** dst, const std::vector<T>& v)
    {
        const size_t n = v.size() * sizeof(T);
        if (n > kMost)
            return false;
        const size_t at = (host_.size() + 255) / 256 * 256;
        host_.resize(at + (n > 0 ? n : 1));
        if (n > 0)
            std::memcpy(host_.data() + at, v.data(), n);
        dst_.emplace_back(reinterpret_cast<void**>(dst), at);
        wanted_ += n > 0 ? n : 1;
        return true;
    }
    size_t bytes() const { return host_.size(); }
    size_t wanted() const { return wanted_; }   // without the padding

    // block: bytes() bytes on the device; sets the pointers of every table
    hipError_t send(void* block, hipStream_t s) const
    {
        for (const auto& d : dst_)
            *d.first = static_cast<char*>(block) + d.second;
        return hipMemcpyAsync(block, host_.data(), host_.size(), hipMemcpyHostToDevice, s);
    }
    // empty, for the next set of tables (the last copy has ended)
    void clear()
    {
        host_.clear();
        dst_.clear();
        wanted_ = 0;
    }

private:
    std::vector<char> host_;
    std::vector<std::pair<void**, size_t>> dst_;
    size_t wanted_ = 0;
};

}  // namespace bltc
