// Pinned host staging blocks, reused across calls: a call takes one, uploads
// from it and lets a kernel write its results into it, and returns it after
// its stream is drained. Allocating and freeing one takes longer (24 us) than
// a small count's kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <mutex>
#include <vector>

namespace tn {

class PinnedPool {
  public:
    static constexpr size_t kUpload = size_t(256) << 10;  // staging bytes
    static constexpr size_t kResults = 128 * 8;           // result words of one call
    static constexpr size_t kKeep = 8;                    // free blocks held (2 MiB)

    static PinnedPool& get() {
        static PinnedPool* p = new PinnedPool;  // outlives every thread's use
        return *p;
    }
    // nullptr: no pinned memory to be had (the caller takes another way)
    uint8_t* take() {
        {
            std::lock_guard<std::mutex> lk(mu_);
            if (!free_.empty()) {
                uint8_t* b = free_.back();
                free_.pop_back();
                return b;
            }
        }
        void* p = nullptr;
        // portable: usable from every device of the process
        if (hipHostMalloc(&p, kUpload + kResults, hipHostMallocPortable) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        return static_cast<uint8_t*>(p);
    }
    void give(uint8_t* b) {
        {
            std::lock_guard<std::mutex> lk(mu_);
            if (free_.size() < kKeep) {
                free_.push_back(b);
                return;
            }
        }
        (void)hipHostFree(b);
    }

  private:
    std::mutex mu_;
    std::vector<uint8_t*> free_;
};

// A block for the length of a call. Between in_use and drained a stream may
// read and write it: a call that ends in between waits for the stream, and
// where even that fails the block stays out of the pool, since the next call's
// results would lie where the stream may still write.
struct PinnedBlock {
    uint8_t* p = nullptr;
    explicit PinnedBlock(bool want) : p(want ? PinnedPool::get().take() : nullptr) {}
    ~PinnedBlock() {
        if (!p || (busy_ && hipStreamSynchronize(stream_) != hipSuccess)) return;
        PinnedPool::get().give(p);
    }
    void in_use(hipStream_t s) {
        stream_ = s;
        busy_ = true;
    }
    void drained() { busy_ = false; }
    PinnedBlock(const PinnedBlock&) = delete;
    PinnedBlock& operator=(const PinnedBlock&) = delete;
    uint64_t* results() const { return reinterpret_cast<uint64_t*>(p + PinnedPool::kUpload); }

  private:
    hipStream_t stream_ = nullptr;
    bool busy_ = false;
};

}  // namespace tn
