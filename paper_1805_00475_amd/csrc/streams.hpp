// Side streams for independent work of one call, reused across calls: a call
// takes some for its length and returns them drained. Creating one takes
// longer than a small batch.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <mutex>
#include <utility>
#include <vector>

namespace tn {

struct SideStream {
    hipStream_t stream = nullptr;
    hipEvent_t event = nullptr;
};

class StreamPool {
  public:
    static constexpr size_t kKeep = 16;  // idle streams held, all devices together

    static StreamPool& get() {
        static StreamPool* p = new StreamPool;  // outlives every thread's use
        return *p;
    }
    // a stream of the current device (stream null: none to be had)
    SideStream take(int device) {
        {
            std::lock_guard<std::mutex> lk(mu_);
            for (size_t i = 0; i < idle_.size(); ++i)
                if (idle_[i].first == device) {
                    const SideStream s = idle_[i].second;
                    idle_.erase(idle_.begin() + std::ptrdiff_t(i));
                    return s;
                }
        }
        SideStream s;
        if (hipStreamCreateWithFlags(&s.stream, hipStreamNonBlocking) != hipSuccess) {
            (void)hipGetLastError();
            return SideStream{};
        }
        if (hipEventCreateWithFlags(&s.event, hipEventDisableTiming) != hipSuccess) {
            (void)hipGetLastError();
            (void)hipStreamDestroy(s.stream);
            return SideStream{};
        }
        return s;
    }
    void give(int device, const SideStream& s) {
        {
            std::lock_guard<std::mutex> lk(mu_);
            if (idle_.size() < kKeep) {
                idle_.push_back({device, s});
                return;
            }
        }
        (void)hipEventDestroy(s.event);
        (void)hipStreamDestroy(s.stream);
    }

  private:
    std::mutex mu_;
    std::vector<std::pair<int, SideStream>> idle_;
};

// Waits for a stream where a scope ends before drained(): by an error's return
// or an exception. Declared after the host buffers that the stream's copies
// use, so that they go away behind it.
class DrainGuard {
  public:
    explicit DrainGuard(hipStream_t s) : stream_(s) {}
    ~DrainGuard() {
        if (!drained_) (void)hipStreamSynchronize(stream_);
    }
    DrainGuard(const DrainGuard&) = delete;
    DrainGuard& operator=(const DrainGuard&) = delete;
    void drained() { drained_ = true; }

  private:
    hipStream_t stream_;
    bool drained_ = false;
};

// Up to n side streams for the length of a call; they are drained before
// they go back.
class SideStreams {
  public:
    explicit SideStreams(int n) {
        if (n <= 0 || hipGetDevice(&device_) != hipSuccess) return;
        s_.reserve(size_t(n));
        for (int i = 0; i < n; ++i) {
            const SideStream s = StreamPool::get().take(device_);
            if (!s.stream) break;
            s_.push_back(s);
        }
    }
    ~SideStreams() {
        for (const SideStream& s : s_) {
            (void)hipStreamSynchronize(s.stream);
            StreamPool::get().give(device_, s);
        }
    }
    SideStreams(const SideStreams&) = delete;
    SideStreams& operator=(const SideStreams&) = delete;
    size_t size() const { return s_.size(); }
    const SideStream& operator[](size_t i) const { return s_[i]; }

  private:
    int device_ = 0;
    std::vector<SideStream> s_;
};

}  // namespace tn
