// First-fit allocator over [0, inf) with a coalescing free list, used to lay
// out tensors of known lifetimes (global arenas and a work-group's LDS).
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <utility>
#include <vector>

namespace tn {

struct Arena {
    std::vector<std::pair<int64_t, int64_t>> free_;  // (offset, size), by offset
    int64_t top = 0;
    int64_t high = 0;
    int64_t alloc(int64_t n) {
        for (size_t i = 0; i < free_.size(); ++i)
            if (free_[i].second >= n) {
                const int64_t off = free_[i].first;
                if (free_[i].second == n) {
                    free_.erase(free_.begin() + std::ptrdiff_t(i));
                } else {
                    free_[i].first += n;
                    free_[i].second -= n;
                }
                return off;
            }
        const int64_t off = top;
        top = off + n;
        high = std::max(high, top);
        return off;
    }
    void release(int64_t off, int64_t n) {
        size_t i = size_t(std::lower_bound(free_.begin(), free_.end(), std::make_pair(off, int64_t(0))) - free_.begin());
        free_.insert(free_.begin() + std::ptrdiff_t(i), {off, n});
        if (i + 1 < free_.size() && free_[i].first + free_[i].second == free_[i + 1].first) {
            free_[i].second += free_[i + 1].second;
            free_.erase(free_.begin() + std::ptrdiff_t(i) + 1);
        }
        if (i > 0 && free_[i - 1].first + free_[i - 1].second == free_[i].first) {
            free_[i - 1].second += free_[i].second;
            free_.erase(free_.begin() + std::ptrdiff_t(i));
            --i;
        }
        if (free_[i].first + free_[i].second == top) {
            top = free_[i].first;
            free_.erase(free_.begin() + std::ptrdiff_t(i));
        }
    }
};

}  // namespace tn
