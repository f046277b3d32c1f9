// Host side: small reports in pinned memory that kernels write and calls read.
#pragma once

#include "common.h"

#include <mutex>
#include <vector>

namespace jitdb {

// A call takes a report and gives it back when its kernels are done with it; at most kKept stay allocated between calls.
template <typename R>
struct PinnedPool {
    static constexpr size_t kKept = 16;
    std::mutex lock;
    std::vector<R *> free_list;
    R *take() {
        {
            std::lock_guard<std::mutex> g(lock);
            if (!free_list.empty()) {
                R *r = free_list.back();
                free_list.pop_back();
                return r;
            }
        }
        void *p = nullptr;
        if (hipHostMalloc(&p, sizeof(R), hipHostMallocPortable | hipHostMallocMapped) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        return static_cast<R *>(p);
    }
    void give(R *r) {
        {
            std::lock_guard<std::mutex> g(lock);
            if (free_list.size() < kKept) {
                free_list.push_back(r);
                return;
            }
        }
        (void)hipHostFree(r);
    }
};

// Waits until ready() sees its word of the report.  A word in pinned memory is seen about 4 us sooner than hipStreamSynchronize returns (8.3
// against 12 us for an empty kernel), which is a large part of a small forest's analysis; work that takes longer
// than the spin is waited for in the ordinary way, which also reports a failed kernel.
template <typename Ready>
inline hipError_t wait_for_report(hipStream_t st, Ready &&ready) {
    for (int i = 0; i < 20000; ++i) {
        if (ready()) return hipSuccess;
        __builtin_ia32_pause();
    }
    return hipStreamSynchronize(st);
}

}  // namespace jitdb
