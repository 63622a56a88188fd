// A step that each device needs once before the first launch of a kernel.  Plain C++: nothing here needs HIP.
#pragma once
#include <atomic>
#include <mutex>

// hipFuncSetAttribute acts on the current device: a launcher keeps one of these per kernel and raises the kernel's dynamic LDS
// limit the first time it runs on each device (devices 0 .. 63).  Whoever comes while that is under way waits for it: a launch
// before the limit is raised is refused.  A step that failed is tried again by the next call.
class gvq_once_per_device {
public:
    template <typename F> int call(int device, F step)   // step: 0 = done; returns what it returned
    {
        const unsigned long long bit = 1ull << (device & 63);
        if (done.load(std::memory_order_acquire) & bit) return 0;
        std::lock_guard<std::mutex> guard(lock);
        if (done.load(std::memory_order_relaxed) & bit) return 0;
        const int rc = step();
        if (rc == 0) done.fetch_or(bit, std::memory_order_release);
        return rc;
    }

private:
    std::atomic<unsigned long long> done{0};
    std::mutex lock;
};
