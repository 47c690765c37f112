// Host-only helper, free of HIP so that it can be tested by itself.
#pragma once
#include <atomic>
#include <cstddef>
#include <mutex>

namespace gcn {

// Remembers the largest value that `ask` was called with.  A caller that needs more asks first, so that whoever returns
// from reach() may rely on `value` having been asked for, and on nothing smaller having been asked for since: compare,
// call and store are one step for all threads (with the call outside the lock, of two threads the one with the smaller
// value could ask last and the larger one be remembered).
class LargestAsked {
public:
    template <class Ask>
    void reach(size_t value, const Ask& ask) {
        if (largest_.load(std::memory_order_acquire) >= value) return;
        std::lock_guard<std::mutex> lk(mu_);
        if (largest_.load(std::memory_order_relaxed) >= value) return;
        if (ask(value)) largest_.store(value, std::memory_order_release);
    }

private:
    std::mutex mu_;
    std::atomic<size_t> largest_{0};
};

}  // namespace gcn
