// What the library has seen of a run's arrival (host side, plain C++).
#pragma once
#include <stdint.h>

#include <mutex>

namespace agg {

// The shards that copy kernels on one stream have been enqueued for, in one epoch.  keeps_order(): that stream runs what it is given in order,
// once; it asks the runtime, so it is called only where the answer counts.
class Delivered {
public:
    template <class F>
    void note(uint64_t ranks, int epoch, const void* stream, F&& keeps_order)
    {
        const bool kept = keeps_order();
        std::lock_guard<std::mutex> lock(mutex_);
        if (!kept || epoch_ != epoch || stream_ != stream) ranks_ = 0;
        epoch_ = epoch;
        stream_ = stream;
        if (kept) ranks_ |= ranks;
    }
    // All of W shards, in this epoch, on this stream.
    template <class F>
    bool all(int W, int epoch, const void* stream, F&& keeps_order)
    {
        {
            std::lock_guard<std::mutex> lock(mutex_);
            if (ranks_ != ~0ull >> (64 - W) || epoch_ != epoch || stream_ != stream) return false;
        }
        return keeps_order();
    }

private:
    std::mutex mutex_;
    uint64_t ranks_ = 0;       // a bit per rank
    int epoch_ = 0;
    const void* stream_ = nullptr;
};

}  // namespace agg
