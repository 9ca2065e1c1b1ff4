// Pinned host buffers that wait for the next call of any handle and thread:
// which of them a call gets, and which are kept when it ends.  No HIP in here.
#pragma once

#include <cstddef>
#include <mutex>

namespace mcl {

struct PinnedBuffer {
    void* host = nullptr;
    void* dev = nullptr;
    size_t bytes = 0;
    int device = 0;
};

class PinnedPool {
public:
    // At most kKept buffers of at most kMost bytes each.
    static constexpr int kKept = 8;
    static constexpr size_t kMost = size_t(4) << 20;

    // The smallest kept buffer of the device with room for `bytes` (so that a
    // small call leaves the large ones to those that need them), if any.
    bool take(size_t bytes, int device, PinnedBuffer& out)
    {
        std::lock_guard<std::mutex> lk(mu_);
        int best = -1;
        for (int i = 0; i < n_; ++i)
            if (b_[i].bytes >= bytes && b_[i].device == device && (best < 0 || b_[i].bytes < b_[best].bytes)) best = i;
        if (best < 0) return false;
        out = b_[best];
        b_[best] = b_[--n_];
        return true;
    }

    // Keeps b; when there are kKept already, in place of the smallest one if that
    // is smaller.  Returns the buffer that is to be freed (host null: none).
    PinnedBuffer give(const PinnedBuffer& b)
    {
        if (b.bytes > kMost) return b;
        std::lock_guard<std::mutex> lk(mu_);
        if (n_ < kKept) {
            b_[n_++] = b;
            return PinnedBuffer();
        }
        int least = 0;
        for (int i = 1; i < n_; ++i)
            if (b_[i].bytes < b_[least].bytes) least = i;
        if (b_[least].bytes >= b.bytes) return b;
        const PinnedBuffer out = b_[least];
        b_[least] = b;
        return out;
    }

private:
    std::mutex mu_;
    PinnedBuffer b_[kKept];
    int n_ = 0;
};

}  // namespace mcl
