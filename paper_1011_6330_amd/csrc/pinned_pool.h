// pinned_pool.h -- page-locked staging buffers of the read-outs (host code only).
//
// A read-out takes a buffer for the duration of its call (it waits for the GPU
// before it returns), so calls on several threads and streams each hold their
// own, allocated by a handle's second read-out.  At most PINNED_KEEP idle buffers
// of at most PINNED_MAX bytes are kept, and none once the last handle is gone.
// Buffers are allocated and freed in the relaxed capture mode, so that neither
// counts against a stream capture of another thread (an unsafe call during a capture
// in the global mode ends it); where an allocation fails the caller copies into its
// own pageable memory instead.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <stdint.h>

#include <mutex>

namespace pcpic {

// The calling thread's capture mode, relaxed for a scope.
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    RelaxedCapture(const RelaxedCapture &) = delete;
    RelaxedCapture &operator=(const RelaxedCapture &) = delete;
};

constexpr size_t PINNED_MIN = 64 << 10, PINNED_MAX = 4 << 20;
constexpr size_t PINNED_KEEP = 8;

class PinnedPool {
public:
    struct Block {
        void *p;
        size_t n;
    };
    void add_handle()
    {
        std::lock_guard<std::mutex> lock(mu_);
        ++handles_;
    }
    void drop_handle()
    {
        Block gone[PINNED_KEEP];
        size_t n = 0;
        {
            std::lock_guard<std::mutex> lock(mu_);
            if (--handles_ == 0) {
                for (; n < n_idle_; ++n) gone[n] = idle_[n];
                n_idle_ = 0;
            }
        }
        for (size_t k = 0; k < n; ++k) release(gone[k]);
    }
    // An idle buffer of at least n bytes, else (with `fresh`) a new one, else none.
    Block take(size_t n, bool fresh)
    {
        {
            std::lock_guard<std::mutex> lock(mu_);
            size_t best = n_idle_;
            for (size_t k = 0; k < n_idle_; ++k)
                if (idle_[k].n >= n && (best == n_idle_ || idle_[k].n < idle_[best].n)) best = k;
            if (best < n_idle_) {
                const Block b = idle_[best];
                idle_[best] = idle_[--n_idle_];
                return b;
            }
        }
        if (!fresh) return Block{nullptr, 0};
        size_t sz = PINNED_MIN;
        while (sz < n) sz *= 2;
        void *p = nullptr;
        RelaxedCapture relaxed;
        if (hipHostMalloc(&p, sz, hipHostMallocPortable) != hipSuccess) {
            (void)hipGetLastError();
            p = nullptr;
        }
        return Block{p, p ? sz : 0};
    }
    void give(const Block &b)
    {
        if (!b.p) return;
        {
            std::lock_guard<std::mutex> lock(mu_);
            if (handles_ > 0 && n_idle_ < PINNED_KEEP) {
                idle_[n_idle_++] = b;
                return;
            }
        }
        release(b);
    }

private:
    static void release(const Block &b)
    {
        RelaxedCapture relaxed;
        if (hipHostFree(b.p) != hipSuccess) (void)hipGetLastError();
    }

    std::mutex mu_;
    Block idle_[PINNED_KEEP] = {};
    size_t n_idle_ = 0;
    int64_t handles_ = 0;
};

}  // namespace pcpic
