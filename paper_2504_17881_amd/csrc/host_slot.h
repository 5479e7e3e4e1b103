// Results of a reduction in pinned host memory (host code).
#pragma once

#include <cstdlib>
#include <mutex>

#include "internal.h"

namespace prx {

// Two doubles of pinned host memory that a kernel writes a result to: read
// after the stream's synchronisation, it saves the copy of a few bytes to
// pageable memory (15 of a small overlap's 27 us).  One page per process, made
// on first use; a slot is held for one call, and a call that finds none free
// takes the copy.  A slot comes back only through done(): where the wait for
// its kernel failed the kernel may still write to it, and nobody else gets it.
// The page is freed at exit (the handler is registered after the HIP runtime's
// own, so it runs before them) unless a slot is still held, by a thread that is
// inside a call or for good.
class HostSlot {
  public:
    HostSlot() {
        Pool &p = pool();
        std::lock_guard<std::mutex> lk(p.mu);
        if (!p.tried) {
            p.tried = true;
            // (allowed while another thread captures a stream)
            hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
            const bool swapped = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
            void *q = nullptr;
            if (hipHostMalloc(&q, kSlots * kStride,
                              hipHostMallocPortable | hipHostMallocCoherent) == hipSuccess) {
                p.base = (char *)q;
                std::atexit([] {
                    std::lock_guard<std::mutex> l(pool().mu);
                    if (pool().free == ~0ull) (void)hipHostFree(pool().base);
                    pool().base = nullptr;
                });
            } else {
                (void)hipGetLastError();
            }
            if (swapped) (void)hipThreadExchangeStreamCaptureMode(&mode);
        }
        if (p.base && p.free) {
            at_ = __builtin_ctzll(p.free);
            p.free &= p.free - 1;
            ptr_ = (double *)(p.base + kStride * at_);
        }
    }
    HostSlot(const HostSlot &) = delete;
    HostSlot &operator=(const HostSlot &) = delete;
    double *ptr() const { return ptr_; }
    // The kernel that writes the slot has ended and its result is read.
    void done() {
        if (!ptr_) return;
        std::lock_guard<std::mutex> lk(pool().mu);
        pool().free |= 1ull << at_;
        ptr_ = nullptr;
    }

  private:
    static constexpr size_t kSlots = 64, kStride = 64;
    struct Pool {
        std::mutex mu;
        char *base = nullptr;
        uint64_t free = ~0ull;
        bool tried = false;
    };
    static Pool &pool() {
        static Pool *p = new Pool;  // outlives the exit handler
        return *p;
    }
    double *ptr_ = nullptr;
    int at_ = 0;
};

// Runs `launch(out)` with a host slot, or with `dev` where none is free, and
// waits for the two doubles it writes.
template <class F>
static prx_status read_back(F launch, double *dev, double h[2], hipStream_t s, const char *what) {
    HostSlot slot;
    double *out = slot.ptr() ? slot.ptr() : dev;
    hipError_t e = launch(out);
    if (e != hipSuccess) {
        // (part of the launches may be under way)
        if (hipStreamSynchronize(s) == hipSuccess) slot.done();
        return hip_fail(e, what);
    }
    if (!slot.ptr())
        PRX_HIP(hipMemcpyAsync(h, dev, 2 * sizeof(double), hipMemcpyDeviceToHost, s));
    PRX_HIP(hipStreamSynchronize(s));
    if (slot.ptr()) {
        h[0] = ((volatile double *)out)[0];
        h[1] = ((volatile double *)out)[1];
        slot.done();
    }
    return PRX_OK;
}

}  // namespace prx
