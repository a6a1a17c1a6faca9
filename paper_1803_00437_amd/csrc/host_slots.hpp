// Slots of pinned host memory that results of a few numbers are written to: a copy to pageable memory is
// one more operation on the stream, staged through a buffer of the runtime (a read of 64^2 takes 26 us
// with the copy, 17.5 without).
//
// All slots of a process lie in one page.  It takes 85 to 150 us to allocate, so it pays after 10 to 18
// reads: it is allocated at the FIRST_READS-th read without one, whichever contexts read, and kept until
// the process ends (freeing it could wait for other streams' work, and destroying a context would be a
// device call).  A context holds its slot until it is destroyed; contexts beyond SLOTS, or all if the
// page cannot be had, go without.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <mutex>

namespace fdlbm {

class HostSlots {
public:
    static constexpr int FIRST_READS = 20, SLOTS = 64;
    // alloc(bytes): the page, or null
    HostSlots(size_t doubles, double *(*alloc)(size_t)) : doubles_(doubles), alloc_(alloc) {}

    // at a read of a context that has no slot: one, or null
    double *take()
    {
        std::lock_guard<std::mutex> lock(mu_);
        if (used_ == ~uint64_t(0) || reads_ > FIRST_READS) return nullptr;
        if (!page_) {
            if (++reads_ < FIRST_READS) return nullptr;
            page_ = alloc_(SLOTS * doubles_ * sizeof(double));
            if (!page_) {
                reads_ = FIRST_READS + 1;  // not again
                return nullptr;
            }
        }
        const int i = __builtin_ctzll(~used_);
        used_ |= uint64_t(1) << i;
        return page_ + (size_t)i * doubles_;
    }

    void give(double *slot)
    {
        if (!slot) return;
        std::lock_guard<std::mutex> lock(mu_);
        used_ &= ~(uint64_t(1) << ((size_t)(slot - page_) / doubles_));
    }

private:
    const size_t doubles_;
    double *(*const alloc_)(size_t);
    std::mutex mu_;
    double *page_ = nullptr;
    uint64_t used_ = 0;  // one bit per slot
    int reads_ = 0;
};

}  // namespace fdlbm
