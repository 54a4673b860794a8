// pc_slabs.h -- host memory of the RA/DEC conversion's slabs (host code only).
//
// Pinned where the system gives pinned memory, so that copies run beside the
// conversion; pageable where it refuses, as the columns were converted before
// they were slabs (the caller then waits for every copy).
#pragma once
#include <stddef.h>
#include <stdlib.h>

namespace pc {

class HostSlabs {
public:
    // At least `want` bytes, contents lost when it grows; false when there is
    // neither kind.  pin(void **, size_t) and unpin(void *) return 0 on success.
    template <class Pin, class Unpin>
    bool grow(size_t want, Pin pin, Unpin unpin)
    {
        if (cap_ >= want)
            return true;
        release(unpin);
        pinned_ = pin(&p_, want) == 0;
        if (!pinned_)
            p_ = malloc(want);
        if (!p_)
            return false;
        cap_ = want;
        return true;
    }
    template <class Unpin>
    void release(Unpin unpin)
    {
        if (p_ && pinned_)
            (void)unpin(p_);
        else
            free(p_);
        p_ = nullptr;
        cap_ = 0;
    }
    char *data() const { return static_cast<char *>(p_); }
    size_t size() const { return cap_; }
    bool pinned() const { return pinned_; }

private:
    void *p_ = nullptr;
    size_t cap_ = 0;
    bool pinned_ = false;
};

}  // namespace pc
