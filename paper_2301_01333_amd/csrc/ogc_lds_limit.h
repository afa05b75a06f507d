// The LDS limit of one kernel, which the runtime holds for each device by itself: raised when a launch needs more than any
// launch on that device did before.  One object per kernel, shared by all threads; the lock keeps raising and remembering
// together.  (Host C++ only, so that it can be tested without a device.)
#ifndef OGC_LDS_LIMIT_H
#define OGC_LDS_LIMIT_H

#include <stddef.h>
#include <mutex>

class OgcLdsLimit {
public:
    // set() raises the limit of `device` to `bytes` and returns 0, or an error, which is passed on and not remembered.
    template <class Set> int raise(int device, size_t bytes, Set set) {
        std::lock_guard<std::mutex> hold(mu_);
        const bool kept = device >= 0 && device < DEVICES;
        if (kept && bytes <= most_[device]) return 0;
        const int rc = set();
        if (rc == 0 && kept) most_[device] = bytes;
        return rc;
    }

private:
    enum { DEVICES = 64 };  // beyond them the limit is raised at every launch
    std::mutex mu_;
    size_t most_[DEVICES] = {};
};

#endif
