// Which copy streams a context uses.  Contexts whose copies wait for the same compute stream share a
// pair: a copy of one is not ready before the copies another has already enqueued for that stream, so
// sharing costs next to nothing, and a process keeps within the device's few hardware queues (nets
// that each had a pair, swapping in turn on one stream at 128^3: 16.0 ms a step, 7.6 with a shared
// one -- some pair's waits stood in the compute stream's own queue).  Contexts of different compute
// streams have pairs of their own: a copy that waits for one stream holds up no other's.  No GPU
// dependency.
#pragma once
#include <mutex>
#include <vector>

#include "lms_engine.h"

namespace k3lms {

struct CopyPair {
    int device = -1;
    stream_t compute = nullptr;                 // the stream its copies wait for
    stream_t d2h = nullptr, h2d = nullptr;
    int users = 0;                              // contexts that use it now
    std::mutex enqueue;                         // held over operations that have to stay together
};

class CopyPool {
public:
    // The pair for copies that wait for `compute`, in exchange for `have` (null: none yet).  A pair that
    // nobody else uses follows its context to another stream; one that nobody uses at all is taken over.
    // create(pair) makes the streams of a new one and returns non-zero on failure (lease: null).
    template <class Create>
    CopyPair *lease(CopyPair *have, int device, stream_t compute, Create create)
    {
        if (have && have->compute == compute) return have;
        std::lock_guard<std::mutex> g(lock_);
        CopyPair *to = nullptr, *spare = nullptr;
        for (CopyPair *p : pairs_) {
            if (p->device != device) continue;
            if (p->users == 0) spare = p;
            else if (p->compute == compute) to = p;
        }
        if (!to && have && have->users == 1) {
            have->compute = compute;
            return have;
        }
        if (!to) to = spare;
        if (!to) {
            to = new CopyPair;
            to->device = device;
            if (create(*to)) {
                delete to;
                return nullptr;
            }
            pairs_.push_back(to);
        }
        to->compute = compute;
        ++to->users;
        if (have) --have->users;
        return to;
    }
    // Ends a context's use; returns the device's pairs without users, for the caller to wait for, destroy
    // and delete.
    std::vector<CopyPair *> give_back(CopyPair *have, int device)
    {
        std::lock_guard<std::mutex> g(lock_);
        if (have) --have->users;
        std::vector<CopyPair *> keep, out;
        for (CopyPair *p : pairs_) (p->device == device && p->users == 0 ? out : keep).push_back(p);
        pairs_.swap(keep);
        return out;
    }

private:
    std::mutex lock_;
    std::vector<CopyPair *> pairs_;
};

}  // namespace k3lms
