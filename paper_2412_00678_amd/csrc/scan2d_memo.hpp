// The launch plans a thread has used last.  Choosing a plan ranks dozens of kernel variants (5 us for a forward, with
// the workspace query 15 to 30 us per call: more than the kernels of a small map take) and depends on the descriptor, a
// few flags, the device and the tuning overrides only.  Each thread keeps its own few (no lock, bounded, gone with the
// thread); they hold no device memory.  A forward shape takes up to four of the sixteen entries (the workspace query ranks
// with and without the softplus step and aligned mask rows), a backward shape one per form: a loop over more than four
// grids ranks again on every call.
#pragma once

#include <hip/hip_runtime.h>

#include "../../include/scan2d.h"
#include "scan2d_tuning.hpp"

namespace scan2d {

template <typename Plan>
class PlanMemo {
public:
    // make(&plan) -> int (0: the plan is valid); its result is kept either way.
    template <typename Make>
    int get(const scan2d_desc& d, unsigned flags, Plan* out, Make make) {
        int dev = -1;
        (void)hipGetDevice(&dev);
        const unsigned gen = tune_generation();
        for (int i = 0; i < used_; ++i) {
            const Entry& e = e_[i];
            if (e.d.Bt == d.Bt && e.d.Dc == d.Dc && e.d.H == d.H && e.d.W == d.W && e.d.N == d.N && e.d.dtype == d.dtype && e.d.flags == d.flags &&
                e.flags == flags && e.dev == dev && e.gen == gen) {
                if (e.rc == 0) *out = e.plan;
                return e.rc;
            }
        }
        Entry& e = e_[next_];
        next_ = (next_ + 1) % kEntries;
        if (used_ < kEntries) ++used_;
        e.d = d; e.flags = flags; e.dev = dev; e.gen = gen;
        e.plan = Plan();
        e.rc = make(&e.plan);
        if (e.rc == 0) *out = e.plan;
        return e.rc;
    }

private:
    static constexpr int kEntries = 16;
    struct Entry {
        scan2d_desc d;
        unsigned flags, gen;
        int dev, rc;
        Plan plan;
    };
    Entry e_[kEntries];
    int used_ = 0, next_ = 0;
};

}  // namespace scan2d
