// partition.h -- the integer arithmetic of the work partition: where a
// worker's range of global pages starts, which worker holds a page, and which
// workers and workspace slots hold the pieces of a unit.  Plain C++, so that it
// is the same function on the host (launches, tests) and in the kernels.
#pragma once

#include <stdint.h>

#ifdef __HIP__
#define TS_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define TS_HOST_DEVICE inline
#endif

namespace tsattn {

TS_HOST_DEVICE int64_t worker_begin(int64_t ptot, int w, int W) { return (ptot * (int64_t)w) / (int64_t)W; }

// floor((2^32 - 1) / ranges), for range_start.
TS_HOST_DEVICE uint32_t range_reciprocal(int ranges) { return 0xffffffffu / (uint32_t)ranges; }

// worker_begin(ptot, w, ranges) with inv = range_reciprocal(ranges): in 32 bits
// the high word of the product with it is at most one below the quotient, since
// it differs from the exact value by at most x / 2^32 < 1 (exactly that for
// ranges = 1).
TS_HOST_DEVICE int64_t range_start(int64_t ptot, int w, int ranges, uint32_t inv) {
    const uint64_t x = (uint64_t)ptot * (uint32_t)w;
    if (x >> 32)
        return worker_begin(ptot, w, ranges);
    const uint32_t q = (uint32_t)(((uint64_t)(uint32_t)x * inv) >> 32);
    return q + ((uint32_t)x - q * (uint32_t)ranges >= (uint32_t)ranges);
}

// Worker whose range holds global page x (0 <= x < ptot).
TS_HOST_DEVICE int worker_of(int64_t ptot, int64_t x, int W) { return (int)(((x + 1) * (int64_t)W - 1) / ptot); }

// The workers whose ranges meet the unit that occupies global pages
// [us, us + np), and the workspace slot of the k-th piece (k = 0 .. nparts-1,
// in worker order).  When every worker has at least one page (ptot >= W),
// worker wlo + k, k > 0, began inside the unit (slot 2 (wlo + k)) and only
// wlo's start needs comparing with us.  Otherwise every range holds at most
// one page, so page us + k of the unit is the whole range of worker
// worker_of(us + k), which began there (slot 2 worker_of(us + k)).
struct UnitSplit {
    int64_t ptot;     // pages of the whole call
    int64_t us;       // global index of the unit's first page
    int W;            // workers
    int wlo, whi;     // first and last worker whose range meets the unit
    int first_slot;   // slot of worker wlo's piece
    bool dense;       // ptot >= W
    int nparts;       // workers with a non-empty piece of the unit
    TS_HOST_DEVICE int slot(int k) const {
        if (dense)
            return k == 0 ? first_slot : 2 * (wlo + k);
        return 2 * worker_of(ptot, us + k, W);
    }
};

TS_HOST_DEVICE UnitSplit unit_split(int64_t ptot, int64_t us, int np, int W) {
    UnitSplit u;
    u.ptot = ptot;
    u.us = us;
    u.W = W;
    u.wlo = worker_of(ptot, us, W);
    u.whi = worker_of(ptot, us + np - 1, W);
    u.dense = ptot >= W;
    u.first_slot = worker_begin(ptot, u.wlo, W) >= us ? 2 * u.wlo : 2 * u.wlo + 1;
    u.nparts = u.dense ? u.whi - u.wlo + 1 : np;
    return u;
}

}  // namespace tsattn
