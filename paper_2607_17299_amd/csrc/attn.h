// Device helpers shared by the verify and the prefill attention.
#pragma once

#include "kernels.h"

// Keep the first n (0..8) bf16 elements of a fragment, zero the rest.  Slots at
// or beyond a sequence's end are never written and may hold any bit pattern;
// their softmax weight is 0, but 0 * NaN would still poison the product.
WAR_DEV uint4 keep_first(uint4 v, int n) {
  auto m = [n](int i) { return 2 * i + 1 < n ? 0xffffffffu : 2 * i < n ? 0x0000ffffu : 0u; };
  return make_uint4(v.x & m(0), v.y & m(1), v.z & m(2), v.w & m(3));
}

// The units a workgroup takes.  Its first one is its own id; the next ones come
// from per-class counters (class = workgroup id mod NC), so units of unequal
// length balance over the workgroups.  Workgroups are dealt to the 8 XCDs
// round-robin, so with 8 kv-heads every unit of one kv-head runs on the same
// XCD, and items that are neighbours in the work order (the same prefix chunk of
// sibling requests) share its L2.  The combine kernel that follows every launch
// resets the counters.  Atomics of the whole grid are slow (eight counters on one
// line, first units taken from them too: 384 units of up to 1024 keys 44.8 us
// against 34.9; 64 requests at 8192 tokens, 3 rows, over four layers 2541 ->
// 2510), so the counters are a line apart and a launch with no more units than
// workgroups uses none.
struct UnitQueue {
  int NC, cls, first, total;
  __device__ explicit UnitQueue(int total_) : total(total_) {
    NC = min(8, (int)gridDim.x);
    cls = blockIdx.x % NC;
    first = ((int)gridDim.x - cls + NC - 1) / NC;  // workgroups of the class
  }
  __device__ int next(int32_t* ctr) const {
    if (total <= (int)gridDim.x) return total;
    return (atomicAdd(&ctr[cls * kCtrStride], 1) + first) * NC + cls;
  }
};
