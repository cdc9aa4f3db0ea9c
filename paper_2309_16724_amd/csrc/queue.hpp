// Device side of the per-XCD work queues (see XcdQueues in plan.hpp).
#pragma once
#include <hip/hip_runtime.h>
#include "plan.hpp"

namespace dmrg {

// Work list of one worker (a wavefront or a work group) of a tile launch.
//
// Range r = blockIdx % NXCD of the list belongs to the workers of the blocks
// with that remainder, which the dispatcher places on one XCD.  A worker's
// first chunk (`chunk` consecutive tiles) is fixed by its index; the rest of
// the range is handed out through the range's atomic counter, and a worker
// whose range is used up helps the others.  Atomics on one address run one
// after the other (measured: about 60 per microsecond over eight counters in
// one 64-byte line, where every take and every failing probe of 16384
// wavefronts made the L=24, D=512 first stage take 4.9 ms for 292,000
// tiles).  So the counters lie QUEUE_STRIDE ints apart, ranges that the fixed
// chunks cover are never asked, the next chunk is requested before the
// current one is computed, and a worker without work reads all counters
// with one load before it takes from another range.
struct WorkQueue {
  const XcdQueues &q;
  int32_t *counters;
  int range, workers, chunk;   // current range, workers per range, tiles per chunk
  int t, tend;                 // current chunk [t, tend)
  int pend = 0;                // lane 0: chunk index the pending request returned
  bool asked = false;

  // tiles of range r that the counters hand out
  __device__ __forceinline__ int dynamic(int r) const {
    return max(0, q.start[r + 1] - q.start[r] - workers * chunk);
  }
  __device__ __forceinline__ WorkQueue(const XcdQueues &q_, int32_t *c, int w, int workers_, int chunk_)
      : q(q_), counters(c), range(blockIdx.x & (NXCD - 1)), workers(workers_), chunk(chunk_) {
    t = q.start[range] + w * chunk;
    tend = min(q.start[range + 1], t + chunk);
  }
  // request the next chunk of the current range (result used by next())
  __device__ __forceinline__ void request(bool leader) {
    asked = dynamic(range) > 0;
    if (asked && leader) pend = atomicAdd(counters + range * QUEUE_STRIDE, 1);
  }
  // called by a whole wavefront after its chunk: the next chunk, false at the
  // end.  Every index is handed out exactly once.
  __device__ __forceinline__ bool next(int lane) {
    if (asked && take(range, __builtin_amdgcn_readfirstlane(pend))) return true;
    for (;;) {
      // ranges with tiles left: lane r looks at range r
      bool left = false;
      if (lane < NXCD) {
        const int k = __hip_atomic_load(counters + lane * QUEUE_STRIDE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        left = (int64_t)k * chunk < dynamic(lane);
      }
      const unsigned m = (unsigned)__ballot(left) & ((1u << NXCD) - 1);
      if (!m) return false;
      // the first one at or after the current range, cyclically
      const unsigned rot = ((m >> range) | (m << (NXCD - range))) & ((1u << NXCD) - 1);
      range = (range + __ffs(rot) - 1) & (NXCD - 1);
      int k = 0;
      if (lane == 0) k = atomicAdd(counters + range * QUEUE_STRIDE, 1);
      if (take(range, __builtin_amdgcn_readfirstlane(k))) return true;
    }
  }

 private:
  __device__ __forceinline__ bool take(int r, int k) {
    const int64_t d = dynamic(r), o = (int64_t)k * chunk;
    if (o >= d) return false;
    t = q.start[r] + workers * chunk + (int)o;
    tend = min(q.start[r + 1], t + chunk);
    return true;
  }
};

// Every launch clears the counters of the next one (the two sets of a
// QueueSets alternate), so that no launch is spent on it.
__device__ __forceinline__ void clear_counters(int32_t *next) {
  if (blockIdx.x == 0 && threadIdx.x < NXCD) next[threadIdx.x * QUEUE_STRIDE] = 0;
}

}  // namespace dmrg
