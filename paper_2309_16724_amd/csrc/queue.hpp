// Device side of the per-XCD work queues (see XcdQueues in plan.hpp).
#pragma once
#include <hip/hip_runtime.h>
#include "plan.hpp"

namespace dmrg {

// Work list of one worker (a wavefront or a work group) of a tile launch.
//
// Range r = blockIdx % NXCD of the list belongs to the workers of the blocks
// with that remainder, which the dispatcher places on one XCD.  Atomics on one
// address run one after the other, about 100 ns each (measured: 60 to 80 per
// microsecond over all counters, in one line or in a line each), and short
// tiles end faster than that: one atomic per tile made the L=24, D=512 first
// stage take 4.9 ms for 292,000 tiles.  So most of a range is dealt out in
// turn, worker w taking tiles w, w + workers, ... of it (side by side, so that
// the workers of an XCD share operand bands in its L2), and only its rest
// [dyn, end) through the range's counter, `chunk` tiles at a time, requested
// one tile ahead.  A worker without work reads all counters with one load
// before it takes from another range.
struct WorkQueue {
  const XcdQueues &q;
  int32_t *counters;
  int range, chunk;   // current range, tiles per dynamic chunk
  int t, tend, step;  // current tiles t, t + step, ... < tend
  int pend = 0;       // lane 0: chunk index the pending request returned
  bool asked = false;

  // tiles of range r that its counter hands out
  __device__ __forceinline__ int dynamic(int r) const { return q.start[r + 1] - q.dyn[r]; }
  __device__ __forceinline__ WorkQueue(const XcdQueues &q_, int32_t *c, int w, int workers, int chunk_)
      : q(q_), counters(c), range(blockIdx.x & (NXCD - 1)), chunk(chunk_) {
    t = q.start[range] + w;
    tend = q.dyn[range];
    step = workers;
  }
  __device__ __forceinline__ bool last() const { return t + step >= tend; }
  // request the next chunk of the current range (result used by next())
  __device__ __forceinline__ void request(bool leader) {
    asked = dynamic(range) > 0;
    if (asked && leader) pend = atomicAdd(counters + range * QUEUE_STRIDE, 1);
  }
  // called by a whole wavefront after its last tile: the next chunk, false at
  // the end.  Every index is handed out exactly once.
  __device__ __forceinline__ bool next(int lane) {
    const bool a = asked;
    asked = false;
    if (a && take(range, __builtin_amdgcn_readfirstlane(pend))) return true;
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
      range = __builtin_amdgcn_readfirstlane((range + __ffs(rot) - 1) & (NXCD - 1));
      int k = 0;
      if (lane == 0) k = atomicAdd(counters + range * QUEUE_STRIDE, 1);
      if (take(range, __builtin_amdgcn_readfirstlane(k))) return true;
    }
  }

 private:
  __device__ __forceinline__ bool take(int r, int k) {
    const int64_t o = (int64_t)k * chunk;
    if (o >= dynamic(r)) return false;
    // (wave-uniform, and said to be: the descriptors of a tile are scalar loads)
    t = __builtin_amdgcn_readfirstlane(q.dyn[r] + (int)o);
    tend = __builtin_amdgcn_readfirstlane(min(q.start[r + 1], t + chunk));
    step = 1;
    return true;
  }
};

// Every launch clears the counters of the next one (the two sets of a
// QueueSets alternate), so that no launch is spent on it.
__device__ __forceinline__ void clear_counters(int32_t *next) {
  if (blockIdx.x == 0 && threadIdx.x < NXCD) next[threadIdx.x * QUEUE_STRIDE] = 0;
}

}  // namespace dmrg
