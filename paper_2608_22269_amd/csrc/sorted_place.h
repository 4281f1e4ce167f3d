// Place of a particle in the sorted order (grid.hip).
#pragma once

#include "kernels.h"

namespace wb {

// Sorted place of the particle at arrival place t (from: its index before the
// sort and its original index): its cell's first place plus the number of the
// cell's particles with a lower original index.  A cell of more than 1,024 (particles parked after a domain
// error) keeps arrival order rather than spend quadratic time.  One thread per
// particle with independent loads: one thread per cell that sorted its run by
// insertion took 93 us at 660,000 particles in cells of 2h (17.6 per cell),
// this 12 us of the reorder.
__device__ __forceinline__ uint32_t sorted_place(const uint32_t *__restrict__ keys, const uint32_t *__restrict__ start,
                                                 const uint2 *__restrict__ perm, uint32_t t, uint2 from) {
  const uint32_t key = keys[from.x];
  const uint32_t b = start[key], e = start[key + 1];
  if (e - b > 1024u) return t;
  uint32_t rank = 0;
  for (uint32_t q = b; q < e; q += 4u) {  // four loads in flight; past the end the last one again
    uint32_t id[4];
#pragma unroll
    for (uint32_t u = 0; u < 4u; ++u) id[u] = perm[min(q + u, e - 1u)].y;
#pragma unroll
    for (uint32_t u = 0; u < 4u; ++u) rank += q + u < e && id[u] < from.y ? 1u : 0u;
  }
  return b + rank;
}

}  // namespace wb
