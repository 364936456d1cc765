// The final reduction of (max, sum) pairs, by a kernel of its own or by one
// more workgroup of the launch that follows the kernel which wrote the pairs.
#pragma once

#include "mgfem_internal.h"

namespace mgfem {

// the maximum that a NaN wins
__device__ inline double nanmax2(double a, double b) { return (b > a || b != b) ? b : a; }

// nb pairs of `part` into out (device) and the record of pinned host memory
// that the count kept in seq points at (part null: nothing to reduce)
struct Reduce {
  const double* part;
  int nb;
  double* out;
  double* host;
  double* seq;
};

// All BS threads of a workgroup, in a fixed order: each thread takes the pairs
// in chunks of U, the loads of a chunk issued together (a lane beyond nb
// reads pair 0 and drops it: loads under a branch would wait for one another),
// then a wave reduction and the waves in order.  sh: 2 BS / 64 doubles of LDS.
template <int BS, int U>
__device__ inline void reduce_block(const Reduce& R, double* sh) {
  double mx = 0.0, sm = 0.0;
  for (int base = 0; base < R.nb; base += U * BS) {
    double lm[U], ls[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int q = base + threadIdx.x + u * BS;
      const int qq = q < R.nb ? q : 0;
      lm[u] = R.part[2 * qq];
      ls[u] = R.part[2 * qq + 1];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = base + (int)threadIdx.x + u * BS < R.nb;
      mx = nanmax2(mx, in ? lm[u] : 0.0);
      sm += in ? ls[u] : 0.0;
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    mx = nanmax2(mx, __shfl_xor(mx, o));
    sm += __shfl_xor(sm, o);
  }
  if ((threadIdx.x & 63) == 0) {
    sh[2 * (threadIdx.x >> 6)] = mx;
    sh[2 * (threadIdx.x >> 6) + 1] = sm;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < BS / 64; ++w) {
      mx = nanmax2(mx, sh[2 * w]);
      sm += sh[2 * w + 1];
    }
    R.out[0] = mx;
    R.out[1] = sm;
    const double q = R.seq[0] + 1.0;  // counted on the device (graph replays)
    R.seq[0] = q;
    double* rec = R.host + 4 * (int)((long long)q % kRedSlots);
    rec[0] = mx;  // straight to pinned host memory; the sequence number goes last
    rec[1] = sm;
    __threadfence_system();
    rec[2] = q;
    __threadfence_system();
  }
}

}  // namespace mgfem
