// Arguments of the hashing launch, and the part of it that puts the call's random draws into the workspace.
#pragma once

#include "ha_common.h"

namespace ha {

// One launch hashes the rows of Q and of K (one tensor: X[1] null) and, in the forward calls, also stores the
// hyperplane matrix R (Definition 1) and the per-node sample indices l_1..l_m (Algorithm 2), derived from the seed or
// copied from the caller's device arrays.  A seed's R travels in the arguments, so hashing waits for no launch
// before it.  Measured (MI355X) against a launch for the draws and one per tensor: forward, 12 heads, n = 4096,
// d = 64: 44 -> 36 us; 15 heads, n = 6300, d = 128: 69 -> 60 us; fp32, one head, n = 1024: 38 -> 27 us.
struct HashArgs {
  const void* X[2];
  uint8_t* codes[2];
  int64_t rows;            // per tensor
  const float* R;          // device R [d][r]; null: Rb
  int32_t r;
  int32_t store_draws;     // whether to fill R_ws and samples_ws
  float* R_ws;
  int32_t* samples_ws;
  const int32_t* samples_dev;
  int32_t* tau_rows_ws;    // Algorithm 2: [total_nodes][m] rows of T, node-local query indices; null: not wanted
  Geometry g;
  uint64_t seed;
  alignas(16) uint16_t Rb[8][128];  // seed-derived R as bf16 bit patterns, hyperplane by hyperplane, zero beyond r and d
};

// Every thread of the launch calls it once.
__device__ inline void store_draws(const HashArgs& a) {
  const int64_t nthreads = (int64_t)gridDim.x * blockDim.x;
  const int nR = a.g.d * a.g.r;
  const int64_t nS = (int64_t)a.g.total_nodes * a.g.m;
  // (by the last workgroups: where the rows do not come out even, they have a trip less)
  for (int64_t i = (int64_t)(gridDim.x - 1 - blockIdx.x) * blockDim.x + threadIdx.x; i < nR || i < nS; i += nthreads) {
    if (i < nR) a.R_ws[i] = a.R ? a.R[i] : __uint_as_float((uint32_t)a.Rb[i % a.g.r][i / a.g.r] << 16);
    if (i < nS) {
      const int heap = (int)(i / a.g.m);
      const int j = (int)(i % a.g.m);
      const int level = 31 - __clz(heap + 1);
      const int node = heap + 1 - (1 << level);
      const NodeRef nr = node_ref(a.g, level, node);
      int32_t v;
      if (a.samples_dev) {
        v = a.samples_dev[i];
        v = v < 0 ? 0 : (v >= nr.s ? nr.s - 1 : v);  // never index outside the node
      } else {
        v = sample_index(a.seed, level, node, nr.s, j);
      }
      a.samples_ws[i] = v;
      if (a.tau_rows_ws) {
        const uint64_t hi = rand_u64(a.seed, kStreamTauRows, (uint64_t)heap * a.g.m + j) >> 32;
        a.tau_rows_ws[i] = (int32_t)((hi * (uint64_t)nr.s) >> 32);
      }
    }
  }
}

int launch_lsh_hash(const HashArgs& a, int d, int dtype, hipStream_t st);
int launch_lsh_hash_mfma(const HashArgs& a, int d, hipStream_t st);

}  // namespace ha
