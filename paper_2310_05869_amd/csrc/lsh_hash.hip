// sortLSH hashing of fp32 rows (Definition 1 of the paper; Algorithm 1, "hash rows of Q, K").
//
// code(x) = Gray-sequence position of the word whose bit k is [<x, R[:,k]> > 0].
//
// The stage is a pure stream over X (d*esz bytes in, 1 byte out per row), so the
// layout is chosen for HBM: every lane issues 16-byte loads, a row is spread
// over LPR = d*esz/16 consecutive lanes and a wave covers 64/LPR whole rows per
// load instruction (fully coalesced 1 KiB).  Each lane multiplies its 16 bytes
// of the row with its slice of R held in registers as fp64 and the LPR partial
// sums of the (up to 8) projections are combined by a transposing butterfly:
// each exchange halves the number of values a lane carries, so 8 values cost 8
// exchanges instead of 8*log2(LPR).
//
// Accumulation is fp64: inputs and R are fp32, so every product
// is exact in fp64 and the sum carries a relative error of about d * 2^-53.  A
// sign can therefore differ from an infinitely precise evaluation only for
// projections that are zero to ~1e-13, which keeps bucket codes reproducible
// against any fp64 reference.
#include "hash_common.h"

namespace ha {

// Sum v[k] over the LPR lanes of a row; lane l ends with projection (l / (LPR/8)) & 7.
template <int LPR>
__device__ inline double reduce_transposed(const double* v, int l) {
  constexpr int W1 = LPR / 2, W2 = LPR / 4, W3 = LPR / 8;
  const bool u1 = (l & W1) != 0;
  double w4[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const double keep = u1 ? v[4 + j] : v[j];
    const double send = u1 ? v[j] : v[4 + j];
    w4[j] = keep + __shfl_xor(send, W1);
  }
  const bool u2 = (l & W2) != 0;
  double w2[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const double keep = u2 ? w4[2 + j] : w4[j];
    const double send = u2 ? w4[j] : w4[2 + j];
    w2[j] = keep + __shfl_xor(send, W2);
  }
  const bool u3 = (l & W3) != 0;
  const double keep = u3 ? w2[1] : w2[0];
  const double send = u3 ? w2[0] : w2[1];
  double w = keep + __shfl_xor(send, W3);
#pragma unroll
  for (int o = W3 / 2; o >= 1; o >>= 1) w += __shfl_xor(w, o);
  return w;
}

template <int D>
__global__ __launch_bounds__(256) void lsh_hash_kernel(HashArgs a) {
  constexpr int EPL = 4;
  constexpr int LPR = D / EPL;   // lanes per row: 16 or 32
  constexpr int RPW = 64 / LPR;  // rows per wave and load
  constexpr int W3 = LPR / 8;
  constexpr int U = 4;           // loads in flight per lane
  const int lane = threadIdx.x & 63;
  const int l = lane % LPR;
  const int jrow = lane / LPR;
  const int c0 = l * EPL;
  const int r = a.r;

  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  const int64_t gpt = (a.rows + RPW - 1) / RPW;  // groups per tensor
  const int64_t ngroups = a.X[1] ? 2 * gpt : gpt;
  uint4 raw[U];
  auto load = [&](int64_t g0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t g = g0 + u * nwaves;
      const int t = g >= gpt;
      const int64_t row = (g - t * gpt) * RPW + jrow;
      raw[u] = make_uint4(0, 0, 0, 0);
      if (g < ngroups && row < a.rows)
        raw[u] = *reinterpret_cast<const uint4*>(reinterpret_cast<const float*>(t ? a.X[1] : a.X[0]) + row * D + c0);
    }
  };
  load(wave);  // in flight while R is converted (forward, 4 heads, n = 4096, d = 64, b = m = 64: 27.1 -> 24.6 us)

  double Rr[EPL][8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    if (a.R) {
#pragma unroll
      for (int e = 0; e < EPL; ++e) Rr[e][k] = (k < r) ? (double)a.R[(c0 + e) * r + k] : 0.0;
    } else {
      const uint2 b = *reinterpret_cast<const uint2*>(&a.Rb[k][c0]);
      Rr[0][k] = (double)__uint_as_float(b.x << 16);
      Rr[1][k] = (double)__uint_as_float(b.x & 0xFFFF0000u);
      Rr[2][k] = (double)__uint_as_float(b.y << 16);
      Rr[3][k] = (double)__uint_as_float(b.y & 0xFFFF0000u);
    }
  }
  if (a.store_draws) store_draws(a);

  for (int64_t g0 = wave; g0 < ngroups; g0 += nwaves * U) {
    if (g0 != wave) load(g0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t grp = g0 + u * nwaves;
      if (grp >= ngroups) break;  // wave-uniform
      const double x[EPL] = {(double)__uint_as_float(raw[u].x), (double)__uint_as_float(raw[u].y),
                             (double)__uint_as_float(raw[u].z), (double)__uint_as_float(raw[u].w)};
      double acc[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) acc[k] = 0.0;
#pragma unroll
      for (int e = 0; e < EPL; ++e)
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] = __builtin_fma(x[e], Rr[e][k], acc[k]);
      const double p = reduce_transposed<LPR>(acc, l);
      const unsigned long long bal = __ballot(p > 0.0);  // 0 and NaN give bit 0
      if (l == 0) {
        const int t = grp >= gpt;
        const int64_t row = (grp - t * gpt) * RPW + jrow;
        if (row < a.rows) {
          const uint32_t rowbits = (uint32_t)(bal >> (jrow * LPR));
          uint32_t word = 0;
          for (int k = 0; k < r; ++k) word |= ((rowbits >> (k * W3)) & 1u) << k;
          // position in the reflected Gray sequence: the i with i ^ (i >> 1) == word
          uint32_t idx = word;
          idx ^= idx >> 1;
          idx ^= idx >> 2;
          idx ^= idx >> 4;
          (t ? a.codes[1] : a.codes[0])[row] = (uint8_t)idx;
        }
      }
    }
  }
}

int launch_lsh_hash(const HashArgs& a, int d, int dtype, hipStream_t st) {
  if (a.rows <= 0) return HA_OK;
  if (dtype == HA_BF16) return launch_lsh_hash_mfma(a, d, st);  // matrix-core path
  const int rpw = 256 / d;
  const int64_t ngroups = (a.rows + rpw - 1) / rpw * (a.X[1] ? 2 : 1);
  // one group per wave while that leaves the chip four waves per SIMD, then up to the four of a trip
  int64_t blocks = (ngroups + 3) / 4;
  if (blocks > 1024) blocks = (ngroups + 15) / 16 > 1024 ? (ngroups + 15) / 16 : 1024;
  if (blocks > 4096) blocks = 4096;
  dim3 grid((unsigned)blocks), block(256);
  if (d == 128)
    hipLaunchKernelGGL((lsh_hash_kernel<128>), grid, block, 0, st, a);
  else if (d == 64)
    hipLaunchKernelGGL((lsh_hash_kernel<64>), grid, block, 0, st, a);
  else
    return HA_ERR_SHAPE;
  return check_launch();
}

}  // namespace ha
