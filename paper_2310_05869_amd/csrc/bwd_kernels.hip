// Small kernels around the backward passes: delta_i = <dO_i, O_i>, and the ordered reduction of the sampled keys'
// gradients: of all levels or one into the accumulated key rows (causal), over the query chunks (unmasked).
// Every sum is taken in a fixed order: results are bit-reproducible.
#include "attn_common.h"
#include "bwd_common.h"

namespace ha {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// One group of D/8 lanes per row; 8 elements per lane.  O is read from its
// unrounded fp32 copy when there is one: with the bf16 tensor, delta carries the
// output's rounding error, which matters where <dO_i, v_j> - delta_i cancels
// (rows whose weight sits on few keys).
template <int D>
__global__ __launch_bounds__(256) void bwd_delta_kernel(const uint16_t* __restrict__ O, const float* __restrict__ O32,
                                                        const uint16_t* __restrict__ G, float* __restrict__ delta,
                                                        int64_t rows) {
  constexpr int LPR = D / 8;  // lanes per row
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t row = t / LPR;
  const int part = (int)(t % LPR);
  float s = 0.f;
  if (row < rows) {
    const u32x4 g = *reinterpret_cast<const u32x4*>(G + row * D + part * 8);
    float o[8];
    if (O32 != nullptr) {
      const f32x4 a = *reinterpret_cast<const f32x4*>(O32 + row * D + part * 8);
      const f32x4 b = *reinterpret_cast<const f32x4*>(O32 + row * D + part * 8 + 4);
      o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
      o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
    } else {
      const u32x4 ob = *reinterpret_cast<const u32x4*>(O + row * D + part * 8);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        o[2 * e] = __uint_as_float(ob[e] << 16);
        o[2 * e + 1] = __uint_as_float(ob[e] & 0xFFFF0000u);
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s = __builtin_fmaf(o[2 * e], __uint_as_float(g[e] << 16), s);
      s = __builtin_fmaf(o[2 * e + 1], __uint_as_float(g[e] & 0xFFFF0000u), s);
    }
  }
#pragma unroll
  for (int off = LPR / 2; off >= 1; off >>= 1) s += __shfl_xor(s, off);
  if (row < rows && part == 0) delta[row] = s;
}

// fp32 tensors: the same dot product, straight from O and dO.
template <int D>
__global__ __launch_bounds__(256) void bwd_delta_f32_kernel(const float* __restrict__ O, const float* __restrict__ G,
                                                            float* __restrict__ delta, int64_t rows) {
  constexpr int LPR = D / 8;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t row = t / LPR;
  const int part = (int)(t % LPR);
  float s = 0.f;
  if (row < rows) {
#pragma unroll
    for (int e = 0; e < 8; ++e) s = __builtin_fmaf(O[row * D + part * 8 + e], G[row * D + part * 8 + e], s);
  }
#pragma unroll
  for (int off = LPR / 2; off >= 1; off >>= 1) s += __shfl_xor(s, off);
  if (row < rows && part == 0) delta[row] = s;
}

int launch_bwd_delta(const void* O, const float* O_f32, const void* dO, float* delta, int64_t rows, int d, int dtype,
                     hipStream_t st) {
  if (rows <= 0) return HA_OK;
  const int lpr = d / 8;
  const int64_t threads = rows * lpr;
  const unsigned grid = (unsigned)((threads + 255) / 256);
  if (dtype == HA_FP32) {
    if (d == 128)
      hipLaunchKernelGGL((bwd_delta_f32_kernel<128>), dim3(grid), dim3(256), 0, st, (const float*)O, (const float*)dO, delta, rows);
    else if (d == 64)
      hipLaunchKernelGGL((bwd_delta_f32_kernel<64>), dim3(grid), dim3(256), 0, st, (const float*)O, (const float*)dO, delta, rows);
    else
      return HA_ERR_SHAPE;
    return check_launch();
  }
  if (d == 128)
    hipLaunchKernelGGL((bwd_delta_kernel<128>), dim3(grid), dim3(256), 0, st, (const uint16_t*)O, O_f32, (const uint16_t*)dO, delta, rows);
  else if (d == 64)
    hipLaunchKernelGGL((bwd_delta_kernel<64>), dim3(grid), dim3(256), 0, st, (const uint16_t*)O, O_f32, (const uint16_t*)dO, delta, rows);
  else
    return HA_ERR_SHAPE;
  return check_launch();
}

// Sampled keys' gradients of levels [level0, level1) into the accumulated key rows.  One wave per sample j
// of a (head, node); a lane owns four columns of dK (lanes < d/4) or of dV (the
// next d/4 lanes).  A key may be drawn more than once, by its node and by the nodes of the other levels that hold it: the
// FIRST sample that drew a key ("owner": lowest level, then lowest sample) adds, level by level and in increasing sample
// order, the sums of every sample of that key, each taken over the node's query chunks in a fixed order;
// the other samples of the key do nothing.  One writer per row and a fixed
// order of additions: reproducible bit for bit.
//
// All levels go in one launch where it is small, else level by level: a launch is 5 us of a small problem, whose upper
// levels have a few workgroups that wait for their chunks, but a wave then looks through the samples of every level's node.
// Forward + backward, a launch per level -> one (MI355X, us; workgroups of the one): fp32, m = 64: 4 heads, n = 4096, two levels (192)
// 214.5 -> 211.8; 1 head, n = 8192, three (112) 183.0 -> 176.4; 3 heads, n = 1024, two (144) 90.0 -> 87.3; bf16, m = 256: 1 head, n = 16384,
// d = 64, five (1984) 222.6 -> 208.0; 4 heads, two (768) 332 -> 329; 8 heads, n = 8192, d = 128, three (3584) 409 -> 405; 32 heads, n = 32768, three (14336)
// 7967 -> 7987; n = 131072, five (63488) 39250 -> 39440; m = 1000, 4 heads, n = 16384, four (15000) 559 -> 578.
constexpr int kScatterOneLaunchSamples = 256;
constexpr int64_t kScatterOneLaunchGrid = 4096;
constexpr int kScatterWaves = 4;

// LEVELS: several; else one, whose samples the waves look through in LDS.
template <bool LEVELS>
__global__ __launch_bounds__(64 * kScatterWaves) void bwd_sample_scatter_kernel(BwdArgs a, int level0, int level1, int hn_first,
                                                                                const float* __restrict__ samp_k,
                                                                                const float* __restrict__ samp_v,
                                                                                float* part_k, float* part_v) {
  const Geometry& g = a.f.g;
  const int d = g.d, m = g.m;
  const int groups = (m + kScatterWaves - 1) / kScatterWaves;
  const int grp = (int)blockIdx.x % groups;
  const int hn = hn_first + (int)blockIdx.x / groups;
  const int heap = (1 << level0) - 1 + hn / g.BH, bh = hn % g.BH;  // the upper levels, of more chunks, first
  const int level = 31 - __builtin_clz(heap + 1);
  const NodeRef nr = node_ref(g, level, heap + 1 - (1 << level));
  const int lane = threadIdx.x & 63;
  const int j = grp * kScatterWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  __shared__ int32_t keys[LEVELS ? 1 : 4096];
  if constexpr (!LEVELS) {
    for (int i = threadIdx.x; i < m; i += blockDim.x) keys[i] = a.f.samples[(int64_t)heap * m + i];
    __syncthreads();
  }
  if (j >= m) return;
  auto drawn_by = [&](const NodeRef& o, int i) {
    if constexpr (LEVELS) return a.f.samples[(int64_t)o.heap * m + i];
    else return keys[i];
  };
  const int row = nr.k_start + drawn_by(nr, j);  // within the head

  // the level's node that holds the row among its keys, if one does
  auto holder = [&](int l, NodeRef* out) {
    *out = node_ref(g, l, row / (g.n >> l));
    return row - out->k_start < out->s;
  };
  // whether one of a node's samples [0, end) is the row; several loads in flight
  auto drawn_in = [&](const NodeRef& o, int end) {
    const int key = row - o.k_start;
    bool hit = false;
#pragma unroll 4
    for (int base = 0; base < end; base += 64) hit |= base + lane < end && drawn_by(o, min(base + lane, m - 1)) == key;
    return __any(hit);
  };
  // an earlier sample of the same key owns it
  for (int l = level0; l <= level; ++l) {
    NodeRef o;
    if (holder(l, &o) && drawn_in(o, l < level ? m : j)) return;
  }

  const int q4 = d / 4;  // column quads per row
  const bool active = lane < 2 * q4;
  const float* src = lane < q4 ? samp_k : samp_v;
  const int c4 = (lane % q4) * 4;
  f32x4* out = reinterpret_cast<f32x4*>((lane < q4 ? part_k : part_v) + ((int64_t)bh * g.n + row) * d + c4);
  f32x4 sum = {0.f, 0.f, 0.f, 0.f};
  if (active) sum = *out;
  int64_t lvl_row0 = 0;  // rows of the levels before
  for (int l = 0; l < level1; ++l) {
    const int cpn = bwd_chunks_per_node(g, a.chunk, l), nodes = 1 << l;
    NodeRef o;
    if (l >= level && holder(l, &o)) {
      const int key = row - o.k_start;
      const int64_t row0 = lvl_row0 + ((int64_t)bh * nodes + (o.heap + 1 - nodes)) * cpn * m;
      f32x4 total = {0.f, 0.f, 0.f, 0.f};
      for (int base = l == level ? j : 0; base < m; base += 64) {
        const int jl = base + lane;
        unsigned long long same = __ballot(jl < m && drawn_by(o, min(jl, m - 1)) == key);
        while (same) {
          const int jj = base + __builtin_ctzll(same);
          same &= same - 1;
          if (active) {
            const float* p = src + (row0 + jj) * d + c4;
            const int64_t step = (int64_t)m * d;
            f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0, s2 = s0, s3 = s0;
            int qc = 0;
            for (; qc + 4 <= cpn; qc += 4) {
              s0 += *reinterpret_cast<const f32x4*>(p + (qc + 0) * step);
              s1 += *reinterpret_cast<const f32x4*>(p + (qc + 1) * step);
              s2 += *reinterpret_cast<const f32x4*>(p + (qc + 2) * step);
              s3 += *reinterpret_cast<const f32x4*>(p + (qc + 3) * step);
            }
            for (; qc < cpn; ++qc) s0 += *reinterpret_cast<const f32x4*>(p + qc * step);
            total += (s0 + s1) + (s2 + s3);
          }
        }
      }
      sum += total;
    }
    lvl_row0 += (int64_t)g.BH * nodes * cpn * m;
  }
  if (active) *out = sum;
}

int launch_bwd_sample_scatter(const BwdArgs& a, const float* samp_k, const float* samp_v, float* acc_k, float* acc_v, hipStream_t st) {
  const Geometry& g = a.f.g;
  if (g.m <= 0 || g.levels <= 0) return HA_OK;
  const int groups = (g.m + kScatterWaves - 1) / kScatterWaves;
  if ((int64_t)g.BH * (1 << (g.levels - 1)) * groups > kMaxGrid) return HA_ERR_SHAPE;
  const bool one_launch = g.m <= kScatterOneLaunchSamples && (int64_t)g.BH * g.total_nodes * groups <= kScatterOneLaunchGrid;
  const int step = one_launch ? g.levels : 1;
  const int64_t most = kMaxLaunch / groups;  // (heads, nodes) per launch; groups <= 1024
  for (int l = 0; l < g.levels; l += step) {
    const int64_t nodes = (int64_t)g.BH * ((1 << (l + step)) - (1 << l));
    for (int64_t first = 0; first < nodes; first += most) {
      const unsigned count = (unsigned)((nodes - first < most ? nodes - first : most) * groups);
      if (step > 1)
        hipLaunchKernelGGL((bwd_sample_scatter_kernel<true>), dim3(count), dim3(64 * kScatterWaves), 0, st, a, l, l + step, (int)first, samp_k,
                           samp_v, acc_k, acc_v);
      else
        hipLaunchKernelGGL((bwd_sample_scatter_kernel<false>), dim3(count), dim3(64 * kScatterWaves), 0, st, a, l, l + step, (int)first, samp_k,
                           samp_v, acc_k, acc_v);
      const int rc = check_launch();
      if (rc != HA_OK) return rc;
    }
  }
  return HA_OK;
}

// Unmasked problems, whose block-key pass adds the sampled sums itself: the rows of the sampled-key pass summed over the
// query chunks, one thread per four columns of a (head, sample) row of dK or dV, in place into the first chunk's row.
// U: the rows that a thread has in flight (sums in one order for each).  With fewer than 256 workgroups their round trips are the
// launch, and U is as many as there are chunks, up to 32; from there on the requests past the last chunk cost more than
// that.  8 -> 32 (MI355X, backward, us; workgroups): 2 heads, n = 65536, d = 64 (64) 112.7 -> 105.2, n = 33792 82.0 -> 79.4, 4 heads, n = 65536 (128) 184.8 ->
// 177.5, d = 128, 2 heads, n = 65536 (128) 181.1 -> 175.4, n = 33792 133.0 -> 131.1; 4 heads, n = 65536 (256) 367.4 -> 372.6; d = 64, 12 heads,
// n = 20480 (384) 175.0 -> 176.1, 40 heads, n = 8448, m = 100 (500) 197.2 -> 200.2.
// Bound by the rows it reads (12 heads, n = 16384, m = 256, d = 64: 50 MB in 9.8 us); left to the block-key pass,
// where few waves hold a sampled key and wait for its chunks one after the other, that pass took 76 instead of 46 us.
template <int U>
__global__ __launch_bounds__(256) void bwd_sample_reduce_kernel(float* samp_k, float* samp_v, int cpn, int m, int d, int64_t total) {
  int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= total) return;
  const int q4 = d / 4;
  const int c4 = (int)(t % q4) * 4;
  t /= q4;
  float* samp = (t & 1) ? samp_v : samp_k;
  t >>= 1;
  float* p = samp + (t / m * cpn * m + t % m) * d + c4;
  const int64_t step = (int64_t)m * d;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 part[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) part[u] = zero;
  for (int q = 0; q < cpn; q += U) {  // U rows in flight: requested unconditionally (a load under a branch is waited for alone)
    f32x4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const f32x4*>(p + min(q + u, cpn - 1) * step);
#pragma unroll
    for (int u = 0; u < U; ++u) part[u % 8] += q + u < cpn ? v[u] : zero;
  }
  *reinterpret_cast<f32x4*>(p) = ((part[0] + part[1]) + (part[2] + part[3])) + ((part[4] + part[5]) + (part[6] + part[7]));
}

int launch_bwd_sample_reduce(const BwdArgs& a, float* samp_k, float* samp_v, hipStream_t st) {
  const Geometry& g = a.f.g;
  const int cpn = bwd_chunks_per_node(g, a.chunk, 0);
  if (cpn == 1) return HA_OK;
  const int64_t total = (int64_t)g.BH * g.m * 2 * (g.d / 4), grid = (total + 255) / 256;
  if (grid > kMaxGrid) return HA_ERR_SHAPE;
  if (grid < 256 && cpn > 16) hipLaunchKernelGGL((bwd_sample_reduce_kernel<32>), dim3((unsigned)grid), dim3(256), 0, st, samp_k, samp_v, cpn, g.m, g.d, total);
  else if (grid < 256 && cpn > 8) hipLaunchKernelGGL((bwd_sample_reduce_kernel<16>), dim3((unsigned)grid), dim3(256), 0, st, samp_k, samp_v, cpn, g.m, g.d, total);
  else hipLaunchKernelGGL((bwd_sample_reduce_kernel<8>), dim3((unsigned)grid), dim3(256), 0, st, samp_k, samp_v, cpn, g.m, g.d, total);
  return check_launch();
}

}  // namespace ha
