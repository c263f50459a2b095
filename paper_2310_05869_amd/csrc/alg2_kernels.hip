// The estimator of Algorithm 2 as printed, and Lemma 2 / Algorithm 3's value
// product, as options beside the Section 4 form the main path implements:
//   tau      = max over a random row subset T of the unmasked row sum <1 - M^H_j, A_j>
//   C_i      = cap_scale * m / (n ln n) * (masked row sum_i + tau / kappa)
//   d_i      = (n/m) sum_j (1 - M_{i,l_j}) min(exp<q_i,k_{l_j}>, C_i)
//   d~_i     = masked row sum_i + max(d_i, tau / kappa)
//   out_i    = (1 / d~_i) sum_r exp<q_i,k_{l'_r}> v_{l'_r} / (m p_{l'_r}),  l'_r ~ p_l ~ |V_l|^2   (Lemma 2)
//         or = (1 / d~_i) (masked part + (n/m) sum_j (1 - M) exp<q_i,k_{l_j}> v_{l_j})                (Section 4)
// The constants the paper leaves open (the Theta in C_i, kappa) are the caller's.
// A launch sequence handles one level of nodes (alg2_common.h): the unmasked problem, or one
// level of Algorithm 4's off-diagonal nodes, every node with its own draws.  The draws, weights and prefix sums are
// computed here for both dtypes, the sums of the rows of T for fp32 tensors (bf16: alg2_mfma.hip).  The caps are a mode of
// either dtype's forward kernel, with value sampling a mode of the fp32 one and a kernel of alg2_mfma.hip.
//
// Lemma 2's rows are drawn with p_l = |V_l|^2 / |V|_F^2 (V the node's value rows) by inverting
// the cumulative distribution in fp64: draw r of head bh at the node with heap index h takes the
// uniform u in (0, 1) formed by the top 53 bits of counter (h * heads + bh) * m + r of stream 2
// and is the first l whose inclusive prefix sum of squared norms exceeds u |V|_F^2.
#include "attn_common.h"
#include "alg2_common.h"

namespace ha {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr uint64_t kStreamVnorm = 2;

template <typename T>
__device__ inline float elem(const T* p);
template <>
__device__ inline float elem<float>(const float* p) { return *p; }
template <>
__device__ inline float elem<uint16_t>(const uint16_t* p) { return __uint_as_float((uint32_t)(*p) << 16); }

// pos_q = P_Q^-1 of one level's nodes, node-local (problems of several levels; where there is one, the sort writes it).
__global__ void alg2_pos_kernel(Alg2Args a) {
  const Geometry& g = a.g;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)g.BH * g.n) return;
  const int vh = (int)(t / g.n);
  const Alg2Node nd = alg2_node(a, vh);
  a.pos_q[(int64_t)vh * g.n + (a.perm_q[t] - nd.q_start)] = (int32_t)(t % g.n);
}

// Squared row norms of V in fp64 (one thread per row); 64 rows per workgroup come in through LDS
// so that the global loads are coalesced.
constexpr int kVwRows = 64;

template <typename T, int D>
__global__ __launch_bounds__(256) void vnorm_weight_kernel(Alg2Args a) {
  constexpr int kRowBytes = D * (int)sizeof(T);
  constexpr int kStride = kRowBytes + 4;  // odd number of words: the 64 row readers hit 64 banks
  __shared__ __attribute__((aligned(16))) unsigned char tile[kVwRows * kStride];
  const Geometry& g = a.g;
  // one workgroup per 64 consecutive keys of one node (g.n need not be a multiple of 64)
  const int per_node = (g.n + kVwRows - 1) / kVwRows;
  const int vh = blockIdx.x / per_node;
  const int l0 = (blockIdx.x % per_node) * kVwRows;
  const Alg2Node nd = alg2_node(a, vh);
  const int nrows = min(kVwRows, g.n - l0);
  const int64_t row0 = (int64_t)vh * g.n + l0;   // in the view
  const unsigned char* src = reinterpret_cast<const unsigned char*>(a.V) +
                             ((int64_t)nd.head * a.n_full + nd.k_start + l0) * kRowBytes;
  for (int e = threadIdx.x; e < nrows * (kRowBytes / 4); e += 256) {
    const int r = e / (kRowBytes / 4), w = e % (kRowBytes / 4);
    *reinterpret_cast<uint32_t*>(tile + r * kStride + 4 * w) = *reinterpret_cast<const uint32_t*>(src + (int64_t)e * 4);
  }
  __syncthreads();
  if (threadIdx.x >= 64) return;  // the first wave sums the rows (whole waves leave; no partial wave)
  const bool active = (int)threadIdx.x < nrows;
  const T* v = reinterpret_cast<const T*>(tile + (active ? threadIdx.x : 0) * kStride);
  double w = 0.0;
  for (int c = 0; c < D; ++c) {
    const double x = (double)elem<T>(v + c);
    w = w + x * x;  // the product of two fp32-representable values is exact in fp64
  }
  const int64_t row = row0 + (active ? threadIdx.x : 0);
  if (active) a.vw[row] = w;
}

constexpr int kScanThreads = 1024;

// Inclusive prefix sums of the squared norms of one head, in fp64 and in a fixed order (a thread
// sums its run of rows, the threads' sums are scanned, every thread then walks its run again).
__global__ __launch_bounds__(kScanThreads) void vnorm_scan_kernel(Alg2Args a) {
  __shared__ double part[kScanThreads];
  const Geometry& g = a.g;
  const int bh = blockIdx.x;
  const int tid = threadIdx.x;
  const int per = (g.n + kScanThreads - 1) / kScanThreads;
  const int lo = min(g.n, tid * per), hi = min(g.n, lo + per);
  const double* w = a.vw + (int64_t)bh * g.n;
  double sum = 0.0;
  for (int l = lo; l < hi; ++l) sum += w[l];
  part[tid] = sum;
  __syncthreads();
  for (int off = 1; off < kScanThreads; off <<= 1) {
    double v = 0.0;
    if (tid >= off) v = part[tid - off];
    __syncthreads();
    part[tid] += v;
    __syncthreads();
  }
  double run = tid > 0 ? part[tid - 1] : 0.0;
  for (int l = lo; l < hi; ++l) {
    run += w[l];
    a.vprefix[(int64_t)bh * g.n + l] = run;
  }
}

__global__ void vnorm_sample_kernel(Alg2Args a) {
  const Geometry& g = a.g;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)g.BH * g.m) return;
  const int vh = (int)(t / g.m), r = (int)(t % g.m);
  const Alg2Node nd = alg2_node(a, vh);
  const double* prefix = a.vprefix + (int64_t)vh * g.n;
  const double total = prefix[g.n - 1];
  const uint64_t ctr = ((uint64_t)nd.heap * a.heads + nd.head) * g.m + r;
  const double u = ((double)(rand_u64(a.seed, kStreamVnorm, ctr) >> 11) + 0.5) * 0x1.0p-53;
  int lo;
  double p;
  if (total > 0.0) {
    const double target = u * total;
    int hi = g.n - 1;  // first l with prefix[l] > target
    lo = 0;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (prefix[mid] > target) hi = mid;
      else lo = mid + 1;
    }
    p = a.vw[(int64_t)vh * g.n + lo] / total;
  } else {  // V = 0: every choice gives the same (zero) product; uniform
    lo = min(g.n - 1, (int)(u * (double)g.n));
    p = 1.0 / (double)g.n;
  }
  const int64_t at = ((int64_t)nd.head * a.total_nodes + nd.heap) * g.m + r;
  a.vsamp[at] = lo;
  a.vlogw[at] = (float)(-log((double)g.m * p));
}

// log of the unmasked row sum of the rows T_j over a range of the keys, on the fp32 matrix cores: a workgroup per head, range and
// 32 rows of T, whose four waves take every fourth tile of 32 keys, as in attn_f32.hip (S^T = K Q^T: a lane holds 16 keys of one
// row; K fragments straight from the caches; sums merged through LDS at the end).  Bound by latency: a wave has a few tiles.
// 64 rows of two heads, n = 4096, d = 128: one thread per key and two rows, a head's keys in one range 582 us, in eight 55,
// this form 19; 4 heads, n = 2048, m = 256: 84 -> 14.
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kTauRows = 32, kTauKeys = 32, kTauWaves = 4;

template <int D>
__global__ __launch_bounds__(64 * kTauWaves, 2) void alg2_tau_kernel(Alg2Args a) {
  constexpr int KJ = D / 8;
  __shared__ float red_m[2 * kTauWaves][kTauRows], red_s[2 * kTauWaves][kTauRows];
  const Geometry& g = a.g;
  const int groups_per_head = (g.m + kTauRows - 1) / kTauRows;
  const int idx = a.wg_first + (int)blockIdx.x;
  const int split = idx % kAlg2TauSplits, row_group = idx / kAlg2TauSplits;
  const int bh = row_group / groups_per_head, j0 = (row_group % groups_per_head) * kTauRows;
  const int nr = min(kTauRows, g.m - j0);
  const int64_t hb = (int64_t)bh * g.n;   // bh: view head (one node)
  const Alg2Node nd = alg2_node(a, bh);
  const float* Qh = reinterpret_cast<const float*>(a.Q) + ((int64_t)nd.head * a.n_full + nd.q_start) * D;
  const float* Kh = reinterpret_cast<const float*>(a.K) + ((int64_t)nd.head * a.n_full + nd.k_start) * D;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lq = tid & 31, h = (tid >> 5) & 1;
  const int ntiles = (g.n + kTauKeys - 1) / kTauKeys;
  const int t_lo = (int)((int64_t)ntiles * split / kAlg2TauSplits), t_hi = (int)((int64_t)ntiles * (split + 1) / kAlg2TauSplits);

  f32x4 kf[KJ];
  auto load_k = [&](int kt) {  // (rows past the end: the last one, masked below)
    const float* kr = Kh + (int64_t)min(kt * kTauKeys + lq, g.n - 1) * D + 4 * h;
#pragma unroll
    for (int j = 0; j < KJ; ++j) kf[j] = *reinterpret_cast<const f32x4*>(kr + 8 * j);
  };
  if (t_lo + wave < t_hi) load_k(t_lo + wave);
  const int row = a.tau_rows[(int64_t)nd.heap * g.m + j0 + (lq < nr ? lq : 0)];
  const int blk0 = a.pos_q[hb + row] / g.b * g.b;  // first sorted position of the row's block
  f32x4 q[KJ];
#pragma unroll
  for (int j = 0; j < KJ; ++j) q[j] = *reinterpret_cast<const f32x4*>(Qh + (int64_t)row * D + 8 * j + 4 * h);

  float mx = -INFINITY, sum = 0.f;
  for (int kt = t_lo + wave; kt < t_hi; kt += kTauWaves) {
    const int base = kt * kTauKeys + 4 * h;  // accumulator register i: key base + 8 (i / 4) + i % 4
    int pos[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) pos[i] = a.pos_k[hb + min(base + 8 * (i / 4) + i % 4, g.n - 1)];
    f32x16 c;
#pragma unroll
    for (int i = 0; i < 16; ++i) c[i] = 0.f;
#pragma unroll
    for (int j = 0; j < KJ; ++j)
#pragma unroll
      for (int z = 0; z < 4; ++z) c = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[j][z], q[j][z], c, 0, 0, 0);
    if (kt + kTauWaves < t_hi) load_k(kt + kTauWaves);
    float top = mx;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const bool out = base + 8 * (i / 4) + i % 4 >= g.n || (uint32_t)(pos[i] - blk0) < (uint32_t)g.b;  // 1 - M
      c[i] = out ? -INFINITY : c[i];
      top = fmaxf(top, c[i]);
    }
    if (top > mx) {
      sum *= expf(mx - top);
      mx = top;
    }
    const float ref = mx == -INFINITY ? 0.f : mx;
#pragma unroll
    for (int i = 0; i < 16; ++i) sum += exp_split(c[i] - ref);
  }
  red_m[2 * wave + h][lq] = mx;
  red_s[2 * wave + h][lq] = sum;
  __syncthreads();
  if (tid < nr) {
    float M = -INFINITY;
#pragma unroll
    for (int t = 0; t < 2 * kTauWaves; ++t) M = fmaxf(M, red_m[t][tid]);
    float S = 0.f;
#pragma unroll
    for (int t = 0; t < 2 * kTauWaves; ++t)
      if (red_m[t][tid] > -INFINITY) S += red_s[t][tid] * expf(red_m[t][tid] - M);
    a.log_unm_parts[((int64_t)split * g.BH + bh) * g.m + j0 + tid] = (M == -INFINITY) ? -INFINITY : M + logf(S);
  }
}

// log tau = the largest log unmasked row sum over the rows of T, one workgroup per head; the sums over ranges of keys are
// added up first (and kept in log_unm_t).
__global__ __launch_bounds__(256) void alg2_tau_max_kernel(Alg2Args a) {
  __shared__ float red[256];
  const Geometry& g = a.g;
  const int bh = blockIdx.x;
  float mx = -INFINITY;
  for (int j = threadIdx.x; j < g.m; j += 256) {
    float p[kAlg2TauSplits];  // all requested at once: one after the other, with a logarithm each, they were most of 7 us
    float top = -INFINITY, sum = 0.f;
#pragma unroll
    for (int sp = 0; sp < kAlg2TauSplits; ++sp) p[sp] = a.log_unm_parts[((int64_t)sp * g.BH + bh) * g.m + j];
#pragma unroll
    for (int sp = 0; sp < kAlg2TauSplits; ++sp) top = fmaxf(top, p[sp]);
#pragma unroll
    for (int sp = 0; sp < kAlg2TauSplits; ++sp) sum += expf(p[sp] - (top == -INFINITY ? 0.f : top));
    const float v = top == -INFINITY ? -INFINITY : top + logf(sum);
    a.log_unm_t[(int64_t)bh * g.m + j] = v;
    mx = fmaxf(mx, v);
  }
  red[threadIdx.x] = mx;
  __syncthreads();
  for (int s = 128; s >= 1; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const Alg2Node nd = alg2_node(a, bh);
    a.log_tau[(int64_t)nd.head * a.total_nodes + nd.heap] = red[0];
  }
}

template <typename T>
static int launch_alg2_t(const Alg2Args& a_in, hipStream_t st) {
  const Geometry& g = a_in.g;
  Alg2Args a = a_in;
  constexpr bool mfma = sizeof(T) == 2;
  if (!a.pos_q_done) {
    const int64_t rows = (int64_t)g.BH * g.n;
    hipLaunchKernelGGL(alg2_pos_kernel, dim3((unsigned)((rows + 255) / 256)), dim3(256), 0, st, a);
  }
  if (a.vnorm && g.m > 0) {
    const unsigned vw_grid = (unsigned)((int64_t)g.BH * ((g.n + kVwRows - 1) / kVwRows));
    if (g.d == 128) hipLaunchKernelGGL((vnorm_weight_kernel<T, 128>), dim3(vw_grid), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((vnorm_weight_kernel<T, 64>), dim3(vw_grid), dim3(256), 0, st, a);
    hipLaunchKernelGGL(vnorm_scan_kernel, dim3((unsigned)g.BH), dim3(kScanThreads), 0, st, a);
    hipLaunchKernelGGL(vnorm_sample_kernel, dim3((unsigned)(((int64_t)g.BH * g.m + 255) / 256)), dim3(256), 0, st, a);
  }
  if constexpr (mfma) {
    if (g.m > 0) {
      const int rc = launch_alg2_tau_mfma(a, st);
      if (rc != HA_OK) return rc;
    }
    hipLaunchKernelGGL(alg2_tau_max_kernel, dim3((unsigned)g.BH), dim3(256), 0, st, a);
    return a.vnorm ? launch_alg2_main_mfma(a, st) : check_launch();  // (without value sampling: the caller's node launch)
  } else {
    if (g.m > 0) {
      const int64_t tau_grid = (int64_t)g.BH * ((g.m + kTauRows - 1) / kTauRows) * kAlg2TauSplits;
      if (tau_grid > 0x7fffffff) return HA_ERR_SHAPE;
      for (int64_t first = 0; first < tau_grid; first += kMaxLaunch) {
        a.wg_first = (int32_t)first;
        const unsigned count = (unsigned)(tau_grid - first < kMaxLaunch ? tau_grid - first : kMaxLaunch);
        if (g.d == 128) hipLaunchKernelGGL((alg2_tau_kernel<128>), dim3(count), dim3(256), 0, st, a);
        else hipLaunchKernelGGL((alg2_tau_kernel<64>), dim3(count), dim3(256), 0, st, a);
      }
    }
    hipLaunchKernelGGL(alg2_tau_max_kernel, dim3((unsigned)g.BH), dim3(256), 0, st, a);
    return check_launch();  // (then the caller's node launch)
  }
}

int launch_alg2(const Alg2Args& a, hipStream_t st) {
  if (a.g.d != 64 && a.g.d != 128) return HA_ERR_SHAPE;
  if (a.g.dtype == HA_BF16) return launch_alg2_t<uint16_t>(a, st);
  if (a.g.dtype == HA_FP32) return launch_alg2_t<float>(a, st);
  return HA_ERR_DTYPE;
}

}  // namespace ha
