// fp32 attention on the fp32 matrix cores: the arithmetic path for HA_FP32 tensors
// (v_mfma_f32_32x32x2_f32: fp32 products, fp32 sums), with the same node / cap / exact
// modes and the same outputs as the bf16 kernel (attn_mfma.hip).
//
// What bounds it: the matrix pipe where the chip is full (4 heads, n = 4096 in blocks of 1024, two waves per SIMD: busy 46 %
// of the cycles).  At d = 128, 32 to 64 bytes per lane spill (256 registers).  One 32 x 32 tile of scores and its product with V
// take D/2 + D/2 instructions of 64 cycles each, against 8 KiB of K and 8 KiB of V
// fragments at d = 64 that every wave reads straight from the caches into the operand
// layout (16 B/clk per CU where four waves share nothing): no LDS staging, hence no
// barrier in the loop and waves that run independently of each other.
//
// A wave owns 32 query rows and computes S^T = K Q^T, so that a lane holds 16 keys of
// ONE query (as in the bf16 kernel) and an accumulator register, exponentiated, is
// directly the B operand of O^T += V^T P^T: the two lanes of a query hold the keys
// 8 g + z and 8 g + 4 + z of the instruction's pair.  The columns of d are walked in
// the order the lanes load them (lane half h: columns 8 j + 4 h ... + 3), which the
// K and the Q fragments share.
//
// KW waves of a workgroup share one group of 32 queries, every wave taking each KW-th
// key tile, and their results are merged through LDS.  KW = 4 quarters the serial
// chain of a small problem (the one-head n = 1024 call has 32 groups of queries for
// 1024 SIMDs) and lets a workgroup fit blocks of 32 rows.
//
// Measured (MI355X; fp32 matrix peak 157 TFLOP/s, library product of 8192^3: 154), against
// one thread per query row with LDS-broadcast keys, the form before: exact attention,
// 32 heads, n = 8192: d = 64 14.8 -> 4.8 ms (114 TFLOP/s), d = 128 95 -> 8.9 ms (124);
// n = 1024, one head, d = 64, b = m = 64: whole forward call 124 -> 35 us.  Then the vector work beside the products:
// the wave's number is a scalar (with a per-lane key loop the compiler wrapped every buffer load in a loop over
// possible descriptors), exponentials in seven instructions, fewer rescales: 32 heads, n = 1024, d = 64, unmasked:
// 111 -> 79 us; 4 heads, n = 4096 in causal blocks of 1024: 50 -> 39 us.  Errors against 64 bits as before.
#include "attn_common.h"
#include "node_sort.h"

namespace ha {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

constexpr int kFKT = 32;   // keys per tile
constexpr int f32_waves(int kw) { return kw == 8 ? 8 : 4; }  // of a workgroup, by the waves that share 32 queries

template <int D, int NW = 4>
struct F32Lds {
  static constexpr int ROW = D + 4;                // floats per staged output row
  static constexpr int BYTES = NW * 32 * ROW * 4 + NW * 32 * 2 * 4;
};

template <int D>
__host__ __device__ inline size_t f32_lds_bytes(int b, int m, int mode) {
  const size_t list = mode != kModeExact ? (size_t)(((b + m + 63) & ~63) + 64) * 4 + 64 : 0;
  // behind the list: the rows drawn by value norm with their weights, the waves' masked sums; two more values per staged row
  const size_t cap = mode == kModeCap || mode == kModeValue ? 4 * 32 * 2 * 4 : 0;
  const size_t drawn = mode == kModeValue ? 2 * (size_t)((m + 63) & ~63) * 4 : 0;
  return list + drawn + cap > (size_t)F32Lds<D>::BYTES + cap ? list + drawn + cap : (size_t)F32Lds<D>::BYTES + cap;
}

// SORT: the sort's tables lie behind the list, the tile's query rows behind all else
template <int D>
__host__ __device__ inline size_t f32_qrows_at(const Geometry& g) {
  const size_t list = ((size_t)(((g.b + g.m + 63) & ~63) + 64) * 4 + 64 + 15) & ~(size_t)15;
  const size_t both = list + ((node_sort_lds_bytes<4>(g) + 15) & ~(size_t)15);
  return both > (size_t)F32Lds<D>::BYTES ? both : (size_t)F32Lds<D>::BYTES;
}

// m + ln l to one rounding of the result: l = f 2^k with f in [1/2, 1), m + k ln 2 kept in two parts.  The reference m only
// moves by steps, so ln l can be as large as the result, and logf of all of it had an error of that size beside the
// result's own: log row sums of blocks and samples (n = 2048, b = m = 128, d = 64) 5.4e-8 off against 64 bits where a
// reference at the row's maximum had 4.6e-8; now 3.2e-8.
__device__ inline float add_log(float m, float l) {
  int k;
  const float f = frexpf(l, &k);
  const float hi = (float)k * 0.693145752f;  // ln 2 in 12 bits: exact for |k| < 4096
  const float s = m + hi, t = s - m;
  const float left = (m - (s - t)) + (hi - t);  // what the rounding of m + hi left out
  return s + (left + __builtin_fmaf((float)k, 1.42860677e-6f, logf(f)));
}

// FAR (node mode): a head's rows pass the reach of a buffer load's 32-bit offset, so they are addressed in 64 bits.
// SORT (node mode): the workgroup finds its rows from the node's bucket codes (node_sort.h).
template <int D, int MODE, int KW, bool FAR, bool SORT>
__global__ __launch_bounds__(64 * f32_waves(KW), D == 64 && KW < 8 ? 3 : 2) void attn_f32_kernel(AttnArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int NW = f32_waves(KW), kFNT = 64 * NW;
  constexpr int kQT = 32 * (NW / KW);
  constexpr bool kValue = MODE == kModeValue, kCap = MODE == kModeCap || kValue, kNode = MODE == kModeNode || kCap;
  constexpr int KJ = D / 8;    // 16-byte pieces of a row per lane
  constexpr int DT = D / 32;
  constexpr int DTA = DT < 2 ? DT : 2;  // V columns are fetched 64 at a time
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // a scalar: so are the key loop and the descriptors
  const int lq = lane & 31, h = lane >> 5;
  const int kw = wave % KW;

  int32_t* scratch = reinterpret_cast<int32_t*>(smem);
  int32_t* list = scratch + 16;

  const int bid = a.wg_first + (kNode ? logical_block(blockIdx.x, gridDim.x) : (int)blockIdx.x);
  TileWork w;
  int nb, nkeys;
  int32_t* qrows = reinterpret_cast<int32_t*>(smem + (SORT ? f32_qrows_at<D>(a.g) : 0));
  if constexpr (SORT) {
    w = decode_node_tile<kQT>(a, bid);
    const int l0 = first_node_sample(a, w);
    unsigned char* sort_lds = reinterpret_cast<unsigned char*>(list) + (((((a.g.b + a.g.m + 63) & ~63) + 64) * 4 + 15) & ~15);
    sort_node_tile<4>(a, w, sort_lds, list, qrows);
    nb = a.g.b;
    nkeys = append_node_samples<4>(a, w, sort_lds, list, scratch, l0);
  } else if (kNode) {
    w = decode_node_tile<kQT>(a, bid);
    nkeys = build_key_list<kFNT, kCap>(a, w, list, scratch, &nb, key_list_fetch<kFNT>(a, w));
  } else {
    w = decode_exact_tile<kQT>(a, bid);
    nkeys = max(0, w.k1 - w.k0);
    nb = 0x7fffffff;
  }
  int ntiles = (nkeys + kFKT - 1) / kFKT;
  // causal: a wave ends with the tile that holds its own last row.  Tiles wholly behind its rows are not only idle work:
  // weight 0 times a V that is Inf or NaN is NaN.
  if (MODE == kModeExact && a.exact_causal) ntiles = min(ntiles, (w.q0 - w.k0) / kFKT + wave / KW + 1);
  // value mode: the rows drawn by value norm, all m of them for every block, follow in tiles of their own
  const int vt0 = ntiles, drawn_at = (((a.g.b + a.g.m + 63) & ~63) + 64) + ((a.g.m + 63) & ~63);
  float* drawn_w = reinterpret_cast<float*>(list + drawn_at);  // -log(m p); -inf past the end
  if constexpr (kValue) {
    const int64_t draws = ((int64_t)w.bh * a.g.total_nodes + w.nr.heap) * a.g.m;
    for (int j = tid; j < ((a.g.m + 31) & ~31); j += kFNT) {
      list[vt0 * kFKT + j] = w.nr.k_start + a.vsamp[draws + min(j, a.g.m - 1)];
      drawn_w[j] = j < a.g.m ? a.vlogw[draws + j] : -INFINITY;
    }
    ntiles += (a.g.m + 31) / kFKT;
    __syncthreads();
  }
  const float nat_bias = (kNode && a.g.m > 0) ? logf((float)w.nr.s / (float)a.g.m) : 0.f;

  const float* Qh = reinterpret_cast<const float*>(a.Q) + (int64_t)w.bh * a.q_bh_stride;
  const float* Kh = reinterpret_cast<const float*>(a.K) + (int64_t)w.bh * a.k_bh_stride;
  const float* Vh = reinterpret_cast<const float*>(a.V) + (int64_t)w.bh * a.k_bh_stride;
  const int r_in_tile = (wave / KW) * 32 + lq;
  const int r_use = r_in_tile < w.rows_valid ? r_in_tile : 0;
  int qrow, q_global = 0;
  if constexpr (SORT) {
    qrow = qrows[r_use];
  } else if (kNode) {
    qrow = a.perm_q ? a.perm_q[w.seg_off + w.p0 + r_use] : w.nr.q_start + w.p0 + r_use;
  } else {
    q_global = w.q0 + r_in_tile;
    qrow = w.q0 + r_use;
  }
  f32x4 q[KJ];
#pragma unroll
  for (int j = 0; j < KJ; ++j) q[j] = *reinterpret_cast<const f32x4*>(Qh + (int64_t)qrow * D + 8 * j + 4 * h);

  // rows past the end of the keys read as zeros (such keys are masked by position)
  const uint32_t bytes = (uint32_t)(kNode ? a.g.n : w.k1) * (uint32_t)(D * 4);
  const __amdgpu_buffer_rsrc_t krsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Kh, 0, (int)bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t vrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Vh, 0, (int)bytes, 0x00020000);
  f32x4 kf[KJ];
  auto load_k = [&](int kt) {
    const int row = kNode ? list[kt * kFKT + lq] : w.k0 + kt * kFKT + lq;
    if constexpr (FAR) {  // (every row of the list exists)
#pragma unroll
      for (int j = 0; j < KJ; ++j) kf[j] = *reinterpret_cast<const f32x4*>(Kh + (int64_t)row * D + 8 * j + 4 * h);
      return;
    }
    const int off = row * (D * 4) + 16 * h;
#pragma unroll
    for (int j = 0; j < KJ; ++j)
      kf[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(krsrc, off, 32 * j, 0));
  };
  // V rows of the tile, columns 32 dt + lq for dt in [dt0, dt0 + DTA): element i of a lane is key
  // 8 (i / 4) + 4 h + i % 4, the key of accumulator register i
  auto load_v = [&](int kt, int dt0, float (&v)[16][DTA]) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      i32x4 rows;
      if (kNode) {
        rows = *reinterpret_cast<const i32x4*>(list + kt * kFKT + 8 * g + 4 * h);
      } else {
        const int r0 = w.k0 + kt * kFKT + 8 * g + 4 * h;
        rows = (i32x4){r0, r0 + 1, r0 + 2, r0 + 3};
      }
#pragma unroll
      for (int z = 0; z < 4; ++z)
#pragma unroll
        for (int dt = 0; dt < DTA; ++dt)
          v[4 * g + z][dt] = FAR ? Vh[(int64_t)rows[z] * D + 32 * (dt0 + dt) + lq]
                                 : __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(vrsrc, rows[z] * (D * 4) + 4 * lq,
                                                                                       128 * (dt0 + dt), 0));
    }
  };

  f32x16 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[dt][i] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;

  // Cap mode (Algorithm 2 as printed): the block's keys, padded to whole tiles, come first; then every sample's weight
  // counts at most C_i in the row sum, whose cap follows from the masked sum of all waves of the row.  One thread per query row
  // had walked both parts before: whole calls with the launch for tau of that time 950 -> 98 us (2 heads, n = 4096, d = 128, b = m = 64;
  // this launch 23), 4 heads, n = 2048, b = m = 256 1590 -> 149 (44), 8 heads, n = 1024, d = 64, b = m = 256 609 -> 72 (21); with the sums of
  // alg2_tau_kernel as they are 62, 73 and 46.
  // Value mode (Lemma 2's rows carry the output): block and samples only sum, the drawn rows, with their log weights, only
  // add to the output.  One thread per query row before: 4 heads, n = 2048, d = 128, b = m = 256 1287 -> 88 us; 8 heads, n = 1024, d = 64
  // 551 -> 60; 2 heads, n = 4096, d = 128, b = 512, m = 1000 3871 -> 203 (the first two now 84 and 58).
  // The switch to the samples sits in the one loop: a loop per part, shared with the other modes, cost those up to 4 %.
  // Scores of one row can lie hundreds apart, so no sum may hang on another's reference: the masked sum is final, as a logarithm,
  // before the first sample counts.  The samples' sum (l_run) is taken against sum_ref: the output's reference m_run, or the cap
  // where that is far below, since no capped term exceeds it.  Value mode, whose output has no part in the samples, begins each
  // part with a reference of its own and keeps the samples' in d_ref.  (With all sums on m_run, rows of clustered inputs lost
  // log d~ to underflow: 150 of 2048, d = 64, b = m = 64, cap 8.  Time: 32 heads, n = 8192, b = m = 256, d = 64 590 -> 578 us, d = 128 1134 ->
  // 1122, with value sampling 1214 -> 1210, 4 heads, n = 2048 82.3 -> 83.7.)
  const int nbt = kCap ? ((nb + 63) & ~63) / kFKT : 0;
  float log_masked = -INFINITY, log_capw = INFINITY;  // log of the row's masked sum, of (s / m) C_i
  float d_ref = -INFINITY;
  constexpr float kFarCap = 40.f;  // a term that underflows against m_run is then e^-47 of the cap or less
  auto sum_ref = [&](float m) { return kCap && !kValue && m > log_capw + kFarCap ? log_capw : m; };
  auto finite_ref = [](float m) { return m == -INFINITY ? 0.f : m; };
  const float floor_term = kCap && a.kappa > 0.f ? a.log_tau[(int64_t)w.bh * a.g.total_nodes + w.nr.heap] - logf(a.kappa) : -INFINITY;
  bool sampled = false, drawn = false;
  auto to_samples = [&]() {  // every wave comes here once
    float* ex = reinterpret_cast<float*>(list + (kValue ? drawn_at + ((a.g.m + 63) & ~63) : ((a.g.b + a.g.m + 63) & ~63) + 64));  // [4 waves][32][2]
    const float mine = l_run + __shfl_xor(l_run, 32);
    if (h == 0) {
      ex[(wave * 32 + lq) * 2] = m_run;
      ex[(wave * 32 + lq) * 2 + 1] = mine;
    }
    __syncthreads();
    float top = -INFINITY, sum = 0.f;
#pragma unroll
    for (int k = 0; k < KW; ++k) top = fmaxf(top, ex[((wave / KW * KW + k) * 32 + lq) * 2]);
#pragma unroll
    for (int k = 0; k < KW; ++k) {
      const float* e = ex + ((wave / KW * KW + k) * 32 + lq) * 2;
      sum += e[1] * (top == -INFINITY ? 0.f : expf(e[0] - top));
    }
    log_masked = sum > 0.f ? add_log(top, sum) : -INFINITY;
    if (a.cap_scale > 0.f) {
      const float n = (float)w.nr.s;
      log_capw = logf(a.cap_scale * (float)a.g.m / (n * logf(n))) + logaddexpf(log_masked, floor_term) + nat_bias;
    }
    l_run = 0.f;
    if (kValue) m_run = -INFINITY;
    sampled = true;
  };
  if (kw < ntiles) load_k(kw);
  for (int kt = kw; kt < ntiles; kt += KW) {
    float va[16][DTA];
    if constexpr (DT == 2 && !kValue) load_v(kt, 0, va);
    f32x16 c;
#pragma unroll
    for (int i = 0; i < 16; ++i) c[i] = 0.f;
#pragma unroll
    for (int j = 0; j < KJ; ++j) {
      if (DT > 2 && !kValue && j == KJ / 2) {  // d = 128: V takes the registers of the K pieces already multiplied
        __builtin_amdgcn_sched_barrier(0);
        load_v(kt, 0, va);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[j][e], q[j][e], c, 0, 0, 0);
    }

    const int base = kt * kFKT;
    if constexpr (kCap) {
      if (kt >= nbt && !sampled) to_samples();
      const int lim = sampled ? nkeys : nb;
      if (kValue && kt >= vt0) {
        if (!drawn) {
          d_ref = m_run;
          m_run = -INFINITY;
          drawn = true;
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 lw = *reinterpret_cast<const f32x4*>(drawn_w + (kt - vt0) * kFKT + 8 * g + 4 * h);
#pragma unroll
          for (int z = 0; z < 4; ++z) c[4 * g + z] = lw[z] == -INFINITY ? -INFINITY : c[4 * g + z] + lw[z];
        }
      } else if (sampled || base + kFKT > lim) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int pos = base + 8 * (i / 4) + 4 * h + (i % 4);
          c[i] = pos >= lim ? -INFINITY : c[i] + (sampled ? nat_bias : 0.f);
          if (kValue && sampled && a.cap_scale > 0.f) c[i] = fminf(c[i], log_capw);
        }
      }
    }
    const bool plain = kCap || base + kFKT <= min(nkeys, nb) &&
                       !(MODE == kModeExact && a.exact_causal && w.k0 + base + kFKT - 1 > w.q0 + (wave / KW) * 32);
    if (!plain) {
      int lim = nkeys;
      if (MODE == kModeExact && a.exact_causal) lim = min(lim, q_global - w.k0 + 1);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int pos = base + 8 * (i / 4) + 4 * h + (i % 4);
        const float s = c[i] + (pos >= nb ? nat_bias : 0.f);
        c[i] = pos >= lim ? -INFINITY : s;
      }
    }
    float mx = c[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = fmaxf(mx, c[i]);
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    // (the reference only moves by steps of 2^8, as in the bf16 kernel: a rescale is a twelfth of a tile's vector work)
    if (__any(mx > m_run + 5.5f)) {
      const float m_new = fmaxf(m_run, mx);
      const float alpha = expf(m_run - finite_ref(m_new));
      if (!kValue || kt < vt0) l_run *= kCap ? expf(sum_ref(m_run) - finite_ref(sum_ref(m_new))) : alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[dt][i] *= alpha;
      m_run = m_new;
    }
    const float m_use = finite_ref(m_run);
    float capw = INFINITY;
    if constexpr (kCap && !kValue) {
      if (sampled) capw = expf(log_capw - m_use);
      if (sampled && __any(m_run > log_capw + kFarCap)) {  // rare: exponentials of the sum's own
        const float ref = finite_ref(sum_ref(m_run));
#pragma unroll
        for (int i = 0; i < 16; ++i) l_run += exp_split(fminf(c[i], log_capw) - ref);
        capw = 0.f;
      }
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      c[i] = exp_split(c[i] - m_use);
      if (!kValue || kt < vt0) l_run += kCap ? fminf(c[i], capw) : c[i];
    }
    if constexpr (DT == 2) {
      if (kt + KW < ntiles) load_k(kt + KW);
    }
    float vb[16][DTA];
    if constexpr (kValue) {  // V behind the sums, 64 columns at a time (fetched amid the products, under a branch: 168 spills at d = 128)
      if (DT > 2 && kt + KW < ntiles) load_k(kt + KW);
      if (kt < vt0) continue;
#pragma unroll
      for (int dt0 = 0; dt0 < DT; dt0 += 2) {
        load_v(kt, dt0, va);
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
          for (int dt = 0; dt < DTA; ++dt)
            o[dt0 + dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[i][dt], c[i], o[dt0 + dt], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      continue;
    }
    if constexpr (DT > 2) load_v(kt, 2, vb);
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
      for (int dt = 0; dt < DTA; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[i][dt], c[i], o[dt], 0, 0, 0);
    if constexpr (DT > 2) {
      __builtin_amdgcn_sched_barrier(0);  // the next K rows take the registers of the first half of V
      if (kt + KW < ntiles) load_k(kt + KW);
#pragma unroll
      for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int dt = 0; dt < DTA; ++dt)
          o[2 + dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(vb[i][dt], c[i], o[2 + dt], 0, 0, 0);
    }
  }
  if constexpr (kCap) {
    if (!sampled) to_samples();
  }

  // ---- results: every wave's rows through LDS, where the KW parts of a row are merged and rows
  // leave as whole 16-byte pieces of consecutive lanes ----
  constexpr int RS = F32Lds<D>::ROW;
  float* orow = reinterpret_cast<float*>(smem);   // [waves][32][RS]
  float* ml = orow + NW * 32 * RS;                // [waves][32][ML]: reference, row sum; cap mode: of the samples, its reference, log of the masked sum
  constexpr int ML = kCap ? 4 : 2;
  const float l_tot = l_run + __shfl_xor(l_run, 32);
  if (kCap && !drawn) d_ref = sum_ref(m_run);
  __syncthreads();  // the key list is read no more
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<f32x4*>(orow + (wave * 32 + lq) * RS + 32 * dt + 8 * g + 4 * h) =
          (f32x4){o[dt][4 * g], o[dt][4 * g + 1], o[dt][4 * g + 2], o[dt][4 * g + 3]};
  if (h == 0) {
    ml[(wave * 32 + lq) * ML] = m_run;
    ml[(wave * 32 + lq) * ML + 1] = l_tot;
    if (kCap) {
      ml[(wave * 32 + lq) * ML + 2] = d_ref;
      ml[(wave * 32 + lq) * ML + 3] = log_masked;  // (the same in all waves of a row)
    }
  }
  __syncthreads();
  constexpr int LPR = D / 4;  // lanes per row
  const bool to_partial = kNode && a.part_o != nullptr;
  for (int idx = tid; idx < w.rows_valid * LPR; idx += kFNT) {
    const int r = idx / LPR, col = (idx % LPR) * 4;
    const int w0 = (r / 32) * KW;  // first of the waves that hold the row
    float mx = -INFINITY, dmx = -INFINITY;
#pragma unroll
    for (int k = 0; k < KW; ++k) {
      mx = fmaxf(mx, ml[((w0 + k) * 32 + (r & 31)) * ML]);
      if (kCap) dmx = fmaxf(dmx, ml[((w0 + k) * 32 + (r & 31)) * ML + 2]);
    }
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float l = 0.f;
#pragma unroll
    for (int k = 0; k < KW; ++k) {
      const int at = (w0 + k) * 32 + (r & 31);
      const float wk = KW == 1 ? 1.f : (mx == -INFINITY ? 0.f : expf(ml[at * ML] - mx));
      l += (kCap && KW > 1 ? expf(ml[at * ML + 2] - finite_ref(dmx)) : wk) * ml[at * ML + 1];
      acc += wk * *reinterpret_cast<const f32x4*>(orow + at * RS + col);
    }
    const bool empty = !(l > 0.f);
    float lse = empty ? -INFINITY : add_log(kCap ? dmx : mx, l);
    float ref = lse;  // of a partial row
    if constexpr (kCap) {  // d~_i = masked + max(d_i, tau / kappa)
      lse = logaddexpf(ml[(w0 * 32 + (r & 31)) * ML + 3], fmaxf(lse, floor_term));
      ref = to_partial && a.part_ref != nullptr && lse != -INFINITY ? fmaxf(lse, mx) : lse;
      acc *= (mx == -INFINITY || lse == -INFINITY) ? 0.f : expf(mx - ref);
    } else {
      acc *= empty ? 0.f : 1.f / l;
    }
    RowDest dest{};
    if constexpr (SORT) {
      dest.out_row = (int64_t)w.bh * a.g.n + qrows[r];
      dest.part_row = w.seg_off + (qrows[r] - w.nr.q_start);
    } else if (kNode) {
      dest = node_row_dest(a, w, r);
    } else {
      dest.row_in_head = w.q0 + r;
      dest.out_row = (int64_t)w.bh * (a.out_bh_stride / D) + w.q0 + r;
    }
    if (to_partial) {
      *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.part_o) + dest.part_row * D + col) = acc;
      if (col == 0) a.part_l[dest.part_row] = lse;
      if (kCap && col == 0 && a.part_ref != nullptr) a.part_ref[dest.part_row] = ref;
      continue;
    }
    if (MODE == kModeExact && a.merge_levels > 0) {
      float rmx, den;
      const float Lm = merged_lse(a, w.bh, dest.row_in_head, lse, &rmx, &den);
      acc *= lse == -INFINITY ? 0.f : expf(lse - rmx) / den;
      for (int l2 = 0; l2 < a.merge_levels; ++l2) {
        int64_t pr;
        if (!level_touches(a.g, w.bh, dest.row_in_head, l2, &pr)) continue;
        const float lp = a.part_l[pr];
        if (lp == -INFINITY) continue;
        const float rp = a.part_ref != nullptr ? a.part_ref[pr] : lp;
        acc += (expf(rp - rmx) / den) * *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(a.part_o) + pr * D + col);
      }
      lse = Lm;
    }
    if (a.out != nullptr) *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.out) + dest.out_row * D + col) = acc;
    if (a.lse != nullptr && col == 0) a.lse[dest.out_row] = lse;
  }
}

template <int D, int MODE, int KW, bool FAR = false, bool SORT = false>
static int launch_f32_one(const AttnArgs& args, hipStream_t st) {
  constexpr int NW = f32_waves(KW), kQT = 32 * (NW / KW);
  AttnArgs a = args;
  if (MODE != kModeExact) set_node_divs<kQT>(a);
  else set_exact_divs<kQT>(a);
  a.exact_lpt = KW == 8;
  const int64_t grid = MODE != kModeExact ? node_grid<kQT>(a.g) : exact_grid<kQT>(a);
  if (grid <= 0) return HA_OK;
  if (grid > kMaxGrid) return HA_ERR_SHAPE;
  const size_t lds = KW == 8 ? (size_t)F32Lds<D, NW>::BYTES : SORT ? f32_qrows_at<D>(a.g) + kQT * 4 : f32_lds_bytes<D>(a.g.b, a.g.m, MODE);
  static std::atomic<uint64_t> lds_set{0};  // per instantiation: devices on which the LDS limit is raised
  if (allow_full_lds(reinterpret_cast<const void*>(&attn_f32_kernel<D, MODE, KW, FAR, SORT>), lds_set) != HA_OK) return HA_ERR_LAUNCH;
  for (int64_t first = 0; first < grid; first += kMaxLaunch) {
    a.wg_first = (int32_t)first;
    const int64_t count = grid - first < kMaxLaunch ? grid - first : kMaxLaunch;
    hipLaunchKernelGGL((attn_f32_kernel<D, MODE, KW, FAR, SORT>), dim3((unsigned)count), dim3(64 * NW), lds, st, a);
    const int rc = check_launch();
    if (rc != HA_OK) return rc;
  }
  return HA_OK;
}

// Waves that share a group of 32 queries: as few as leave the chip's 1024 SIMDs two waves each, but
// enough that a workgroup's 128 / KW rows do not outgrow the run of rows it is cut from (a block of b
// sorted positions, an exact diagonal block) by more than a third: idle rows cost matrix time like real
// ones, while the merge of KW results costs a few LDS reads per row.
static int f32_waves_per_group(int run, int64_t grid128) {
  auto padded = [&](int qt) { return (int64_t)((run + qt - 1) / qt) * qt; };
  const int64_t waves = 4 * grid128;
  if (waves >= 2048 && 3 * padded(128) <= 4 * (int64_t)run) return 1;
  return waves >= 1024 && 3 * padded(64) <= 4 * (int64_t)run ? 2 : 4;
}

int64_t attn_f32_node_grid(const Geometry& g) {
  const int kw = f32_waves_per_group(g.b, node_grid<128>(g));
  return kw == 1 ? node_grid<128>(g) : kw == 2 ? node_grid<64>(g) : node_grid<32>(g);
}

// Whether a node launch sorts by itself (attn_mfma_sorts, for the kernel without it).  d = 64: up to 1024 workgroups.  d = 128 has 512
// places, two to a CU; past them, from some 580 to 768 workgroups, calls whose workgroups sort take up to a fifth longer (they start and
// end together, and the second round seems to fall on the CUs unevenly: its places were not recorded).  Sorting launch -> in the attention (MI355X, us; workgroups, of
// 128 rows, of 64, of 32):
//   d = 64, b = m = 64: one head, n = 1024 (32) 21.2 -> 17.2; 24 heads, n = 2048 (768) 51.4 -> 46.8; 16 heads, n = 4096 (1024) 66.7 -> 62.7,
//     32 (2048) 106.1 -> 108.1; 64 heads, n = 1024 (1024) 65.3 -> 61.8; 6 heads, n = 4100, b = 82 (900) 48.6 -> 49.1
//   d = 128, 128 rows: 32 heads, n = 2048, b = m = 128 (512) 134.0 -> 128.3, 36 (576) 179.9 -> 173.6, 44 (704) 189.2 -> 183.7, 48 (768) 196.7 ->
//     223.8, 52 (832) 238.0 -> 231.8, 64 (1024) 254.4 -> 247.4; b = m = 256: 40 (640) 287.9 -> 280.0, 48 (768) 334.2 -> 348.1; n = 512, b = 128, m =
//     32: 180 heads (720) 152.7 -> 158.2; n = 1000, b = 100, m = 64: 56 heads (560) 133.7 -> 129.8, 61 (610) 137.4 -> 151.0, 90 (900) 180.4 -> 175.3
//   64 rows: 16 heads, n = 2048, b = m = 64 (512) 60.6 -> 59.1, 18 (576) 79.9 -> 78.7, 20 (640) 81.1 -> 80.2, 23 (736) 85.0 -> 87.8, 24 (768) 86.0 ->
//     97.2, 32 (1024) 109.3 -> 110.2; b = m = 256: 18 (576) 156.8 -> 156.0, 20 (640) 167.7 -> 183.5; n = 6144, b = 64: 4 heads (384) 59.0 -> 58.8,
//     n = 8192: 2 heads (256) 42.2 -> 38.3, 3 (384) 58.9 -> 60.4; b = 128: 4 heads (512) 80.5 -> 85.2
//   32 rows, of long blocks: 4 heads, n = 4096, b = m = 256 (512) 70.1 -> 67.0, 6 (768) 99.0 -> 108.2; 8 heads, n = 2100, b = 100 (672) 67.9 -> 68.2;
//     2 heads, n = 8192, b = 256 (512) 70.8 -> 75.1; of blocks that 64 rows do not fill: 24 heads, n = 1024, b = 32 (768) 57.0 -> 55.0, 32
//     (1024) 63.9 -> 62.8; 8 heads, n = 4096, b = 32 (1024) 65.1 -> 64.7
// Where the sort's tables cost a CU one of its workgroups, calls that need it lose more the longer the attention is: d = 64, b = m = 64: 7 heads,
// n = 6144 (672) 52.7 -> 51.9, m = 256 74.1 -> 73.5; b = m = 256, 11 heads (528) 152.9 -> 154.4; b = 64, m = 1000: 6 heads (576) 152.9 -> 160.0; r = 8: 9
// heads, n = 4096 (576) 152.0 -> 157.7; b = 128, m = 2000, 8 heads, n = 8192 (512, one to a CU) 352 -> 396; d = 128, the same 643 -> 723.
template <int D>
static bool f32_tables_cost(const Geometry& g, int64_t wgs, int kw) {
  const int64_t sorting = lds_workgroups(f32_qrows_at<D>(g) + 128 / kw * 4, D == 64 ? 3 : 2);
  return wgs > 256 * sorting && sorting < lds_workgroups(f32_lds_bytes<D>(g.b, g.m, kModeNode), D == 64 ? 3 : 2);
}

bool attn_f32_sorts(const Geometry& g) {
  const int rows = node_sort_rows(g);
  const int64_t wgs = attn_f32_node_grid(g);
  if (rows > kNodeSortMax || wgs > 1024 || wgs * rows > 4 << 20) return false;
  const int kw = f32_waves_per_group(g.b, node_grid<128>(g));
  if (g.b + g.m > 320 && (g.d == 64 ? f32_tables_cost<64>(g, wgs, kw) : f32_tables_cost<128>(g, wgs, kw))) return false;
  if (g.d == 64 || 4 * g.b < 3 * 64) return true;
  if (kw > 1 && wgs * rows > 5 << 19) return false;
  return wgs <= (kw == 4 ? 512 : kw == 1 && g.b % 128 == 0 ? 704 : 576) || (kw == 1 && wgs > 768);
}

// Exact launches of few workgroups and long rows are bound by the longest chain of key tiles: eight waves then share 32 queries,
// two per SIMD where four left one, a workgroup that fills a CU (causal: up to one and a half or two rounds of those, heaviest first).
// Four waves -> eight (MI355X, us; groups of 32 rows in brackets): d = 128: causal, 16 heads, n = 512 (256) 29.9 -> 28.8; 12 heads,
// n = 1024 (384) 54.7 -> 49.5, 16 (512) 55.1 -> 58.9; 8 heads, n = 2048 (512) 96.4 -> 92.9; 4 heads, n = 4000 (500) 176 -> 162, 1 head 179 -> 141;
// unmasked, 8 heads, n = 1024 (256) 52.1 -> 48.2, 12 (384) 79.8 -> 87.9; 1 head, n = 4000 181 -> 146, 3 (375) 275 -> 285.
// d = 64: causal, 8 heads, n = 1024 (256) 24.0 -> 25.0; 6 heads, n = 2048 (384) 48.9 -> 41.8, 8 (512) 49.0 -> 50.6; 3 heads, n = 4000 (375)
// 84.5 -> 75.1; unmasked, 1 head, n = 2048 (64) 42.4 -> 41.9, 4 (256) 42.7 -> 42.6.
bool f32_exact_eight(const AttnArgs& a) {
  const int rows = a.exact_block < a.exact_rows_q ? a.exact_block : a.exact_rows_q;
  const int64_t groups = exact_grid<32>(a);
  if (a.g.d == 128) return rows >= 512 && groups <= (!a.exact_causal ? 256 : rows < 2048 ? 384 : 512);
  return rows >= 2048 && groups <= (a.exact_causal ? 384 : 128);
}

template <int D, int MODE>
static int launch_f32_mode(const AttnArgs& a, hipStream_t st) {
  if constexpr (MODE == kModeNode)  // stage calls alone: the whole-call entry points take up to 2^22 rows per head
    if ((int64_t)a.g.n * (D * 4) > 0x7fffffff + 1ll) return launch_f32_one<D, MODE, 4, true>(a, st);
  const int run = MODE != kModeExact ? a.g.b : (a.exact_block < a.exact_rows_q ? a.exact_block : a.exact_rows_q);
  const int kw = f32_waves_per_group(run, MODE != kModeExact ? node_grid<128>(a.g) : exact_grid<128>(a));
  if constexpr (MODE == kModeNode)
    if (a.codes_q) {
      if (kw == 1) return launch_f32_one<D, MODE, 1, false, true>(a, st);
      return kw == 2 ? launch_f32_one<D, MODE, 2, false, true>(a, st) : launch_f32_one<D, MODE, 4, false, true>(a, st);
    }
  if constexpr (MODE == kModeExact)
    if (f32_exact_eight(a)) return launch_f32_one<D, MODE, 8>(a, st);
  if (kw == 1) return launch_f32_one<D, MODE, 1>(a, st);
  return kw == 2 ? launch_f32_one<D, MODE, 2>(a, st) : launch_f32_one<D, MODE, 4>(a, st);
}

int launch_attn_f32(const AttnArgs& a, int mode, hipStream_t st) {
  if (a.g.dtype != HA_FP32) return HA_ERR_DTYPE;
  if (a.g.d != 64 && a.g.d != 128) return HA_ERR_SHAPE;
  if (mode == kModeNode) return a.g.d == 128 ? launch_f32_mode<128, kModeNode>(a, st) : launch_f32_mode<64, kModeNode>(a, st);
  if (mode == kModeCap) return a.g.d == 128 ? launch_f32_mode<128, kModeCap>(a, st) : launch_f32_mode<64, kModeCap>(a, st);
  if (mode == kModeValue) return a.g.d == 128 ? launch_f32_mode<128, kModeValue>(a, st) : launch_f32_mode<64, kModeValue>(a, st);
  if (mode == kModeExact) return a.g.d == 128 ? launch_f32_mode<128, kModeExact>(a, st) : launch_f32_mode<64, kModeExact>(a, st);
  return HA_ERR_SHAPE;
}

}  // namespace ha
