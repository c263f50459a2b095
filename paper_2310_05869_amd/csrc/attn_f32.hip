// fp32 attention: the arithmetic path for HA_FP32 tensors, with the same node / cap / exact modes and the same outputs as the
// bf16 kernel (attn_mfma.hip).  Its products run on the bf16 matrix cores, every operand split in three (split_f32.h).
//
// What bounds it: in large launches the matrix pipe at the clock that the chip's power leaves it (32 heads, n = 8192, d = 64: 178 TFLOP/s, 1070
// of bf16 products), in small ones the vector work of the splits and the chain of one wave's tiles (4 heads, n = 4096 in causal blocks of
// 1024, 512 workgroups: matrix pipe 21 %, vector issue 59 % of the cycles).
//
// A wave owns 32 query rows and computes S^T = K Q^T, so that a lane holds 16 keys of
// ONE query (as in the bf16 kernel) and accumulator registers, exponentiated and split, are
// directly the B operand of O^T += V^T P^T: the eight of a step hold the lane's keys
// 8 g + 4 h + z, g = 0, 1, in the order that V's operand has them too.
//
// A workgroup has KW ways, every way taking each KW-th key tile, and their results are merged through LDS; the other waves of a way hold
// further queries and share its tiles.  KW = 1 or 2 (KW = 2 at d = 64): a tile of K and V is split once, by all threads of its way, into LDS (a
// wave's splits are otherwise a third to a half of its vector work), and read from there, V through the transposing read.  KW = 4 or 8:
// small problems, one group of 32 queries per workgroup (the one-head n = 1024 call has 32 groups of queries for 1024 SIMDs), where no
// two waves share a tile: K and V come straight from the caches in operand layout and are split in registers, no barrier
// in the loop, and the queries lie split in LDS.
//
// Measured (MI355X, us; fp32 matrix instructions, K and V always from the caches -> this form): exact attention, 32 heads, n = 8192:
// d = 64 4220 -> 3090; 16 heads, d = 128 4210 -> 3490; causal, 16 heads, n = 1024 d = 64 30.7 -> 23.8, d = 128 54.1 -> 41.7; 8 heads, n = 4096
// 166 -> 135, 349 -> 251; one head, n = 1024 23.7 -> 17.8, 43.2 -> 30.5; whole calls: one head, n = 1024, d = 64, b = m = 64 17.5 -> 16.6, 8 heads, n = 4096,
// b = m = 256 67.6 -> 55.8, d = 128 115 -> 94; 16 causal heads, n = 4096 in blocks of 1024, b = m = 128 192 -> 149, 352 -> 294.
// Tried: the next step's split in slices between the products, by the compiler's issue-order hints (+-1 %: the other waves fill the gaps);
// KW = 2 at d = 128 (one wave per SIMD: 16 heads, n = 2048, causal 138 -> 187).
#include <type_traits>

#include "attn_common.h"
#include "node_sort.h"
#include "split_f32.h"

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

// What the loop keeps in front of the tiles: the key list, and behind it the rows drawn by value norm with their weights and the waves'
// masked sums.
__host__ __device__ inline size_t f32_list_bytes(int b, int m, int mode) {
  if (mode == kModeExact) return 0;
  const size_t list = (size_t)(((b + m + 63) & ~63) + 64) * 4 + 64;
  const size_t cap = mode == kModeCap || mode == kModeValue ? 4 * 32 * 2 * 4 : 0;
  const size_t drawn = mode == kModeValue ? 2 * (size_t)((m + 63) & ~63) * 4 : 0;
  return (list + drawn + cap + 15) & ~(size_t)15;
}

// K and V tiles of every way, or, where the waves of a workgroup share one group of queries, its rows
template <int D, int KW>
__host__ __device__ constexpr size_t f32_tile_bytes() {
  return (size_t)SplitTile<D>::BYTES * (KW < 4 ? 2 * KW : 1);
}

template <int D, int KW>
__host__ __device__ inline size_t f32_finite_at(int b, int m, int mode) {
  constexpr int NW = f32_waves(KW);
  const size_t loop = f32_list_bytes(b, m, mode) + f32_tile_bytes<D, KW>();
  // staged rows: two more values each in cap mode
  const size_t rows = (size_t)F32Lds<D, NW>::BYTES + (mode == kModeCap || mode == kModeValue ? NW * 32 * 2 * 4 : 0);
  return loop > rows ? loop : rows;
}

template <int D, int KW>
__host__ __device__ inline size_t f32_lds_bytes(int b, int m, int mode) {
  return f32_finite_at<D, KW>(b, m, mode) + SplitFinite<f32_waves(KW)>::BYTES;
}

// SORT: the sort's tables lie behind the list, where the tiles come later, the tile's query rows behind all else
__host__ __device__ inline size_t f32_sort_end(const Geometry& g) {
  return f32_list_bytes(g.b, g.m, kModeNode) + ((node_sort_lds_bytes<4>(g) + 15) & ~(size_t)15);
}
template <int D, int KW>
__host__ __device__ inline size_t f32_qrows_at(const Geometry& g) {
  const size_t sort = f32_sort_end(g), rest = f32_lds_bytes<D, KW>(g.b, g.m, kModeNode);
  return sort > rest ? sort : rest;
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
__global__ __launch_bounds__(64 * f32_waves(KW), D == 128 && KW < 4 ? 1 : D == 64 && KW == 4 ? 3 : 2) void attn_f32_kernel(AttnArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int NW = f32_waves(KW), kFNT = 64 * NW;
  constexpr int RG = NW / KW;  // waves that share the tiles of a way
  constexpr bool kShared = RG > 1;
  constexpr int kQT = 32 * RG;
  using T = SplitTile<D>;
  constexpr bool kValue = MODE == kModeValue, kCap = MODE == kModeCap || kValue, kNode = MODE == kModeNode || kCap;
  constexpr int KJ = D / 8;    // 16-byte pieces of a row per lane
  constexpr int KS = D / 16;   // steps of a score's product
  constexpr int DT = D / 32;
  constexpr int DTA = DT < 2 ? DT : 2;  // V columns are fetched 64 at a time
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // a scalar: so are the key loop and the descriptors
  const int lq = lane & 31, h = lane >> 5;
  const int grp = wave % RG, kw = wave / RG;

  int32_t* scratch = reinterpret_cast<int32_t*>(smem);
  int32_t* list = scratch + 16;

  const int bid = a.wg_first + (kNode ? logical_block(blockIdx.x, gridDim.x) : (int)blockIdx.x);
  TileWork w;
  int nb, nkeys;
  int32_t* qrows = reinterpret_cast<int32_t*>(smem + (SORT ? f32_qrows_at<D, KW>(a.g) : 0));
  unsigned char* tiles_at = smem + f32_list_bytes(a.g.b, a.g.m, MODE);
  if constexpr (SORT) {
    w = decode_node_tile<kQT>(a, bid);
    const int l0 = first_node_sample(a, w);
    unsigned char* sort_lds = smem + f32_list_bytes(a.g.b, a.g.m, MODE);
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
  int wg_tiles = ntiles;  // of the workgroup
  if (MODE == kModeExact && a.exact_causal) ntiles = min(ntiles, (w.q0 - w.k0) / kFKT + grp + 1);
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
    wg_tiles = ntiles;
    __syncthreads();
  }
  const float nat_bias = (kNode && a.g.m > 0) ? logf((float)w.nr.s / (float)a.g.m) : 0.f;

  const float* Qh = reinterpret_cast<const float*>(a.Q) + (int64_t)w.bh * a.q_bh_stride;
  const float* Kh = reinterpret_cast<const float*>(a.K) + (int64_t)w.bh * a.k_bh_stride;
  const float* Vh = reinterpret_cast<const float*>(a.V) + (int64_t)w.bh * a.k_bh_stride;
  const int r_in_tile = grp * 32 + lq;
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
  // Columns 16 s + 8 h ... + 7 are the lane's eight of step s, of Q and of K.  Where a workgroup's waves share the queries, these lie
  // split in LDS.
  Split8 q[kShared ? KS : 1];
  if constexpr (kShared) {
    f32x4 qf[KJ];
#pragma unroll
    for (int j = 0; j < KJ; ++j) qf[j] = *reinterpret_cast<const f32x4*>(Qh + (int64_t)qrow * D + 16 * (j / 2) + 8 * h + 4 * (j % 2));
#pragma unroll
    for (int s = 0; s < KS; ++s) q[s] = split8_raw([&](int e) { return qf[2 * s + e / 4][e % 4]; });
  } else {
    for (int i = tid; i < 32 * T::PPR; i += kFNT) {
      const int r = i / T::PPR, piece = i % T::PPR, ru = r < w.rows_valid ? r : 0;
      const int row = SORT ? qrows[ru] : kNode && a.perm_q ? a.perm_q[w.seg_off + w.p0 + ru] : kNode ? w.nr.q_start + w.p0 + ru : w.q0 + ru;
      const f32x4* at = reinterpret_cast<const f32x4*>(Qh + (int64_t)row * D + piece * 8);
      T::store(tiles_at, r, piece, at[0], at[1]);
    }
  }

  // rows past the end of the keys read as zeros (such keys are masked by position)
  const uint32_t bytes = (uint32_t)(kNode ? a.g.n : w.k1) * (uint32_t)(D * 4);
  const __amdgpu_buffer_rsrc_t krsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Kh, 0, (int)bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t vrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Vh, 0, (int)bytes, 0x00020000);
  f32x4 kf[kShared ? 1 : KJ];
  auto load_k = [&](int kt, int j0 = 0, int j1 = D / 8) {
    if constexpr (kShared) return;
    const int row = kNode ? list[kt * kFKT + lq] : w.k0 + kt * kFKT + lq;
    if constexpr (FAR) {  // (every row of the list exists)
#pragma unroll
      for (int j = j0; j < j1; ++j) kf[kShared ? 0 : j] = *reinterpret_cast<const f32x4*>(Kh + (int64_t)row * D + 16 * (j / 2) + 8 * h + 4 * (j % 2));
      return;
    }
    const int off = row * (D * 4) + 32 * h;
#pragma unroll
    for (int j = j0; j < j1; ++j)
      kf[kShared ? 0 : j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(krsrc, off + 16 * (j % 2), 64 * (j / 2), 0));
  };
  // V rows of the tile, columns 32 dt + lq for dt in [dt0, dt0 + DTA): element i of a lane is key
  // 8 (i / 4) + 4 h + i % 4, the key of accumulator register i
  auto load_v = [&](int kt, int dt0, float (&v)[kShared ? 1 : 16][DTA]) {
    if constexpr (kShared) return;
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
          v[kShared ? 0 : 4 * g + z][dt] = FAR ? Vh[(int64_t)rows[z] * D + 32 * (dt0 + dt) + lq]
                                 : __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(vrsrc, rows[z] * (D * 4) + 4 * lq,
                                                                                       128 * (dt0 + dt), 0));
    }
  };

  // Shared tiles: a thread fetches pieces of eight floats, splits them and puts them into its way's tiles.
  constexpr int NP = kShared ? kFKT * T::PPR / (64 * RG) : 1;  // pieces per thread and tensor
  const int wtid = tid % (64 * RG);
  unsigned char* ktile = tiles_at + (kShared ? kw * 2 * T::BYTES : 0);
  unsigned char* vtile = ktile + T::BYTES;
  f32x4 ks[NP][2], vs[NP][2];
  auto fetch = [&](int kt) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int r = (wtid + i * 64 * RG) / T::PPR, piece = (wtid + i * 64 * RG) % T::PPR;
      const int off = (kNode ? list[kt * kFKT + r] : w.k0 + kt * kFKT + r) * (D * 4) + piece * 32;
      ks[i][0] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(krsrc, off, 0, 0));
      ks[i][1] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(krsrc, off + 16, 0, 0));
      if (kValue && kt < vt0) continue;
      vs[i][0] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(vrsrc, off, 0, 0));
      vs[i][1] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(vrsrc, off + 16, 0, 0));
    }
  };
  auto store = [&](int kt) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int r = (wtid + i * 64 * RG) / T::PPR, piece = (wtid + i * 64 * RG) % T::PPR;
      T::store(ktile, r, piece, ks[i][0], ks[i][1]);
      if (kValue && kt < vt0) continue;
      T::store(vtile, r, piece, vs[i][0], vs[i][1]);
    }
  };
  const int row_at = T::row_at(lane), col_at = T::col_at(lane);

  f32x16 o[DT];
  float m_run, l_run;

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
  float log_masked, log_capw;  // log of the row's masked sum, of (s / m) C_i
  float d_ref;
  constexpr float kFarCap = 40.f;  // a term that underflows against m_run is then e^-47 of the cap or less
  auto sum_ref = [&](float m) { return kCap && !kValue && m > log_capw + kFarCap ? log_capw : m; };
  auto finite_ref = [](float m) { return m == -INFINITY ? 0.f : m; };
  const float floor_term = kCap && a.kappa > 0.f ? a.log_tau[(int64_t)w.bh * a.g.total_nodes + w.nr.heap] - logf(a.kappa) : -INFINITY;
  bool sampled, drawn;
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
    for (int k = 0; k < KW; ++k) top = fmaxf(top, ex[((k * RG + grp) * 32 + lq) * 2]);
#pragma unroll
    for (int k = 0; k < KW; ++k) {
      const float* e = ex + ((k * RG + grp) * 32 + lq) * 2;
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
  // BOUND: split_tile_products'; tiles are then not fetched ahead, so that this form needs no more registers.
  auto run = [&](auto bound) {
    constexpr bool BOUND = decltype(bound)::value;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[dt][i] = 0.f;
    m_run = log_masked = d_ref = -INFINITY;
    l_run = 0.f;
    log_capw = INFINITY;
    sampled = drawn = false;
    if constexpr (kShared) {
      if (!BOUND && kw < wg_tiles) fetch(kw);
    } else if (!BOUND && kw < ntiles) {
      load_k(kw);
    }
    // (shared tiles: the same trips for all ways, the barriers are the workgroup's)
    const int kt_end = kShared ? (wg_tiles + KW - 1) / KW * KW : ntiles;
    for (int kt = kw; kt < kt_end; kt += KW) {
      if constexpr (kShared) {
        if (kt >= KW) __syncthreads();  // the tiles before are read no more
        if (BOUND && kt < wg_tiles) fetch(kt);
        if (kt < wg_tiles) store(kt);
        __syncthreads();
        if (!BOUND && kt + KW < wg_tiles) fetch(kt + KW);
        if (kt >= ntiles) continue;
      } else if (BOUND) {
        load_k(kt);
      }
      float va[kShared ? 1 : 16][DTA];
      if constexpr (!kShared && DT == 2 && !kValue) load_v(kt, 0, va);
      f32x16 c, small;
#pragma unroll
      for (int i = 0; i < 16; ++i) c[i] = small[i] = 0.f;
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        if constexpr (kShared) {
          split_product(T::row_frag(ktile, row_at, s), q[s], c, small);
        } else {
          if constexpr (DT > 2 && !kValue) {
            if (s == KS / 2) {  // d = 128: V takes the registers of the K pieces already multiplied
              __builtin_amdgcn_sched_barrier(0);
              load_v(kt, 0, va);
            }
          }
          split_product(split8_raw([&](int e) { return kf[2 * s + e / 4][e % 4]; }), T::row_frag(tiles_at, row_at, s), c, small);
        }
      }
      split_sum<BOUND || kCap>(c, small);

      const int base = kt * kFKT;
      constexpr float kUnit = kCap ? 1.f : kSplitScore;  // of c: biases are divided by it, what is read of c multiplied
      if constexpr (kCap) {
#pragma unroll
        for (int i = 0; i < 16; ++i) c[i] *= kSplitScore;
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
                         !(MODE == kModeExact && a.exact_causal && w.k0 + base + kFKT - 1 > w.q0 + grp * 32);
      if (!plain) {
        int lim = nkeys;
        if (MODE == kModeExact && a.exact_causal) lim = min(lim, q_global - w.k0 + 1);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int pos = base + 8 * (i / 4) + 4 * h + (i % 4);
          const float s = c[i] + (pos >= nb ? nat_bias * (1.f / kUnit) : 0.f);
          c[i] = pos >= lim ? -INFINITY : s;
        }
      }
      float mx = c[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) mx = fmaxf(mx, c[i]);
      mx = fmaxf(mx, __shfl_xor(mx, 32)) * kUnit;
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
      float ls[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        c[i] = exp_split(__builtin_fmaf(c[i], kUnit, -m_use));
        ls[i % 4] += kCap ? fminf(c[i], capw) : c[i];
      }
      if (!kValue || kt < vt0) l_run += (ls[0] + ls[1]) + (ls[2] + ls[3]);
      if constexpr (DT == 2) {
        if (!BOUND && kt + KW < ntiles) load_k(kt + KW);
      }
      float vb[kShared ? 1 : 16][DTA];
      Split8 p[2];  // the weights: elements 8 s ... 8 s + 7 are the lane's keys of step s
#pragma unroll
      for (int s = 0; s < 2; ++s) p[s] = split8([&](int e) { return c[8 * s + e]; });
      auto add_pv = [&](const float (&v)[kShared ? 1 : 16][DTA], int dt0) {
        if constexpr (!kShared)
          split_tile_products<DTA, kSumEach, BOUND>([&](int dt, int s) { return split8_raw([&](int e) { return v[8 * s + e][dt]; }); }, p, o + dt0);
      };
      if constexpr (kShared) {
        if (!kValue || kt >= vt0) split_tile_products<DT, kSumTile, BOUND>([&](int dt, int s) { return T::col_frag(vtile, col_at, s, dt); }, p, o);
        continue;
      }
      if constexpr (kValue) {  // V behind the sums, 64 columns at a time (fetched amid the products, under a branch: 168 spills at d = 128)
        if (DT > 2 && !BOUND && kt + KW < ntiles) load_k(kt + KW);
        if (kt < vt0) continue;
#pragma unroll
        for (int dt0 = 0; dt0 < DT; dt0 += 2) {
          load_v(kt, dt0, va);
          add_pv(va, dt0);
          __builtin_amdgcn_sched_barrier(0);
        }
        continue;
      }
      if constexpr (DT > 2) load_v(kt, 2, vb);
      add_pv(va, 0);
      if constexpr (DT > 2) {
        __builtin_amdgcn_sched_barrier(0);  // the next K rows take the registers of the first half of V
        if (!BOUND && kt + KW < ntiles) load_k(kt + KW, 0, KJ / 2);
        add_pv(vb, 2);
        if (!BOUND && kt + KW < ntiles) load_k(kt + KW, KJ / 2);
      }
    }
    if constexpr (kCap) {
      if (!sampled) to_samples();
    }
    split_settle();
  };
  if constexpr (!kShared) __syncthreads();  // the queries stand
  run(std::false_type{});
  if constexpr (kShared || kCap) {
    const SplitFinite<NW> finite{reinterpret_cast<int32_t*>(smem + f32_finite_at<D, KW>(a.g.b, a.g.m, MODE))};
    finite.post(wave, split_finite(o));
    __syncthreads();  // the key list is read no more
    if (__builtin_expect(!finite.all(), 0)) {
      run(std::true_type{});
      __syncthreads();
    }
  } else {
    if (__builtin_expect(!__all(split_finite(o)), 0)) run(std::true_type{});
    __syncthreads();  // the key list is read no more
  }

  // ---- results: every wave's rows through LDS, where the KW parts of a row are merged and rows
  // leave as whole 16-byte pieces of consecutive lanes ----
  constexpr int RS = F32Lds<D>::ROW;
  float* orow = reinterpret_cast<float*>(smem);   // [waves][32][RS]
  float* ml = orow + NW * 32 * RS;                // [waves][32][ML]: reference, row sum; cap mode: of the samples, its reference, log of the masked sum
  constexpr int ML = kCap ? 4 : 2;
  const float l_tot = l_run + __shfl_xor(l_run, 32);
  if (kCap && !drawn) d_ref = sum_ref(m_run);
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<f32x4*>(orow + (wave * 32 + lq) * RS + 32 * dt + 8 * g + 4 * h) =
          (f32x4){o[dt][4 * g], o[dt][4 * g + 1], o[dt][4 * g + 2], o[dt][4 * g + 3]} * (1.f / kSplitRaw);
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
    float mx = -INFINITY, dmx = -INFINITY;
#pragma unroll
    for (int k = 0; k < KW; ++k) {
      mx = fmaxf(mx, ml[(k * kQT + r) * ML]);
      if (kCap) dmx = fmaxf(dmx, ml[(k * kQT + r) * ML + 2]);
    }
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float l = 0.f;
#pragma unroll
    for (int k = 0; k < KW; ++k) {
      const int at = k * kQT + r;
      const float wk = KW == 1 ? 1.f : (mx == -INFINITY ? 0.f : expf(ml[at * ML] - mx));
      l += (kCap && KW > 1 ? expf(ml[at * ML + 2] - finite_ref(dmx)) : wk) * ml[at * ML + 1];
      acc += wk * *reinterpret_cast<const f32x4*>(orow + at * RS + col);
    }
    const bool empty = !(l > 0.f);
    float lse = empty ? -INFINITY : add_log(kCap ? dmx : mx, l);
    float ref = lse;  // of a partial row
    if constexpr (kCap) {  // d~_i = masked + max(d_i, tau / kappa)
      lse = logaddexpf(ml[r * ML + 3], fmaxf(lse, floor_term));
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
  constexpr int kQT = 32 * (f32_waves(KW) / KW), NT = 64 * f32_waves(KW);
  AttnArgs a = args;
  if (MODE != kModeExact) set_node_divs<kQT>(a);
  else set_exact_divs<kQT>(a);
  a.exact_lpt = KW == 8;
  const int64_t grid = MODE != kModeExact ? node_grid<kQT>(a.g) : exact_grid<kQT>(a);
  if (grid <= 0) return HA_OK;
  if (grid > kMaxGrid) return HA_ERR_SHAPE;
  const size_t lds = SORT ? f32_qrows_at<D, KW>(a.g) + kQT * 4 : f32_lds_bytes<D, KW>(a.g.b, a.g.m, MODE);
  static std::atomic<uint64_t> lds_set{0};  // per instantiation: devices on which the LDS limit is raised
  if (allow_full_lds(reinterpret_cast<const void*>(&attn_f32_kernel<D, MODE, KW, FAR, SORT>), lds_set) != HA_OK) return HA_ERR_LAUNCH;
  for (int64_t first = 0; first < grid; first += kMaxLaunch) {
    a.wg_first = (int32_t)first;
    const int64_t count = grid - first < kMaxLaunch ? grid - first : kMaxLaunch;
    hipLaunchKernelGGL((attn_f32_kernel<D, MODE, KW, FAR, SORT>), dim3((unsigned)count), dim3(NT), lds, st, a);
    const int rc = check_launch();
    if (rc != HA_OK) return rc;
  }
  return HA_OK;
}

// Ways of a workgroup of four waves: one where there are workgroups of 128 rows enough for it, four (of 32 rows) where there are not, two in
// between at d = 64 (at d = 128 its two tiles and registers leave one wave per SIMD); but not so few that a workgroup's 128 / KW rows
// outgrow the run of rows it is cut from (a block of b sorted positions, an exact diagonal block) by more than a third: idle rows
// cost matrix time like real ones, while the merge of KW results costs a few LDS reads per row.  Causal tiles differ in length, so workgroups of
// 128 rows pay only where a CU gets several; at d = 128 a CU holds one of them, and a last round that is not nearly full loses what they gain.
// One way / two / four (MI355X, us; workgroups of 128 rows in brackets):
//   d = 64, causal: 32 heads, n = 1024 (256) 66.4 / 44.5 / 41.5, 64 (512) 74.7 / 72.6 / 75.1, 128 (1024) 120 / 139 / 154; 16 heads, n = 4096 (512) 270 / 241 /
//     254; unmasked: 32 heads, n = 1024 (256) 72 / 65 / 69; 16 heads, n = 4000 (500) 415 / 442 / 467; nodes: b = m = 256, 8 heads, n = 4096 (256) 54.6 / 53.1 /
//     56.7, 16 (512) 83.5 / 95.6 / 99.4; b = m = 128, 12 heads, n = 4096 (384) 53.0 / 56.8 / 57.9; b = m = 64, 16 heads, n = 4096 61.4 / 54.7 / 58.1
//   d = 128 (one / four): causal, 64 heads, n = 1024 (512) 158 / 146, 128 (1024) 278 / 296; unmasked, 32 heads (256) 119 / 130; nodes: b = m = 256, 8
//     heads, n = 4096 (256) 91.1 / 98.9; b = m = 128, 12 heads, n = 4096 (384) 109.6 / 98.4, 32 heads, n = 2048 (512) 118.9 / 124.6, 44 (704) 167.5 / 162.0,
//     52 (832) 210 / 185; 24 heads, n = 2000, b = 100 (480) 94.5 / 109.0
static bool f32_fits(int run, int rows) { return 3 * (int64_t)((run + rows - 1) / rows * rows) <= 4 * (int64_t)run; }
static int f32_ways(int d, int run, int64_t grid128, bool causal) {
  const int64_t rounds = (grid128 + 255) / 256;
  const bool full = d == 64 || 100 * grid128 >= 92 * 256 * rounds;  // (d = 128: one workgroup of 128 rows to a CU)
  if (f32_fits(run, 128) && full && grid128 >= (causal ? 1024 : d == 64 ? 384 : 236)) return 1;
  return d == 64 && f32_fits(run, 64) && grid128 >= (causal ? 512 : 256) ? 2 : 4;
}

int attn_f32_node_ways(const Geometry& g) { return f32_ways(g.d, g.b, node_grid<128>(g), false); }

// Workgroups of a node launch that a CU holds by their registers
static constexpr int f32_places(int d, int kw) { return d == 64 ? (kw == 4 ? 3 : 2) : kw == 4 ? 2 : 1; }

// Whether the sort's tables in the LDS cost a CU one of the workgroups that the launch needs it to hold
template <int D, int KW>
static bool f32_tables_cost(const Geometry& g, int64_t wgs) {
  const int64_t sorting = lds_workgroups(f32_qrows_at<D, KW>(g) + 128 / KW * 4, f32_places(D, KW));
  return wgs > 256 * sorting && sorting < lds_workgroups(f32_lds_bytes<D, KW>(g.b, g.m, kModeNode), f32_places(D, KW));
}

// Whether a node launch sorts by itself (attn_mfma_sorts, for the kernel without it): up to 1024 workgroups of the form that is launched
// (attn_f32_node_ways), each of which counts its whole node, and up to 2^22 rows counted.  Sorting launch -> in the attention (MI355X, us; workgroups):
//   d = 64, four ways: b = m = 64: one head, n = 1024 (32) 20.9 -> 17.7; b = m = 256, 6 heads, n = 4096 (768) 48.3 -> 45.0, 3 heads, n = 8192 (768) 48.7 ->
//     51.6; n = 4096, b = 32: 8 heads (1024) 36.1 -> 35.5, 12 (1536) 46.8 -> 46.9, 16 (2048) 54.6 -> 56.7
//   two: b = m = 64: 16 heads, n = 2048 (512) 35.4 -> 31.2, n = 4096: 9 (576) 46.6 -> 45.3, 16 (1024) 56.7 -> 55.1, 17 (1088) 64.9 -> 67.1, 20 (1280) 67.4 ->
//     68.9; n = 8192: 4 (512) 36.7 -> 33.4, 6 (768) 49.5 -> 49.6; n = 6144: 7 (672) 47.8 -> 48.1, 12 (1152) 65.7 -> 69.6
//   one: b = m = 128: 32 heads, n = 2048 (512) 62.6 -> 58.0, 64 (1024) 106.1 -> 103.6, 48, n = 4096 (1536) 145.3 -> 145.5; b = m = 256, 6 heads, n = 8192
//     (384) 80.6 -> 76.8; n = 2000, b = 100, 64 heads (1280) 101.3 -> 101.5, 90 (1800) 138.9 -> 140.7
//   d = 128, four: b = m = 64: one head, n = 1024 (32) 24.6 -> 20.9; 16 heads, n = 2048 (1024) 58.6 -> 56.4, 18 (1152) 68.4 -> 68.2, 24 (1536) 79.4 -> 79.6, 32
//     (2048) 100.0 -> 102.2; b = m = 128: 24 (1536) 96.9 -> 96.7, 36 (2304) 135.3 -> 138.7, 44 (2816) 160.7 -> 164.5, 52 (3328) 185.2 -> 192.4; b = m = 256,
//     6 heads, n = 4096 (768) 82.7 -> 80.0, 10 (1280) 119.9 -> 119.8, 20 (2560) 216.0 -> 219.8; b = m = 64, n = 8192: 2 (512) 39.1 -> 35.0, 3 (768)
//     51.0 -> 50.9, 6 (1536) 81.1 -> 83.4
//   one: b = m = 128: 16 heads, n = 2048 (256) 70.2 -> 63.5, 64 (1024) 229.8 -> 223.1, n = 8192: 4 (256) 71.1 -> 65.2, 8 (512) 127.1 -> 122.6
// Not where the tables cost a CU one of its workgroups and the call needs it: b = 128, m = 2000, r = 8, n = 8192: d = 64, 2 heads (four ways, 512) 96.8 ->
// 113.1, 8 (one, 512) 256.8 -> 320.3; d = 128, 2 heads (four, 512) 158.6 -> 182.6, but 8 (one, 512, of which a CU holds one in any case) 546.5 -> 542.3.
bool attn_f32_sorts(const Geometry& g) {
  const int rows = node_sort_rows(g), kw = attn_f32_node_ways(g);
  const int64_t wgs = kw == 1 ? node_grid<128>(g) : kw == 2 ? node_grid<64>(g) : node_grid<32>(g);
  if (rows > kNodeSortMax || wgs > 1024 || wgs * rows > 4 << 20) return false;
  if (g.d == 128) return !(kw == 1 ? f32_tables_cost<128, 1>(g, wgs) : f32_tables_cost<128, 4>(g, wgs));
  return !(kw == 1 ? f32_tables_cost<64, 1>(g, wgs) : kw == 2 ? f32_tables_cost<64, 2>(g, wgs) : f32_tables_cost<64, 4>(g, wgs));
}

// Exact launches of few workgroups and long rows are bound by the longest chain of key tiles: eight waves then share 32 queries,
// two per SIMD where four left one, a workgroup that fills a CU (causal: up to one and a half or two rounds of those, heaviest first).
// Four waves -> eight (MI355X, us; groups of 32 rows in brackets): d = 64: causal, 16 heads, n = 512 (256) 13.5 -> 12.6; n = 1024: one head (32)
// 19.8 -> 17.7, 8 heads (256) 22.0 -> 19.5, 16 (512) 24.5 -> 26.1; n = 2048: 4 heads (256) 37.9 -> 32.3, 8 (512) 42.0 -> 41.3; 3 heads, n = 4000 (375)
// 71.2 -> 61.5; unmasked: 8 heads, n = 1024 (256) 23.0 -> 21.7, 4 heads, n = 2048 (256) 40.0 -> 38.5, 4 heads, n = 4000 (500) 127.4 -> 131.5.  d = 128:
// causal, 16 heads, n = 512 (256) 23.7 -> 21.7; 8 heads, n = 1024 (256) 38.4 -> 34.8, 16 (512) 43.8 -> 45.4; 8 heads, n = 2048 (512) 78.4 -> 76.8; 3 heads,
// n = 4000 (375) 135 -> 113; unmasked, 8 heads, n = 1024 (256) 40.5 -> 39.8, 4 heads, n = 4000 (500) 235.9 -> 242.5.
bool f32_exact_eight(const AttnArgs& a) {
  const int rows = a.exact_block < a.exact_rows_q ? a.exact_block : a.exact_rows_q;
  return rows >= 512 && exact_grid<32>(a) <= (!a.exact_causal ? 256 : rows < 2048 ? 384 : 512);
}

template <int D, int MODE>
static int launch_f32_mode(const AttnArgs& a, hipStream_t st) {
  if constexpr (MODE == kModeNode)  // stage calls alone: the whole-call entry points take up to 2^22 rows per head
    if ((int64_t)a.g.n * (D * 4) > 0x7fffffff + 1ll) return launch_f32_one<D, MODE, 4, true>(a, st);
  if constexpr (MODE == kModeExact)
    if (f32_exact_eight(a)) return launch_f32_one<D, MODE, 8>(a, st);
  const int run = a.exact_block < a.exact_rows_q ? a.exact_block : a.exact_rows_q;
  const int kw = MODE != kModeExact ? attn_f32_node_ways(a.g) : f32_ways(D, run, exact_grid<128>(a), a.exact_causal);
  if constexpr (MODE == kModeNode)
    if (a.codes_q) {
      if (kw == 1) return launch_f32_one<D, MODE, 1, false, true>(a, st);
      if constexpr (D == 64)
        if (kw == 2) return launch_f32_one<D, MODE, 2, false, true>(a, st);
      return launch_f32_one<D, MODE, 4, false, true>(a, st);
    }
  if (kw == 1) return launch_f32_one<D, MODE, 1>(a, st);
  if constexpr (D == 64)
    if (kw == 2) return launch_f32_one<D, MODE, 2>(a, st);
  return launch_f32_one<D, MODE, 4>(a, st);
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
