// bf16 MFMA attention kernel for gfx950: one online-softmax pass of a tile of
// 128 queries over a list of keys.
//
//   node mode   the b x b diagonal block of the sorted attention matrix
//               (Algorithm 1's mask M^H; Section 4, Implementation Detail) and
//               the kept sampled columns of Algorithm 2 in ONE pass with a
//               shared normaliser; rows of Q, K, V are fetched through the
//               sort permutations (the "permute" is fused into the loads) and
//               the result is written back through P_Q (the inverse permute is
//               fused into the store).
//   exact mode  plain tiled softmax attention over contiguous keys with an
//               optional causal mask (Section 1.1 / 3.1): the exact baseline
//               and the n_min base case of Algorithm 4, whose epilogue also
//               folds in the per-level partial results of the recursion
//               (row sum = D_21 + D_C22 at every split).
//
// Tiling (wave64, v_mfma_f32_32x32x16_bf16):
//   * 4 waves per workgroup, 32 queries per wave, 64 keys per step.
//   * S^T = K Q^T is computed, not S: keys run along the MFMA's M dimension and
//     queries along N, so in the accumulator a lane holds 16 keys of ONE query.
//     Row max and row sum are then in-lane reductions plus a single exchange
//     with lane^32, and the accumulator registers, converted to bf16, are
//     already the B operand of O^T += V^T P^T (no LDS round trip for P).
//   * Q stays in registers for the whole pass; K (row-major, padded rows) and
//     V^T (d-major, padded rows, keys stored in the order the P registers have
//     them) are staged in LDS, double buffered; the next tile's global loads
//     are issued before the current tile's MFMAs.
//   * softmax runs in the exp2 domain in fp32; P is rounded to bf16 only as the
//     MFMA operand, the row sum uses the unrounded fp32 values.
#include <type_traits>

#include "attn_common.h"
#include "node_sort.h"

namespace ha {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kKT = 64;       // keys per step

template <int D>
struct Lds {
  static constexpr int KSTR = (D + 8) * 2;        // bytes per K row (+16: conflict-free 16-byte row reads)
  static constexpr int VSTR = (D + 32) * 2;       // bytes per V row (+64: conflict-free transposing reads)
  static constexpr int K_BYTES = kKT * KSTR;
  static constexpr int V_BYTES = kKT * VSTR;
  static constexpr int BUF = K_BYTES + V_BYTES;
};

// Epilogue staging per wave: 32 fp32 rows (padded), 32 x kMaxFold merge weights, 32 row ids,
// kMaxFold partial-row bases.
constexpr int kMaxFold = 8;
template <int D>
struct EpLds {
  static constexpr int ROW = D * 4 + 16;
  static constexpr int WAVE = 32 * ROW + 32 * kMaxFold * 4 + 32 * 8 + kMaxFold * 8;
};

__host__ __device__ inline int list_capacity(int b, int m) { return ((b + m + 63) & ~63) + 64; }

template <int D>
__host__ __device__ inline size_t mfma_lds_bytes(int b, int m, int mode) {
  size_t s = 2 * (size_t)Lds<D>::BUF + 64;  // + wave counters
  if (mode != kModeExact) s += (size_t)list_capacity(b, m) * 4;
  return s;
}

// SORT: the sort's tables lie where the tiles will, and push the list back where they are larger; the tile's query rows
// lie behind the list
template <int D, int NW>
__host__ __device__ inline size_t sort_pushes_list(const Geometry& g) {
  const size_t sort = (node_sort_lds_bytes<NW>(g) + 15) & ~(size_t)15;
  return sort > 2 * (size_t)Lds<D>::BUF ? sort - 2 * (size_t)Lds<D>::BUF : 0;
}

__device__ inline float max3f(float a, float b, float c) { return __builtin_fmaxf(__builtin_fmaxf(a, b), c); }

template <int D, int NT>
struct TileRegs {
  static constexpr int CPR = D / 8;              // 16-byte chunks per K row
  static constexpr int NKC = kKT * CPR / NT;     // K (and V) chunks per thread
};

// NW waves per workgroup (32 queries each); two waves per SIMD at d = 128, three (four-wave workgroups) at d = 64.
// STAMPS: the measuring instantiation, which also records counter readings at its phase
// boundaries (a.stamps); the product launches use STAMPS = false and carry none of it.
// NG = 2 (exact mode): two groups of NW waves take the key tiles in turn, each with tile buffers of its own, and their
// results are merged through LDS.
// SORT (node mode): the workgroup finds its rows from the node's bucket codes (node_sort.h).
template <int D, int MODE, int NW, bool STAMPS = false, int NG = 1, bool SORT = false>
__global__ __launch_bounds__(64 * NW * NG, (D == 64 && NW == 4 && NG == 1) ? 3 : 2) void attn_mfma_kernel(AttnArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr bool kCap = MODE == kModeCap;
  constexpr bool kNode = MODE == kModeNode || kCap;
  constexpr int kQT = 32 * NW;  // queries per workgroup
  constexpr int kNT = 64 * NW;  // threads of a group
  using L = Lds<D>;
  using TR = TileRegs<D, kNT>;
  constexpr int KS = D / 16;  // MFMA k-steps of the score product
  constexpr int DT = D / 32;  // 32-wide d tiles of the output

  const int tid = NG == 1 ? threadIdx.x : threadIdx.x % kNT;
  const int grp = NG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / kNT);
  const int lane = tid & 63, wave = tid >> 6;
  const int lq = lane & 31, h = lane >> 5;

  unsigned char* bufs = smem + grp * 2 * L::BUF;
  int32_t* scratch = reinterpret_cast<int32_t*>(smem + NG * 2 * L::BUF + (SORT ? sort_pushes_list<D, NW>(a.g) : 0));
  int32_t* list = scratch + 16;
  int32_t* qrows = list + (SORT ? list_capacity(a.g.b, a.g.m) : 0);

  long long stamp_c[5] = {0, 0, 0, 0, 0}, stamp_w = 0;
  auto stamp = [&](int i) {
    if constexpr (STAMPS) {
      __builtin_amdgcn_sched_barrier(0);
      stamp_c[i] = (long long)__builtin_readcyclecounter();
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  if constexpr (STAMPS) stamp_w = (long long)wall_clock64();
  stamp(0);

  const int bid = (kCap ? a.wg_first : 0) + (kNode ? logical_block(blockIdx.x, gridDim.x) : (int)blockIdx.x);
  TileWork w;
  if (kNode) w = decode_node_tile<kQT>(a, bid);
  else w = decode_exact_tile<kQT>(a, bid);

  const uint16_t* Qh = reinterpret_cast<const uint16_t*>(a.Q) + (int64_t)w.bh * a.q_bh_stride;
  const uint16_t* Kh = reinterpret_cast<const uint16_t*>(a.K) + (int64_t)w.bh * a.k_bh_stride;
  const uint16_t* Vh = reinterpret_cast<const uint16_t*>(a.V) + (int64_t)w.bh * a.k_bh_stride;

  // ---- this lane's query row: B operand of S^T = K Q^T, kept in registers.
  // Node mode: the key list's first index values and the row's own index (through P_Q) travel
  // in one round trip; the (gathered) row is then in flight while the key list is built.
  KeyListHead klh{0, 0, 0};
  if (kNode && !SORT) klh = key_list_fetch<kNT>(a, w);
  if constexpr (SORT) {
    klh.l0 = first_node_sample(a, w);
    sort_node_tile<NW>(a, w, smem, list, qrows);
  }
  const int r_in_tile = wave * 32 + lq;
  RowDest dest;
  int qrow_load;   // row to load (always a valid row)
  int q_global;    // exact mode: row index within the head, for the causal mask
  if constexpr (SORT) {
    dest = RowDest{};
    dest.valid = r_in_tile < w.rows_valid;
    // A lane past the tile's end repeats a valid row, and counts where its wave decides whether references move.  It is the row that
    // a tile of 128 rows would repeat, so that eight waves give the bits of four (blocks of b = 200, d = 128, 16 heads, n = 3200: the
    // last eight rows of one block in 256 differed by a rounding while it was the tile's first row).
    const int spare = (r_in_tile & ~127) < w.rows_valid ? r_in_tile & ~127 : 0;
    qrow_load = qrows[dest.valid ? r_in_tile : spare];
    dest.row_in_head = qrow_load;
    dest.out_row = (int64_t)w.bh * a.g.n + qrow_load;
    dest.part_row = w.seg_off + (qrow_load - w.nr.q_start);
    q_global = 0;
  } else if (kNode) {
    dest = node_row_dest(a, w, r_in_tile);
    const int p = w.p0 + (dest.valid ? r_in_tile : 0);
    qrow_load = a.perm_q ? a.perm_q[w.seg_off + p] : w.nr.q_start + p;
    q_global = 0;
  } else {
    dest = RowDest{};
    dest.valid = r_in_tile < w.rows_valid;
    q_global = w.q0 + r_in_tile;
    qrow_load = dest.valid ? q_global : w.q0;
    dest.row_in_head = q_global;
    dest.out_row = (int64_t)w.bh * (a.out_bh_stride / D) + q_global;
  }
  bf16x8 qreg[KS];
  {
    const u32x4* qp = reinterpret_cast<const u32x4*>(Qh + (int64_t)qrow_load * D + 8 * h);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qreg[ks] = __builtin_bit_cast(bf16x8, qp[2 * ks]);
  }

  int nb, nkeys;
  if constexpr (SORT) {
    nb = a.g.b;
    nkeys = append_node_samples<NW>(a, w, smem, list, scratch, klh.l0);
  } else if (kNode) {
    nkeys = build_key_list<kNT, kCap>(a, w, list, scratch, &nb, klh);
  } else {
    nkeys = max(0, w.k1 - w.k0);
    nb = 0x7fffffff;
  }
  const int ntiles = (nkeys + NG * kKT - 1) / (NG * kKT);  // of the group; its tile t is tile NG t + grp of the keys
  const float bias2 = (kNode && a.g.m > 0) ? log2f((float)w.nr.s / (float)a.g.m) : 0.f;
  stamp(1);

  // ---- tile movers ----
  // K and V rows are fetched with buffer loads at a 32-bit per-lane byte offset.  Node mode: the key list's rows, all of
  // them rows of the head.  Exact mode: the tile's descriptor starts at the tile's first row and ends with the
  // workgroup's keys, so the lane's offset, the one part of an address that the bounds check covers for certain, is checked
  // against what is left: rows past the keys (the next diagonal block, the next head, the end of the
  // tensor) are not read and count as zeros.  Masking their scores alone would not do: weight 0 times a V that is Inf or
  // NaN is NaN, and with two wave groups a whole tile can lie there.  A descriptor is six scalar instructions per tile: 1 %
  // where one chain of tiles is the launch (7 heads, n = 3328, d = 64: 35.05 -> 35.5 us), nothing where the chip is full.
  auto rows_rsrc = [&](const uint16_t* head, int kt) {
    if (kNode) return __builtin_amdgcn_make_buffer_rsrc((void*)head, 0, (int)((uint32_t)a.g.n * (D * 2)), 0x00020000);
    const int off = (w.k0 + (NG * kt + grp) * kKT) * (D * 2);
    return __builtin_amdgcn_make_buffer_rsrc((void*)(reinterpret_cast<const unsigned char*>(head) + (uint32_t)off), 0,
                                             max(0, w.k1 * (D * 2) - off), 0x00020000);
  };
  u32x4 kreg[TR::NKC], vreg[TR::NKC];
  auto load_rows = [&](int kt, const uint16_t* head, u32x4 (&reg)[TR::NKC]) {
    const __amdgpu_buffer_rsrc_t rsrc = rows_rsrc(head, kt);
#pragma unroll
    for (int i = 0; i < TR::NKC; ++i) {
      const int c = tid + i * kNT;
      const int key = c / TR::CPR, col = c % TR::CPR;
      const int row = kNode ? list[kt * kKT + key] : key;
      reg[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, row * (D * 2) + col * 16, 0, 0);
    }
  };
  auto store_rows = [&](unsigned char* dst, int stride, const u32x4 (&reg)[TR::NKC]) {
#pragma unroll
    for (int i = 0; i < TR::NKC; ++i) {
      const int c = tid + i * kNT;
      const int key = c / TR::CPR, col = c % TR::CPR;
      *reinterpret_cast<u32x4*>(dst + key * stride + col * 16) = reg[i];
    }
  };
  auto kbuf_at = [&](int t) -> unsigned char* { return bufs + (t & 1) * L::BUF; };
  auto vbuf_at = [&](int t) -> unsigned char* { return bufs + (t & 1) * L::BUF + L::K_BYTES; };
  // V^T fragments come from the row-major V tile through the transposing LDS
  // read: the 16 lanes of a group fetch a 4-key x 16-d patch (lane i: key i/4,
  // d 4*(i%4)..+3) and lane n receives the 4 keys of column n.
  const int vtr_off = ((lane & 15) >> 2) * L::VSTR + ((lane & 3) * 4 + ((lane >> 4) & 1) * 16) * 2 + (4 * h) * L::VSTR;

  // ---- state ----
  f32x16 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[dt][i] = 0.f;
  // m_run is a reference for the exponentials, not necessarily the running
  // maximum: it is only moved (and the accumulators rescaled) when a row's tile
  // maximum exceeds it by more than 2^8, so after the first tiles the rescale is
  // skipped.  Log2 domain.
  float m_run = -INFINITY;
  float m_ref = 0.f;  // m_run, 0 where that is -inf
  float l_run = 0.f;  // this lane's share of the row sum
  // Cap mode (Algorithm 2 as printed): once the block's keys are done (tile nb_tiles on) l_run becomes the capped sum of
  // the samples and log_masked keeps the masked row sum, from which the row's cap C_i follows.  Scores of one row can lie hundreds
  // apart, so neither may hang on the output's reference: the masked sum is a logarithm before the first sample's reference
  // is formed, and the samples' sum is taken against sum_ref, the cap where that is far below m_run, since no capped term exceeds it.
  // One more vector instruction per score than the plain node mode (32 heads, n = 32768, d = 128, b = m = 256: 8 % more
  // cycles, vector issue 50 against 44 % of them; 414 to 487 us, by the clock of the run, where a kernel of its own without
  // the software pipeline below took 600).  At d = 64 the 168 registers that three workgroups per CU leave cost it 40 bytes of scratch
  // per lane, at d = 128 the 256 of two 16.  (With the masked and the capped sum on m_run, 20 and none, rows of clustered inputs lost log d~ to
  // underflow; calls of 32 heads, n = 32768 with it -> without, three sessions: d = 128 623 -> 622, 622 -> 623, 627 -> 629 us, d = 64 370 -> 367,
  // 376 -> 376.)
  const int nb_tiles = kCap ? (nb + kKT - 1) / kKT : 0;
  float log_masked = -INFINITY, log2capw = INFINITY;  // log2 of (s / m) C_i
  constexpr float kFarCap = 60.f;  // a term that underflows against m_run is then 2^-66 of the cap or less
  auto sum_ref = [&](float m) { return kCap && m > log2capw + kFarCap ? log2capw : m; };
  auto finite_ref = [](float m) { return m == -INFINITY ? 0.f : m; };
  auto end_masked = [&]() {
    const float mt = l_run + __shfl_xor(l_run, 32);
    log_masked = (mt > 0.f) ? (m_run + log2f(mt)) * kLn2 : -INFINITY;
    l_run = 0.f;
  };
  const float floor_term = kCap && a.kappa > 0.f ? a.log_tau[(int64_t)w.bh * a.g.total_nodes + w.nr.heap] - logf(a.kappa) : -INFINITY;

  // Masks of a score tile (rare tiles only): tail of the key list, causal
  // diagonal, and a tile that straddles the block / sampled boundary.  `bias` is
  // the tile-uniform log2-domain bias (log2(s/m) on sampled tiles).
  auto mask_tile = [&](f32x16 (&c)[2], int t, float& bias) {
    const int key_base = (NG * t + grp) * kKT;
    const bool tail = key_base + kKT > nkeys;
    const bool mixed = (key_base < nb) && (key_base + kKT > nb);  // (cap mode: the block's last, padded tile)
    const bool diag = (MODE == kModeExact) && a.exact_causal && (w.k0 + key_base + kKT - 1 > w.q0 + wave * 32);
    bias = (key_base >= nb) ? bias2 : 0.f;
    if (tail || mixed || diag) {
      int lim = kCap && mixed ? nb : nkeys;
      if (MODE == kModeExact && a.exact_causal) lim = min(lim, q_global - w.k0 + 1);
      const int lim2 = lim - key_base - 4 * h;  // element i is masked iff koff_i >= lim2
      const int nb2 = !kCap && mixed ? nb - key_base - 4 * h : 0x7fffffff;
      const float nat_bias = bias2 * kLn2;
#pragma unroll
      for (int sub = 0; sub < 2; ++sub)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int koff = 32 * sub + 8 * (i / 4) + (i % 4);
          float v = c[sub][i];
          if (koff >= nb2) v += nat_bias;
          c[sub][i] = (koff >= lim2) ? -INFINITY : v;
        }
      if (mixed) bias = 0.f;
    }
  };
  // Row maximum of a score tile in the log2 domain, in-lane and then over lane ^ 32.  d = 64: of the lane's own keys; whether any
  // row's reference has to move takes no exchange, so it waits for the branch that moves it, and what the exponentials subtract
  // is formed there too.  Same bits; 12 heads, n = 4096 25.6 -> 25.3 us, causal, n = 8192 99.6 -> 98.7, 64 heads, n = 65536 1357 -> 1350.
  // At d = 128 the node kernel then spills (12 bytes per lane) and the calls differ by +-0.4 %.
  constexpr bool kLaneMax = D == 64;
  auto row_max = [](float mx) { return kLaneMax ? fmaxf(mx, __shfl_xor(mx, 32)) : mx; };
  auto tile_max = [&](const f32x16 (&c)[2], float bias) -> float {
    float mx = max3f(c[0][0], c[1][0], c[0][1]);
#pragma unroll
    for (int i = 1; i < 16; ++i) {
      if (i + 1 < 16) mx = max3f(mx, c[1][i], c[0][i + 1]);
      else mx = fmaxf(mx, c[1][i]);
    }
    if constexpr (!kLaneMax) mx = fmaxf(mx, __shfl_xor(mx, 32));
    return __builtin_fmaf(mx, kLog2e, bias);
  };

  // Software pipeline over key tiles: while the matrix cores compute the scores
  // of tile kt+1, the vector ALU turns the scores of tile kt into bf16 weights;
  // while they accumulate P V of tile kt, the vector ALU reduces the row maximum
  // of tile kt+1.  K tile t and V tile t live in buffer (t & 1) of their kind;
  // K runs one tile ahead of V.
  f32x16 c[2];
  float bias = 0.f, t_max = -INFINITY;
  if (ntiles > 0) {
    // all three tiles are requested before any is stored: one global round trip
    u32x4 kreg1[TR::NKC];
    load_rows(0, Kh, kreg);
    load_rows(0, Vh, vreg);
    if (ntiles > 1) load_rows(1, Kh, kreg1);
    store_rows(kbuf_at(0), L::KSTR, kreg);
    store_rows(vbuf_at(0), L::VSTR, vreg);
    if (ntiles > 1) store_rows(kbuf_at(1), L::KSTR, kreg1);
  }
  __syncthreads();
  if (ntiles > 0) {
#pragma unroll
    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
      for (int i = 0; i < 16; ++i) c[sub][i] = 0.f;
    const unsigned char* kp0 = kbuf_at(0) + lq * L::KSTR + 16 * h;
    const unsigned char* kp1 = kp0 + 32 * L::KSTR;
#pragma unroll
    for (int j = 0; j < KS; ++j) {
      c[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(kp0 + 32 * j), qreg[j], c[0], 0, 0, 0);
      c[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(kp1 + 32 * j), qreg[j], c[1], 0, 0, 0);
    }
    mask_tile(c, 0, bias);
    t_max = tile_max(c, bias);
    m_run = row_max(t_max);  // the first tile sets the reference: the accumulators are still zero, nothing to rescale
    m_ref = finite_ref(m_run);
  }

  auto body = [&](int kt, f32x16 (&c)[2], float& bias, f32x16 (&cn)[2], float& bias_n, auto has_next) {
    constexpr bool HN = decltype(has_next)::value;
    const bool more_k = kt + 2 < ntiles;
    // The d = 64 kernels request the next tiles inside the score block (below), in the shadow of its MFMAs:
    // they then fit 168 registers (the node kernel with five spilled ones), a third workgroup per CU, and
    // take 8-10 % less (node launch, base case and exact attention alike).  At d = 128 the same move
    // measures +-0.5 % in exact mode and +7 % in node mode, whose requests first read the key list from
    // LDS: there they are issued here, ahead of the block.
    constexpr bool kRequestInBlock = D == 64;
    if constexpr (!kRequestInBlock) {
      if (more_k) load_rows(kt + 2, Kh, kreg);
      if (HN) load_rows(kt + 1, Vh, vreg);
    }

    if constexpr (kCap) {
      if (kt == nb_tiles) {
        end_masked();
        if (a.cap_scale > 0.f) {
          const float n = (float)w.nr.s;
          log2capw = (logf(a.cap_scale * (float)a.g.m / (n * logf(n))) + logaddexpf(log_masked, floor_term)) * kLog2e + bias2;
        }
      }
    }
    if (__any(t_max > m_run + 8.0f)) {
      const float m_new = fmaxf(m_run, row_max(t_max));
      const float alpha = __builtin_amdgcn_exp2f(m_run - ((m_new == -INFINITY) ? 0.f : m_new));
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[dt][i] *= alpha;
      l_run *= kCap ? __builtin_amdgcn_exp2f(sum_ref(m_run) - finite_ref(sum_ref(m_new))) : alpha;
      m_run = m_new;
      m_ref = finite_ref(m_new);
    }
    float capw = INFINITY;
    if constexpr (kCap) {
      if (kt >= nb_tiles) {
        capw = __builtin_amdgcn_exp2f(fminf(log2capw - finite_ref(m_run), 120.f));
        if (__any(m_run > log2capw + kFarCap)) {  // rare: exponentials of the sum's own
          const float ref = finite_ref(sum_ref(m_run));
#pragma unroll
          for (int sub = 0; sub < 2; ++sub)
#pragma unroll
            for (int i = 0; i < 16; ++i)
              l_run += __builtin_amdgcn_exp2f(fminf(__builtin_fmaf(c[sub][i], kLog2e, bias), log2capw) - ref);
          capw = 0.f;
        }
      }
    }
    const float shift = bias - (kLaneMax ? m_ref : finite_ref(m_run));

    // ---- scores of tile kt+1 (matrix cores)  ||  weights of tile kt (vector ALU) ----
    // The wave takes issue priority over its SIMD neighbour for this block, its densest one (an MFMA and a
    // slice of exponentials per slot), and gives it back for the P V block, whose slots the neighbour's
    // vector work fills: measured -3 % on the causal base case, -2 % on the node launch (any of the
    // neighbouring placements of the two instructions measured the same; priority during P V alone: no gain;
    // the d = 64 node launch, where vector issue binds, loses 2 % with it and goes without).
    constexpr bool kPrio = D == 128 || MODE == kModeExact;
    bf16x8 pf[4];
    if constexpr (kPrio) __builtin_amdgcn_s_setprio(1);
    if constexpr (kRequestInBlock && HN) {
      // no branch here: past the end the last tile is requested again (and not stored)
      load_rows(min(kt + 2, ntiles - 1), Kh, kreg);
      load_rows(kt + 1, Vh, vreg);
    }
    {
      if (HN) {
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
          for (int i = 0; i < 16; ++i) cn[sub][i] = 0.f;
        const unsigned char* kp0 = kbuf_at(kt + 1) + lq * L::KSTR + 16 * h;
        const unsigned char* kp1 = kp0 + 32 * L::KSTR;
        bf16x8 kf[2 * KS];
#pragma unroll
        for (int j = 0; j < KS; ++j) {
          kf[2 * j] = *reinterpret_cast<const bf16x8*>(kp0 + 32 * j);
          kf[2 * j + 1] = *reinterpret_cast<const bf16x8*>(kp1 + 32 * j);
        }
#pragma unroll
        for (int j = 0; j < KS; ++j) {
          cn[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[2 * j], qreg[j], cn[0], 0, 0, 0);
          cn[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[2 * j + 1], qreg[j], cn[1], 0, 0, 0);
        }
      }
      float ls[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int sub = 0; sub < 2; ++sub)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
          u32x4 pk;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(c[sub][8 * jj + 2 * e], kLog2e, shift));
            const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(c[sub][8 * jj + 2 * e + 1], kLog2e, shift));
            ls[e] += kCap ? fminf(p0, capw) + fminf(p1, capw) : p0 + p1;
            pk[e] = pack_bf16x2(p0, p1);
          }
          pf[2 * sub + jj] = __builtin_bit_cast(bf16x8, pk);
        }
      l_run += (ls[0] + ls[1]) + (ls[2] + ls[3]);
      // keep the weights' computation in this block, next to the MFMAs it hides behind
#pragma unroll
      for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(pf[j]));
      asm volatile("" : "+v"(l_run));
      if (HN) {
        // issue order: a few fragment reads ahead, then per MFMA one more read and
        // a slice of the vector work, which fits inside the MFMA's 32 cycles
        constexpr int kPre = 4;
        constexpr int kValu = (KS == 8) ? 5 : 18;  // d = 128: 5 measured best of 2 ... 9 (by half a percent); d = 64: 18 of 7 ... 26 (by 2 %)
        __builtin_amdgcn_sched_group_barrier(0x100, kPre, 0);
#pragma unroll
        for (int j = 0; j < 2 * KS; ++j) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          if (j < 2 * KS - kPre) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, kValu, 0);
        }
      }
    }
    if constexpr (kPrio) __builtin_amdgcn_s_setprio(0);
    if (HN) mask_tile(cn, kt + 1, bias_n);

    // ---- O^T += V^T P^T of tile kt (matrix cores)  ||  row maximum of tile kt+1 ----
    // slot e of a lane's P registers holds key 8*(e/4) + 4*h + e%4 of the 16-key step
    {
      typedef short s16x4 __attribute__((ext_vector_type(4)));
      typedef short s16x8 __attribute__((ext_vector_type(8)));
      typedef s16x4 __attribute__((address_space(3))) * lds_s16x4_ptr;
      const unsigned char* vb = vbuf_at(kt) + vtr_off;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          const unsigned char* vp = vb + (16 * j) * L::VSTR + (32 * dt) * 2;
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(vp));
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(vp + 8 * L::VSTR));
          const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), pf[j], o[dt], 0, 0, 0);
        }
      }
      if (HN) t_max = tile_max(cn, bias_n);
      constexpr int kPreV = 8;
      __builtin_amdgcn_sched_group_barrier(0x100, kPreV, 0);
#pragma unroll
      for (int j = 0; j < 4 * DT; ++j) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if (2 * j < 8 * DT - kPreV) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        if (HN) __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
      }
    }
    if (more_k) store_rows(kbuf_at(kt + 2), L::KSTR, kreg);
    if (HN) store_rows(vbuf_at(kt + 1), L::VSTR, vreg);
    __syncthreads();
  };
  // two tiles per trip so the score registers swap roles without copies.  The read / MFMA / vector-slice pipeline
  // that the sched_group_barrier calls ask for is formed where a block starts with its first fragment reads: the
  // ISA shows it for the two bodies inside the loop (kt's parity, hence every buffer address, is a constant
  // there), not for the copies of the body after the loop, which handle a list's last one or two tiles.
  f32x16 c2[2];
  float bias_b = 0.f;
  int kt = 0;
  stamp(2);
  for (; kt + 2 < ntiles; kt += 2) {
    body(kt, c, bias, c2, bias_b, std::true_type{});
    body(kt + 1, c2, bias_b, c, bias, std::true_type{});
  }
  if (kt + 2 == ntiles) {
    body(kt, c, bias, c2, bias_b, std::true_type{});
    body(kt + 1, c2, bias_b, c, bias, std::false_type{});
  } else if (kt + 1 == ntiles) {
    body(kt, c, bias, c2, bias_b, std::false_type{});
  }
  stamp(3);

  if constexpr (NG == 2) {  // the second group's sums through LDS (the tiles are read no more)
    f32x4* part = reinterpret_cast<f32x4*>(smem + NW * EpLds<D>::WAVE) + tid;  // [4 DT][kNT], then references and row sums
    float* ml = reinterpret_cast<float*>(reinterpret_cast<f32x4*>(smem + NW * EpLds<D>::WAVE) + 4 * DT * kNT) + tid;
    if (grp == 1) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4)
          part[(4 * dt + g4) * kNT] = (f32x4){o[dt][4 * g4], o[dt][4 * g4 + 1], o[dt][4 * g4 + 2], o[dt][4 * g4 + 3]};
      ml[0] = m_run;
      ml[kNT] = l_run;
    }
    __syncthreads();
    if (grp == 1) return;
    const float m1 = ml[0], m = fmaxf(m_run, m1), ref = (m == -INFINITY) ? 0.f : m;
    const float w0 = __builtin_amdgcn_exp2f(m_run - ref), w1 = __builtin_amdgcn_exp2f(m1 - ref);
    l_run = l_run * w0 + ml[kNT] * w1;
    m_run = m;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const f32x4 v = part[(4 * dt + g4) * kNT];
#pragma unroll
        for (int z = 0; z < 4; ++z) o[dt][4 * g4 + z] = o[dt][4 * g4 + z] * w0 + v[z] * w1;
      }
  }

  // ---- epilogue ----
  if (kCap && ntiles <= nb_tiles) end_masked();  // no sample was kept
  const float l_tot = l_run + __shfl_xor(l_run, 32);
  const bool empty = !(l_tot > 0.f);
  float inv = empty ? 0.f : 1.f / l_tot;
  float lse_own = empty ? -INFINITY : (sum_ref(m_run) + log2f(l_tot)) * kLn2;
  if constexpr (kCap) {  // d~_i = masked + max(d_i, tau / kappa)
    lse_own = logaddexpf(log_masked, fmaxf(lse_own, floor_term));
    float ref = lse_own;
    if (a.part_ref != nullptr) {
      if (lse_own != -INFINITY) ref = fmaxf(lse_own, m_run * kLn2);
      if (dest.valid && h == 0) a.part_ref[dest.part_row] = ref;
    }
    inv = (m_run == -INFINITY || lse_own == -INFINITY) ? 0.f : expf(m_run * kLn2 - ref);
  }
  // Where the row goes: a partial result of the causal recursion (node mode) or
  // the final output; in exact mode the partial results of every level of
  // Algorithm 4 are folded in first (row sum = D_21 + D_C22 at every split).
  //
  // The wave's 32 rows are transposed through LDS in fp32 (free now: the last
  // barrier of the loop is behind every wave), so that rows leave, and partial
  // rows arrive, as whole 16-byte pieces on consecutive lanes.
  const bool to_partial = (kNode) && a.part_o != nullptr;
  unsigned char* ep = smem + wave * EpLds<D>::WAVE;
  float* ep_w = reinterpret_cast<float*>(ep + 32 * EpLds<D>::ROW);
  int64_t* ep_rows = reinterpret_cast<int64_t*>(ep + 32 * EpLds<D>::ROW + 32 * kMaxFold * 4);
  int64_t* ep_pr = ep_rows + 32;

  // Levels folded row-major below (up to kMaxFold of them).  The 32 rows of a wave
  // lie in one n_min block, so every level treats them alike: either none of
  // them belongs to its off-diagonal node, or they are 32 consecutive partial rows.
  const bool fold = MODE == kModeExact && a.merge_levels > 0;
  const bool fold_rows = fold && a.merge_levels <= kMaxFold;
  uint32_t touched = 0;
  int nfold = 0;  // number of touched levels
  int64_t pr0[kMaxFold];
  float scale_own = inv;
  if (fold_rows) {
    const int i0 = w.q0 + 32 * __builtin_amdgcn_readfirstlane(wave);
    float lp[kMaxFold];
#pragma unroll
    for (int u = 0; u < kMaxFold; ++u) {
      lp[u] = -INFINITY;
      pr0[u] = 0;
      int64_t pr;
      if (u < a.merge_levels && level_touches(a.g, w.bh, i0, u, &pr)) {
        touched |= 1u << u;
        pr0[u] = pr;
        if (dest.valid) lp[u] = a.part_l[pr + lq];
      }
    }
    float mx = lse_own;
#pragma unroll
    for (int u = 0; u < kMaxFold; ++u) mx = fmaxf(mx, lp[u]);
    float w_own = 0.f, wl[kMaxFold];
#pragma unroll
    for (int u = 0; u < kMaxFold; ++u) wl[u] = 0.f;
    if (mx != -INFINITY) {
      const float e_own = expf(lse_own - mx);
      float den = e_own;
#pragma unroll
      for (int u = 0; u < kMaxFold; ++u) {
        wl[u] = expf(lp[u] - mx);
        den += wl[u];
      }
      const float rden = 1.f / den;
      w_own = e_own * rden;
#pragma unroll
      for (int u = 0; u < kMaxFold; ++u) wl[u] *= rden;
      if (a.part_ref != nullptr) {
#pragma unroll
        for (int u = 0; u < kMaxFold; ++u)
          if (((touched >> u) & 1u) && dest.valid) wl[u] = expf(a.part_ref[pr0[u] + lq] - mx) * rden;
      }
      lse_own = mx + logf(den);
    }
    scale_own = inv * w_own;
    // weights and partial-row bases of the touched levels, compacted (the set
    // of touched levels is the same for the whole wave)
#pragma unroll
    for (int u = 0; u < kMaxFold; ++u)
      if ((touched >> u) & 1u) {
        if (h == 0) ep_w[lq * kMaxFold + nfold] = wl[u];
        if (lane == 0) ep_pr[nfold] = pr0[u];
        ++nfold;
      }
  }
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[dt][i] *= scale_own;

  if (fold && !fold_rows && dest.valid) {
    // deeper recursions than kMaxFold levels: fold in the accumulator layout
    float mx, den;
    const float Lm = merged_lse(a, w.bh, dest.row_in_head, lse_own, &mx, &den);
    const float w_own = (lse_own == -INFINITY) ? 0.f : expf(lse_own - mx) / den;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[dt][i] *= w_own;
    for (int l = 0; l < a.merge_levels; ++l) {
      int64_t pr;
      if (!level_touches(a.g, w.bh, dest.row_in_head, l, &pr)) continue;
      const float lp = a.part_l[pr];
      if (lp == -INFINITY) continue;
      const float wl = expf((a.part_ref != nullptr ? a.part_ref[pr] : lp) - mx) / den;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          const int64_t at = pr * D + 32 * dt + 8 * g4 + 4 * h;
          const u32x2 raw = *reinterpret_cast<const u32x2*>(reinterpret_cast<const uint16_t*>(a.part_o) + at);
          const f32x4 v = {__uint_as_float(raw.x << 16), __uint_as_float(raw.x & 0xFFFF0000u),
                           __uint_as_float(raw.y << 16), __uint_as_float(raw.y & 0xFFFF0000u)};
          o[dt][4 * g4] += wl * v.x;
          o[dt][4 * g4 + 1] += wl * v.y;
          o[dt][4 * g4 + 2] += wl * v.z;
          o[dt][4 * g4 + 3] += wl * v.w;
        }
    }
    lse_own = Lm;
  }
  float* lse_dst = to_partial ? a.part_l : a.lse;
  const int64_t row_dst = to_partial ? dest.part_row : dest.out_row;
  if (lse_dst != nullptr && dest.valid && h == 0) lse_dst[row_dst] = lse_own;

  unsigned char* dst_base = to_partial ? reinterpret_cast<unsigned char*>(a.part_o) : reinterpret_cast<unsigned char*>(a.out);
  if (dst_base == nullptr) return;
  const bool out_fp32 = to_partial && !a.part_bf16;  // the stage calls take their partial rows in fp32
  constexpr int rs = EpLds<D>::ROW;
  if (h == 0) ep_rows[lq] = dest.valid ? row_dst : (int64_t)-1;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const int col = 32 * dt + 8 * g4 + 4 * h;
      const f32x4 v = {o[dt][4 * g4], o[dt][4 * g4 + 1], o[dt][4 * g4 + 2], o[dt][4 * g4 + 3]};
      *reinterpret_cast<f32x4*>(ep + lq * rs + col * 4) = v;
    }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  constexpr int CH = D / 8;  // 8-element pieces per row
  // NF = number of partial rows folded into every row (bf16 rows of the node launch); a compile-time
  // count, and the pieces of a lane walked in groups whose partial-row loads are ALL issued before
  // the first is consumed: one global round trip per group instead of one per piece.  The loads are
  // unconditional (a row that is not stored re-reads the wave's first row) and only the stores are
  // guarded: with loads under a branch the compiler's wait counts fall back to "everything", which
  // also waits for the previous piece's stores to reach memory.
  // Rows that the launch reads or writes once are non-temporal and leave the caches to the tiles: the folded partial rows, the fp32 copy,
  // the results of the exact pass; not those of the node pass (nor its partial rows), which gained nothing.  Forward (MI355X, us): 12
  // causal heads, n = 8192, d = 128 150.9 -> 150.0, 8 heads, n = 32768 454.3 -> 448.1, 32, n = 65536 3960 -> 3940; with the fp32 copy
  // 475.9 -> 461.8 and 4054 -> 4031; 32 unmasked heads, n = 32768 547.8 -> 540.6, d = 64 292.8 -> 287.6, 12, n = 4096 30.4 -> 29.2.
  if (ep_rows[0] < 0) return;  // a wave whose rows all lie past the end (valid rows are a prefix)
  auto drain = [&](auto nf_tag) {
    constexpr int NF = decltype(nf_tag)::value;
    constexpr int IT = 32 * CH / 64;                 // pieces per lane
    constexpr int GROUP = NF <= 4 ? IT : IT / 2;     // 16-byte loads in flight per lane: GROUP * NF <= 32
    const uint16_t* prow[NF > 0 ? NF : 1];
#pragma unroll
    for (int c = 0; c < NF; ++c) prow[c] = reinterpret_cast<const uint16_t*>(a.part_o) + ep_pr[c] * D;
#pragma unroll
    for (int g0 = 0; g0 < IT; g0 += GROUP) {
      int64_t r64[GROUP];
      u32x4 raw[GROUP][NF > 0 ? NF : 1];
#pragma unroll
      for (int it = 0; it < GROUP; ++it) {
        const int idx = lane + 64 * (g0 + it);
        const int row = idx / CH, ch = idx % CH;
        r64[it] = ep_rows[row];
        const int row_ld = r64[it] >= 0 ? row : 0;
#pragma unroll
        for (int c = 0; c < NF; ++c) raw[it][c] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(prow[c] + row_ld * D + ch * 8));
      }
#pragma unroll
      for (int it = 0; it < GROUP; ++it) {
        const int idx = lane + 64 * (g0 + it);
        const int row = idx / CH, ch = idx % CH;
        f32x4 v0 = *reinterpret_cast<const f32x4*>(ep + row * rs + ch * 32);
        f32x4 v1 = *reinterpret_cast<const f32x4*>(ep + row * rs + ch * 32 + 16);
#pragma unroll
        for (int c = 0; c < NF; ++c) {
          float wl = ep_w[row * kMaxFold + c];
          const u32x4 q = raw[it][c];
          f32x4 p0 = {__uint_as_float(q.x << 16), __uint_as_float(q.x & 0xFFFF0000u),
                      __uint_as_float(q.y << 16), __uint_as_float(q.y & 0xFFFF0000u)};
          f32x4 p1 = {__uint_as_float(q.z << 16), __uint_as_float(q.z & 0xFFFF0000u),
                      __uint_as_float(q.w << 16), __uint_as_float(q.w & 0xFFFF0000u)};
          if (!(wl != 0.f)) {  // a partial with an empty row sum carries no defined values
            p0 = (f32x4){0.f, 0.f, 0.f, 0.f};
            p1 = p0;
            wl = 0.f;
          }
          v0 += wl * p0;
          v1 += wl * p1;
        }
        if (r64[it] < 0) continue;
        if (out_fp32) {
          f32x4* dp = reinterpret_cast<f32x4*>(dst_base + (r64[it] * D + ch * 8) * 4);
          dp[0] = v0;
          dp[1] = v1;
          continue;
        }
        const u32x4 pk = {pack_bf16x2(v0.x, v0.y), pack_bf16x2(v0.z, v0.w), pack_bf16x2(v1.x, v1.y), pack_bf16x2(v1.z, v1.w)};
        u32x4* to = reinterpret_cast<u32x4*>(dst_base + (r64[it] * D + ch * 8) * 2);
        if (MODE == kModeExact) __builtin_nontemporal_store(pk, to);
        else *to = pk;
        if (!to_partial && a.out_f32 != nullptr) {  // unrounded copy of the final output, for the backward's delta
          f32x4* fp = reinterpret_cast<f32x4*>(a.out_f32 + r64[it] * D + ch * 8);
          __builtin_nontemporal_store(v0, fp);
          __builtin_nontemporal_store(v1, fp + 1);
        }
      }
    }
  };
  if (MODE == kModeExact) {
    switch (nfold) {
      case 0: drain(std::integral_constant<int, 0>{}); break;
      case 1: drain(std::integral_constant<int, 1>{}); break;
      case 2: drain(std::integral_constant<int, 2>{}); break;
      case 3: drain(std::integral_constant<int, 3>{}); break;
      case 4: drain(std::integral_constant<int, 4>{}); break;
      case 5: drain(std::integral_constant<int, 5>{}); break;
      case 6: drain(std::integral_constant<int, 6>{}); break;
      case 7: drain(std::integral_constant<int, 7>{}); break;
      default: drain(std::integral_constant<int, 8>{}); break;
    }
  } else {
    drain(std::integral_constant<int, 0>{});
  }
  if constexpr (STAMPS) {
    stamp(4);
    if (tid == 0 && a.stamps != nullptr) {
      long long* rec = a.stamps + (int64_t)kStampWords * bid;
#pragma unroll
      for (int i = 0; i < 5; ++i) rec[i] = stamp_c[i];
      rec[5] = stamp_w;
      rec[6] = (long long)wall_clock64();
      // where it ran: the hardware id register (wave, SIMD, CU, shader engine) and the XCD number
      const unsigned hw = __builtin_amdgcn_s_getreg(4 | (0 << 6) | (31 << 11));   // HW_ID, all 32 bits
      const unsigned xcc = __builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11));  // XCC_ID, bits 0-3
      rec[7] = (long long)(((nkeys + kKT - 1) / kKT) & 0xffff) | ((long long)hw << 16) | ((long long)(xcc & 15u) << 48);
    }
  }
}

template <int D, int MODE, int NW, bool STAMPS = false, int NG = 1, bool SORT = false>
static int launch_one(const AttnArgs& args, hipStream_t st) {
  AttnArgs a = args;
  if (MODE != kModeExact) set_node_divs<32 * NW>(a);
  else set_exact_divs<32 * NW>(a);
  a.exact_lpt = NG == 2;
  const int64_t grid = MODE != kModeExact ? node_grid<32 * NW>(a.g) : exact_grid<32 * NW>(a);
  if (grid <= 0) return HA_OK;
  if (grid > kMaxGrid) return HA_ERR_SHAPE;
  size_t lds = mfma_lds_bytes<D>(a.g.b, a.g.m, MODE) + (NG - 1) * 2 * (size_t)Lds<D>::BUF;
  const size_t ep = (size_t)NW * EpLds<D>::WAVE + (NG - 1) * (size_t)(D / 8 * 16 + 8) * 64 * NW;
  if (SORT) lds += sort_pushes_list<D, NW>(a.g) + 32 * NW * 4;
  if (lds < ep) lds = ep;
  static std::atomic<uint64_t> lds_set{0};  // per instantiation: devices on which the LDS limit is raised
  if (allow_full_lds(reinterpret_cast<const void*>(&attn_mfma_kernel<D, MODE, NW, STAMPS, NG, SORT>), lds_set) != HA_OK) return HA_ERR_LAUNCH;
  if constexpr (MODE == kModeCap) {  // all levels in one launch, or in as many as their workgroups take
    for (int64_t first = 0; first < grid; first += kMaxLaunch) {
      a.wg_first = (int32_t)first;
      const int64_t count = grid - first < kMaxLaunch ? grid - first : kMaxLaunch;
      hipLaunchKernelGGL((attn_mfma_kernel<D, MODE, NW, STAMPS, NG, SORT>), dim3((unsigned)count), dim3(64 * NW * NG), lds, st, a);
      const int rc = check_launch();
      if (rc != HA_OK) return rc;
    }
    return HA_OK;
  }
  hipLaunchKernelGGL((attn_mfma_kernel<D, MODE, NW, STAMPS, NG, SORT>), dim3((unsigned)grid), dim3(64 * NW * NG), lds, st, a);
  return check_launch();
}

// Waves per workgroup: node tiles (short key loops) use 4, two workgroups per
// CU, so one workgroup's gathers overlap the other's MFMAs; exact attention and
// the causal base case (long key loops) can share each K / V tile among 8 waves.
#ifndef HA_NW_NODE
#define HA_NW_NODE 4
#endif
#ifndef HA_NW_EXACT
#define HA_NW_EXACT 4
#endif

// Exact attention over long key ranges shares each K / V tile among 8 waves (one workgroup per CU) at d = 128.  Unmasked:
// wherever the 4-wave form would put two workgroups on some CUs, which all then wait for (up to 256 of them, 128 wide
// ones, two wave groups share the keys instead); causal, of unequal length: where every CU gets several.
// 8 waves -> 4 waves (MI355X, d = 128), unmasked, n = 8192: 8 heads (256 wide workgroups) 243 -> 259 us, 5 heads (160) 188 ->
// 198, 7 heads (224) 224 -> 233; 2 heads, n = 16384 (128) 361 -> 288, 3 heads (192) 400 -> 416, one head (64) 358 -> 268;
// causal: 4 heads, n = 16384 (256) 370 -> 310, 8 heads (512) 578 -> 540, 16 heads (1024) 1032 -> 1029.
// The short loops of the base case prefer two 4-wave workgroups per CU.
constexpr int kWideExactMinRows = 8192;
// Launches that leave a CU at most one or two workgroups are bound by the longest chain of key tiles of a workgroup: two groups
// of four waves then share it.  One such workgroup fills a CU, so past 256 a second round begins, whose workgroups start as
// CUs become free: causal tiles then come heaviest first throughout (exact_lpt), and up to two rounds are worth it, the more
// the longer the rows.  Short rows gain nothing.  One group -> two (MI355X, us):
//   unmasked: 4 heads, n = 4096, d = 64 54.4 -> 42.0, d = 128 73.0 -> 60.6; 32 heads (256), n = 1024: 17.3 -> 15.4, 23.7 -> 23.5;
//     32 heads (192), n = 768: 13.7 -> 12.4, 18.4 -> 17.5; 42 heads (252): 15.9 -> 14.9, but d = 128 22.1 -> 23.1; 64 heads (192),
//     n = 384: 11.2 -> 11.7, 12.0 -> 12.2
//   causal (in brackets, where measured: every second round of 32 backwards, the order of the one-group form), d = 64:
//     8 heads (512), n = 8192 107.5 -> 92.4 (109.8), 9 heads (576) 118.7 -> 113.8, 10 (640) 124.9 -> 123.7; 16 heads (512), n = 4096
//     56.0 -> 50.8 (60.5), 18 (576) 61.8 -> 62.2; 24 heads (384), n = 2048 30.4 -> 24.5 (29.1), 32 (512) 30.9 -> 29.9, 36 (576) 34.0 ->
//     38.7; 48 heads (384), n = 1024 18.2 -> 17.5 (20.3), 56 (448) 18.2 -> 19.6; 64 heads (320), n = 640 13.1 -> 12.7, 77 (385) 15.0 -> 16.5
//   d = 128: 8 heads (512), n = 8192 159 -> 144 (170), 9 (576) 177 -> 178; 16 heads (512), n = 4096 83.2 -> 78.7 (90.8), 17 (544) 89.4 ->
//     93.6; 19 heads (456), n = 3072 63.4 -> 60.9, 21 (504) 65.8 -> 67.1; 28 heads (448), n = 2048 43.5 -> 42.8, 32 (512) 45.5 -> 45.1; 32
//     heads (384), n = 1536 33.1 -> 30.4, 37 (444) 38.5 -> 39.1; 40 heads (320), n = 1024 24.4 -> 22.0, 48 (384) 25.0 -> 25.8; 51
//     heads (255), n = 640 18.6 -> 18.3, 64 (320) 18.4 -> 19.6
// The groups' references differ, so weights are rounded to bf16 at other points than in the one-group form: results differ by 1.8e-3 (2-norm; 12
// causal heads, n = 5000, d = 128; unmasked, 4 heads, n = 4096, 2.5e-3), errors against 64 bits do not: 2.13e-3 -> 2.10e-3, 2.334e-3 ->
// 2.331e-3.
constexpr int kSplitExactMinRows = 640;
static bool split_exact(const AttnArgs& a) {
  const int rows = a.exact_block < a.exact_rows_q ? a.exact_block : a.exact_rows_q;
  if (rows < kSplitExactMinRows) return false;
  const int64_t grid = exact_grid<128>(a);
  if (!a.exact_causal) return grid <= (a.g.d == 128 && rows < 1024 ? 160 : 256);
  if (a.g.d == 64) return grid <= (rows < 1024 ? 320 : rows < 1536 ? 384 : rows < 8192 ? 512 : 576);
  return grid <= (rows < 1024 ? 256 : rows < 1536 ? 320 : rows < 2048 ? 384 : rows < 4096 ? 448 : 512);
}
constexpr int64_t kWideExactMinGrid = 129, kWideExactMinGridCausal = 1024;

// Node launches that sort by themselves: with more than one workgroup of 128 rows per CU some CUs hold two, which count the same node twice
// side by side and end last (33 k cycles of life where one has a CU, 43 k where two share it).  Where tiles of 256 rows fit
// the chip once, eight waves do that work once per CU.  Four waves -> eight (MI355X, us; b = m = 256): d = 64: 12 heads, n = 4096 26.4 ->
// 25.4, 9 heads 25.8 -> 24.8, 16 heads 27.9 -> 27.1; 64 heads, n = 1024 27.8 -> 27.1; 32 heads, n = 2048 28.2 -> 27.3; 8 heads, n = 3900,
// b = 300 27.7 -> 26.2; other blocks and samples: 24 heads, n = 2048, b = m = 512 34.0 -> 32.0, m = 32 22.3 -> 21.2; 25 heads, n = 1500, b = 150 21.3 ->
// 20.2, n = 1300, b = 130 19.3 -> 17.8; 8 heads, n = 8192, m = 64 25.6 -> 24.5; causal, 12 heads, n = 8192 102.9 -> 101.5; d = 128: 12 heads,
// n = 4096 36.9 -> 35.4, 16 heads 43.4 both; 32 heads, n = 2048, m = 64 34.6 -> 34.0; 14 heads, n = 1300, b = 130 23.3 -> 23.5; causal, 16 heads,
// n = 8192 192.8 -> 193.0.
static bool wide_sorting_node(const Geometry& g) { return node_grid<128>(g) > 256 && node_grid<256>(g) <= 256; }

// Whether a node launch sorts by itself.  Every workgroup then counts its whole node, some 4 us of its life at 4096 keys,
// against a sorting launch of 6.5 to 8 us and 2.5 us of the host's time for it: worth it while the workgroups fit the chip at
// once, eight-wave ones by their rule.  At d = 64 three of a CU's 160 KB fit beside each other until the sort's tables take them past a
// third of it, and the launch that drops to two loses more than the sort.  Sorting launch -> in the attention (MI355X, us; workgroups of 128 rows):
//   d = 64, one round: 12 heads, n = 4096 (384) 29.8 -> 25.5, 16 (512) 31.9 -> 27.7, 20 (640) 37.2 -> 33.8, 24 (768) 39.3 -> 35.9; b = m = 64:
//     40 heads, n = 1024 (640) 21.9 -> 18.6, 24 heads, n = 2048 (768) 22.3 -> 19.6, 12 heads, n = 4096 (768) 23.3 -> 20.5, 4 heads, n = 8192
//     (512) 21.1 -> 19.6; b = m = 128: 24 heads, n = 4096 (768) 32.3 -> 28.7, 8 heads, n = 8192 (512) 27.5 -> 24.5; b = 100, m = 77: 34
//     heads, n = 2100 (714) 29.1 -> 26.9, 13 heads, n = 5600 (728) 29.7 -> 27.0; causal, 12 heads, n = 8192, n_min = 2048 (768) 80.4 -> 76.3
//   d = 64, 512 places: b = m = 64: 8 heads, n = 5760 (720, three to a CU) 23.5 -> 22.2, 7 heads, n = 5888 (644) 23.8 -> 27.7; n = 6144: 10 heads (480)
//     31.5 -> 27.2, 11 (528) 36.3 -> 40.9; n = 4096, m = 1024: 17 heads (544) r = 7 56.3 -> 52.8, r = 8 56.5 -> 63.2
//   d = 128, 512 places: 16 heads, n = 4096 (512) 44.1 -> 41.2, 20 (640) 55.2 both, 24 (768) 58.6 -> 59.7; 8 heads, n = 8192 (512) 44.8 ->
//     42.2; b = m = 64: 16 heads, n = 2048 (512) 25.7 -> 23.1, 4 heads, n = 8192 (512) 27.3 -> 24.9; 15 heads, n = 6300, b = 100, m = 77 (945)
//     50.4 -> 55.0
// A second round of up to 1024 workgroups at d = 64 gains where a sort's threads hold few keys (up to 8 each, n <= 2048), or nearly the 16
// they are dealt, loaded 16 bytes at a time: n = 1000, b = 40 (900) 25.8 -> 25.0, n = 1600, b = 100 (800) 31.8 -> 31.3, n = 2048, b = 64 (1024)
// 26.6 -> 26.2, b = 128 36.3 -> 35.6; n = 1152, b = 128 (990) 36.7 -> 37.2; n = 2112, b = 96 (880) 32.1 -> 32.6; n = 2304, b = 256 (774)
// 44.1 -> 45.5; n = 3072, b = 128 (792) 36.0 -> 35.5, b = 192 (800) 35.4 -> 35.7, b = 256 (792) 44.1 -> 44.2; n = 3328, b = 128 (780) 37.6 ->
// 36.1; n = 3500, b = 100, whose heads do not start at 16 bytes (770) 32.8 -> 33.3; n = 4096, b = 32 (896) 25.5 -> 25.6, b = 64 (1024) 27.8 -> 27.3, b = 256
// (1024) 46.7 -> 45.7; n = 5120, b = 64 (800) 27.0 -> 28.6, b = 256 45.6 -> 47.4.  Past 1024: 128 heads, n = 1024, b = m = 64 (2048) 37.5 -> 39.0.
bool attn_mfma_sorts(const Geometry& g) {
  const int rows = node_sort_rows(g);
  const int64_t wgs = node_grid<128>(g);
  if (rows > kNodeSortMax || wgs * rows > 4 << 20) return false;
  if (wide_sorting_node(g)) return true;
  if (g.d == 128) return wgs <= 512;
  const size_t plain = mfma_lds_bytes<64>(g.b, g.m, kModeNode), sorting = plain + sort_pushes_list<64, 4>(g) + 32 * 4 * 4;
  const int64_t per_cu = lds_workgroups(sorting, 3);  // (a fourth has no registers)
  if (wgs <= 256 * per_cu) return true;
  if (per_cu < lds_workgroups(plain, 3) || wgs > 1024) return false;
  const bool whole_words = (g.causal ? g.n_min : g.n) % 16 == 0;
  return rows <= 2048 || (rows > 3200 && rows <= 4096 && whole_words);
}

int64_t attn_mfma_grid(const AttnArgs& a, int mode) {
  return mode == kModeNode ? node_grid<32 * HA_NW_NODE>(a.g) : exact_grid<32 * HA_NW_EXACT>(a);
}

int launch_attn_mfma(const AttnArgs& a, int mode, hipStream_t st) {
  if (a.g.dtype != HA_BF16) return HA_ERR_DTYPE;
  if (mode == kModeExact && a.merge_levels > 0 && !a.part_bf16) return HA_ERR_DTYPE;  // this kernel folds bf16 partial rows
  const bool split = mode == kModeExact && split_exact(a);
  if (a.stamps != nullptr) {  // the measuring instantiations: the node launch behind a sorting launch, the base case
    if (a.g.d == 128) {
      if (mode == kModeNode) return launch_one<128, kModeNode, HA_NW_NODE, true>(a, st);
      return split ? launch_one<128, kModeExact, 4, true, 2>(a, st) : launch_one<128, kModeExact, HA_NW_EXACT, true>(a, st);
    }
    if (a.g.d == 64) {
      if (mode == kModeNode) return launch_one<64, kModeNode, HA_NW_NODE, true>(a, st);
      return split ? launch_one<64, kModeExact, 4, true, 2>(a, st) : launch_one<64, kModeExact, HA_NW_EXACT, true>(a, st);
    }
    return HA_ERR_SHAPE;
  }
  const bool wide_node = a.codes_q && wide_sorting_node(a.g);
  const bool wide = mode == kModeExact && a.merge_levels == 0 &&
                    a.exact_block >= kWideExactMinRows && a.exact_rows_q >= kWideExactMinRows &&
                    exact_grid<256>(a) >= (a.exact_causal ? kWideExactMinGridCausal : kWideExactMinGrid);
  if (a.g.d == 128) {
    if (mode == kModeNode && wide_node) return launch_one<128, kModeNode, 8, false, 1, true>(a, st);
    if (mode == kModeNode && a.codes_q) return launch_one<128, kModeNode, 4, false, 1, true>(a, st);
    if (mode == kModeNode) return launch_one<128, kModeNode, HA_NW_NODE>(a, st);
    if (mode == kModeCap) return launch_one<128, kModeCap, HA_NW_NODE>(a, st);
    if (split) return launch_one<128, kModeExact, 4, false, 2>(a, st);
    return wide ? launch_one<128, kModeExact, 8>(a, st) : launch_one<128, kModeExact, HA_NW_EXACT>(a, st);
  }
  if (a.g.d == 64) {
    if (mode == kModeNode && wide_node) return launch_one<64, kModeNode, 8, false, 1, true>(a, st);
    if (mode == kModeNode && a.codes_q) return launch_one<64, kModeNode, 4, false, 1, true>(a, st);
    if (mode == kModeNode) return launch_one<64, kModeNode, HA_NW_NODE>(a, st);
    if (mode == kModeCap) return launch_one<64, kModeCap, HA_NW_NODE>(a, st);
    if (split) return launch_one<64, kModeExact, 4, false, 2>(a, st);
    return launch_one<64, kModeExact, HA_NW_EXACT>(a, st);  // no gain from the wide form at d = 64
  }
  return HA_ERR_SHAPE;
}

}  // namespace ha
