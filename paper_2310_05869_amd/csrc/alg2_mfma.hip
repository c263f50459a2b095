// bf16 MFMA kernels for the estimator of Algorithm 2 as printed and the value
// product of Lemma 2 / Algorithm 3 (the options beside the Section 4 form):
//
//   tau         log of the unmasked row sum <1 - M^H_j, A_j> of the rows j in T
//               (Algorithm 2's tau is their maximum): 128 rows of T per
//               workgroup against a range of the node's keys in sorted order,
//               keys of the row's own sorted block left out.
//   main        with Lemma 2's value product: for 128 queries of one sorted block
//               the masked row sum over the block's keys, the capped estimate d_i
//               over the uniform samples, d~_i = masked + max(d_i, tau / kappa),
//               and the numerator over rows of V drawn by squared norm, each with
//               its 1 / (m p_l).  (Section 4's value product with the caps is a
//               mode of the forward kernel: the same keys feed sums and numerator.)
//
// Tiling as in the forward kernel: 4 waves x 32 queries, 64 keys per step,
// S^T = K Q^T with v_mfma_f32_32x32x16_bf16 so that a lane holds 16 keys of one
// query, weights converted to bf16 in place as the B operand of O^T += V^T P^T,
// V^T fragments from the transposing LDS read.  The main loop is not software
// pipelined: the next tile's rows are fetched into registers while the current
// tile is computed.
//
// The key list of the main kernel has three segments, each padded to whole tiles:
// A the block's keys, B the m uniform samples, C the m rows drawn
// by squared norm.  An entry is a row index, or its complement when the key is
// to be left out (padding; a sample that falls into the row's own block, the
// factor 1 - M_{i,l_j}); segment C carries a log weight per key.  The exponentials'
// reference (log2 domain, lazily moved as in the forward kernel) begins anew with
// every segment.
#include "alg2_common.h"
#include "attn_common.h"

namespace ha {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

constexpr int kA2KT = 64;    // keys per step
constexpr int kA2QT = 128;   // queries per workgroup
constexpr int kA2NT = 256;   // threads

template <int D>
struct A2Lds {
  static constexpr int KSTR = (D + 8) * 2;    // bytes per K row (conflict-free 16-byte row reads)
  static constexpr int VSTR = (D + 32) * 2;   // bytes per V row (conflict-free transposing reads)
  static constexpr int K_BYTES = kA2KT * KSTR;
  static constexpr int V_BYTES = kA2KT * VSTR;
  static constexpr int BUF = K_BYTES + V_BYTES;
  static constexpr int EP_ROW = D * 4 + 16;
  static constexpr int EP_WAVE = 32 * EP_ROW + 32 * 8;
};

__host__ __device__ inline int a2_tiles(int count) { return (count + kA2KT - 1) / kA2KT; }

// list entries: segments A, B, C (the log weights of C follow)
__host__ __device__ inline int a2_list_entries(const Geometry& g) { return (a2_tiles(g.b) + 2 * a2_tiles(g.m)) * kA2KT; }

template <int D>
__host__ __device__ inline size_t a2_lds_bytes(const Geometry& g) {
  const size_t s = 2 * (size_t)A2Lds<D>::BUF + (size_t)a2_list_entries(g) * 4 + (size_t)a2_tiles(g.m) * kA2KT * 4;
  const size_t ep = 4 * (size_t)A2Lds<D>::EP_WAVE;
  return s > ep ? s : ep;
}

// Row sums of the rows of T.  Keys are walked in sorted order, so that a row's own block is one run of positions and
// only the tiles that touch the run of one of a wave's rows carry a mask; in storage order every score of every
// tile had to be compared with its key's block (two of seven vector instructions per score), and vector issue is
// what bounds a kernel with one product per score.  A range of keys is shared by two groups of RW waves, tile about,
// whose sums are merged through LDS: with kAlg2TauSplits ranges alone 32 heads of 256 rows are two waves per
// SIMD, which cannot cover each other.  The row tiles of a range are neighbours on one XCD (its keys meet in one L2).
// Measured (MI355X, 32 heads, n = 32768, d = 128, m = 256): 171 -> 134 us.
//
// A trip ends for all waves at one barrier, and waves that all begin with their products leave the vector units idle, then the matrix
// cores: the second group adds up its previous tile first.  (Vector instructions were 59 % of the kernel's cycles, products 32 %, and they added
// up.)  Tiles come by DMA, NB - 1 of them ahead, into LDS in rows of D * 2 bytes, unpadded: piece c (16 bytes) of row r at place c ^ swz(r), free
// of bank conflicts for the row reads.  The positions' rows are kept ahead of them in LDS too, in chunks of four trips, and come by DMA
// as well: a load of an index into a register is waited for with every tile requested before it (twice a chunk, the compiler's count
// knowing nothing of the DMA; 16 heads, n = 16384, d = 128 165.1 -> 163.0, 24 heads, m = 512 312.7 -> 309.7, d = 64 1 %).
// Forward with the caps (MI355X, us), tiles through registers, in step and with the maxima of every tile -> this; d = 128, m = 256: 16
// heads, n = 16384 173 -> 166, 8 heads 115 -> 106, 4 heads, n = 4096 46.5 -> 45.8; 24 heads, n = 16384, m = 512 325 -> 309; 12 causal heads,
// n = 32768 849 -> 830; 32 heads, n = 32768, whose keys come from HBM, 1 %; d = 64: 8 heads, n = 16384 84.2 -> 79.9, m = 512 208 -> 196, 12
// causal heads, n = 32768 526 -> 512.
// Clustered inputs (64 clusters, scores to 250), whose references move often: 16 heads, n = 16384, d = 128 170.3 -> 163.6, 8 heads 114.5 -> 108.5, 12 causal
// heads, n = 32768 845 -> 822; d = 64: 8 heads, n = 16384 84.8 -> 81.8, 12 heads, n = 4096 47.6 -> 47.5 (weights formed twice where one moves: 49.0).
// Eight waves to a tile, whose groups of 1024 threads read every key once and four tiles ahead: 1 to 14 % slower than this.
template <int D>
struct TauLds {
  static constexpr int RW = 4;                       // waves of a group
  static constexpr int NT = 2 * RW * 64;             // threads; also the positions of a chunk of the list
  static constexpr int ROWB = D * 2, CPR = D / 8;
  static constexpr int TILE = kA2KT * ROWB;
  static constexpr int RPI = 64 / CPR;               // rows per DMA instruction
  static constexpr int DPW = kA2KT / RPI / RW;       // DMA instructions per wave and tile
  static constexpr int NB = D == 64 ? 4 : 2;        // tile buffers of a group (two workgroups per CU)
  static constexpr int LIST_AT = 2 * NB * TILE;
  static constexpr int BYTES = LIST_AT + 4 * NT * 4;  // (a ring of four chunks)
  static_assert(DPW >= 1 && (NB == 2 || NB == 4) && NB <= RW && NT == 4 * 2 * kA2KT);
  __device__ static int swz(int row) { return D == 128 ? row & 15 : (row >> 1) & 7; }
};

template <int D>
__global__ __launch_bounds__(TauLds<D>::NT, 4) void alg2_tau_mfma_kernel(Alg2Args a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  using L = TauLds<D>;
  constexpr int KS = D / 16;
  constexpr int RW = L::RW;
  const Geometry& g = a.g;
  const int grp = __builtin_amdgcn_readfirstlane(threadIdx.x / (64 * RW));
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((threadIdx.x / 64) % RW);
  const int lq = lane & 31, h = lane >> 5;
  unsigned char* bufs = smem + grp * L::NB * L::TILE;
  int32_t* list = reinterpret_cast<int32_t*>(smem + L::LIST_AT);

  const int row_tiles = (g.m + kA2QT - 1) / kA2QT;
  const int idx = a.wg_first + logical_block(blockIdx.x, gridDim.x);
  const int j0 = (idx % row_tiles) * kA2QT;
  const int split = idx / row_tiles % kAlg2TauSplits;
  const int bh = idx / row_tiles / kAlg2TauSplits;
  const int rows_valid = min(kA2QT, g.m - j0);
  const int64_t hb = (int64_t)bh * g.n;
  const Alg2Node nd = alg2_node(a, bh);
  const uint16_t* Qh = reinterpret_cast<const uint16_t*>(a.Q) + (int64_t)nd.head * a.n_full * D;
  const uint16_t* Kh = reinterpret_cast<const uint16_t*>(a.K) + (int64_t)nd.head * a.n_full * D;

  const int ntiles = a2_tiles(g.n);
  const int kt_lo = (int)((int64_t)ntiles * split / kAlg2TauSplits);
  const int kt_hi = (int)((int64_t)ntiles * (split + 1) / kAlg2TauSplits);
  const int trips = (kt_hi - kt_lo + 1) / 2;
  // chunk c of the list: the rows at positions 64 kt_lo + NT c ... (past the end: the last position, masked)
  const int32_t* keys = a.perm_k + hb;
  auto chunk_at = [&](int c) { return min(kt_lo * kA2KT + c * L::NT + (int)threadIdx.x, g.n - 1); };
  const int row0 = keys[chunk_at(0)], row1 = keys[chunk_at(1)];

  const int r_in_tile = wave * 32 + lq;
  const int r_use = r_in_tile < rows_valid ? r_in_tile : 0;
  const int q_in_node = a.tau_rows[(int64_t)nd.heap * g.m + j0 + r_use];
  int own = a.pos_q[hb + q_in_node] / g.b * g.b;  // first position of the row's own block
  bf16x8 qreg[KS];
  {
    const u32x4* qp = reinterpret_cast<const u32x4*>(Qh + (int64_t)(nd.q_start + q_in_node) * D + 8 * h);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qreg[ks] = __builtin_bit_cast(bf16x8, qp[2 * ks]);
  }

  const __amdgpu_buffer_rsrc_t krsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Kh, 0, (int)(uint32_t)(a.n_full * L::ROWB), 0x00020000);
  // instruction ii of this wave fills rows RPI (RW ii + wave) ... of the tile
  const int drow = L::RPI * wave + lane / L::CPR;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)bufs + 1024 * wave;
  auto request_tile = [&](int it) {  // of this trip; past the range: rows that exist and are not used
    const uint32_t at = lds0 + (it & (L::NB - 1)) * L::TILE;
#pragma unroll
    for (int ii = 0; ii < L::DPW; ++ii) {
      const int t = RW * L::RPI * ii + drow;
      const int row = list[((2 * it + grp) * kA2KT + t) & (4 * L::NT - 1)];
      const int voff = row * L::ROWB + (((lane % L::CPR) ^ L::swz(t)) << 4);
      const uint32_t to = at + 1024 * RW * ii;
      asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"{m0}"(to), "v"(voff), "s"(krsrc) : "memory");
    }
  };
  const __amdgpu_buffer_rsrc_t lrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)keys, 0, g.n * 4, 0x00020000);
  const uint32_t list0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int32_t*)list + 256 * (grp * RW + wave);
  auto request_chunk = [&](int c) {
    const int voff = chunk_at(c) * 4;
    const uint32_t to = list0 + (c & 3) * (L::NT * 4);
    asm volatile("s_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"{m0}"(to), "v"(voff), "s"(lrsrc) : "memory");
  };
  list[threadIdx.x] = row0;
  list[L::NT + threadIdx.x] = row1;
  __syncthreads();
#pragma unroll
  for (int it = 0; it < L::NB - 1; ++it) request_tile(it);
  // (used in registers, so that the loop does not wait for these loads again)
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qreg[ks]));
  asm volatile("" : "+v"(own));

  f32x16 c[2];  // element i of c[sub]: position 32 sub + 8 (i / 4) + 4 h + i % 4 of the tile
  auto scores = [&](int it) {
    const unsigned char* kp = bufs + (it & (L::NB - 1)) * L::TILE + lq * L::ROWB;
    auto frag = [&](int sub, int j) {  // (rows lq and lq + 32 have the same swizzle)
      return *reinterpret_cast<const bf16x8*>(kp + sub * 32 * L::ROWB + (((2 * j + h) ^ L::swz(lq)) << 4));
    };
#pragma unroll
    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
      for (int i = 0; i < 16; ++i) c[sub][i] = 0.f;
#pragma unroll
    for (int j = 0; j < KS; ++j) {
      c[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(0, j), qreg[j], c[0], 0, 0, 0);
      c[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(1, j), qreg[j], c[1], 0, 0, 0);
    }
  };
  float m_run = -INFINITY, sum = 0.f;  // reference (log2 domain) and this lane's share of the row sum / 2^m_run
  auto add_tile = [&](int kt) {
    // a tile that lies in the row's own block as a whole is left out as a whole
    const int mlo = own - kt * kA2KT, tail = g.n - kt * kA2KT;
    const bool out = mlo <= 0 && mlo + g.b >= kA2KT;
    if (tail < kA2KT || __any(!out && mlo < kA2KT && mlo + g.b > 0)) {
#pragma unroll
      for (int sub = 0; sub < 2; ++sub)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int koff = 32 * sub + 8 * (i / 4) + (i % 4);
          if (koff >= tail - 4 * h || (unsigned)(koff - (mlo - 4 * h)) < (unsigned)g.b) c[sub][i] = -INFINITY;
        }
    }
    auto weigh = [&]() {
      const float shift = (m_run == -INFINITY) ? 0.f : -m_run;
      float s4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int sub = 0; sub < 2; ++sub)
#pragma unroll
        for (int i = 0; i < 16; ++i) s4[i & 3] += __builtin_amdgcn_exp2f(__builtin_fmaf(c[sub][i], kLog2e, shift));
      return (s4[0] + s4[1]) + (s4[2] + s4[3]);
    };
    // The reference moves when a weight exceeds 2^8: a sum below that has none, and the maxima, a seventh of a tile's vector
    // instructions, need not be formed.  Where it moves, a sum of weights in range is taken to the new reference as a whole, and the
    // weights are formed again only where they left it.
    auto move = [&]() {  // returns the factor of sums against the reference before
      float mx = fmaxf(c[0][0], c[1][0]);
#pragma unroll
      for (int i = 1; i < 16; ++i) mx = __builtin_fmaxf(__builtin_fmaxf(mx, c[0][i]), c[1][i]);
      mx = fmaxf(mx, __shfl_xor(mx, 32)) * kLog2e;
      if (out) mx = -INFINITY;
      const float m_new = fmaxf(m_run, mx);
      const float factor = __builtin_amdgcn_exp2f(m_run - ((m_new == -INFINITY) ? 0.f : m_new));
      sum *= factor;
      m_run = m_new;
      return factor;
    };
    float s;
    if (__any(m_run == -INFINITY)) {
      move();
      s = weigh();
    } else {
      s = weigh();
      if (__any(!(out || s < 256.f))) {
        const float factor = move();
        if (__any(!(out || s < 0x1p100f))) s = weigh();
        else s *= factor;
      }
    }
    sum += out ? 0.f : s;
  };
  const int mine = (kt_hi - kt_lo + 1 - grp) / 2;  // the group's tiles
  for (int it = 0; it < trips; ++it) {
    // the trip's tile has landed, for the whole workgroup, and the one before it is read no more
    // (the list's chunk of a trip that RW divides was requested ahead of its tile: one request more lies behind the tiles of the next two)
    if (L::NB == 4 && (unsigned)(it % RW - 1) < 2u) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(L::DPW * (L::NB - 2) + 1) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(L::DPW * (L::NB - 2)) : "memory");
    __syncthreads();
    if (it % RW == 0) request_chunk(it / RW + 2);
    request_tile(it + L::NB - 1);
    const int kt = kt_lo + grp + 2 * it;
    if (grp == 1 && it > 0) add_tile(kt - 2);
    if (it < mine) scores(it);
    if (grp == 0) add_tile(kt);
  }
  if (grp == 1 && mine == trips && trips > 0) add_tile(kt_lo + 1 + 2 * (trips - 1));
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  sum += __shfl_xor(sum, 32);
  float* part = reinterpret_cast<float*>(smem);  // [2][kA2QT]: the tiles are read no more
  if (grp == 1 && h == 0) {
    part[r_in_tile] = m_run;
    part[kA2QT + r_in_tile] = sum;
  }
  __syncthreads();
  if (grp == 0 && h == 0 && r_in_tile < rows_valid) {
    const float m1 = part[r_in_tile], m = fmaxf(m_run, m1);
    const float ref = (m == -INFINITY) ? 0.f : m;
    const float total = sum * __builtin_amdgcn_exp2f(m_run - ref) + part[kA2QT + r_in_tile] * __builtin_amdgcn_exp2f(m1 - ref);
    a.log_unm_parts[((int64_t)split * g.BH + bh) * g.m + j0 + r_in_tile] = (total > 0.f) ? (m + log2f(total)) * kLn2 : -INFINITY;
  }
}

template <int D>
__global__ __launch_bounds__(kA2NT, 2) void alg2_mfma_kernel(Alg2Args a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  using L = A2Lds<D>;
  constexpr int KS = D / 16;                 // MFMA k-steps of the score product
  constexpr int DT = D / 32;                 // 32-wide d tiles of the numerator
  constexpr int CPR = D / 8;                 // 16-byte chunks per row
  constexpr int NKC = kA2KT * CPR / kA2NT;   // chunks per thread and tensor
  const Geometry& g = a.g;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int lq = lane & 31, h = lane >> 5;

  unsigned char* bufs = smem;
  int32_t* list = reinterpret_cast<int32_t*>(smem + 2 * L::BUF);

  // ---- which rows this workgroup owns ----
  const int tpb = (g.b + kA2QT - 1) / kA2QT;
  const int per_head = (g.n / g.b) * tpb;
  const int tile = blockIdx.x % per_head;
  const int bh = blockIdx.x / per_head;
  const int t = tile / tpb;
  const int chunk = tile % tpb;
  const int p0 = t * g.b + chunk * kA2QT;
  const int rows_valid = min(kA2QT, g.b - chunk * kA2QT);
  // bh is a view head: one node of the level (alg2_common.h).  Row indices below are rows of the
  // real head (permutation entries already are; node-local draws get the node's first row added).
  const int64_t hb = (int64_t)bh * g.n;
  const Alg2Node nd = alg2_node(a, bh);
  const int64_t draws = ((int64_t)nd.head * a.total_nodes + nd.heap) * g.m;
  const uint16_t* Qh = reinterpret_cast<const uint16_t*>(a.Q) + (int64_t)nd.head * a.n_full * D;
  const uint16_t* Kh = reinterpret_cast<const uint16_t*>(a.K) + (int64_t)nd.head * a.n_full * D;
  const uint16_t* Vh = reinterpret_cast<const uint16_t*>(a.V) + (int64_t)nd.head * a.n_full * D;

  // ---- this lane's query row: B operand of S^T = K Q^T, kept in registers ----
  const int r_in_tile = wave * 32 + lq;
  const bool valid = r_in_tile < rows_valid;
  const int r_use = valid ? r_in_tile : 0;
  const int qrow = a.perm_q[hb + p0 + r_use];
  bf16x8 qreg[KS];
  {
    const u32x4* qp = reinterpret_cast<const u32x4*>(Qh + (int64_t)qrow * D + 8 * h);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qreg[ks] = __builtin_bit_cast(bf16x8, qp[2 * ks]);
  }

  // ---- the keys ----
  const int nA = a2_tiles(g.b), nB = a2_tiles(g.m), nC = nB;
  const int ntiles = nA + nB + nC;
  const float* bias_c = reinterpret_cast<const float*>(list + (nA + nB + nC) * kA2KT);  // log2-domain weights of segment C
  {
    int32_t* la = list;
    int32_t* lb = la + nA * kA2KT;
    int32_t* lc = lb + nB * kA2KT;
    float* bc = reinterpret_cast<float*>(lc + nC * kA2KT);
    for (int i = tid; i < nA * kA2KT; i += kA2NT) la[i] = (i < g.b) ? a.perm_k[hb + (int64_t)t * g.b + i] : ~0;
    for (int j = tid; j < nB * kA2KT; j += kA2NT) {
      int e = ~0;
      if (j < g.m) {
        const int row = nd.k_start + a.samples[(int64_t)nd.heap * g.m + j];
        e = (a.samp_blk[draws + j] == t) ? ~row : row;  // factor 1 - M_{i,l_j}
      }
      lb[j] = e;
    }
    for (int j = tid; j < nC * kA2KT; j += kA2NT) {
      lc[j] = (j < g.m) ? nd.k_start + a.vsamp[draws + j] : ~0;
      bc[j] = (j < g.m) ? a.vlogw[draws + j] * kLog2e : 0.f;
    }
    __syncthreads();
  }
  const float ratio = g.m > 0 ? (float)g.n / (float)g.m : 1.f;
  const float log2ratio = log2f(ratio);
  const float floor_term = (a.kappa > 0.f)
                               ? a.log_tau[(int64_t)nd.head * a.total_nodes + nd.heap] - logf(a.kappa) : -INFINITY;
  auto need_v = [&](int kt) -> bool { return kt >= nA + nB; };

  // ---- tile movers (buffer loads: rows past the head read as zeros and are left out by their entries) ----
  const uint32_t head_bytes = (uint32_t)(a.n_full * (D * 2));
  const __amdgpu_buffer_rsrc_t krsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Kh, 0, (int)head_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t vrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Vh, 0, (int)head_bytes, 0x00020000);
  u32x4 kreg[NKC], vreg[NKC];
  auto load_tile = [&](int kt) {
    const bool with_v = need_v(kt);
#pragma unroll
    for (int i = 0; i < NKC; ++i) {
      const int c = tid + i * kA2NT;
      const int key = c / CPR, col = c % CPR;
      const int e = list[kt * kA2KT + key];
      const int voff = (e < 0 ? ~e : e) * (D * 2) + col * 16;
      kreg[i] = __builtin_amdgcn_raw_buffer_load_b128(krsrc, voff, 0, 0);
      if (with_v) vreg[i] = __builtin_amdgcn_raw_buffer_load_b128(vrsrc, voff, 0, 0);
    }
  };
  auto store_tile = [&](int kt) {
    unsigned char* kbuf = bufs + (kt & 1) * L::BUF;
    unsigned char* vbuf = kbuf + L::K_BYTES;
    const bool with_v = need_v(kt);
#pragma unroll
    for (int i = 0; i < NKC; ++i) {
      const int c = tid + i * kA2NT;
      const int key = c / CPR, col = c % CPR;
      *reinterpret_cast<u32x4*>(kbuf + key * L::KSTR + col * 16) = kreg[i];
      if (with_v) *reinterpret_cast<u32x4*>(vbuf + key * L::VSTR + col * 16) = vreg[i];
    }
  };
  const int vtr_off = ((lane & 15) >> 2) * L::VSTR + ((lane & 3) * 4 + ((lane >> 4) & 1) * 16) * 2 + (4 * h) * L::VSTR;

  // ---- state ----
  f32x16 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[dt][i] = 0.f;
  // Scores of one row can lie hundreds apart, so every segment has a reference of its own: the sums of A and B are kept as
  // logarithms when the next segment begins, and no sample of B counts (or moves the reference) beyond its cap.
  float m_run = -INFINITY;  // reference of the segment's exponentials, log2 domain
  float l_run = 0.f;        // this lane's share of the segment's row sum / 2^m_run
  float log_masked = -INFINITY, log_d = -INFINITY;  // of the block; of (n/m) sum of capped kept samples
  float log2capw = 3e38f;  // log2 of (n/m) C_i, known once segment A is done; no cap: above every finite score
  auto end_segment = [&]() -> float {
    const float l = l_run + __shfl_xor(l_run, 32);
    const float r = (l > 0.f) ? (m_run + log2f(l)) * kLn2 : -INFINITY;
    l_run = 0.f;
    m_run = -INFINITY;
    return r;
  };

  load_tile(0);
  store_tile(0);
  __syncthreads();

  for (int kt = 0; kt < ntiles; ++kt) {
    const bool more = kt + 1 < ntiles;
    if (more) load_tile(kt + 1);

    if (kt == nA) {
      // the masked row sum is complete: the cap C_i of Algorithm 2
      log_masked = end_segment();
      if (a.cap_scale > 0.f) {
        const float log_cap = logf(a.cap_scale * (float)g.m / ((float)g.n * logf((float)g.n))) + logaddexpf(log_masked, floor_term);
        log2capw = log_cap * kLog2e + log2ratio;
      }
    }
    if (kt == nA + nB) log_d = end_segment();

    const unsigned char* kbuf = bufs + (kt & 1) * L::BUF;
    const unsigned char* vbuf = kbuf + L::K_BYTES;
    // ---- scores ----
    f32x16 c[2];
#pragma unroll
    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
      for (int i = 0; i < 16; ++i) c[sub][i] = 0.f;
    {
      const unsigned char* kp0 = kbuf + lq * L::KSTR + 16 * h;
      const unsigned char* kp1 = kp0 + 32 * L::KSTR;
#pragma unroll
      for (int j = 0; j < KS; ++j) {
        c[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(kp0 + 32 * j), qreg[j], c[0], 0, 0, 0);
        c[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(kp1 + 32 * j), qreg[j], c[1], 0, 0, 0);
      }
    }
    // ---- log2-domain arguments: score + the key's log weight, -inf where the key is left out.
    // Element i of c[sub] is key 32 sub + 8 (i / 4) + 4 h + i % 4 of the tile.
    const int seg = kt < nA ? 0 : (kt < nA + nB ? 1 : 2);
    const float segbias = (seg == 1) ? log2ratio : 0.f;
    float tmax = -INFINITY;
#pragma unroll
    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const int at = 32 * sub + 8 * g4 + 4 * h;
        f32x4 b4 = {segbias, segbias, segbias, segbias};
        const i32x4 e4 = *reinterpret_cast<const i32x4*>(list + kt * kA2KT + at);
        if (seg == 2) b4 = *reinterpret_cast<const f32x4*>(bias_c + (kt - nA - nB) * kA2KT + at);
#pragma unroll
        for (int z = 0; z < 4; ++z) {
          float v = e4[z] < 0 ? -INFINITY : __builtin_fmaf(c[sub][4 * g4 + z], kLog2e, b4[z]);
          if (seg == 1) v = fminf(v, log2capw);
          c[sub][4 * g4 + z] = v;
          tmax = fmaxf(tmax, v);
        }
      }
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
    if (__any(tmax > m_run + 8.0f)) {
      const float m_new = fmaxf(m_run, tmax);
      const float alpha = __builtin_amdgcn_exp2f(m_run - ((m_new == -INFINITY) ? 0.f : m_new));
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[dt][i] *= alpha;
      l_run *= alpha;
      m_run = m_new;
    }
    const float mref = (m_run == -INFINITY) ? 0.f : m_run;
    // ---- weights, sums, and the B operand of the numerator ----
    bf16x8 pf[4];
    float sp = 0.f;
#pragma unroll
    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        u32x4 pk;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float p0w = __builtin_amdgcn_exp2f(c[sub][8 * jj + 2 * e] - mref);
          const float p1w = __builtin_amdgcn_exp2f(c[sub][8 * jj + 2 * e + 1] - mref);
          sp += p0w + p1w;
          pk[e] = pack_bf16x2(p0w, p1w);
        }
        pf[2 * sub + jj] = __builtin_bit_cast(bf16x8, pk);
      }
    l_run += sp;
    // ---- numerator: O^T += V^T P^T ----
    if (need_v(kt)) {
      typedef short s16x4 __attribute__((ext_vector_type(4)));
      typedef short s16x8 __attribute__((ext_vector_type(8)));
      typedef s16x4 __attribute__((address_space(3))) * lds_s16x4_ptr;
      const unsigned char* vb = vbuf + vtr_off;
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
    }
    if (more) store_tile(kt + 1);
    __syncthreads();
  }

  // ---- results ----
  if (g.m == 0) log_masked = end_segment();
  const float log_dt = logaddexpf(log_masked, fmaxf(log_d, floor_term));   // d~_i = masked + max(d_i, tau / kappa)
  const float ref = a.part_ref != nullptr && log_dt != -INFINITY ? fmaxf(log_dt, m_run * kLn2) : log_dt;
  const float f = (m_run == -INFINITY || log_dt == -INFINITY) ? 0.f : expf(m_run * kLn2 - ref);
  const int64_t out_row = hb + (qrow - nd.q_start);
  if (valid && h == 0) {
    a.lse[out_row] = log_dt;
    if (a.part_ref != nullptr) a.part_ref[out_row] = ref;
  }

  // the wave's 32 rows leave through an fp32 LDS transpose as whole 16-byte pieces
  unsigned char* ep = smem + wave * L::EP_WAVE;
  int64_t* ep_rows = reinterpret_cast<int64_t*>(ep + 32 * L::EP_ROW);
  if (h == 0) ep_rows[lq] = valid ? out_row : (int64_t)-1;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const int col = 32 * dt + 8 * g4 + 4 * h;
      const f32x4 v = {o[dt][4 * g4] * f, o[dt][4 * g4 + 1] * f, o[dt][4 * g4 + 2] * f, o[dt][4 * g4 + 3] * f};
      *reinterpret_cast<f32x4*>(ep + lq * L::EP_ROW + col * 4) = v;
    }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  constexpr int CH = D / 8;  // 8-element pieces per row
  uint16_t* outp = reinterpret_cast<uint16_t*>(a.out);
  for (int idx = lane; idx < 32 * CH; idx += 64) {
    const int row = idx / CH, ch = idx % CH;
    const int64_t r64 = ep_rows[row];
    if (r64 < 0) continue;
    const f32x4 v0 = *reinterpret_cast<const f32x4*>(ep + row * L::EP_ROW + ch * 32);
    const f32x4 v1 = *reinterpret_cast<const f32x4*>(ep + row * L::EP_ROW + ch * 32 + 16);
    const u32x4 pk = {pack_bf16x2(v0.x, v0.y), pack_bf16x2(v0.z, v0.w), pack_bf16x2(v1.x, v1.y), pack_bf16x2(v1.z, v1.w)};
    *reinterpret_cast<u32x4*>(outp + r64 * D + ch * 8) = pk;
  }
}

template <int D>
static int launch_tau(const Alg2Args& args, int64_t grid, hipStream_t st) {
  static std::atomic<uint64_t> lds_set{0};  // per instantiation: devices on which the LDS limit is raised
  if (allow_full_lds(reinterpret_cast<const void*>(&alg2_tau_mfma_kernel<D>), lds_set) != HA_OK) return HA_ERR_LAUNCH;
  Alg2Args a = args;
  constexpr int64_t kStep = kMaxLaunch / 2;  // (512 threads)
  for (int64_t first = 0; first < grid; first += kStep) {
    a.wg_first = (int32_t)first;
    const unsigned count = (unsigned)(grid - first < kStep ? grid - first : kStep);
    hipLaunchKernelGGL((alg2_tau_mfma_kernel<D>), dim3(count), dim3(TauLds<D>::NT), TauLds<D>::BYTES, st, a);
    const int rc = check_launch();
    if (rc != HA_OK) return rc;
  }
  return HA_OK;
}

int launch_alg2_tau_mfma(const Alg2Args& a, hipStream_t st) {
  const Geometry& g = a.g;
  const int64_t grid = (int64_t)g.BH * ((g.m + kA2QT - 1) / kA2QT) * kAlg2TauSplits;
  if (grid <= 0) return HA_OK;
  if (grid > kMaxGrid) return HA_ERR_SHAPE;
  return g.d == 128 ? launch_tau<128>(a, grid, st) : launch_tau<64>(a, grid, st);
}

template <int D>
static int launch_a2(const Alg2Args& a, hipStream_t st) {
  const Geometry& g = a.g;
  const int64_t grid = (int64_t)g.BH * (g.n / g.b) * ((g.b + kA2QT - 1) / kA2QT);
  if (grid <= 0) return HA_OK;
  if (grid > kMaxGrid) return HA_ERR_SHAPE;
  static std::atomic<uint64_t> lds_set{0};  // per instantiation: devices on which the LDS limit is raised
  if (allow_full_lds(reinterpret_cast<const void*>(&alg2_mfma_kernel<D>), lds_set) != HA_OK) return HA_ERR_LAUNCH;
  hipLaunchKernelGGL((alg2_mfma_kernel<D>), dim3((unsigned)grid), dim3(kA2NT), a2_lds_bytes<D>(g), st, a);
  return check_launch();
}

int launch_alg2_main_mfma(const Alg2Args& a, hipStream_t st) {
  return a.g.d == 128 ? launch_a2<128>(a, st) : launch_a2<64>(a, st);
}

}  // namespace ha
