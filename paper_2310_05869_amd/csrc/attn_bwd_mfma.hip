// bf16 MFMA backward kernel for gfx950: gradients of the HyperAttention forward
// with respect to Q, K and V, the random draws (hyperplanes, sample indices)
// and hence the permutations held fixed.
//
// Every output row of the forward is ONE softmax over a multiset of keys with
// weights: its block keys (weight 1) and its kept sampled keys (weight s/m) in
// every node the row belongs to, plus, when causal, the keys of its base-case
// block (Algorithms 1, 2 and 4 with the row sums added up).  With the final
// log row sum L_i and delta_i = <dO_i, O_i>, the gradient therefore splits into
// independent contributions of every (query, key) pair that occurs:
//   P_ij  = w_ij exp(<q_i, k_j> - L_i)
//   dV_j += P_ij dO_i
//   dS_ij = P_ij (<dO_i, v_j> - delta_i)
//   dQ_i += dS_ij k_j          dK_j += dS_ij q_i
// and each part (node block, node samples, base block) can be processed on its
// own, with the same tiles, lists and masks as in the forward.
//
// One kernel, two roles.  32 "R rows" per wave stay in registers for the whole
// pass and own the accumulators; "T rows" stream through LDS in tiles of 64:
//   dQ passes   R = queries (Q, dO, L, delta in registers), T = keys (K, V)
//   dK/dV passes R = keys (K, V in registers),  T = queries (Q, dO; L, delta in LDS)
// As in the forward the transposed products are formed (T rows along the MFMA's
// M dimension), so a lane holds 16 T rows of ONE R row, and P^T, dS^T converted
// to bf16 are directly the B operands of the accumulating products, whose A
// operands (T tile transposed) come from the transposing LDS read.
//
// The dK / dV passes form S and dP once and accumulate both gradients (4 products; 3 in the dQ passes).
// At d = 128 that is 128 accumulator registers, 64 of R rows and 32 of scores out of the 256 that two waves
// per SIMD leave each, so the T tiles go to LDS by DMA (buffer loads with an LDS destination) and never
// pass through registers.  A DMA instruction fills 1 KiB of consecutive LDS, so rows cannot be padded
// against bank conflicts; instead the 16-byte pieces of a row are swizzled (BwdLds), which the lanes do
// by choosing which piece of the row they fetch.
// The budget does not quite close: at d = 128 the compiler spills 28 (sampled keys), 12 (exact) and 24 bytes per lane (block keys
// of an unmasked problem); at d = 64 every form of one wave group gets three workgroups per CU, the exact dQ pass four where
// it has more than three to place (bwd_four_workgroups).  The compiler gave the sampled-key pass 173
// registers by itself, five too many; asked for three workgroups it needs 168, without spills (forward + backward, 12 heads:
// n = 16384 234 -> 227 us, where its 768 workgroups then are one round; n = 32768 451 -> 439 us).
// What bounds it: the order in which a wave issues reads, products and vector work (two waves per SIMD, 64 products
// of 32 cycles per tile and wave in the dK / dV passes).  So that order is written out and pinned (below), the rare
// masks sit behind a branch, and nothing in the loop waits for memory but the one wait per tile.  Counters (32 causal
// heads, n = 32768, d = 128): matrix pipe busy 60 % at 1.73 GHz in the exact dK / dV pass, 55 % in the exact dQ pass, 48 % with the
// sampled keys (the steady loop of the forward: 62 % at 1.65 GHz); the block keys move 4.4 TB/s, a copy 4.9.
// Measured (MI355X, 32 causal heads, n = 131072, d = 128, b = m = 256).  First form: dK and dV in passes of their own,
// tiles staged through registers; second: one pass, tiles by DMA; third: this one, pinned order.
//   dK / dV of the base case 13.9 -> 10.0 -> 8.2 ms, of the sampled keys 5.5 -> 4.1 -> 2.9 ms, of the blocks
//   7.65 -> 6.25 -> 5.75 ms, dQ of the base case 7.1 -> 6.8 -> 6.6 ms, of the nodes 6.0 -> 5.95 -> 5.6 ms;
//   forward + backward 50.5 -> 43.5 -> 39.3 ms.
//
// Sums over parts are taken in a fixed order, never by floating-point atomics: the node passes run
// level by level and add their fp32 rows to one accumulated row per tensor row (the first level
// that holds a row writes it), the sampled keys' rows go through a reduction of their own, and the
// base-case passes add the accumulated rows in their epilogue and write the final gradient.
#include <type_traits>

#include "attn_common.h"
#include "bwd_common.h"

namespace ha {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kTT = 64;    // T rows per step
constexpr int kRT = 128;   // R rows per workgroup (4 waves x 32)
constexpr int kBNT = 256;  // threads

// A T tile: 64 rows of D * 2 bytes, unpadded; piece c (16 bytes) of row r sits at place c ^ swz(r).
// Both readers are conflict-free: the row-major reads take one piece of 16 rows at a time (swz is a
// bijection on 16 rows, together with the row's parity at d = 64), the transposing reads 64
// consecutive bytes of four rows (which swz sends to four different quarters of the banks).
template <int D>
struct BwdLds {
  static constexpr int ROWB = D * 2;
  static constexpr int TILE = kTT * ROWB;       // one tensor's tile
  static constexpr int BUF = 2 * TILE;          // y tile + bt tile
  static constexpr int SC = 2 * kTT * 4;        // per buffer: bias - L and -delta of the T rows
  static constexpr int EP_ROW = D * 4 + 16;
  static constexpr int EP_WAVE = 32 * EP_ROW + 256;  // rows, row ids
  __device__ static int swz(int row) {
    if (D == 128) return ((row & 3) << 2) | ((row >> 2) & 3);
    return ((row & 2) << 1) | ((row >> 2) & 3);
  }
};

// rows of the T positions, where they are not consecutive: the key list (dQ of a node), the block's or the chunk's
// queries (dK / dV of a node)
__host__ __device__ inline int bwd_list_capacity(const BwdArgs& a, int mode) {
  const Geometry& g = a.f.g;
  if (mode == kBwdDqNode) return ((g.b + g.m + 63) & ~63) + 64;
  if (mode == kBwdDkvBlock) return (g.b + 63) & ~63;
  if (mode == kBwdDkvSamp) return ((a.chunk < g.n_cov ? a.chunk : g.n_cov) + 63) & ~63;
  return 0;
}

// block-key pass: the workgroup's sampled keys lie behind all else, from the prologue to the end
template <int D, int NG>
__host__ __device__ inline size_t bwd_hits_at(const BwdArgs& a, int mode) {
  const size_t s = NG * (2 * (size_t)BwdLds<D>::BUF + 2 * BwdLds<D>::SC) + 64 + (size_t)bwd_list_capacity(a, mode) * 4;
  return s > (size_t)4 * NG * BwdLds<D>::EP_WAVE ? s : (size_t)4 * NG * BwdLds<D>::EP_WAVE;
}

template <int D, int NG>
__host__ __device__ inline size_t bwd_lds_bytes(const BwdArgs& a, int mode) {
  return bwd_hits_at<D, NG>(a, mode) + (mode == kBwdDkvBlock && !a.f.g.causal ? sample_hits_bytes(a.f.g) : 0);
}

// 16 bytes per lane from buffer memory to 1 KiB of LDS starting at byte lds_at (wave-uniform).  Inline assembly
// because the compiler's wait counts would serialise the builtin with every LDS read; the kernel
// waits for these requests itself, once per tile.
__device__ inline void dma_1k(const __amdgpu_buffer_rsrc_t& rsrc, uint32_t lds_at, int voff) {
  // (m0 as an operand: the compiler writes it and knows; it takes no clobber of a reserved register)
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"{m0}"(lds_at), "v"(voff), "s"(rsrc) : "memory");
}

// Waves per SIMD that the compiler is asked for.
constexpr int bwd_waves_per_simd(int d, int mode) { return d == 64 && mode == kBwdDkvSamp ? 3 : 2; }

// FINAL: the node passes of an unmasked problem, which write the final gradients.
// NG = 2 (exact passes): two groups of four waves take the T tiles in turn, each with tile buffers of its own; their sums are
// added through LDS.
// FOUR: held to the registers of four waves per SIMD (bwd_four_workgroups).
template <int D, int MODE, bool FINAL, int NG, bool FOUR>
__global__ __launch_bounds__(kBNT * NG, FOUR ? 4 : bwd_waves_per_simd(D, MODE)) void attn_bwd_kernel(BwdArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  using L = BwdLds<D>;
  constexpr bool kDq = (MODE == kBwdDqNode || MODE == kBwdDqExact);
  constexpr bool kExact = (MODE == kBwdDqExact || MODE == kBwdDkvExact);
  constexpr bool kSorted = (MODE == kBwdDkvBlock || MODE == kBwdDkvSamp);  // T rows = a run of sorted query positions
  constexpr bool kHits = FINAL && MODE == kBwdDkvBlock;  // sampled keys' sums added here
  constexpr int KS = D / 16;
  constexpr int DT = D / 32;
  constexpr int CPR = D / 8;                 // 16-byte pieces per row
  constexpr int RPI = 64 / CPR;              // rows per DMA instruction
  constexpr int NDMA = kTT / RPI / 4;        // instructions per wave and tensor tile
  static_assert(NG == 1 || kExact);          // the lists, sampled keys and accumulated rows of the node passes are one group's

  const AttnArgs& f = a.f;
  const Geometry& g = f.g;
  const int tid = NG == 1 ? threadIdx.x : threadIdx.x % kBNT;  // within the group
  const int grp = NG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / kBNT);
  const int lane = tid & 63, wave = tid >> 6;
  const int lq = lane & 31, h = lane >> 5;

  unsigned char* bufs = smem + grp * 2 * L::BUF;
  float* sc = reinterpret_cast<float*>(smem + NG * 2 * L::BUF + grp * 2 * L::SC);
  int32_t* scratch = reinterpret_cast<int32_t*>(smem + NG * (2 * L::BUF + 2 * L::SC));
  int32_t* list = scratch + 16;

  // ---- which part of the problem this workgroup owns ----
  const BwdWork b = decode_bwd_work<kRT, MODE>(a, kExact ? (int)blockIdx.x : logical_block(blockIdx.x, gridDim.x), (int)gridDim.x);
  const TileWork& w = b.w;

  const int64_t hs = f.q_bh_stride;
  const uint16_t* Qh = reinterpret_cast<const uint16_t*>(f.Q) + (int64_t)w.bh * hs;
  const uint16_t* Kh = reinterpret_cast<const uint16_t*>(f.K) + (int64_t)w.bh * hs;
  const uint16_t* Vh = reinterpret_cast<const uint16_t*>(f.V) + (int64_t)w.bh * hs;
  const uint16_t* Gh = reinterpret_cast<const uint16_t*>(a.dO) + (int64_t)w.bh * hs;
  const float* lse_h = a.lse + (int64_t)w.bh * g.n;
  const float* del_h = a.delta + (int64_t)w.bh * g.n;
  const uint16_t* Xh = kDq ? Qh : Kh;   // R rows: x operand of the scores
  const uint16_t* Ah = kDq ? Gh : Vh;   // R rows: operand of dP
  const uint16_t* Yh = kDq ? Kh : Qh;   // T rows: y operand of the scores
  const uint16_t* Bh = kDq ? Vh : Gh;   // T rows: operand of dP

  // ---- this lane's R row ----
  const int r_in_tile = wave * 32 + lq;
  const int r_use = r_in_tile < w.rows_valid ? r_in_tile : 0;
  int blk_r = -1;        // sampled-key pass: sorted block of this key
  const int r_row = bwd_r_row<MODE>(a, b, r_use, &blk_r);           // row within the head
  SampleHead shead{-1, 0};
  if (kHits) shead = fetch_sample_head(a, b, tid);
  // What the first tile waits for comes first: the entries of the T rows' list, then, while the R rows are on their way, the list and the
  // tile's requests; only then are the R rows waited for.  (With the R rows awaited ahead of the list, MI355X, us: forward + backward, 12
  // heads, n = 16384, d = 64 231.9 -> 229.6; backward, d = 128 295.8 -> 288.8, 16 causal heads, n = 32768 3146 -> 3123, d = 64 1704 ->
  // 1687; exact passes, which have no list, +-0.5 %.)
  KeyListHead khead{};
  if (MODE == kBwdDqNode) khead = key_list_fetch<kBNT>(f, w);
  const int nsorted = MODE == kBwdDkvBlock ? g.b : b.chunk_len;
  const int32_t* tperm = kSorted ? f.perm_q + w.seg_off + (MODE == kBwdDkvBlock ? (int64_t)w.t * g.b : (int64_t)b.chunk_start) : nullptr;
  const int t_first = kSorted ? tperm[min(tid, nsorted - 1)] : 0;
  bf16x8 xreg[KS], areg[KS];
  {
    const u32x4* xp = reinterpret_cast<const u32x4*>(Xh + (int64_t)r_row * D + 8 * h);
    const u32x4* ap = reinterpret_cast<const u32x4*>(Ah + (int64_t)r_row * D + 8 * h);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      xreg[ks] = __builtin_bit_cast(bf16x8, xp[2 * ks]);
      areg[ks] = __builtin_bit_cast(bf16x8, ap[2 * ks]);
    }
  }
  // ---- the T rows: the key list in LDS (dQ of a node), a run of sorted query
  // positions through P_Q, listed in LDS too (dK/dV of a node), or a contiguous range ----
  int nT, nb = 0x7fffffff;
  if (MODE == kBwdDqNode) {
    nT = build_key_list<kBNT>(f, w, list, scratch, &nb, khead);
  } else if (kSorted) {
    nT = nsorted;
    for (int i = tid; i < ((nT + 63) & ~63); i += kBNT) list[i] = i == tid ? t_first : tperm[min(i, nT - 1)];
    __syncthreads();
  } else {
    nT = max(0, w.k1 - w.k0);
  }
  const int ntiles = (nT + NG * kTT - 1) / (NG * kTT);  // of the group; its tile kt is tile NG kt + grp of the T rows
  const float bias2 = ((MODE == kBwdDqNode || MODE == kBwdDkvSamp) && g.m > 0) ? log2f((float)w.nr.s / (float)g.m) : 0.f;
  const float nat_bias = bias2 * kLn2;

  // ---- tile movers: DMA from buffer memory ----
  const uint32_t head_bytes = (uint32_t)(g.n * (D * 2));
  const __amdgpu_buffer_rsrc_t yrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Yh, 0, (int)head_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t brsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Bh, 0, (int)head_bytes, 0x00020000);
  // instruction ii of this wave fills rows RPI (4 ii + wave) ... of the tile; this lane fetches the piece of its row
  // that belongs at its place (the row's swizzle does not depend on ii)
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const int drow = RPI * wave_s + lane / CPR;
  const int dcol = ((lane % CPR) ^ L::swz(drow)) * 16;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)bufs + 1024 * wave_s;
  float sc_l = 0.f, sc_d = 0.f;
  auto request_tile = [&](int kt) {
    const int t0 = (NG * kt + grp) * kTT;
    if (NG == 2 && t0 >= nT) return;  // (the other group has the last tile)
    if (!kDq && tid < kTT) {
      const int row = kSorted ? list[t0 + tid] : min(w.k0 + t0 + tid, g.n - 1);
      sc_l = lse_h[row];
      sc_d = del_h[row];
    }
    const uint32_t at = lds0 + (kt & 1) * L::BUF;
#pragma unroll
    for (int ii = 0; ii < NDMA; ++ii) {
      const int t = t0 + 4 * RPI * ii + drow;
      const int row = kExact ? min(w.k0 + t, g.n - 1) : list[t];  // past the end: some existing row, masked
      const int voff = row * (D * 2) + dcol;
      dma_1k(yrsrc, at + 4096 * ii, voff);
      dma_1k(brsrc, at + L::TILE + 4096 * ii, voff);
    }
  };
  auto finish_tile = [&](int kt) {  // everything requested for tile kt has landed, for the whole workgroup on return
    if (!kDq && tid < kTT) {
      float* s = sc + (kt & 1) * (2 * kTT);
      s[tid] = (sc_l == -INFINITY) ? -INFINITY : nat_bias - sc_l;
      s[kTT + tid] = -sc_d;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };
  // row-major fragments: piece 2 j + h of row lq (+ 32 sub); transposed: 4 rows x 16 columns per 16-lane group, lane i of
  // a group at row i / 4, columns 4 (i % 4) ...
  const int rd_row = lq * L::ROWB + ((h ^ L::swz(lq)) << 4);   // ^ 32 j
  const int r4 = (lane & 15) >> 2;
  const int rd_col = (4 * h + r4) * L::ROWB + (((((lane >> 4) & 1) * 2 + ((lane & 3) >> 1)) ^ L::swz(4 * h + r4)) << 4) +
                     (lane & 1) * 8;                            // ^ (64 dt + 32 hi)

  f32x16 acc1[DT], acc2[kDq ? 1 : DT];  // dQ or dK; dV
#pragma unroll
  for (int i = 0; i < 16; ++i) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) acc1[dt][i] = 0.f;
#pragma unroll
    for (int dt = 0; dt < (kDq ? 1 : DT); ++dt) acc2[dt][i] = 0.f;
  }
  if (ntiles > 0) request_tile(0);
  // (a use in registers, so that the loop does not wait for these loads again: behind the tile requests such a
  // wait would be one for the whole next tile)
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    asm volatile("" : "+v"(xreg[ks]));
    asm volatile("" : "+v"(areg[ks]));
  }
  float nl2_r = 0.f, del_r = 0.f;  // dQ passes: -L log2(e) and delta of the R row
  if (kDq) {
    const float lv = lse_h[r_row];
    nl2_r = (lv == -INFINITY) ? -INFINITY : -lv * kLog2e;
    if (a.delta_out == nullptr) {
      del_r = del_h[r_row];
    } else {
      // The lane's half of the row.  A launch of its own read dO once more.  Forward + backward, with it -> without (MI355X, us):
      // 12 heads, n = 16384, d = 64 217 -> 209; n = 32768, d = 128 820 -> 805; 2 heads, n = 4096 74.4 -> 73.8; exact, 12 heads, n =
      // 5000, d = 128 375 -> 373.
      const int64_t at = ((int64_t)w.bh * g.n + r_row) * D + 8 * h;
      f32x4 s = {0.f, 0.f, 0.f, 0.f};
      auto add = [&](int ks, f32x4 o0, f32x4 o1) {
        const u32x4 dv = __builtin_bit_cast(u32x4, areg[ks]);
        s[0] = __builtin_fmaf(o0[0], __uint_as_float(dv[0] << 16), s[0]);
        s[1] = __builtin_fmaf(o0[1], __uint_as_float(dv[0] & 0xFFFF0000u), s[1]);
        s[2] = __builtin_fmaf(o0[2], __uint_as_float(dv[1] << 16), s[2]);
        s[3] = __builtin_fmaf(o0[3], __uint_as_float(dv[1] & 0xFFFF0000u), s[3]);
        s[0] = __builtin_fmaf(o1[0], __uint_as_float(dv[2] << 16), s[0]);
        s[1] = __builtin_fmaf(o1[1], __uint_as_float(dv[2] & 0xFFFF0000u), s[1]);
        s[2] = __builtin_fmaf(o1[2], __uint_as_float(dv[3] << 16), s[2]);
        s[3] = __builtin_fmaf(o1[3], __uint_as_float(dv[3] & 0xFFFF0000u), s[3]);
      };
      if (a.O32 != nullptr) {
        f32x4 o[2 * KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          o[2 * ks] = *reinterpret_cast<const f32x4*>(a.O32 + at + 16 * ks);
          o[2 * ks + 1] = *reinterpret_cast<const f32x4*>(a.O32 + at + 16 * ks + 4);
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) add(ks, o[2 * ks], o[2 * ks + 1]);
      } else {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const u32x4 ob = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(a.O) + at + 16 * ks);
          add(ks, (f32x4){__uint_as_float(ob[0] << 16), __uint_as_float(ob[0] & 0xFFFF0000u), __uint_as_float(ob[1] << 16), __uint_as_float(ob[1] & 0xFFFF0000u)},
              (f32x4){__uint_as_float(ob[2] << 16), __uint_as_float(ob[2] & 0xFFFF0000u), __uint_as_float(ob[3] << 16), __uint_as_float(ob[3] & 0xFFFF0000u)});
        }
      }
      del_r = (s[0] + s[1]) + (s[2] + s[3]);
      del_r += __shfl_xor(del_r, 32);
      if (h == 0 && grp == 0 && r_in_tile < w.rows_valid) a.delta_out[(int64_t)w.bh * g.n + r_row] = del_r;
    }
  }

  asm volatile("" : "+v"(nl2_r), "+v"(del_r));
  if (ntiles > 0) {
    if (kHits) find_sample_hits<kBNT>(a, b, sample_hits(smem + bwd_hits_at<D, NG>(a, MODE)), shead);  // while the first tile is on its way
    finish_tile(0);
  }

  for (int kt = 0; kt < ntiles; ++kt) {
    const bool more = kt + 1 < ntiles;
    if (more) request_tile(kt + 1);

    const unsigned char* yb = bufs + (kt & 1) * L::BUF;
    const unsigned char* bb = yb + L::TILE;
    const float* scb = sc + (kt & 1) * (2 * kTT);

    // ---- P^T and dS^T ----
    // Masks as limits on the in-tile row offset ko = koff - 4 h of an accumulator element
    // (koff = 32 sub + 8 (i / 4) + 4 h + i % 4): masked iff ko >= hi2 (end of the T rows; keys
    // after the query), ko < lo2 (queries before the key) or mlo2 <= ko < mhi2 (queries of
    // the sampled key's own block, factor 1 - M of Algorithm 2).
    // Whether the tile has any is known from scalars, except in the sampled-key pass, whose keys differ by lane;
    // the limits themselves are formed inside the branch, so that they hold no registers across the products.
    const int tbase = (NG * kt + grp) * kTT;
    float nl2_t = nl2_r;
    if (MODE == kBwdDqNode && tbase >= nb) nl2_t += bias2;
    const int r_first = w.q0 + 32 * wave_s;   // exact passes: the wave's first R row
    bool special = tbase + kTT > nT;
    if (MODE == kBwdDqNode) special = special || (tbase < nb && tbase + kTT > nb);
    if (MODE == kBwdDqExact && f.exact_causal) special = special || (w.k0 + tbase + kTT - 1 > r_first);
    if (MODE == kBwdDkvExact && f.exact_causal) special = special || (w.k0 + tbase < r_first + 31);
    if (MODE == kBwdDkvSamp) {
      const int mlo = blk_r * g.b - (b.chunk_start + tbase);
      special = special || __any(mlo < kTT && mlo + g.b > 0);
    }

    // one 32-row half of the tile at a time: S^T = Y X^T and dP^T = Bt A^T, then P^T / dS^T
    if (NG == 1 || tbase < nT)
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      // dK / dV passes start the sums at bias - L and -delta of the T rows, straight from LDS; in the dQ passes,
      // where these belong to the lane, they enter with the exponential and the product below
      f32x16 cs, es;
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        f32x4 l4 = {0.f, 0.f, 0.f, 0.f}, d4 = l4;
        if (!kDq) {
          l4 = *reinterpret_cast<const f32x4*>(scb + 32 * sub + 8 * i4 + 4 * h);
          d4 = *reinterpret_cast<const f32x4*>(scb + kTT + 32 * sub + 8 * i4 + 4 * h);
        }
#pragma unroll
        for (int z = 0; z < 4; ++z) {
          cs[4 * i4 + z] = l4[z];
          es[4 * i4 + z] = d4[z];
        }
      }
      // the wave holds issue priority over its SIMD neighbour while it issues its S^T / dP^T products
      constexpr bool kPrio = kExact || MODE == kBwdDkvSamp;
      if constexpr (kPrio) __builtin_amdgcn_s_setprio(1);
      // the eight addresses are formed where they are used: kept across the loop they would cost eight registers
      int rr = rd_row;
      asm volatile("" : "+v"(rr));
      // Fragment q of the half is piece q / 2 of the Y tile (even q) or the Bt tile (odd q).  The order is written
      // out and pinned: kPre fragments are read ahead and every product is followed by one more read; left to
      // itself the compiler keeps one fragment register and waits for every read in full.
      auto row_frag = [&](int q) {
        return *reinterpret_cast<const bf16x8*>((q & 1 ? bb : yb) + (rr ^ (32 * (q >> 1))) + sub * 32 * L::ROWB);
      };
      constexpr int kPre = (D == 128 && !kDq) ? 3 : 4;
      bf16x8 fr[kPre];
#pragma unroll
      for (int q = 0; q < kPre; ++q) fr[q] = row_frag(q);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < 2 * KS; ++q) {
        if (q & 1) es = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[q % kPre], areg[q >> 1], es, 0, 0, 0);
        else cs = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[q % kPre], xreg[q >> 1], cs, 0, 0, 0);
        if (q + kPre < 2 * KS) fr[q % kPre] = row_frag(q + kPre);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (kPrio) __builtin_amdgcn_s_setprio(0);
      if (special) {  // rare tiles, behind a branch: folded into the weights' code the tests would double it
        int hi2 = nT - tbase - 4 * h, lo2 = 0;
        if (MODE == kBwdDqExact && f.exact_causal) hi2 = min(hi2, r_row - w.k0 - tbase + 1 - 4 * h);
        if (MODE == kBwdDkvExact && f.exact_causal) lo2 = r_row - w.k0 - tbase - 4 * h;
        const int mlo2 = blk_r * g.b - (b.chunk_start + tbase) - 4 * h;
        const int nb2 = (tbase < nb ? nb : 0x40000000) - tbase - 4 * h;  // a tile past nb has its bias already
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int ko = 32 * sub + 8 * (i / 4) + (i % 4);
          if (MODE == kBwdDqNode && ko >= nb2) cs[i] += nat_bias;
          bool msk = ko >= hi2;
          if (MODE == kBwdDkvExact) msk = msk || (ko < lo2);
          if (MODE == kBwdDkvSamp) msk = msk || ((unsigned)(ko - mlo2) < (unsigned)g.b);
          if (msk) cs[i] = -INFINITY;
        }
      }
      // weights of elements 2 e, 2 e + 1, as bf16: the B operands of the accumulating products
      uint32_t pw[8], dw[8];
      auto weights = [&](int e) {
        float pv[2], dv[2];
#pragma unroll
        for (int z = 0; z < 2; ++z) {
          const int i = 2 * e + z;
          pv[z] = __builtin_amdgcn_exp2f(kDq ? __builtin_fmaf(cs[i], kLog2e, nl2_t) : cs[i] * kLog2e);
          dv[z] = pv[z] * (kDq ? es[i] - del_r : es[i]);
        }
        if (!kDq) pw[e] = pack_bf16x2(pv[0], pv[1]);
        dw[e] = pack_bf16x2(dv[0], dv[1]);
      };
      // ---- acc1^T += Y^T dS^T and acc2^T += Bt^T P^T for the 32 rows of this half ----
      typedef short s16x4 __attribute__((ext_vector_type(4)));
      typedef short s16x8 __attribute__((ext_vector_type(8)));
      typedef s16x4 __attribute__((address_space(3))) * lds_s16x4_ptr;
      int rc = rd_col;
      asm volatile("" : "+v"(rc));
      auto column_frag = [&](const unsigned char* tile, int j, int dt) {
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(tile + (rc ^ (64 * dt)) + 16 * j * L::ROWB));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(tile + (rc ^ (64 * dt + 32)) + (16 * j + 8) * L::ROWB));
        return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      };
      // Product q accumulates column tile dt of jj, the 16-row step of the half; again the order is pinned: weights of the first
      // step, kPreC fragments, then per product the next fragment and, during the first step's products, a
      // slice of the second step's weights.
      constexpr int kPer = kDq ? DT : 2 * DT;    // products per step
      constexpr int kAcc = 2 * kPer;
      constexpr int kPreC = (D == 128 && !kDq) ? 3 : 4;
      auto col_frag = [&](int q) {
        const int jj = q / kPer, u = q % kPer;
        return kDq ? column_frag(yb, 2 * sub + jj, u) : column_frag(u & 1 ? yb : bb, 2 * sub + jj, u >> 1);
      };
      bf16x8 fc[kPreC];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (e == (D == 128 && !kDq ? 2 : 0)) {
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int q = 0; q < kPreC; ++q) fc[q] = col_frag(q);
        }
        weights(e);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < kAcc; ++q) {
        const int jj = q / kPer, u = q % kPer;
        const bf16x8 df = __builtin_bit_cast(bf16x8, (u32x4){dw[4 * jj], dw[4 * jj + 1], dw[4 * jj + 2], dw[4 * jj + 3]});
        if constexpr (kDq) {
          acc1[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fc[q % kPreC], df, acc1[u], 0, 0, 0);
        } else {
          const bf16x8 pf = __builtin_bit_cast(bf16x8, (u32x4){pw[4 * jj], pw[4 * jj + 1], pw[4 * jj + 2], pw[4 * jj + 3]});
          if (u & 1) acc1[u >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fc[q % kPreC], df, acc1[u >> 1], 0, 0, 0);
          else acc2[u >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fc[q % kPreC], pf, acc2[u >> 1], 0, 0, 0);
        }
        if (q + kPreC == kPer) asm volatile("" : "+v"(rc));  // the second step forms its addresses anew, as above
        if (q + kPreC < kAcc) fc[q % kPreC] = col_frag(q + kPreC);
        if (q < kPer) {
#pragma unroll
          for (int e = 4 + 4 * q / kPer; e < 4 + 4 * (q + 1) / kPer; ++e) weights(e);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (more) finish_tile(kt + 1);
  }
  __syncthreads();  // the tiles are read no more

  auto staged = [&]() {  // a wave's own staging area, or both groups'
    if (NG == 2) {
      __syncthreads();
      return;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  auto write_out = [&](const auto& acc, float* dst32, const float* samp, uint16_t* dst16, const float* lvl) {
    // ---- epilogue: the wave's 32 rows leave through an LDS transpose as whole rows.
    // Node passes write or add fp32 rows into the accumulated rows (unmasked problems: write the final gradient).
    // Exact passes (the base case of Algorithm 4) write the final gradient in the tensors' dtype, after
    // adding the accumulated row where some level's node holds the row on the pass's
    // side (queries: second half of the node; keys: first half).
    // Two groups: both stage their sums of the rows; each takes half of the rows on and adds the two.
    // No later workgroup of the launch reads a row that it reads or writes here: non-temporal, they leave the caches to the tiles
    // (not the samples' rows, which the next launch reads: 2 heads, n = 4096, d = 64 31.0 -> 31.8 us).  Backward (MI355X, us): 12 heads, n =
    // 16384, d = 128 279.0 -> 266.7, 32 heads, n = 32768 1267 -> 1254, d = 64 673 -> 668; 8 causal heads, n = 32768, d = 128 1577 -> 1561,
    // 32, n = 65536 13460 -> 13360, d = 64 6984 -> 6943; exact passes +-0.3 %.  The accumulated rows that the exact passes fold
    // in: read so, 0.5 % slower.
    unsigned char* ep = smem + wave * L::EP_WAVE;
    unsigned char* ep_own = ep + 4 * grp * L::EP_WAVE;
    int64_t* ep_rows = reinterpret_cast<int64_t*>(ep_own + 32 * L::EP_ROW);
    if (h == 0) {  // (the row's index is fetched again: kept across the loop it would cost registers)
      int r = wave * 32 + lq, blk;
      asm volatile("" : "+v"(r));
      ep_rows[lq] = r < w.rows_valid ? bwd_out_row<MODE>(a, b, r, bwd_r_row<MODE>(a, b, r, &blk)) : (int64_t)-1;
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const int col = 32 * dt + 8 * g4 + 4 * h;
        const f32x4 v = {acc[dt][4 * g4], acc[dt][4 * g4 + 1], acc[dt][4 * g4 + 2], acc[dt][4 * g4 + 3]};
        *reinterpret_cast<f32x4*>(ep_own + lq * L::EP_ROW + col * 4) = v;
      }
    staged();
    const int row0 = NG == 2 ? 16 * grp : 0;  // this wave's first row of the 32
    auto sums_at = [&](int row, int byte) -> f32x4 {
      f32x4 v = *reinterpret_cast<const f32x4*>(ep + row * L::EP_ROW + byte);
      if (NG == 2) v += *reinterpret_cast<const f32x4*>(ep + 4 * L::EP_WAVE + row * L::EP_ROW + byte);
      return v;
    };
    // Rows that are not stored (past the end of the tile; valid rows are a prefix) re-read the wave's first
    // row, so that every load below is unconditional and all of them are requested before the first is
    // used; only the stores sit under a branch.  With loads under a branch the compiler's wait counts
    // fall back to "everything", and each piece would also wait for the previous piece's stores.
    const int64_t row_first = ep_rows[0];
    if (row_first < 0) return;
    // sums of the wave's sampled keys: requested together with the rows' earlier sums below; the further
    // draws of a row are added here, by the lanes of its group (a quarter or half of the wave per row)
    const float* sums = nullptr;  // null: no sampled key in the wave's rows
    const int32_t* first = nullptr;
    if (kHits && samp != nullptr) {
      const SampleHits sh = sample_hits(smem + bwd_hits_at<D, NG>(a, MODE));
      first = sh.first + 32 * wave;
      if (__any(first[lq] != kNoSample)) sums = samp + (int64_t)w.bh * bwd_chunks_per_node(g, a.chunk, 0) * g.m * D;
      const int nm = sums ? *sh.count : 0;
      constexpr int LPR = D / 4, G = 64 / LPR;
      for (int e = 0; e < nm; ++e) {
        const int row = sh.more[e] >> 16;
        if ((row >> 5) != wave || (row & (G - 1)) != lane / LPR) continue;
        f32x4* at = reinterpret_cast<f32x4*>(ep + (row & 31) * L::EP_ROW + (lane % LPR) * 16);
        *at = *at + *reinterpret_cast<const f32x4*>(sums + (int64_t)(sh.more[e] & 0xffff) * D + (lane % LPR) * 4);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    if (!kExact && !FINAL) {
      // node passes add to what earlier levels left in the row; all rows of a node lie on the same side of
      // every ancestor, so the whole workgroup either adds or writes
      bool add = false;
      if (MODE == kBwdDqNode) add = node_levels_hold(g, w.nr.q_start, true, w.level);
      if (MODE == kBwdDkvBlock) add = node_levels_hold(g, w.nr.k_start, false, w.level);
      constexpr int CH = D / 4;            // 16-byte pieces per fp32 row
      constexpr int IT = 32 * CH / 64;     // pieces per lane
      int64_t r64[IT];
      f32x4 prev[IT];
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int idx = lane + 64 * it;
        r64[it] = ep_rows[idx / CH];
        prev[it] = (f32x4){0.f, 0.f, 0.f, 0.f};
      }
      if (add) {
#pragma unroll
        for (int it = 0; it < IT; ++it) {
          const int ch = (lane + 64 * it) % CH;
          const int64_t rr = r64[it] >= 0 ? r64[it] : row_first;
          prev[it] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(dst32 + rr * D + ch * 4));
        }
      }
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        const int idx = lane + 64 * it;
        const int row = idx / CH, ch = idx % CH;
        const f32x4 v = *reinterpret_cast<const f32x4*>(ep + row * L::EP_ROW + ch * 16) + prev[it];
        if (r64[it] < 0) continue;
        f32x4* to = reinterpret_cast<f32x4*>(dst32 + r64[it] * D + ch * 4);
        if (MODE == kBwdDkvSamp) *to = v;  // (read again by the launch that adds the samples' sums)
        else __builtin_nontemporal_store(v, to);
      }
      return;
    }
    // the 32 rows of a wave lie in one n_min block: the node passes hold all of them or none
    const int i0 = w.q0 + 32 * __builtin_amdgcn_readfirstlane(wave);
    const bool fold = kExact && lvl != nullptr && node_levels_hold(g, i0, kDq, g.levels);
    const float* acc_rows = lvl + ((int64_t)w.bh * g.n + i0) * D;
    constexpr int CH8 = D / 8;             // 8-element pieces per row
    constexpr int IT8 = 32 / NG * CH8 / 64;  // pieces per lane
    int64_t r64[IT8];
    f32x4 p0[IT8], p1[IT8];
#pragma unroll
    for (int it = 0; it < IT8; ++it) {
      r64[it] = ep_rows[row0 + (lane + 64 * it) / CH8];
      p0[it] = (f32x4){0.f, 0.f, 0.f, 0.f};
      p1[it] = p0[it];
    }
    if (fold) {
#pragma unroll
      for (int it = 0; it < IT8; ++it) {
        const int idx = lane + 64 * it;
        const int row = r64[it] >= 0 ? row0 + idx / CH8 : 0, ch = idx % CH8;
        const float* pp = acc_rows + (int64_t)row * D + ch * 8;
        p0[it] = *reinterpret_cast<const f32x4*>(pp);
        p1[it] = *reinterpret_cast<const f32x4*>(pp + 4);
      }
    }
    if (kHits && sums != nullptr) {  // (a row without a sample reads sample 0's sums and drops them)
#pragma unroll
      for (int it = 0; it < IT8; ++it) {
        const int idx = lane + 64 * it, j = first[idx / CH8];
        const float* pp = sums + (int64_t)(j != kNoSample ? j : 0) * D + (idx % CH8) * 8;
        p0[it] = *reinterpret_cast<const f32x4*>(pp);
        p1[it] = *reinterpret_cast<const f32x4*>(pp + 4);
      }
#pragma unroll
      for (int it = 0; it < IT8; ++it) {
        const bool none = first[(lane + 64 * it) / CH8] == kNoSample;
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        p0[it] = none ? zero : p0[it];
        p1[it] = none ? zero : p1[it];
      }
    }
#pragma unroll
    for (int it = 0; it < IT8; ++it) {
      const int idx = lane + 64 * it;
      const int row = row0 + idx / CH8, ch = idx % CH8;
      const f32x4 v0 = sums_at(row, ch * 32) + p0[it];
      const f32x4 v1 = sums_at(row, ch * 32 + 16) + p1[it];
      const u32x4 pk = {pack_bf16x2(v0.x, v0.y), pack_bf16x2(v0.z, v0.w), pack_bf16x2(v1.x, v1.y), pack_bf16x2(v1.z, v1.w)};
      if (r64[it] >= 0) __builtin_nontemporal_store(pk, reinterpret_cast<u32x4*>(dst16 + r64[it] * D + ch * 8));
    }
  };
  write_out(acc1, a.out1, a.samp1, reinterpret_cast<uint16_t*>(a.fin1), a.lvl1);
  if constexpr (!kDq) {
    staged();  // (one group: a wave rewrites only its own staging area, which its own reads above have left)
    write_out(acc2, a.out2, a.samp2, reinterpret_cast<uint16_t*>(a.fin2), a.lvl2);
  }
}

template <int D, int MODE, bool FINAL, int NG, bool FOUR = false>
static int launch_bwd_form(const BwdArgs& args, int grid, hipStream_t st) {
  BwdArgs a = args;
  if (MODE == kBwdDqNode || MODE == kBwdDkvBlock) set_node_divs<kRT>(a.f);
  if (MODE == kBwdDqExact || MODE == kBwdDkvExact) set_exact_divs<kRT>(a.f);
  a.f.exact_lpt = NG == 2;
  const size_t lds = bwd_lds_bytes<D, NG>(a, MODE);
  static std::atomic<uint64_t> lds_set{0};  // per instantiation: devices on which the LDS limit is raised
  if (allow_full_lds(reinterpret_cast<const void*>(&attn_bwd_kernel<D, MODE, FINAL, NG, FOUR>), lds_set) != HA_OK) return HA_ERR_LAUNCH;
  hipLaunchKernelGGL((attn_bwd_kernel<D, MODE, FINAL, NG, FOUR>), dim3((unsigned)grid), dim3(kBNT * NG), lds, st, a);
  return check_launch();
}

// Exact passes of few workgroups are bound by the longest chain of T tiles of one of them, as in the forward (split_exact,
// attn_mfma.hip): two groups of four waves then share it, a workgroup that fills a CU.  Up to one round of those unmasked, up
// to two in causal launches, whose second round's are the lightest.  Forward + backward of exact attention, one group -> two
// in the backward's passes (MI355X, us; in brackets the workgroups of a pass):
//   causal, d = 64: 8 heads, n = 8192 (512) 399 -> 359, 9 heads (576) 446 -> 437, 10 (640) 478 -> 487; 16 heads, n = 4096 (512) 215 ->
//     196, 18 (576) 240 -> 243; 32 heads, n = 2048 (512) 122 -> 116, 36 (576) 134 -> 141; 37 heads, n = 1536 (444) 97.1 -> 94.3, 43 (516)
//     103 -> 112; 48 heads, n = 1024 (384) 71.4 -> 69.0, 56 (448) 72.7 -> 75.7; 64 heads, n = 640 (320) 54.8 -> 51.8, 77 (385) 57.3 -> 61.1
//   causal, d = 128: 8 heads, n = 8192 (512) 656 -> 605, 9 (576) 738 -> 733, 10 (640) 791 -> 811; 12 heads, n = 4096 (384) 318 -> 287, 16
//     (512) 352 -> 328, 18 (576) 393 -> 402; 32 heads, n = 2048 (512) 198 -> 190, 36 (576) 219 -> 232; 48 heads, n = 1024 (384) 108 -> 106;
//     64 heads, n = 512 (256) 65.5 -> 62.9, 96 (384) 75.3 -> 82.4
//   unmasked, n = 8192: 4 heads (256) d = 64 362 -> 336, d = 128 601 -> 569, 5 heads (320) 540 -> 587, 888 -> 937; 51 heads, n = 640
//     (255): d = 64 50.2 -> 48.6, d = 128 77.8 -> 79.3; 64 heads, n = 384 (192): 36.9 -> 36.6, 55.0 -> 55.3
// Errors against 64 bits, forward and backward of one group each -> of two (12 causal heads, n = 5000, d = 128): dQ 2.387e-3 -> 2.386e-3, dK
// 2.364e-3 -> 2.365e-3, dV 2.306e-3 both.
constexpr int kSplitBwdMinRows = 512;
static bool split_bwd_exact(const BwdArgs& a, int grid) {
  const int rows = a.f.exact_block < a.f.exact_rows_q ? a.f.exact_block : a.f.exact_rows_q;
  if (rows < kSplitBwdMinRows) return false;
  if (!a.f.exact_causal) return grid <= (a.f.g.d == 128 && rows < 1024 ? 160 : 256);
  return grid <= (rows < 1024 ? 320 : rows < 1536 ? 384 : rows < 2048 ? 448 : 512);
}

// dQ of exact attention at d = 64 takes 135 registers by itself, three workgroups per CU; at 128, with 16 bytes of scratch per lane, a
// fourth fits.  It pays from the 769th workgroup on, where three per CU need a second round.  Forward + backward, three -> four (MI355X, us;
// workgroups of the pass): causal, 96 heads, n = 1024 (768) 93.7 -> 94.2, 128 (1024) 128.6 -> 124.1; 120 heads, n = 700 (720) 72.8 -> 73.2; 200 heads,
// n = 600 (1000) 103.4 -> 99.7; 48 heads, n = 2048 (768) 153.3 -> 153.0, 64 (1024) 198.4 -> 196.6; 32 heads, n = 4096 (1024) 346.7 -> 340.4; 16
// heads, n = 8192 (1024) 648.0 -> 635.8, 24 (1536) 934.0 -> 927.4; 8 heads, n = 16384 (1024) 1272 -> 1243; unmasked, 128 heads, n = 1024 (1024) 185.8 -> 185.7,
// 16 heads, n = 8192 (1024) 1221 -> 1210; causal HyperAttention, 32 heads, n = 65536 9519 -> 9461.  The same of the nodes' dQ pass, 20 bytes of
// scratch, loses (12 heads, n = 16384 215 -> 220; n = 32768 425 -> 442).
static bool bwd_four_workgroups(int grid) { return grid > 768; }

template <int D, int MODE>
static int launch_bwd_one(const BwdArgs& a, int grid, hipStream_t st) {
  if (grid <= 0) return HA_OK;
  if constexpr (MODE == kBwdDqExact || MODE == kBwdDkvExact)
    if (split_bwd_exact(a, grid)) return launch_bwd_form<D, MODE, false, 2>(a, grid, st);
  if constexpr (D == 64 && MODE == kBwdDqExact)
    if (bwd_four_workgroups(grid)) return launch_bwd_form<D, MODE, false, 1, true>(a, grid, st);
  if constexpr (MODE == kBwdDqNode || MODE == kBwdDkvBlock)
    if (!a.f.g.causal) return launch_bwd_form<D, MODE, true, 1>(a, grid, st);
  return launch_bwd_form<D, MODE, false, 1>(a, grid, st);
}

template <int D>
static int launch_bwd_d(const BwdArgs& a, int mode, int grid, hipStream_t st) {
  switch (mode) {
    case kBwdDqNode: return launch_bwd_one<D, kBwdDqNode>(a, grid, st);
    case kBwdDqExact: return launch_bwd_one<D, kBwdDqExact>(a, grid, st);
    case kBwdDkvBlock: return launch_bwd_one<D, kBwdDkvBlock>(a, grid, st);
    case kBwdDkvSamp: return launch_bwd_one<D, kBwdDkvSamp>(a, grid, st);
    case kBwdDkvExact: return launch_bwd_one<D, kBwdDkvExact>(a, grid, st);
    default: return HA_ERR_SHAPE;
  }
}

int launch_attn_bwd_mfma(const BwdArgs& a, int mode, hipStream_t st) {
  if (a.f.g.dtype != HA_BF16) return HA_ERR_DTYPE;
  const int64_t grid64 = bwd_grid<kRT>(a, mode);
  if (grid64 > kMaxGrid) return HA_ERR_SHAPE;
  const int grid = (int)grid64;
  if (a.f.g.d == 128) return launch_bwd_d<128>(a, mode, grid, st);
  if (a.f.g.d == 64) return launch_bwd_d<64>(a, mode, grid, st);
  return HA_ERR_SHAPE;
}

}  // namespace ha
