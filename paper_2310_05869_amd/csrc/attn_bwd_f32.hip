// Backward pass of HA_FP32 tensors, with the same passes and the same buffers as the bf16 backward kernel, so that the host sequence is
// one and the same.  Its products run on the bf16 matrix cores, every operand split in three (split_f32.h).
//
// As there, a row of the forward is one softmax over its block keys, its kept sampled keys (weight
// s/m) and, when causal, the keys of its base-case block (Algorithms 1, 2, 4), and with the final
// log row sum L_i and delta_i = <dO_i, O_i> every (query, key) pair contributes on its own:
//   P_ij = w_ij exp(<q_i, k_j> - L_i),  dV_j += P_ij dO_i,  dS_ij = P_ij (<dO_i, v_j> - delta_i),
//   dQ_i += dS_ij k_j,  dK_j += dS_ij q_i.
//
// A wave owns 32 "R rows" (queries in the dQ passes, keys in the dK / dV passes) and their accumulators.  The "T rows" (keys, resp.
// queries) come in tiles of 32, row-major for the scores and dP and transposed for the accumulating products (attn_f32.hip has
// the layouts).  The dK / dV passes form S and dP once and accumulate both gradients: 4 products, 3 in the dQ passes.  The scores are formed
// as the forward forms them, step by step (P = exp(S - L) then cancels their rounding where scores are large: with the columns of d in
// another order than the forward's, 64 clusters, scores to 250, dQ's error was 7.3e-5 instead of 1.2e-5).
//
// KW ways share a group of R rows, each taking every KW-th tile; their sums are added through LDS in
// order, so results are bit-reproducible.  KW = 1: four waves of different R rows share the tiles, split once into LDS.  KW = 4 or 8: one group of
// 32 R rows per workgroup, which lie split in LDS; a wave's T rows come straight from the caches in operand layout and are split in
// registers, B's in the dK / dV passes twice (as rows and in columns); the split rows of Y go to a tile of the wave's own for the product
// that takes them in columns (24 KB with R, 12 KB a wave: both tensors' tiles would leave a CU one workgroup).  Fetched and split twice as
// well (backward, MI355X, us): causal, 4 heads, n = 4096 in blocks of 1024, b = m = 64 116 -> 108, d = 128 248 -> 235; exact, causal, 8 heads, n = 4096 482 ->
// 457, 1012 -> 951, one head, n = 1024 60.0 -> 56.0, 119 -> 112; 8 heads, n = 4096, b = m = 256 152 -> 142.
//
// What bounds it: in large launches the matrix pipe at the clock that the chip's power leaves it (32 heads, n = 8192, d = 64: the seven products
// of a pair at 1120 TFLOP/s of bf16 products); in small ones (4 heads, n = 4096 in causal blocks of 1024, base case with the sampled keys, 1152
// workgroups) vector issue, half of the cycles, the splits being about half of it, and workgroups of unequal length (matrix pipe 32 %; 1.4 waves
// per SIMD of two).  The dK / dV passes of one way spill 176 to 204 bytes per lane at d = 64, 100 to 180 at d = 128, mostly outside the first
// run's loop; with more ways up to 28.
// Measured (MI355X, us; fp32 matrix instructions, T rows always from the caches -> this form), backward of exact attention: 32 heads,
// n = 8192, d = 64 14850 -> 10340, 16 heads, d = 128 16010 -> 10650; causal, 16 heads, n = 1024 91.1 -> 71.2, d = 128 204 -> 166; 8 heads, n = 4096 550 -> 419,
// 1120 -> 913; one head, n = 1024 77.4 -> 53.5, 138 -> 109; of HyperAttention: one head, n = 1024, b = m = 64 45.8 -> 36.9, 8 heads, n = 4096, b = m = 256
// 190 -> 138, d = 128 391 -> 258; causal, 4 heads, n = 4096 in blocks of 1024, b = m = 64 150 -> 106, 278 -> 235.
#include <type_traits>

#include "attn_common.h"
#include "bwd_common.h"
#include "split_f32.h"

namespace ha {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kFTT = 32;   // T rows per tile

// LDS: the ways' tiles (Y and B) and L and delta of their rows, or, RG = 1, the R rows; the key list of a node's dQ pass; in the end the
// staged rows, over the tiles; behind all else a word per wave (SplitFinite) and the sampled keys of a block-key pass.
// (RG = 1: whether a wave keeps the split rows of its Y tile for the accumulating products; the lists of a d = 128 node leave no room,
// nor do 4096 sampled keys of an unmasked problem's block keys)
constexpr bool f32_bwd_keeps_y(int d, int mode, bool causal) {
  return d == 64 || (mode != kBwdDqNode && (mode != kBwdDkvBlock || causal));
}

template <int D, int RG, int KW>
struct F32BwdLds {
  static constexpr int WAY = 2 * SplitTile<D>::BYTES;  // bytes of a way's tiles
  static constexpr int SC_AT = (RG > 1 ? KW : 1) * WAY;
  static constexpr int OWN_AT = SC_AT + (RG > 1 ? KW * 2 * kFTT * 4 : 0);  // RG = 1: the waves' Y tiles
  __host__ __device__ static constexpr int list_at(int mode, bool causal) {
    return OWN_AT + (RG == 1 && f32_bwd_keeps_y(D, mode, causal) ? KW * SplitTile<D>::BYTES : 0);
  }
  static constexpr int ROW = D + 4;  // floats per staged row
  static constexpr int ROWS = RG * KW * 32 * ROW * 4;
  __host__ __device__ static size_t finite_at(const Geometry& g, int mode) {
    const size_t list = mode == kBwdDqNode ? (size_t)(((g.b + g.m + 63) & ~63) + 64) * 4 + 64 : 0;
    const size_t end = list_at(mode, g.causal) + list;
    return end > (size_t)ROWS ? end : (size_t)ROWS;
  }
  __host__ __device__ static size_t hits_at(const Geometry& g, int mode) { return finite_at(g, mode) + SplitFinite<RG * KW>::BYTES; }
  __host__ __device__ static size_t bytes(const Geometry& g, int mode) {
    return hits_at(g, mode) + (mode == kBwdDkvBlock && !g.causal ? sample_hits_bytes(g) : 0);
  }
};

// RG waves, of 32 R rows each, share the T tiles of a way; the KW ways take every KW-th tile.  RG = 1: a wave's tiles are its own
// and come straight from the caches in operand layout, each row twice (as a row and in columns), and the KW waves share the R rows.
// FINAL: the node passes of an unmasked problem, which write the final gradients.
// wg: the workgroup's number among the pass's wgs.
template <int D, int MODE, int RG, int KW, bool FINAL>
__device__ __forceinline__ void bwd_f32_pass(const BwdArgs& a, const int wg, const int wgs, unsigned char* smem) {
  constexpr bool kDq = (MODE == kBwdDqNode || MODE == kBwdDqExact);
  constexpr bool kExact = (MODE == kBwdDqExact || MODE == kBwdDkvExact);
  constexpr bool kSorted = (MODE == kBwdDkvBlock || MODE == kBwdDkvSamp);
  constexpr bool kHits = FINAL && MODE == kBwdDkvBlock;  // sampled keys' sums added here
  constexpr int NW = RG * KW, kFBT = 64 * NW;
  constexpr int kRT = 32 * RG;
  constexpr int KS = D / 16;  // steps of a score's product
  constexpr int DT = D / 32;
  using L = F32BwdLds<D, RG, KW>;
  using T = SplitTile<D>;
  const AttnArgs& f = a.f;
  const Geometry& g = f.g;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, h = lane >> 5;
  const int grp = wave % RG, kw = wave / RG;
  const int wtid = tid % (64 * RG);  // within the way
  constexpr bool kShared = RG > 1, kKeepY = !kShared && f32_bwd_keeps_y(D, MODE, !FINAL);
  unsigned char* ytile = smem + (kShared ? kw * L::WAY : 0);
  unsigned char* btile = ytile + T::BYTES;
  unsigned char* own_y = smem + L::OWN_AT + (kKeepY ? wave * T::BYTES : 0);
  float* sc = reinterpret_cast<float*>(smem + L::SC_AT) + kw * 2 * kFTT;
  int32_t* scratch = reinterpret_cast<int32_t*>(smem + L::list_at(MODE, !FINAL));
  int32_t* list = scratch + 16;

  // ---- which part of the problem this workgroup owns ----
  BwdWork b = decode_bwd_work<kRT, MODE>(a, kExact ? wg : logical_block(wg, wgs), wgs);
  const TileWork& w = b.w;

  const int64_t hs = f.q_bh_stride;
  const float* Qh = reinterpret_cast<const float*>(f.Q) + (int64_t)w.bh * hs;
  const float* Kh = reinterpret_cast<const float*>(f.K) + (int64_t)w.bh * hs;
  const float* Vh = reinterpret_cast<const float*>(f.V) + (int64_t)w.bh * hs;
  const float* Gh = reinterpret_cast<const float*>(a.dO) + (int64_t)w.bh * hs;
  const float* lse_h = a.lse + (int64_t)w.bh * g.n;
  const float* del_h = a.delta + (int64_t)w.bh * g.n;
  const float* Xh = kDq ? Qh : Kh;   // R rows: operand of the scores
  const float* Ah = kDq ? Gh : Vh;   // R rows: operand of dP
  const float* Yh = kDq ? Kh : Qh;   // T rows: operand of the scores and of dQ / dK
  const float* Bh = kDq ? Vh : Gh;   // T rows: operand of dP and of dV

  // ---- this lane's R row ----
  const int r_in_tile = grp * 32 + lq;
  const int r_use = r_in_tile < w.rows_valid ? r_in_tile : 0;
  int blk_r = -1;
  const int r_row = bwd_r_row<MODE>(a, b, r_use, &blk_r);
  Split8 xs[kShared ? KS : 1], as[kShared ? KS : 1];
  float L_r = 0.f, del_r = 0.f;
  auto load_r = [&](f32x4 (&av)[2 * KS]) {  // columns 16 s + 8 h ... + 7 of step s
    f32x4 x[2 * KS];
#pragma unroll
    for (int j = 0; j < 2 * KS; ++j) {
      const int64_t at = (int64_t)r_row * D + 16 * (j / 2) + 8 * h + 4 * (j % 2);
      if (kShared) x[j] = *reinterpret_cast<const f32x4*>(Xh + at);
      av[j] = *reinterpret_cast<const f32x4*>(Ah + at);
    }
    if constexpr (kShared) {
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        xs[s] = split8_raw([&](int e) { return x[2 * s + e / 4][e % 4]; });
        as[s] = split8_raw([&](int e) { return av[2 * s + e / 4][e % 4]; });
      }
    }
  };
  {
    f32x4 av[2 * KS];
    if (kShared || (kDq && a.delta_out != nullptr)) load_r(av);
    if constexpr (!kShared) {
      for (int i = tid; i < 32 * T::PPR; i += kFBT) {
        const int r = i / T::PPR, piece = i % T::PPR;
        int blk;
        const int64_t at = (int64_t)bwd_r_row<MODE>(a, b, r < w.rows_valid ? r : 0, &blk) * D + piece * 8;
        const f32x4 x0 = *reinterpret_cast<const f32x4*>(Xh + at), x1 = *reinterpret_cast<const f32x4*>(Xh + at + 4);
        const f32x4 a0 = *reinterpret_cast<const f32x4*>(Ah + at), a1 = *reinterpret_cast<const f32x4*>(Ah + at + 4);
        T::store(ytile, r, piece, x0, x1);
        T::store(btile, r, piece, a0, a1);
      }
    }
    if (kDq) {
      L_r = lse_h[r_row];
      if (a.delta_out == nullptr) {
        del_r = del_h[r_row];
      } else {
        const float* Oh = reinterpret_cast<const float*>(a.O) + ((int64_t)w.bh * g.n + r_row) * D + 8 * h;
        f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 2 * KS; ++j) {
          const f32x4 o = *reinterpret_cast<const f32x4*>(Oh + 16 * (j / 2) + 4 * (j % 2));
#pragma unroll
          for (int z = 0; z < 4; ++z) s[z] = __builtin_fmaf(o[z], av[j][z], s[z]);
        }
        del_r = (s[0] + s[1]) + (s[2] + s[3]);
        del_r += __shfl_xor(del_r, 32);
        if (h == 0 && kw == 0 && r_in_tile < w.rows_valid) a.delta_out[(int64_t)w.bh * g.n + r_row] = del_r;
      }
    }
  }

  const SampleHits sh = sample_hits(smem + L::hits_at(g, MODE));
  if (kHits) find_sample_hits<kFBT>(a, b, sh, fetch_sample_head(a, b, tid));

  // ---- the T rows ----
  int nT, nb = 0x7fffffff;
  const int32_t* tperm = nullptr;
  if (MODE == kBwdDqNode) {
    nT = build_key_list<kFBT>(f, w, list, scratch, &nb);
  } else if (MODE == kBwdDkvBlock) {
    nT = g.b;
    tperm = f.perm_q + w.seg_off + (int64_t)w.t * g.b;
  } else if (MODE == kBwdDkvSamp) {
    nT = b.chunk_len;
    tperm = f.perm_q + w.seg_off + b.chunk_start;
  } else {
    nT = max(0, w.k1 - w.k0);
  }
  const float nat_bias = ((MODE == kBwdDqNode || MODE == kBwdDkvSamp) && g.m > 0) ? logf((float)w.nr.s / (float)g.m) : 0.f;
  // tiles of the workgroup; in causal passes a wave leaves out those that lie wholly on its masked side
  const int tiles = (nT + kFTT - 1) / kFTT;
  int kt_lo = 0, kt_hi = tiles;
  if (MODE == kBwdDqExact && f.exact_causal) kt_hi = min(kt_hi, (w.q0 - w.k0 + grp * 32 + 31) / kFTT + 1);
  if (MODE == kBwdDkvExact && f.exact_causal) kt_lo = grp;  // T starts at the workgroup's first key

  // ---- tile movers.  Shared tiles: a thread fetches pieces of eight floats, splits them and puts them into its way's tiles ----
  // (exact passes: rows past the T rows' end read as zeros and are masked)
  constexpr int NP = kFTT * T::PPR / (64 * RG);  // pieces per thread and tensor
  const uint32_t bytes = (uint32_t)(kExact ? w.k1 : g.n) * (uint32_t)(D * 4);
  const __amdgpu_buffer_rsrc_t yrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Yh, 0, (int)bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t brsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Bh, 0, (int)bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t lrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)lse_h, 0, (kExact ? w.k1 : g.n) * 4, 0x00020000);
  const __amdgpu_buffer_rsrc_t drsrc = __builtin_amdgcn_make_buffer_rsrc((void*)del_h, 0, (kExact ? w.k1 : g.n) * 4, 0x00020000);
  int trow[NP];  // rows of the tile that is fetched next
  auto find_rows = [&](int kt) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int tp = kt * kFTT + (wtid + i * 64 * RG) / T::PPR;
      if (kExact) trow[i] = w.k0 + tp;
      else trow[i] = kSorted ? tperm[min(tp, nT - 1)] : list[min(tp, nT - 1)];
    }
  };
  f32x4 ys[NP][2], bs[NP][2];
  float sl[NP], sd[NP];  // dK / dV passes: L and delta of the row
  auto fetch = [&]() {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int off = trow[i] * (D * 4) + (wtid + i * 64 * RG) % T::PPR * 32;
      ys[i][0] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(yrsrc, off, 0, 0));
      ys[i][1] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(yrsrc, off + 16, 0, 0));
      bs[i][0] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(brsrc, off, 0, 0));
      bs[i][1] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(brsrc, off + 16, 0, 0));
      if (!kDq) {
        sl[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(lrsrc, trow[i] * 4, 0, 0));
        sd[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(drsrc, trow[i] * 4, 0, 0));
      }
    }
  };
  auto store = [&]() {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int r = (wtid + i * 64 * RG) / T::PPR, piece = (wtid + i * 64 * RG) % T::PPR;
      T::store(ytile, r, piece, ys[i][0], ys[i][1]);
      T::store(btile, r, piece, bs[i][0], bs[i][1]);
      if (!kDq && piece == 0) {
        sc[r] = sl[i];
        sc[kFTT + r] = sd[i];
      }
    }
  };
  const int row_at = T::row_at(lane), col_at = T::col_at(lane);
  // RG = 1: the lane's T row (position 32 kt + lq) in pieces, and columns 32 dt + lq of rows 8 (i / 4) + 4 h + i % 4
  int row = 0;
  float scl = 0.f, scd = 0.f;  // dK / dV of sorted rows: L and delta of the T row this lane holds
  f32x4 yf[kShared ? 1 : 2 * KS];
  auto load_rows = [&](const __amdgpu_buffer_rsrc_t& rsrc, int of, f32x4 (&v)[kShared ? 1 : 2 * KS]) {
    if constexpr (!kShared) {
#pragma unroll
      for (int j = 0; j < 2 * KS; ++j)
        v[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, of * (D * 4) + 32 * h + 16 * (j % 2), 64 * (j / 2), 0));
    }
  };
  auto fetch_own = [&](int kt) {
    const int tp = min(kt * kFTT + lq, nT - 1);
    row = kExact ? w.k0 + kt * kFTT + lq : kSorted ? tperm[tp] : list[tp];
    load_rows(yrsrc, row, yf);
    if (!kDq && !kExact) {
      scl = lse_h[row];
      scd = del_h[row];
    }
  };
  auto of_elem = [&](auto v, int i) { return __shfl(v, 8 * (i / 4) + 4 * h + (i % 4)); };
  auto load_cols = [&](const __amdgpu_buffer_rsrc_t& rsrc, int of, int kt, auto& v, int i0, int count) {
    // Consecutive rows.  All of the row is in the lane's offset: the bounds check covers it, not the scalar one.  One
    // running offset (opaque, or the compiler keeps one register per eight rows across the loop): 241.3 us where constants of
    // one offset take 245.6 (4 heads, n = 4096 in causal blocks of 1024, forward + backward).
    if (kExact) {
      int off = (w.k0 + kt * kFTT + 8 * (i0 / 4) + 4 * h) * (D * 4) + 4 * lq;
#pragma unroll
      for (int i = i0; i < i0 + count; ++i) {
        if (i % 4 == 0 && i > i0) {
          off += 8 * (D * 4);
          asm volatile("" : "+v"(off));
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
          v[i][dt] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, off + (i % 4) * (D * 4) + 128 * dt, 0, 0));
      }
      return;
    }
#pragma unroll
    for (int i = i0; i < i0 + count; ++i) {
      const int off = of_elem(of, i) * (D * 4) + 4 * lq;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) v[i][dt] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, off, 128 * dt, 0));
    }
  };

  f32x16 acc1[DT], acc2[kDq ? 1 : DT];  // dQ or dK; dV
  // BOUND: split_tile_products'; tiles are then not fetched ahead, so that this form needs no more registers.
  auto run = [&](auto bound) {
    constexpr bool BOUND = decltype(bound)::value;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) acc1[dt][i] = 0.f;
#pragma unroll
      for (int dt = 0; dt < (kDq ? 1 : DT); ++dt) acc2[dt][i] = 0.f;
    }

    if constexpr (kShared && BOUND) {  // (kept through the first run, they would take registers that its loop needs)
      f32x4 av[2 * KS];
      load_r(av);
    }
    if constexpr (kShared) {
      if (!BOUND && kw < tiles) {
        find_rows(kw);
        fetch();
        if (!kExact) find_rows(kw + KW);
      }
    } else if (!BOUND && kt_lo + kw < kt_hi) {
      fetch_own(kt_lo + kw);
    }
    // (shared tiles: the same trips for all ways, the barriers are the workgroup's)
    const int kt_end = kShared ? (tiles + KW - 1) / KW * KW : kt_hi;
    for (int kt = (kShared ? 0 : kt_lo) + kw; kt < kt_end; kt += KW) {
      if constexpr (kShared) {
        if (kt >= KW) __syncthreads();  // the tiles before are read no more
        if (BOUND && kt < tiles) {
          find_rows(kt);
          fetch();
        }
        if (kt < tiles) store();
        __syncthreads();
        if (!BOUND && kt + KW < tiles) {
          if (kExact) find_rows(kt + KW);
          fetch();
          if (!kExact) find_rows(kt + 2 * KW);
        }
        if (kt < kt_lo || kt >= kt_hi) continue;
      } else if (BOUND) {
        fetch_own(kt);
      }
      f32x4 l4[4], d4[4];  // dK / dV passes: L and delta of the lane's T rows
      if (!kDq && (kShared || kExact)) {
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int at = (w.k0 + kt * kFTT + 8 * q4 + 4 * h) * 4;
          l4[q4] = kShared ? *reinterpret_cast<const f32x4*>(sc + 8 * q4 + 4 * h) : __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(lrsrc, at, 0, 0));
          d4[q4] = kShared ? *reinterpret_cast<const f32x4*>(sc + kFTT + 8 * q4 + 4 * h) : __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(drsrc, at, 0, 0));
        }
      }
      const int row_c = row;
      const float scl_c = scl, scd_c = scd;
      f32x4 bf[kShared ? 1 : 2 * KS];
      if (!kShared) load_rows(brsrc, row_c, bf);

      f32x16 c, e;
      {
        f32x16 small;
#pragma unroll
        for (int i = 0; i < 16; ++i) c[i] = small[i] = 0.f;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          if constexpr (kShared) split_product(T::row_frag(ytile, row_at, s), xs[s], c, small);
          else {
            const Split8 y = split8_raw([&](int i) { return yf[2 * s + i / 4][i % 4]; });
            if (kKeepY) T::store(own_y, lq, 2 * s + h, y);
            split_product(y, T::row_frag(ytile, row_at, s), c, small);
          }
        }
        split_sum<BOUND>(c, small);
      }
      float tv[kShared ? 1 : 16][DT];
      if constexpr (!kShared && !(kDq && kKeepY)) load_cols(kDq ? yrsrc : brsrc, row_c, kt, tv, 0, 16);
      {
        f32x16 small;
#pragma unroll
        for (int i = 0; i < 16; ++i) e[i] = small[i] = 0.f;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          if constexpr (kShared) split_product(T::row_frag(btile, row_at, s), as[s], e, small);
          else split_product(split8_raw([&](int i) { return bf[2 * s + i / 4][i % 4]; }), T::row_frag(btile, row_at, s), e, small);
        }
        split_sum<BOUND>(e, small);
      }

      // masks, on the tiles that have any: in the sampled-key pass the keys differ by lane
      const int tbase = kt * kFTT;
      bool special = tbase + kFTT > nT;
      if (MODE == kBwdDqNode) special = special || (tbase < nb && tbase + kFTT > nb);
      if (MODE == kBwdDqExact && f.exact_causal) special = special || (w.k0 + tbase + kFTT - 1 > w.q0 + grp * 32);
      if (MODE == kBwdDkvExact && f.exact_causal) special = special || (w.k0 + tbase < w.q0 + grp * 32 + 31);
      if (MODE == kBwdDkvSamp) {
        const int mlo = blk_r * g.b - (b.chunk_start + tbase);
        special = special || __any(mlo < kFTT && mlo + g.b > 0);
      }
      float tile_bias = MODE == kBwdDkvSamp ? nat_bias : 0.f;
      if (MODE == kBwdDqNode && tbase >= nb) tile_bias = nat_bias;
      if (special) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int tpos = tbase + 8 * (i / 4) + 4 * h + (i % 4);
          bool masked = tpos >= nT;
          if (MODE == kBwdDqNode && tbase < nb && tpos >= nb) c[i] += nat_bias * (1.f / kSplitScore);
          // queries of the key's own block: factor 1 - M of Algorithm 2
          if (MODE == kBwdDkvSamp) masked = masked || (unsigned)(b.chunk_start + tpos - blk_r * g.b) < (unsigned)g.b;
          if (MODE == kBwdDqExact && f.exact_causal) masked = masked || (w.k0 + tpos > r_row);   // keys after the query
          if (MODE == kBwdDkvExact && f.exact_causal) masked = masked || (w.k0 + tpos < r_row);  // queries before the key
          if (masked) c[i] = -INFINITY;
          if (kExact && !kDq && masked) {  // (a piece of four values can end past the head's last row)
            l4[i / 4][i % 4] = 0.f;
            d4[i / 4][i % 4] = 0.f;
          }
        }
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const bool quads = kShared || kExact;
        const float L = kDq ? L_r : quads ? l4[i / 4][i % 4] : of_elem(scl_c, i);
        const float dl = kDq ? del_r : quads ? d4[i / 4][i % 4] : of_elem(scd_c, i);
        float p = exp_split(__builtin_fmaf(c[i], kSplitScore, tile_bias) - L);
        if (L == -INFINITY) p = 0.f;  // (a row without keys)
        c[i] = p;
        e[i] = p * __builtin_fmaf(e[i], kSplitScore, -dl);
      }
      Split8 ps[2];  // 16 T rows each
      if constexpr (kShared) {
        if constexpr (!kDq) {
#pragma unroll
          for (int hf = 0; hf < 2; ++hf) ps[hf] = split8([&](int i) { return c[8 * hf + i]; });
          split_tile_products<DT, D == 64 && !kDq ? kSumSmall : kSumTile, BOUND>([&](int dt, int hf) { return T::col_frag(btile, col_at, hf, dt); }, ps, acc2);
        }
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) ps[hf] = split8([&](int i) { return e[8 * hf + i]; });
        split_tile_products<DT, D == 64 && !kDq ? kSumSmall : kSumTile, BOUND>([&](int dt, int hf) { return T::col_frag(ytile, col_at, hf, dt); }, ps, acc1);
      } else {
        // Y^T dS from the wave's own tile, or from the caches: the rows arrive while the dV products run
        float yv[kKeepY || kDq ? 1 : 16][DT];
        if constexpr (!kDq) {
          if constexpr (!kKeepY) load_cols(yrsrc, row_c, kt, yv, 0, 16);
#pragma unroll
          for (int hf = 0; hf < 2; ++hf) ps[hf] = split8([&](int i) { return c[8 * hf + i]; });
          split_tile_products<DT, kSumEach, BOUND>([&](int dt, int hf) { return split8_raw([&](int i) { return tv[8 * hf + i][dt]; }); }, ps, acc2);
        }
        if (!BOUND && kt + KW < kt_hi) fetch_own(kt + KW);
        if constexpr (kKeepY) {  // (the tile's rows came from other lanes of the wave)
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) ps[hf] = split8([&](int i) { return e[8 * hf + i]; });
        split_tile_products<DT, kSumEach, BOUND>([&](int dt, int hf) {
          if constexpr (kKeepY) return T::col_frag(own_y, col_at, hf, dt);
          else return split8_raw([&](int i) { return (kDq ? tv : yv)[kDq || !kKeepY ? 8 * hf + i : 0][dt]; });
        }, ps, acc1);
        if constexpr (kKeepY) {  // (the next tile's rows are written behind these reads)
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
      }
    }
    split_settle();
  };
  if constexpr (!kShared) __syncthreads();  // the R rows stand
  run(std::false_type{});
  const bool sums_finite = split_finite(acc1) && (kDq || split_finite(acc2));
  if constexpr (kShared) {
    const SplitFinite<NW> finite{reinterpret_cast<int32_t*>(smem + L::finite_at(g, MODE))};
    finite.post(wave, sums_finite);
    __syncthreads();  // the key list is read no more
    if (__builtin_expect(!finite.all(), 0)) {
      run(std::true_type{});
      __syncthreads();
    }
  } else {
    if (__builtin_expect(!__all(sums_finite), 0)) run(std::true_type{});
    __syncthreads();  // the key list is read no more
  }

  // ---- results: the waves' rows through LDS, the KW parts of a row added in wave order.  Node passes write
  // (the first level that holds the row on the pass's side) or add (later levels) fp32 rows of the accumulated
  // gradient; exact passes write the final gradient after adding the accumulated row where some level
  // holds this row (queries: second half of the node; keys: first half) ----
  constexpr int RS = L::ROW;
  float* rows_lds = reinterpret_cast<float*>(smem);
  const int64_t srow0 = (int64_t)w.bh * bwd_chunks_per_node(g, a.chunk, 0) * g.m;  // sample 0's sums (kHits)
  auto write_out = [&](const auto& acc, float* node_dst, const float* samp, float* fin, const float* lvl) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        *reinterpret_cast<f32x4*>(rows_lds + (wave * 32 + lq) * RS + 32 * dt + 8 * q4 + 4 * h) =
            (f32x4){acc[dt][4 * q4], acc[dt][4 * q4 + 1], acc[dt][4 * q4 + 2], acc[dt][4 * q4 + 3]} * (1.f / kSplitRaw);
    __syncthreads();
    constexpr int LPR = D / 4;  // lanes per row
    for (int idx = tid; idx < w.rows_valid * LPR; idx += kFBT) {
      const int r = idx / LPR, col = (idx % LPR) * 4;
      const float* src = rows_lds + r * RS + col;
      f32x4 v = *reinterpret_cast<const f32x4*>(src);
#pragma unroll
      for (int k = 1; k < KW; ++k) v += *reinterpret_cast<const f32x4*>(src + k * kRT * RS);
      if (kHits && samp != nullptr) {
        const int j = sh.first[r];
        const f32x4 sv = *reinterpret_cast<const f32x4*>(samp + (srow0 + (j != kNoSample ? j : 0)) * D + col);
        if (j != kNoSample) v += sv;
        const int nm = *sh.count;
        for (int e = 0; e < nm; ++e)
          if (sh.more[e] >> 16 == r) v += *reinterpret_cast<const f32x4*>(samp + (srow0 + (sh.more[e] & 0xffff)) * D + col);
      }
      int dummy;
      const int rr = bwd_r_row<MODE>(a, b, r, &dummy);
      const int64_t out_row = bwd_out_row<MODE>(a, b, r, rr);
      bool add = false;
      if (MODE == kBwdDqNode && !FINAL) add = a.base_first || node_levels_hold(g, rr, true, w.level);
      if (MODE == kBwdDkvBlock && !FINAL) add = a.base_first || node_levels_hold(g, rr, false, w.level);
      if (kExact) add = lvl != nullptr && node_levels_hold(g, rr, kDq, g.levels);
      const float* from = kExact ? lvl : node_dst;
      if (add) v += *reinterpret_cast<const f32x4*>(from + out_row * D + col);
      *reinterpret_cast<f32x4*>((kExact || FINAL ? fin : node_dst) + out_row * D + col) = v;
    }
  };
  write_out(acc1, a.out1, a.samp1, reinterpret_cast<float*>(a.fin1), a.lvl1);
  if constexpr (!kDq) {
    __syncthreads();  // the rows of the other gradient are read no more
    write_out(acc2, a.out2, a.samp2, reinterpret_cast<float*>(a.fin2), a.lvl2);
  }
}

template <int D, int MODE, int RG, int KW, bool FINAL>
__global__ __launch_bounds__(64 * RG * KW, D == 64 ? 2 : 1) void attn_bwd_f32_kernel(BwdArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bwd_f32_pass<D, MODE, RG, KW, FINAL>(a, (int)blockIdx.x, (int)gridDim.x, smem);
}

// Passes of a small causal problem side by side in one launch.  One behind the other each of them leaves the chip half empty and
// pays for its start: the node passes are 256 workgroups of a tile or two (4 heads, n = 4096), the sampled keys 128.  The
// gradients of fp32 tensors can hold the sums over the parts themselves, so the base case, which writes every row, comes
// first, and nothing but the order of additions ties the passes together: the base case's dK / dV and dQ and the sampled
// keys are one launch, longest workgroups first, then each level's dK / dV and dQ another.
// Backward, passes apart -> shared (MI355X, us; d = 64, d = 128): 4 heads, n = 4096, n_min = 1024, b = m = 64 140 -> 109, 293 -> 236; 1 head, n = 2048
// 92 -> 51, 175 -> 89; 1 head, n = 8192 145 -> 92, 266 -> 162; 3 heads, n = 1024, n_min = 256 85 -> 45, 141 -> 72; 12 heads, n = 4096 297 -> 264, 714 -> 650.
// Where the passes fill the chip (small_pass) they stay apart, with the sums in rows of the workspace: d = 64, 16 heads, n = 4096, n_min = 1024, b = m = 128
// (512 workgroups of 128 rows in the base case) 422 -> 391, 24 (768) 593 -> 602; 8 heads, n = 8192, n_min = 2048, b = m = 256 (512) 708 -> 678, 10 heads,
// n_min = 4096 (640) 1149 -> 1270; d = 128: 14 heads, n = 4096 (448) 970 -> 864, 16 (512) 909 -> 963.
template <int D, bool NODES>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void attn_bwd_f32_shared_kernel(BwdShared m) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int wg = (int)blockIdx.x;
  const int first1 = m.part[1].first, first2 = m.part[2].first;
  if constexpr (NODES) {
    if (wg < first1) {
      if (wg < m.part[0].count) bwd_f32_pass<D, kBwdDkvBlock, 1, 4, false>(m.part[0].a, wg, m.part[0].count, smem);
    } else if (wg - first1 < m.part[1].count) {
      bwd_f32_pass<D, kBwdDqNode, 1, 4, false>(m.part[1].a, wg - first1, m.part[1].count, smem);
    }
  } else {
    if (wg < first1) {
      if (wg < m.part[0].count) bwd_f32_pass<D, kBwdDkvExact, 1, 4, false>(m.part[0].a, wg, m.part[0].count, smem);
    } else if (wg < first2) {
      if (wg - first1 < m.part[1].count) bwd_f32_pass<D, kBwdDqExact, 1, 4, false>(m.part[1].a, wg - first1, m.part[1].count, smem);
    } else if (wg - first2 < m.part[2].count) {
      bwd_f32_pass<D, kBwdDkvSamp, 1, 4, false>(m.part[2].a, wg - first2, m.part[2].count, smem);
    }
  }
}

template <int D, int MODE, int RG, int KW, bool FINAL>
static int launch_bwd_f32_form(const BwdArgs& args, int grid, hipStream_t st) {
  BwdArgs a = args;
  if (MODE == kBwdDqNode || MODE == kBwdDkvBlock) set_node_divs<32 * RG>(a.f);
  if (MODE == kBwdDqExact || MODE == kBwdDkvExact) set_exact_divs<32 * RG>(a.f);
  a.f.exact_lpt = KW == 8;
  const size_t lds = F32BwdLds<D, RG, KW>::bytes(a.f.g, MODE);
  static std::atomic<uint64_t> lds_set{0};  // per instantiation: devices on which the LDS limit is raised
  if (allow_full_lds(reinterpret_cast<const void*>(&attn_bwd_f32_kernel<D, MODE, RG, KW, FINAL>), lds_set) != HA_OK) return HA_ERR_LAUNCH;
  hipLaunchKernelGGL((attn_bwd_f32_kernel<D, MODE, RG, KW, FINAL>), dim3((unsigned)grid), dim3(64 * RG * KW), lds, st, a);
  return check_launch();
}

template <int D, int MODE, int RG, int KW>
static int launch_bwd_f32_one(const BwdArgs& a, hipStream_t st) {
  const int64_t grid = bwd_grid<32 * RG>(a, MODE);
  if (grid <= 0) return HA_OK;
  if (grid > kMaxGrid) return HA_ERR_SHAPE;
  if constexpr (MODE == kBwdDqNode || MODE == kBwdDkvBlock)
    if (!a.f.g.causal) return launch_bwd_f32_form<D, MODE, RG, KW, true>(a, (int)grid, st);
  return launch_bwd_f32_form<D, MODE, RG, KW, false>(a, (int)grid, st);
}

// Whether workgroups of 128 R rows fill the runs of rows they are cut from (blocks, sample sets) to three quarters.
template <int MODE>
static bool rows_fit_128(const BwdArgs& a) {
  const Geometry& g = a.f.g;
  const int run = MODE == kBwdDkvSamp ? g.m : (MODE == kBwdDqNode || MODE == kBwdDkvBlock) ? g.b : a.f.exact_block;
  return 3 * (int64_t)((run + 127) / 128 * 128) <= 4 * (int64_t)run;
}

template <int MODE>
static bool small_pass(const BwdArgs& a) {
  return !rows_fit_128<MODE>(a) || bwd_grid<128>(a, MODE) < (a.f.g.d == 64 ? 576 : 512);
}

// a part begins at a multiple of 8, so that its workgroups' XCDs are those of a launch of its own
static int64_t part_span(const BwdArgs& a, int mode) { return (bwd_grid<32>(a, mode) + 7) & ~(int64_t)7; }

// (short blocks: a workgroup each in the level's launch, one per 32 rows in that of the base case)
int64_t bwd_f32_shared_workgroups(const BwdArgs& a) {
  const int64_t base = part_span(a, kBwdDkvExact) + part_span(a, kBwdDqExact) + part_span(a, kBwdDkvSamp);
  const int64_t level = part_span(a, kBwdDkvBlock) + part_span(a, kBwdDqNode);
  return base > level ? base : level;
}

bool bwd_f32_shares(const BwdArgs& a) {
  return small_pass<kBwdDqExact>(a) && small_pass<kBwdDqNode>(a) && (a.f.g.m == 0 || small_pass<kBwdDkvSamp>(a)) &&
         bwd_f32_shared_workgroups(a) <= kMaxLaunch;
}

template <int D, bool NODES>
static int launch_shared_form(const BwdShared& m, int64_t grid, hipStream_t st) {
  size_t lds = 0;  // the most that a part takes
  for (const int mode : {NODES ? kBwdDkvBlock : kBwdDkvExact, NODES ? kBwdDqNode : kBwdDqExact, NODES ? kBwdDqNode : kBwdDkvSamp}) {
    const size_t l = F32BwdLds<D, 1, 4>::bytes(m.part[0].a.f.g, mode);
    lds = l > lds ? l : lds;
  }
  static std::atomic<uint64_t> lds_set{0};  // per instantiation: devices on which the LDS limit is raised
  if (allow_full_lds(reinterpret_cast<const void*>(&attn_bwd_f32_shared_kernel<D, NODES>), lds_set) != HA_OK) return HA_ERR_LAUNCH;
  hipLaunchKernelGGL((attn_bwd_f32_shared_kernel<D, NODES>), dim3((unsigned)grid), dim3(256), lds, st, m);
  return check_launch();
}

// parts one behind the other
static int launch_shared(BwdShared& m, int parts, const int* modes, bool nodes, hipStream_t st) {
  int64_t at = 0;
  for (int i = 0; i < 3; ++i) {
    BwdPart& p = m.part[i];
    p.first = (int32_t)at;
    p.count = 0;
    if (i >= parts) continue;
    const int64_t span = part_span(p.a, modes[i]);
    if (at + span > kMaxLaunch) return HA_ERR_SHAPE;
    p.count = (int32_t)bwd_grid<32>(p.a, modes[i]);
    if (nodes) set_node_divs<32>(p.a.f);
    else if (modes[i] != kBwdDkvSamp) set_exact_divs<32>(p.a.f);
    at += span;
  }
  if (at == 0) return HA_OK;
  const int d = m.part[0].a.f.g.d;
  if (d != 64 && d != 128) return HA_ERR_SHAPE;
  if (nodes) return d == 64 ? launch_shared_form<64, true>(m, at, st) : launch_shared_form<128, true>(m, at, st);
  return d == 64 ? launch_shared_form<64, false>(m, at, st) : launch_shared_form<128, false>(m, at, st);
}

int launch_attn_bwd_f32_base(const BwdArgs& dkv, const BwdArgs& dq, const BwdArgs* samp, hipStream_t st) {
  BwdShared m{};
  m.part[0].a = dkv;
  m.part[1].a = dq;
  m.part[1].a.f.exact_lpt = 1;  // placed as the workgroups before them end
  if (samp) m.part[2].a = *samp;
  const int modes[3] = {kBwdDkvExact, kBwdDqExact, kBwdDkvSamp};
  return launch_shared(m, samp ? 3 : 2, modes, false, st);
}

int launch_attn_bwd_f32_level(const BwdArgs& block, const BwdArgs& dq, hipStream_t st) {
  BwdShared m{};
  m.part[0].a = block;
  m.part[1].a = dq;
  const int modes[2] = {kBwdDkvBlock, kBwdDqNode};
  return launch_shared(m, 2, modes, true, st);
}

// Ways of a workgroup, as in the forward (f32_ways): one where there are workgroups of 128 rows enough, else four, of 32 rows; exact
// launches of few groups and long rows take eight at d = 64 (at d = 128 a wave's registers leave one per SIMD).  One way / four (MI355X, us; backward
// passes, workgroups of 128 rows in brackets):
//   d = 64: exact, causal, 32 heads, n = 1024 (256) 205 / 131, 64 (512) 225 / 240, 16 heads, n = 4096 (512) 819 / 826; unmasked, 32 heads, n = 1024 (256)
//     207 / 220; nodes: b = m = 256, 8 heads, n = 4096 (256) 180 / 149, b = m = 128: 10 heads (320) 129 / 120, 12 (384) 132 / 133, 14 (448) 138 / 153
//   d = 128: exact, causal, 64 heads, n = 1024 (512) 595 / 564, 128 (1024) 1102 / 1184; unmasked, 32 heads (256) 401 / 472; nodes: 8 heads, n = 2048 (128)
//     156 / 114; b = m = 256, 8 heads, n = 4096 (256) 267 / 321; b = m = 128: 10 heads (320) 246 / 272, 18 (576) 404 / 466
//   eight ways, d = 64, causal: one head, n = 1024 56.9 (four: 62.5), 8 heads 61.5 (66.2), 16 80.1 (76.9); 4 heads, n = 2048 103 (120)
template <int MODE>
static int bwd_f32_ways(const BwdArgs& a) {
  constexpr bool kExact = MODE == kBwdDqExact || MODE == kBwdDkvExact;
  const int d = a.f.g.d;
  if (d == 64 && kExact && f32_exact_eight(a.f)) return 8;
  const int64_t enough = kExact && a.f.exact_causal ? (d == 64 ? 512 : 1024) : d == 128 ? 208 : kExact ? 256 : 384;
  return rows_fit_128<MODE>(a) && bwd_grid<128>(a, MODE) >= enough ? 1 : 4;
}

int bwd_f32_node_ways(const BwdArgs& a) { return bwd_f32_ways<kBwdDqNode>(a); }

template <int D, int MODE>
static int launch_bwd_f32_mode(const BwdArgs& a, hipStream_t st) {
  const int kw = bwd_f32_ways<MODE>(a);
  if constexpr (D == 64 && (MODE == kBwdDqExact || MODE == kBwdDkvExact))
    if (kw == 8) return launch_bwd_f32_one<D, MODE, 1, 8>(a, st);
  return kw == 1 ? launch_bwd_f32_one<D, MODE, 4, 1>(a, st) : launch_bwd_f32_one<D, MODE, 1, 4>(a, st);
}

template <int D>
static int launch_bwd_f32_d(const BwdArgs& a, int mode, hipStream_t st) {
  switch (mode) {
    case kBwdDqNode: return launch_bwd_f32_mode<D, kBwdDqNode>(a, st);
    case kBwdDqExact: return launch_bwd_f32_mode<D, kBwdDqExact>(a, st);
    case kBwdDkvBlock: return launch_bwd_f32_mode<D, kBwdDkvBlock>(a, st);
    case kBwdDkvSamp: return launch_bwd_f32_mode<D, kBwdDkvSamp>(a, st);
    case kBwdDkvExact: return launch_bwd_f32_mode<D, kBwdDkvExact>(a, st);
    default: return HA_ERR_SHAPE;
  }
}

int launch_attn_bwd_f32(const BwdArgs& a, int mode, hipStream_t st) {
  if (a.f.g.dtype != HA_FP32) return HA_ERR_DTYPE;
  if (a.f.g.d == 128) return launch_bwd_f32_d<128>(a, mode, st);
  if (a.f.g.d == 64) return launch_bwd_f32_d<64>(a, mode, st);
  return HA_ERR_SHAPE;
}

}  // namespace ha
