// Backward pass on the fp32 matrix cores: the arithmetic path for HA_FP32 tensors
// (v_mfma_f32_32x32x2_f32: every product and sum in fp32), with the same passes and the
// same buffers as the bf16 backward kernel, so that the host sequence is one and the same.
//
// As there, a row of the forward is one softmax over its block keys, its kept sampled keys (weight
// s/m) and, when causal, the keys of its base-case block (Algorithms 1, 2, 4), and with the final
// log row sum L_i and delta_i = <dO_i, O_i> every (query, key) pair contributes on its own:
//   P_ij = w_ij exp(<q_i, k_j> - L_i),  dV_j += P_ij dO_i,  dS_ij = P_ij (<dO_i, v_j> - delta_i),
//   dQ_i += dS_ij k_j,  dK_j += dS_ij q_i.
//
// A wave owns 32 "R rows" (queries in the dQ passes, keys in the dK / dV passes): the row, the operand of
// dP and the accumulators live in its registers.  The "T rows" (keys, resp. queries) come in tiles of 32
// straight from the caches in operand layout, once row-major for the scores and dP and once
// transposed for the accumulating products (attn_f32.hip has the layouts): no LDS staging and no
// barrier, because 64-cycle instructions leave the caches 16 B/clk per CU to deliver.  The dK / dV passes
// form S and dP once and accumulate both gradients: 4 products, 3 in the dQ passes.
//
// KW waves share a group of R rows, each taking every KW-th tile; their sums are added through LDS in
// wave order, so results are bit-reproducible.
//
// What bounds it: the matrix pipe where the chip is full.  At 4 heads, n = 4096 (at most two waves per SIMD) it is busy
// 52 - 57 % of the cycles in the exact passes and 14 - 24 % in the node passes; waves wait for issue 55 - 65 % of their
// time in the former.  The dK / dV passes at d = 64 spill 56 to 108 bytes per lane (two fragments in flight beside rows and
// accumulators in 256 registers), the launches that small causal problems share 144 (base case) and 64 (a level): one allocation serves all
// their passes.
// Measured (MI355X, backward of exact attention, the five algorithmic products
// counted, seven executed), against two lanes per row with fp32 FMA and separate dK and dV passes, the form before:
// 8 heads, n = 4096, d = 64 5.5 -> 1.29 ms, d = 128 12.0 -> 2.4 ms; 32 heads, n = 8192, d = 64 17.1 ms = 80 TFLOP/s
// (112 executed, of 157); 4 causal heads, n = 4096, n_min = 1024, forward + backward 4.07 -> 0.45 ms.  Then the vector
// work beside the products (masks behind a branch; in the exact passes row addresses in the instructions' offsets and
// L, delta as four values per load instead of lane exchanges): there dQ 51 -> 45, dK / dV 68 -> 61 us.
#include "attn_common.h"
#include "bwd_common.h"

namespace ha {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kFTT = 32;   // T rows per tile
constexpr int f32_bwd_waves(int kw) { return kw == 8 ? 8 : 4; }  // of a workgroup, by the waves that share 32 R rows

template <int D, int NW = 4>
struct F32BwdLds {
  static constexpr int ROW = D + 4;  // floats per staged row
  static constexpr int BYTES = NW * 32 * ROW * 4;
};

template <int D>
__host__ __device__ inline size_t bwd_f32_lds_bytes(const Geometry& g, int mode) {
  const size_t list = mode == kBwdDqNode ? (size_t)(((g.b + g.m + 63) & ~63) + 64) * 4 + 64 : 0;
  const size_t hits = mode == kBwdDkvBlock && !g.causal ? sample_hits_bytes(g) : 0;  // behind the rows
  return list > (size_t)F32BwdLds<D>::BYTES ? list : (size_t)F32BwdLds<D>::BYTES + hits;
}

// d = 128 keeps up to 483 registers per lane (two fragments in flight beside rows and accumulators): one wave per SIMD
// FINAL: the node passes of an unmasked problem, which write the final gradients.
// wg: the workgroup's number among the pass's wgs.
template <int D, int MODE, int KW, bool FINAL>
__device__ __forceinline__ void bwd_f32_pass(const BwdArgs& a, const int wg, const int wgs, unsigned char* smem) {
  constexpr bool kDq = (MODE == kBwdDqNode || MODE == kBwdDqExact);
  constexpr bool kExact = (MODE == kBwdDqExact || MODE == kBwdDkvExact);
  constexpr bool kSorted = (MODE == kBwdDkvBlock || MODE == kBwdDkvSamp);
  constexpr bool kHits = FINAL && MODE == kBwdDkvBlock;  // sampled keys' sums added here
  constexpr int NW = f32_bwd_waves(KW), kFBT = 64 * NW;
  constexpr int kRT = 32 * (NW / KW);
  constexpr int KJ = D / 8;
  constexpr int DT = D / 32;
  // dQ: a dP is two sums of half the columns each; as one chain of d products it had dQ's error above that of the half-row
  // sums of the form before (4 blocks of 256 rows, d = 128: 4.8e-7 against 4.2e-7 relative; with this and log row sums of
  // one rounding 4.0e-7).  The scores stay one chain, the forward's: P = exp(S - L) then cancels their rounding where
  // scores are large (64 clusters, scores to 250: dQ's error 2.1e-5, with halves 1.7e-4).  The dK / dV passes have no
  // registers for it, and their errors are below those of the form before.
  constexpr int kChains = kDq ? 2 : 1;
  const AttnArgs& f = a.f;
  const Geometry& g = f.g;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, h = lane >> 5;
  const int kw = wave % KW, grp = wave / KW;
  int32_t* scratch = reinterpret_cast<int32_t*>(smem);
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
  f32x4 x[KJ], av[KJ];
#pragma unroll
  for (int j = 0; j < KJ; ++j) {
    x[j] = *reinterpret_cast<const f32x4*>(Xh + (int64_t)r_row * D + 8 * j + 4 * h);
    av[j] = *reinterpret_cast<const f32x4*>(Ah + (int64_t)r_row * D + 8 * j + 4 * h);
  }
  float L_r = 0.f, del_r = 0.f;
  if (kDq) {
    L_r = lse_h[r_row];
    if (a.delta_out == nullptr) {
      del_r = del_h[r_row];
    } else {
      const float* Oh = reinterpret_cast<const float*>(a.O) + ((int64_t)w.bh * g.n + r_row) * D + 4 * h;
      f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < KJ; ++j) {
        const f32x4 o = *reinterpret_cast<const f32x4*>(Oh + 8 * j);
#pragma unroll
        for (int z = 0; z < 4; ++z) s[z] = __builtin_fmaf(o[z], av[j][z], s[z]);
      }
      del_r = (s[0] + s[1]) + (s[2] + s[3]);
      del_r += __shfl_xor(del_r, 32);
      if (h == 0 && kw == 0 && r_in_tile < w.rows_valid) a.delta_out[(int64_t)w.bh * g.n + r_row] = del_r;
    }
  }

  const SampleHits sh = sample_hits(smem + F32BwdLds<D>::BYTES);
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
  // tiles of this wave's group: causal passes leave out those that lie wholly on the masked side
  int kt_lo = 0, kt_hi = (nT + kFTT - 1) / kFTT;
  if (MODE == kBwdDqExact && f.exact_causal) kt_hi = min(kt_hi, (w.q0 - w.k0 + grp * 32 + 31) / kFTT + 1);
  if (MODE == kBwdDkvExact && f.exact_causal) kt_lo = grp;  // T starts at the workgroup's first key
  auto t_row = [&](int kt) -> int {  // row within the head of T position kt * 32 + lq (clamped to an existing one)
    if (kExact) return w.k0 + kt * kFTT + lq;
    const int tp = min(kt * kFTT + lq, nT - 1);
    if (kSorted) return tperm[tp];
    return list[tp];
  };

  // (exact passes: rows past the T rows' end read as zeros and are masked)
  const uint32_t bytes = (uint32_t)(kExact ? w.k1 : g.n) * (uint32_t)(D * 4);
  const __amdgpu_buffer_rsrc_t yrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Yh, 0, (int)bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t brsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Bh, 0, (int)bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t lrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)lse_h, 0, (kExact ? w.k1 : g.n) * 4, 0x00020000);
  const __amdgpu_buffer_rsrc_t drsrc = __builtin_amdgcn_make_buffer_rsrc((void*)del_h, 0, (kExact ? w.k1 : g.n) * 4, 0x00020000);
  auto load_rows = [&](const __amdgpu_buffer_rsrc_t& rsrc, int row, f32x4 (&v)[KJ]) {
#pragma unroll
    for (int j = 0; j < KJ; ++j)
      v[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, row * (D * 4) + 16 * h, 32 * j, 0));
  };
  // element i of an accumulator is T row 8 (i / 4) + 4 h + i % 4 of the tile; lane l < 32 holds row l's values
  auto of_elem = [&](auto v, int i) { return __shfl(v, 8 * (i / 4) + 4 * h + (i % 4)); };
  auto load_cols = [&](const __amdgpu_buffer_rsrc_t& rsrc, int row, int kt, float (&v)[16][DT], int i0, int count) {
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
      const int off = of_elem(row, i) * (D * 4) + 4 * lq;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) v[i][dt] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, off, 128 * dt, 0));
    }
  };

  f32x16 acc1[DT], acc2[kDq ? 1 : DT];  // dQ or dK; dV
#pragma unroll
  for (int i = 0; i < 16; ++i) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) acc1[dt][i] = 0.f;
#pragma unroll
    for (int dt = 0; dt < (kDq ? 1 : DT); ++dt) acc2[dt][i] = 0.f;
  }

  int row = 0;
  float sc_l = 0.f, sc_d = 0.f;  // dK / dV passes: L and delta of the T row this lane holds
  f32x4 yf[KJ];
  auto fetch = [&](int kt) {
    row = t_row(kt);
    load_rows(yrsrc, row, yf);
    if (!kDq && !kExact) {
      sc_l = lse_h[row];
      sc_d = del_h[row];
    }
  };
  if (kt_lo + kw < kt_hi) fetch(kt_lo + kw);
  for (int kt = kt_lo + kw; kt < kt_hi; kt += KW) {
    const int row_c = row;
    const float scl = sc_l, scd = sc_d;
    f32x4 l4[4], d4[4];  // dK / dV of exact attention: L and delta of the lane's T rows, four consecutive ones at a time
    if (kExact && !kDq) {
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int at = (w.k0 + kt * kFTT + 8 * q4 + 4 * h) * 4;
        l4[q4] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(lrsrc, at, 0, 0));
        d4[q4] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(drsrc, at, 0, 0));
      }
    }
    f32x4 bf[KJ];
    load_rows(brsrc, row_c, bf);
    f32x16 c, es[kChains];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      c[i] = 0.f;
#pragma unroll
      for (int k = 0; k < kChains; ++k) es[k][i] = 0.f;
    }
#pragma unroll
    for (int j = 0; j < KJ; ++j)
#pragma unroll
      for (int z = 0; z < 4; ++z) c = __builtin_amdgcn_mfma_f32_32x32x2f32(yf[j][z], x[j][z], c, 0, 0, 0);
    float tv[16][DT];
    load_cols(kDq ? yrsrc : brsrc, row_c, kt, tv, 0, 16);
#pragma unroll
    for (int j = 0; j < KJ; ++j)
#pragma unroll
      for (int z = 0; z < 4; ++z) es[j % kChains] = __builtin_amdgcn_mfma_f32_32x32x2f32(bf[j][z], av[j][z], es[j % kChains], 0, 0, 0);

    f32x16 e = es[0];
    if constexpr (kChains == 2) e += es[1];

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
        if (MODE == kBwdDqNode && tbase < nb && tpos >= nb) c[i] += nat_bias;
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
      const float L = kDq ? L_r : kExact ? l4[i / 4][i % 4] : of_elem(scl, i);
      const float dl = kDq ? del_r : kExact ? d4[i / 4][i % 4] : of_elem(scd, i);
      float p = exp_split(c[i] + tile_bias - L);
      if (L == -INFINITY) p = 0.f;  // (a row without keys)
      c[i] = p;
      e[i] = p * (e[i] - dl);
    }
    if constexpr (!kDq) {
      // dV and dK half a tile at a time: the Q rows of a half arrive while the other half's dV products run
      float yv[16][DT];
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        load_cols(yrsrc, row_c, kt, yv, 8 * hf, 8);
#pragma unroll
        for (int i = 8 * hf; i < 8 * hf + 8; ++i)
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) acc2[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(tv[i][dt], c[i], acc2[dt], 0, 0, 0);
      }
      if (kt + KW < kt_hi) fetch(kt + KW);
#pragma unroll
      for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) acc1[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(yv[i][dt], e[i], acc1[dt], 0, 0, 0);
    } else {
      if (kt + KW < kt_hi) fetch(kt + KW);
#pragma unroll
      for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) acc1[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(tv[i][dt], e[i], acc1[dt], 0, 0, 0);
    }
  }

  // ---- results: the waves' rows through LDS, the KW parts of a row added in wave order.  Node passes write
  // (the first level that holds the row on the pass's side) or add (later levels) fp32 rows of the accumulated
  // gradient; exact passes write the final gradient after adding the accumulated row where some level
  // holds this row (queries: second half of the node; keys: first half) ----
  constexpr int RS = F32BwdLds<D>::ROW;
  float* rows_lds = reinterpret_cast<float*>(smem);
  const int64_t srow0 = (int64_t)w.bh * bwd_chunks_per_node(g, a.chunk, 0) * g.m;  // sample 0's sums (kHits)
  auto write_out = [&](const auto& acc, float* node_dst, const float* samp, float* fin, const float* lvl) {
    __syncthreads();  // the key list, or the rows of the other gradient, are read no more
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        *reinterpret_cast<f32x4*>(rows_lds + (wave * 32 + lq) * RS + 32 * dt + 8 * q4 + 4 * h) =
            (f32x4){acc[dt][4 * q4], acc[dt][4 * q4 + 1], acc[dt][4 * q4 + 2], acc[dt][4 * q4 + 3]};
    __syncthreads();
    constexpr int LPR = D / 4;  // lanes per row
    for (int idx = tid; idx < w.rows_valid * LPR; idx += kFBT) {
      const int r = idx / LPR, col = (idx % LPR) * 4;
      const float* src = rows_lds + ((r / 32) * KW * 32 + (r & 31)) * RS + col;
      f32x4 v = *reinterpret_cast<const f32x4*>(src);
#pragma unroll
      for (int k = 1; k < KW; ++k) v += *reinterpret_cast<const f32x4*>(src + k * 32 * RS);
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
  if constexpr (!kDq) write_out(acc2, a.out2, a.samp2, reinterpret_cast<float*>(a.fin2), a.lvl2);
}

template <int D, int MODE, int KW, bool FINAL>
__global__ __launch_bounds__(64 * f32_bwd_waves(KW), D == 64 ? 2 : 1) void attn_bwd_f32_kernel(BwdArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bwd_f32_pass<D, MODE, KW, FINAL>(a, (int)blockIdx.x, (int)gridDim.x, smem);
}

// Passes of a small causal problem side by side in one launch.  One behind the other each of them leaves the chip half empty and
// pays for its start: the node passes are 256 workgroups of a tile or two (4 heads, n = 4096), the sampled keys 128.  The
// gradients of fp32 tensors can hold the sums over the parts themselves, so the base case, which writes every row, comes
// first, and nothing but the order of additions ties the passes together: the base case's dK / dV and dQ and the sampled
// keys are one launch, longest workgroups first, then each level's dK / dV and dQ another.
// Forward + backward, passes apart -> shared (MI355X): 4 heads, n = 4096, n_min = 1024, b = m = 64, d = 64 239 -> 214 us, d = 128 447 ->
// 386; 1 head, n = 2048 170 -> 112; 1 head, n = 8192 251 -> 183; 3 heads, n = 1024, n_min = 256 134 -> 85; 12 heads, n = 4096 558 -> 502.
// Where the passes fill the chip (one wave per group of rows) they stay apart, with the sums in rows of the workspace: base
// case first there too, 8 heads, n = 8192, n_min = 2048, b = m = 256 took 1319 instead of 1284 us.
template <int D, bool NODES>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void attn_bwd_f32_shared_kernel(BwdShared m) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int wg = (int)blockIdx.x;
  const int first1 = m.part[1].first, first2 = m.part[2].first;
  if constexpr (NODES) {
    if (wg < first1) {
      if (wg < m.part[0].count) bwd_f32_pass<D, kBwdDkvBlock, 4, false>(m.part[0].a, wg, m.part[0].count, smem);
    } else if (wg - first1 < m.part[1].count) {
      bwd_f32_pass<D, kBwdDqNode, 4, false>(m.part[1].a, wg - first1, m.part[1].count, smem);
    }
  } else {
    if (wg < first1) {
      if (wg < m.part[0].count) bwd_f32_pass<D, kBwdDkvExact, 4, false>(m.part[0].a, wg, m.part[0].count, smem);
    } else if (wg < first2) {
      if (wg - first1 < m.part[1].count) bwd_f32_pass<D, kBwdDqExact, 4, false>(m.part[1].a, wg - first1, m.part[1].count, smem);
    } else if (wg - first2 < m.part[2].count) {
      bwd_f32_pass<D, kBwdDkvSamp, 4, false>(m.part[2].a, wg - first2, m.part[2].count, smem);
    }
  }
}

template <int D, int MODE, int KW, bool FINAL>
static int launch_bwd_f32_form(const BwdArgs& args, int grid, hipStream_t st) {
  BwdArgs a = args;
  constexpr int NW = f32_bwd_waves(KW);
  if (MODE == kBwdDqNode || MODE == kBwdDkvBlock) set_node_divs<32 * (NW / KW)>(a.f);
  if (MODE == kBwdDqExact || MODE == kBwdDkvExact) set_exact_divs<32 * (NW / KW)>(a.f);
  a.f.exact_lpt = KW == 8;
  const size_t lds = KW == 8 ? (size_t)F32BwdLds<D, NW>::BYTES : bwd_f32_lds_bytes<D>(a.f.g, MODE);
  static std::atomic<uint64_t> lds_set{0};  // per instantiation: devices on which the LDS limit is raised
  if (allow_full_lds(reinterpret_cast<const void*>(&attn_bwd_f32_kernel<D, MODE, KW, FINAL>), lds_set) != HA_OK) return HA_ERR_LAUNCH;
  hipLaunchKernelGGL((attn_bwd_f32_kernel<D, MODE, KW, FINAL>), dim3((unsigned)grid), dim3(64 * NW), lds, st, a);
  return check_launch();
}

template <int D, int MODE, int KW>
static int launch_bwd_f32_one(const BwdArgs& a, hipStream_t st) {
  const int64_t grid = bwd_grid<32 * (f32_bwd_waves(KW) / KW)>(a, MODE);
  if (grid <= 0) return HA_OK;
  if (grid > kMaxGrid) return HA_ERR_SHAPE;
  if constexpr (MODE == kBwdDqNode || MODE == kBwdDkvBlock)
    if (!a.f.g.causal) return launch_bwd_f32_form<D, MODE, KW, true>(a, (int)grid, st);
  return launch_bwd_f32_form<D, MODE, KW, false>(a, (int)grid, st);
}

template <int MODE>
static bool four_waves(const BwdArgs& a) {
  const Geometry& g = a.f.g;
  const int run = MODE == kBwdDkvSamp ? g.m : (MODE == kBwdDqNode || MODE == kBwdDkvBlock) ? g.b : a.f.exact_block;
  return 3 * (int64_t)((run + 127) / 128 * 128) > 4 * (int64_t)run || 4 * bwd_grid<128>(a, MODE) < 2048;
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
  return four_waves<kBwdDqExact>(a) && !f32_exact_eight(a.f) && four_waves<kBwdDqNode>(a) && (a.f.g.m == 0 || four_waves<kBwdDkvSamp>(a)) &&
         bwd_f32_shared_workgroups(a) <= kMaxLaunch;
}

template <int D, bool NODES>
static int launch_shared_form(const BwdShared& m, int64_t grid, hipStream_t st) {
  size_t lds = F32BwdLds<D>::BYTES;
  if (NODES) {
    const size_t l = bwd_f32_lds_bytes<D>(m.part[1].a.f.g, kBwdDqNode);
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

// Waves that share a group of 32 R rows, by the rule of the forward (launch_f32_mode): few groups or short runs
// of rows (blocks, sample sets) take four; exact launches of few groups and long rows take eight at d = 64 (forward + backward, 6
// causal heads, n = 2048: 204 -> 183 us; 3 heads, n = 4000: 372 -> 340; at d = 128 a wave's registers leave one per SIMD).
template <int D, int MODE>
static int launch_bwd_f32_mode(const BwdArgs& a, hipStream_t st) {
  const Geometry& g = a.f.g;
  const int run = MODE == kBwdDkvSamp ? g.m : (MODE == kBwdDqNode || MODE == kBwdDkvBlock) ? g.b : a.f.exact_block;
  const bool fits = 3 * (int64_t)((run + 127) / 128 * 128) <= 4 * (int64_t)run;
  if constexpr (D == 64 && (MODE == kBwdDqExact || MODE == kBwdDkvExact))
    if (f32_exact_eight(a.f)) return launch_bwd_f32_one<D, MODE, 8>(a, st);  // the forward's rule
  if (fits && 4 * bwd_grid<128>(a, MODE) >= 2048) return launch_bwd_f32_one<D, MODE, 1>(a, st);
  return launch_bwd_f32_one<D, MODE, 4>(a, st);
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
