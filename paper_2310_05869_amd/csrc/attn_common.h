// Work decomposition and key-list construction shared by the bf16 and the fp32
// attention kernels.
//
// One workgroup = one tile of QT consecutive sorted query positions inside one
// b-block of one node (node mode), or QT consecutive query rows of one diagonal
// block (exact mode).  In node mode the workgroup attends to ONE list of keys:
//   [0, nb)        the b keys of the block, M^H of Algorithm 1, bias 0
//   [nb, nkeys)    the sampled keys l_j of Algorithm 2 that are NOT in the
//                  row's own block (factor 1 - M_{i,l_j}), bias log(s/m)
// so the block part, the residual estimate and their shared normaliser come out
// of a single softmax pass: sum_block exp(S) + (s/m) sum_kept exp(S).
#pragma once

#include "ha_common.h"

namespace ha {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

struct TileWork {
  int bh;
  int rows_valid;    // query rows of this tile that exist
  // node mode
  int level, t, p0;  // block index within the node, first sorted position (node-local) of the tile
  NodeRef nr;
  int64_t seg_off;   // offset of the node in perm_q / perm_k / pos_k / part_*
  // exact mode
  int q0;            // first query row (within the head)
  int k0, k1;        // key rows [k0, k1) this tile attends to (before causal masking)
};

// XCD-aware ordering: consecutive workgroup ids are dealt round-robin to the 8
// XCDs, each with its own L2.  Give every XCD a contiguous range of logical
// tiles so that tiles sharing K/V (same block, same node) meet in one L2.
__device__ inline int logical_block(int bid, int total) {
  if (total % 8 != 0) return bid;
  return (bid & 7) * (total >> 3) + (bid >> 3);
}

template <int QT>
inline void set_node_divs(AttnArgs& a) {
  const Geometry& g = a.g;
  const int tpb = (g.b + QT - 1) / QT;
  a.div_tpl = make_fast_div((int64_t)(g.n_cov / g.b) * tpb);
  a.div_bh = make_fast_div(g.BH);
  a.div_tpb = make_fast_div(tpb);
  a.div_unit = make_fast_div(g.causal ? g.n_min / g.b : g.n / g.b);  // a node of level l: 2^(levels - 1 - l) times as many
}

template <int QT>
__device__ inline TileWork decode_node_tile(const AttnArgs& a, int idx) {
  const Geometry& g = a.g;
  TileWork w{};
  const int rest = a.div_tpl.div(idx);
  const int tile = idx - rest * (int)a.div_tpl.d;
  w.level = a.div_bh.div(rest);
  w.bh = rest - w.level * g.BH;
  const int blk = a.div_tpb.div(tile), chunk = tile - blk * (int)a.div_tpb.d;
  const int below = g.levels - 1 - w.level;
  const int node = a.div_unit.div(blk >> below);
  w.t = blk - ((node * (int)a.div_unit.d) << below);
  w.nr = node_ref(g, w.level, node);
  w.p0 = w.t * g.b + chunk * QT;
  w.rows_valid = min(QT, g.b - chunk * QT);
  w.seg_off = ((int64_t)w.level * g.BH + w.bh) * g.n_cov + (int64_t)node * w.nr.s;
  return w;
}

template <int QT>
__host__ __device__ inline int64_t node_grid(const Geometry& g) {
  const int tpb = (g.b + QT - 1) / QT;
  return (int64_t)g.levels * g.BH * (g.n_cov / g.b) * tpb;
}

// Order of an exact launch's workgroups.  Causal tiles differ in length up to (tiles per block)-fold, and a launch
// that fits the chip at once (two or three workgroups per CU) is placed before any of them has finished: workgroup i
// goes to XCD i mod 8 and, within it, to its 32 CUs in turn, so what a CU gets is fixed by the order.
//
// Causal launches of up to 256 tiles per XCD (in whole blocks): heaviest tiles first ACROSS the blocks; every second round of
// 32 tiles of an XCD runs backwards, so the CU (and the shader engine) that got the heaviest tile of one round gets the
// lightest of the next.  Where the number of blocks is a multiple of 8, block b stays on XCD b mod 8 (its K and V in one
// L2); 12 blocks share two XCDs each, an odd number all eight.
// Block after block, the order before, gave a CU the same rank of several blocks: 186 key tiles on the fullest CU
// against 99 on average at 24 blocks of 32 tiles.  Measured (MI355X): forward, 12 heads, n = 8192, d = 64: 141 ->
// 119 us (122 with every round forwards); forward + backward: fp32, 4 heads, n = 4096: 336 -> 283 (305) us;
// exact, 12 heads, n = 5000, d = 128: 530 -> 408 (437) us.
// Workgroups that take a CU each (exact_lpt: two wave groups) are not all placed at once, and with the rounds backwards the
// last to start would be the second round's heaviest: they come heaviest first throughout.
//
// Unmasked launches, whose tiles are all alike, and larger causal ones, where workgroups are replaced as they finish:
// every XCD takes a contiguous range, block after block (across the blocks an unmasked launch was 1 % slower: 12
// heads, n = 16384, d = 64: 947 -> 955 us), heaviest first, the starting tile rotated from one block to the next: an XCD's
// workgroups are dealt to its four shader engines in turn, and a fixed order would hand one of them every fourth, the
// heaviest, tile of every block.  The causal order above, in groups of 64 tiles per XCD, is 0.8 % slower there (forward, 32
// heads, n = 131072, d = 128: 9.14 against 9.22 ms; 9.31 with 256): more blocks in flight than an L2 holds.
struct ExactPlace {
  int bh, blk;
  int rank;  // tile within the block, heaviest first
};

constexpr int kOrderRound = 32;   // CUs of an XCD
constexpr int kOrderWhole = 256;  // tiles per XCD ordered as one

// The place is decoded with precomputed reciprocals (FastDiv), as a node workgroup's is: its five divisions were a fortieth
// of a small launch (one causal head, n = 512, d = 128: 13.5 -> 13.2 us).
template <int QT>
inline void set_exact_divs(AttnArgs& a) {
  const int eb = a.exact_block;
  const int nblk = (a.exact_rows_q + eb - 1) / eb;
  a.div_tpb = make_fast_div((eb + QT - 1) / QT);
  a.div_unit = make_fast_div(nblk);
  a.div_tpl = make_fast_div((int64_t)nblk * a.g.BH);
}

__device__ inline ExactPlace exact_place(const AttnArgs& a, int wg) {
  const int tpb = (int)a.div_tpb.d, nblk = (int)a.div_unit.d, blocks = (int)a.div_tpl.d;
  ExactPlace e;
  int b;
  if (!a.exact_causal || blocks > 8 * a.div_tpb.div(kOrderWhole + tpb - 1)) {
    const int idx = logical_block(wg, blocks * tpb);
    b = a.div_tpb.div(idx);
    const int r = idx - b * tpb + b;
    e.rank = r - a.div_tpb.div(r) * tpb;
  } else {
    const int xcd = wg & 7, j = wg >> 3;
    const int round = j / kOrderRound;
    int p = wg;
    if ((round & 1) && !a.exact_lpt) {
      const int left = ((blocks * tpb - xcd + 7) >> 3) - round * kOrderRound;  // the XCD's tiles from this round on
      const int cnt = left < kOrderRound ? left : kOrderRound;
      p = (2 * round * kOrderRound + cnt - 1 - j) * 8 + xcd;
    }
    e.rank = a.div_tpl.div(p);
    b = p - e.rank * blocks;
  }
  e.bh = a.div_unit.div(b);
  e.blk = b - e.bh * nblk;
  return e;
}

template <int QT>
__device__ inline TileWork decode_exact_tile(const AttnArgs& a, int wg) {
  TileWork w{};
  const int eb = a.exact_block;
  const ExactPlace e = exact_place(a, wg);
  const int qt = (int)a.div_tpb.d - 1 - e.rank;
  const int blk = e.blk;
  w.bh = e.bh;
  w.q0 = blk * eb + qt * QT;
  const int blk_rows = min(eb, a.exact_rows_q - blk * eb);
  w.rows_valid = max(0, min(QT, blk_rows - qt * QT));
  w.k0 = blk * eb;
  w.k1 = min(a.exact_rows_k, (blk + 1) * eb);
  if (a.exact_causal) w.k1 = min(w.k1, w.q0 + w.rows_valid);
  return w;
}

template <int QT>
__host__ __device__ inline int64_t exact_grid(const AttnArgs& a) {
  const int eb = a.exact_block;
  const int tpb = (eb + QT - 1) / QT;
  const int nblk = (a.exact_rows_q + eb - 1) / eb;
  return (int64_t)a.g.BH * nblk * tpb;
}

constexpr int64_t kMaxGrid = 0x7fffffff;  // workgroup ids are decoded as 32-bit integers

// The first index values a thread contributes to the key list (block key `tid`, sample `tid` and
// its sorted block): fetched ahead of the list's construction so that a caller can put other
// loads of the same round trip in flight beside them.
struct KeyListHead {
  int pk0, l0, blk0;
};

template <int NT>
__device__ inline KeyListHead key_list_fetch(const AttnArgs& a, const TileWork& w) {
  const Geometry& g = a.g;
  const int tid = threadIdx.x;
  const int nb = a.use_block ? g.b : 0;
  const int m = (a.samples != nullptr) ? g.m : 0;
  KeyListHead kh{0, 0, 0};
  if (tid < nb) kh.pk0 = a.perm_k ? a.perm_k[w.seg_off + w.t * g.b + tid] : w.nr.k_start + w.t * g.b + tid;
  if (tid < m) {
    kh.l0 = a.samples[(int64_t)w.nr.heap * g.m + tid];
    if (a.samp_blk) kh.blk0 = a.samp_blk[((int64_t)w.bh * g.total_nodes + w.nr.heap) * g.m + tid];
    else kh.blk0 = (a.pos_k ? a.pos_k[w.seg_off + kh.l0] : kh.l0) / g.b;
  }
  return kh;
}

// Builds the key list of a node tile in LDS.  `list` has room for b + m entries
// rounded up to a multiple of 64; `scratch` for (NT/64 + 1) ints.  All NT
// threads call it; on return (after its final barrier) list[0..pad) holds row
// indices within the head, *nb_out the block keys and the return value nkeys.
// `kh` = key_list_fetch's values of the calling thread.
// PADDED: the block's keys are padded to whole tiles of 64, so that no tile holds both parts.  All padding is then a key
// of the block, one that the rows see anyway: a masked key's weight is 0, but 0 times a V that is Inf or NaN is NaN.
template <int NT, bool PADDED = false>
__device__ inline int build_key_list(const AttnArgs& a, const TileWork& w, int32_t* list, int32_t* scratch,
                                     int* nb_out, const KeyListHead& kh) {
  const Geometry& g = a.g;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  constexpr int NW = NT / 64;
  const int nb = a.use_block ? g.b : 0;
  const int m = (a.samples != nullptr) ? g.m : 0;
  auto block_key = [&](int i) -> int {
    return a.perm_k ? a.perm_k[w.seg_off + w.t * g.b + i] : w.nr.k_start + w.t * g.b + i;
  };
  auto sample_of = [&](int j, int* blk) -> int {
    const int l = a.samples[(int64_t)w.nr.heap * g.m + j];
    if (a.samp_blk) *blk = a.samp_blk[((int64_t)w.bh * g.total_nodes + w.nr.heap) * g.m + j];
    else *blk = (a.pos_k ? a.pos_k[w.seg_off + l] : l) / g.b;
    return l;
  };
  const int pk0 = kh.pk0, l0 = kh.l0, blk0 = kh.blk0;
  if (tid < nb) list[tid] = pk0;
  for (int i = tid + NT; i < nb; i += NT) list[i] = block_key(i);
  int base = PADDED ? (nb + 63) & ~63 : nb;
  if (PADDED)
    for (int i = nb + tid; i < base; i += NT) list[i] = block_key(nb - 1);
  for (int j0 = 0; j0 < m; j0 += NT) {
    const int j = j0 + tid;
    int l = l0, blk = blk0;
    bool keep = false;
    if (j < m) {
      if (j0 > 0) l = sample_of(j, &blk);
      keep = blk != w.t;  // 1 - M_{i, l_j}: same for every row of the block
    }
    const unsigned long long bal = __ballot(keep);
    if (lane == 0) scratch[wave] = __popcll(bal);
    __syncthreads();
    int before = 0, total = 0;
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) {
      const int c = scratch[ww];
      if (ww < wave) before += c;
      total += c;
    }
    if (keep) list[base + before + __popcll(bal & ((1ull << lane) - 1ull))] = w.nr.k_start + l;
    base += total;
    if (j0 + NT < m) __syncthreads();  // before the counters are written again
  }
  const int nkeys = base;
  const int pad = (nkeys + 63) & ~63;
  // loadable, masked by position (PADDED: there are samples, so a barrier lies behind the block's keys)
  for (int i = nkeys + tid; i < pad; i += NT) list[i] = PADDED ? list[nb - 1] : w.nr.k_start;
  __syncthreads();
  *nb_out = nb;
  return nkeys;
}

template <int NT>
__device__ inline int build_key_list(const AttnArgs& a, const TileWork& w, int32_t* list, int32_t* scratch,
                                     int* nb_out) {
  return build_key_list<NT>(a, w, list, scratch, nb_out, key_list_fetch<NT>(a, w));
}

// e^x to one or two units in the last place, like the library's, in seven instructions against its thirteen: the
// hardware's 2^t at t = fl(x log2 e), times 1 + r ln 2 for what the rounding of t left out, r = x log2 e - t.
// (r is bounded so that x = -inf gives 0; results below 2^-126 are 0; NaN stays NaN.)
__device__ inline float exp_split(float x) {
  constexpr float kHi = 1.44269502f, kLo = 1.92596303e-8f;  // log2 e = kHi + kLo
  const float t = x * kHi;
  const float r = __builtin_fmaf(x, kLo, __builtin_fmaf(x, kHi, -t));
  const float e = __builtin_amdgcn_exp2f(t);
  return __builtin_fmaf(e * __builtin_amdgcn_fmed3f(r, -1.f, 1.f), kLn2, e);
}

__device__ inline float logaddexpf(float x, float y) {
  const float hi = fmaxf(x, y), lo = fminf(x, y);
  if (hi == -INFINITY) return -INFINITY;
  return hi + log1pf(expf(lo - hi));
}

__device__ inline uint32_t pack_bf16x2(float lo, float hi) {
  typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
  typedef float f2 __attribute__((ext_vector_type(2)));
  const bf2 p = __builtin_convertvector((f2){lo, hi}, bf2);
  return *reinterpret_cast<const uint32_t*>(&p);
}

// Where a finished query row goes.
struct RowDest {
  bool valid;
  int64_t out_row;   // row index into out / lse (head offset included), final output
  int64_t part_row;  // row index into part_o / part_l (node mode partial)
  int row_in_head;   // exact mode: for the per-level merge
};

__device__ inline RowDest node_row_dest(const AttnArgs& a, const TileWork& w, int r_in_tile) {
  RowDest d{};
  d.valid = r_in_tile < w.rows_valid;
  const int p = w.p0 + (d.valid ? r_in_tile : 0);
  const int row = (a.scatter_out && a.perm_q) ? a.perm_q[w.seg_off + p] : w.nr.q_start + p;
  d.row_in_head = row;
  d.out_row = (int64_t)w.bh * a.g.n + row;
  d.part_row = w.seg_off + (row - w.nr.q_start);
  return d;
}

// Causal merge (Algorithm 4): the row sum of row i is the base-case row sum
// plus the row sums of the off-diagonal nodes it belongs to.  Level l touches
// row i iff i lies in the second half of its level-l node; *prow is then the
// row's index in part_o / part_l.
__device__ inline bool level_touches(const Geometry& g, int bh, int i, int l, int64_t* prow) {
  const int s = g.n >> (l + 1);
  *prow = ((int64_t)l * g.BH + bh) * g.n_cov + (int64_t)(i / (2 * s)) * s + (i % s);
  return ((i / s) & 1) != 0;
}

// Combined log row sum of the base-case result (lse_own) and the partials;
// *mx_out is the reference the weights exp(l - mx) / den are taken against.
__device__ inline float merged_lse(const AttnArgs& a, int bh, int i, float lse_own, float* mx_out,
                                   float* den_out) {
  float mx = lse_own;
  for (int l = 0; l < a.merge_levels; ++l) {
    int64_t pr;
    if (level_touches(a.g, bh, i, l, &pr)) mx = fmaxf(mx, a.part_l[pr]);
  }
  if (mx == -INFINITY) {
    *mx_out = 0.f;
    *den_out = 1.f;
    return -INFINITY;
  }
  float den = expf(lse_own - mx);
  for (int l = 0; l < a.merge_levels; ++l) {
    int64_t pr;
    if (level_touches(a.g, bh, i, l, &pr)) den += expf(a.part_l[pr] - mx);
  }
  *mx_out = mx;
  *den_out = den;
  return mx + logf(den);
}

}  // namespace ha
