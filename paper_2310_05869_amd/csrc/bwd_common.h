// Declarations shared by the backward-pass kernels and their host driver.
#pragma once

#include "attn_common.h"

namespace ha {

// Passes of the backward kernels.
enum BwdMode : int32_t {
  kBwdDqNode = 0,    // dQ of the node parts: query tiles over their key lists (block keys + kept samples)
  kBwdDqExact = 1,   // dQ of exact attention / the causal base case
  kBwdDkvBlock = 2,  // dK, dV of the block keys of every node: key tiles over the queries of their block
  kBwdDkvSamp = 3,   // dK, dV of the sampled keys of every node: sample slabs over chunks of the node's queries
  kBwdDkvExact = 4,  // dK, dV of exact attention / the causal base case
};

constexpr int kBwdMaxLevels = 24;

typedef float f32x4 __attribute__((ext_vector_type(4)));

struct BwdArgs {
  AttnArgs f;          // tensors, permutations, samples and geometry as in the forward
  const void* dO;      // [BH][n][d], dtype of the tensors
  const float* lse;    // final log row sums [BH][n]
  const float* delta;  // <dO_i, O_i> [BH][n]
  // dQ passes that hold every row once (unmasked problems, exact attention) form delta themselves, from rows of dO that they hold
  // anyway, and store it for the passes behind them; null: it is there.  O: the forward's output; O32: its unrounded
  // copy (bf16 tensors; may be null)
  float* delta_out;
  const void* O;
  const float* O32;
  // Node passes (one launch per level, in level order) accumulate fp32 rows [BH][n][d], natural row
  // order: out1 = dQ (dQ pass) or dK (dK/dV passes), out2 = dV.  The first level that holds a row on
  // the pass's side writes it, later levels add to it.  (base_first: the rows are the gradients of fp32 tensors themselves; the
  // exact passes come first and write every row, and all levels add to it.)  The sampled-key pass writes its own rows
  // (per level, head, node, query chunk, sample) into out1 / out2 instead.
  float* out1;
  float* out2;
  int32_t level;       // node passes: the launch's level
  int32_t base_first;
  // exact passes write the final gradients (tensors' dtype): fin1 = dQ or dK, fin2 = dV, after adding
  // the accumulated node rows lvl1 / lvl2 (null: none) where some level holds the row on that side; so do the node
  // passes of an unmasked problem, whose one node is the whole result: its block-key pass runs after the sampled-key
  // pass and adds the sums of the sampled keys from samp1 / samp2 (null: no samples)
  void* fin1;
  void* fin2;
  const float* lvl1;
  const float* lvl2;
  const float* samp1;
  const float* samp2;
  // sampled-key pass: sorted query positions per workgroup, and (head, node, query chunk) triples over all
  // levels, level after level; a triple owns m consecutive output rows
  int32_t chunk;
  int32_t samp_chunks;
};

// Whether row i of a head lies, at some level l in [0, upto), on the given side of its level-l node of
// Algorithm 4 (query side: second half; key side: first half): whether a node pass before level `upto`
// has a contribution for it.  Unmasked problems have one node that holds every row on both sides.
__host__ __device__ inline bool node_levels_hold(const Geometry& g, int i, bool query_side, int upto) {
  if (!g.causal) return upto > 0;
  for (int l = 0; l < upto; ++l) {
    const bool second = ((i / (g.n >> (l + 1))) & 1) != 0;
    if (second == query_side) return true;
  }
  return false;
}

// Chunks of sorted query positions per node at a level, for the sampled-key pass.
__host__ __device__ inline int bwd_chunks_per_node(const Geometry& g, int chunk, int level) {
  const int s = g.causal ? (g.n >> (level + 1)) : g.n;
  const int clen = s < chunk ? s : chunk;
  return (s + clen - 1) / clen;
}

// (head, node, query chunk) triples over all levels
inline int64_t bwd_sample_chunks(const Geometry& g, int chunk) {
  int64_t total = 0;
  for (int l = 0; l < g.levels; ++l) total += (int64_t)g.BH * (g.causal ? (1 << l) : 1) * bwd_chunks_per_node(g, chunk, l);
  return total;
}

// Sorted query positions per workgroup of the sampled-key pass: 2048, halved while the pass has fewer than 1024
// workgroups of 128 samples (two rounds of the two that a CU holds), but not below 2 m: every chunk writes two fp32 rows
// per sample, at 2 m as many bytes as the bf16 query rows it reads.  Measured against 2048 always: 12 heads, n = 16384,
// d = 64, b = m = 256 (192 workgroups of 256 CUs -> 768) forward + backward 411 -> 342 us; fp32, 4 causal heads,
// n = 4096, m = 64: 445 -> 337 us.
inline int bwd_chunk(const Geometry& g) {
  int chunk = 2048;
  const int64_t slabs = (g.m + 127) / 128;
  while (chunk / 2 >= 256 && chunk / 2 >= 2 * g.m && bwd_sample_chunks(g, chunk) * slabs < 1024) chunk /= 2;
  return chunk;
}

// Rows of the sampled-key pass that the workspace holds: at least one per (head, node, query chunk, sample), by a bound
// that never falls when the rows, heads or samples grow, though the chunk does, so that a workspace
// of the largest problem serves the smaller ones.  A chunk below 2048 is at least 256 and 2 m, which bounds a
// node's rows by s / 2 + m, and came from one twice as long with at most 1023 workgroups of up to 128 samples.
inline int64_t bwd_sample_rows(const Geometry& g) {
  const int64_t longest = bwd_sample_chunks(g, 2048) * g.m;
  int64_t rows = bwd_sample_chunks(g, 256) * g.m;
  const int64_t half = (int64_t)g.levels * g.BH * ((g.n_cov + 1) / 2) + (int64_t)g.BH * g.total_nodes * g.m;
  if (rows > half) rows = half;
  if (rows > 2 * 1023 * 128) rows = 2 * 1023 * 128;
  return rows > longest ? rows : longest;
}

// What a workgroup of QT "R rows" owns in each pass (TileWork: the head, the node, the rows; exact dK / dV
// pass: q0 = first KEY row, [k0, k1) = its queries).
struct BwdWork {
  TileWork w;
  int chunk_start, chunk_len;   // sampled-key pass: run of sorted query positions
  int samp0;                    // first sample
  int64_t samp_row0;            // row of sample 0 of this (head, node, chunk) in the pass's output
};

template <int QT, int MODE>
__device__ inline BwdWork decode_bwd_work(const BwdArgs& a, int idx, int wgs) {  // workgroup idx of the pass's wgs
  const AttnArgs& f = a.f;
  const Geometry& g = f.g;
  BwdWork b{};
  if (MODE == kBwdDqNode || MODE == kBwdDkvBlock) {
    b.w = decode_node_tile<QT>(f, a.level * wgs + idx);
  } else if (MODE == kBwdDqExact) {
    b.w = decode_exact_tile<QT>(f, idx);
  } else if (MODE == kBwdDkvExact) {
    // key tiles of the diagonal blocks
    const int eb = f.exact_block;
    const ExactPlace e = exact_place(f, idx);
    const int ktile = e.rank;  // early key tiles see the most queries
    const int blk = e.blk;
    b.w.bh = e.bh;
    b.w.q0 = blk * eb + ktile * QT;  // first KEY row of this tile
    const int blk_rows = min(eb, f.exact_rows_q - blk * eb);
    b.w.rows_valid = max(0, min(QT, blk_rows - ktile * QT));
    b.w.k0 = f.exact_causal ? b.w.q0 : blk * eb;
    b.w.k1 = blk * eb + blk_rows;     // queries [k0, k1)
  } else {  // kBwdDkvSamp: a slab of QT samples over one chunk of the node's sorted queries
    const int spn = (g.m + QT - 1) / QT;              // sample slabs per node
    const int slab = idx % spn;
    const int cidx = idx / spn;
    int level = 0, left = cidx, cpn;
    for (;;) {
      cpn = bwd_chunks_per_node(g, a.chunk, level);
      const int here = g.BH * (g.causal ? (1 << level) : 1) * cpn;
      if (left < here || level + 1 >= g.levels) break;
      left -= here;
      ++level;
    }
    const int nodes = g.causal ? (1 << level) : 1;
    const int qc = left % cpn;
    const int hn = left / cpn;                         // (head, node)
    const int node = hn % nodes;
    b.w.bh = hn / nodes;
    b.w.level = level;
    b.w.nr = node_ref(g, level, node);
    b.w.seg_off = ((int64_t)level * g.BH + b.w.bh) * g.n_cov + (int64_t)node * b.w.nr.s;
    b.chunk_start = qc * a.chunk;
    b.chunk_len = min(a.chunk, b.w.nr.s - b.chunk_start);
    b.samp0 = slab * QT;
    b.w.rows_valid = min(QT, g.m - b.samp0);
    b.samp_row0 = (int64_t)cidx * g.m;
  }
  return b;
}

// Row within the head of the workgroup's R row r; sampled-key pass: *blk_r = the sorted block of that key.
template <int MODE>
__device__ inline int bwd_r_row(const BwdArgs& a, const BwdWork& b, int r, int* blk_r) {
  const AttnArgs& f = a.f;
  if (MODE == kBwdDqNode) return f.perm_q[b.w.seg_off + b.w.p0 + r];
  if (MODE == kBwdDkvBlock) return f.perm_k[b.w.seg_off + b.w.p0 + r];
  if (MODE == kBwdDkvSamp) {
    const int j = b.samp0 + r;
    *blk_r = f.samp_blk[((int64_t)b.w.bh * f.g.total_nodes + b.w.nr.heap) * f.g.m + j];
    return b.w.nr.k_start + f.samples[(int64_t)b.w.nr.heap * f.g.m + j];
  }
  return b.w.q0 + r;
}

// Where its gradient goes: row of out1 / out2 (sampled-key pass: a row of its own per sample) or of fin1 / fin2.
template <int MODE>
__device__ inline int64_t bwd_out_row(const BwdArgs& a, const BwdWork& b, int r, int row) {
  if (MODE == kBwdDkvSamp) return b.samp_row0 + b.samp0 + r;
  return (int64_t)b.w.bh * a.f.g.n + row;
}

// The sampled keys among a workgroup's key rows (block-key pass of an unmasked problem).  A sample belongs to the one workgroup that holds
// its sorted position, which adds its sums to the key's row: one writer per key, a fixed order of additions.  first[r] =
// the lowest sample that drew row r (kNoSample: none), whose sums arrive together with the rows' earlier ones; further
// draws of a row, rare, go to the list `more` in sample order, entries row << 16 | sample, and are added one by one.
// All NT threads call it; the results are visible after the caller's next barrier.
//
// Unmasked only: it takes the place of fp32 rows in memory, a launch that adds the samples' sums to them and three that
// convert them.  Measured (MI355X): forward + backward, 12 heads, n = 16384, d = 64: 286 -> 247 us.  In a
// causal problem the rows accumulate over the levels in memory anyway, and the same form lost: block keys of a level
// 1.21 -> 1.29 ms (32 heads, n = 131072, d = 128) for 0.08 ms less of the samples' launches.
constexpr int kNoSample = 0x7fffffff;
struct SampleHits {
  int32_t* first;   // [128]
  int32_t* more;    // [m]
  int32_t* count;   // more's entries
  int32_t* scratch; // one int per wave
};
__host__ __device__ inline size_t sample_hits_bytes(const Geometry& g) { return (128 + 8 + (size_t)g.m) * 4; }
__device__ inline SampleHits sample_hits(unsigned char* lds) {
  int32_t* p = reinterpret_cast<int32_t*>(lds);
  return SampleHits{p, p + 136, p + 128, p + 132};
}
// `head`: fetch_sample_head's values of the thread, asked for ahead of other waits.
struct SampleHead {
  int blk, key;  // sample `tid`: its sorted block and its index in the node
};
__device__ inline SampleHead fetch_sample_head(const BwdArgs& a, const BwdWork& b, int j) {
  const AttnArgs& f = a.f;
  SampleHead h{-1, 0};
  if (a.samp1 != nullptr && j < f.g.m) {
    h.blk = f.samp_blk[((int64_t)b.w.bh * f.g.total_nodes + b.w.nr.heap) * f.g.m + j];
    h.key = f.samples[(int64_t)b.w.nr.heap * f.g.m + j];
  }
  return h;
}
template <int NT>
__device__ inline void find_sample_hits(const BwdArgs& a, const BwdWork& b, const SampleHits& out, SampleHead head) {
  const AttnArgs& f = a.f;
  const int m = a.samp1 != nullptr ? f.g.m : 0;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid < 128) out.first[tid] = kNoSample;
  __syncthreads();
  int n = 0;
  for (int j0 = 0; j0 < m; j0 += NT) {
    const int j = j0 + tid;
    if (j0 > 0) head = fetch_sample_head(a, b, j);
    int row = head.blk == b.w.t ? f.pos_k[b.w.seg_off + head.key] - b.w.p0 : -1;
    if (row >= b.w.rows_valid) row = -1;
    if (row >= 0) atomicMin(&out.first[row], j);
    __syncthreads();
    const bool again = row >= 0 && out.first[row] != j;
    const unsigned long long bal = __ballot(again);
    if (lane == 0) out.scratch[wave] = __popcll(bal);
    __syncthreads();
    int at = n;
#pragma unroll
    for (int ww = 0; ww < NT / 64; ++ww) {
      if (ww < wave) at += out.scratch[ww];
      n += out.scratch[ww];
    }
    if (again) out.more[at + __popcll(bal & ((1ull << lane) - 1ull))] = row << 16 | j;
    // (the next trip writes scratch only after a barrier)
  }
  if (tid == 0) *out.count = n;
}

// Workgroups of QT R rows in a launch; node passes: of one level.
template <int QT>
inline int64_t bwd_grid(const BwdArgs& a, int mode) {
  const Geometry& g = a.f.g;
  if (mode == kBwdDqNode || mode == kBwdDkvBlock) return g.levels > 0 ? node_grid<QT>(g) / g.levels : 0;
  if (mode == kBwdDqExact || mode == kBwdDkvExact) return exact_grid<QT>(a.f);
  return (int64_t)a.samp_chunks * ((g.m + QT - 1) / QT);
}

int launch_attn_bwd_mfma(const BwdArgs& a, int mode, hipStream_t st);  // bf16 tensors
int launch_attn_bwd_f32(const BwdArgs& a, int mode, hipStream_t st);   // fp32 tensors
// Passes of an fp32 causal problem that do not wait for each other, in one launch: the base case's dK / dV and dQ with the
// sampled keys, or a level's block keys with its dQ (bwd_f32_shares: whether the problem is small enough for it).
struct BwdPart {
  BwdArgs a;
  int32_t first, count;  // workgroups
};
struct BwdShared {
  BwdPart part[3];
};
bool bwd_f32_shares(const BwdArgs& a);
int bwd_f32_node_ways(const BwdArgs& a);  // ways of the node passes' workgroups in launches of their own (attn_bwd_f32.hip)
int64_t bwd_f32_shared_workgroups(const BwdArgs& a);  // of the larger of those launches
int launch_attn_bwd_f32_base(const BwdArgs& dkv, const BwdArgs& dq, const BwdArgs* samp, hipStream_t st);
int launch_attn_bwd_f32_level(const BwdArgs& block, const BwdArgs& dq, hipStream_t st);
// delta_i = <dO_i, O_i>; bf16 tensors: O from its unrounded fp32 copy when O_f32 is non-null, else from the tensor
int launch_bwd_delta(const void* O, const float* O_f32, const void* dO, float* delta, int64_t rows, int d, int dtype,
                     hipStream_t st);
// causal: adds the sampled keys' sums of all levels into the accumulated key rows acc_k / acc_v [BH][n][d]
int launch_bwd_sample_scatter(const BwdArgs& a, const float* samp_k, const float* samp_v, float* acc_k, float* acc_v, hipStream_t st);
// unmasked: the sampled keys' rows summed over the query chunks, into those of the first chunk
int launch_bwd_sample_reduce(const BwdArgs& a, float* samp_k, float* samp_v, hipStream_t st);

}  // namespace ha
