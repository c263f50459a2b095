// Shared declarations of the HIP side of the HyperAttention library (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "hyperattn.h"

namespace ha {

// ---------------------------------------------------------------------------
// Counter-based generator of the method's random draws (hyperplanes of
// Definition 1, sample indices of Algorithm 2).  SplitMix64's output function
// keyed by (seed, stream) and indexed by a counter; integer-only, so the host
// and the device produce the same indices.
// ---------------------------------------------------------------------------
__host__ __device__ inline uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
__host__ __device__ inline uint64_t rand_u64(uint64_t seed, uint64_t stream, uint64_t ctr) {
  const uint64_t g = 0x9E3779B97F4A7C15ull;
  const uint64_t key = mix64(seed + g * (stream + 1));
  return mix64(key + g * (ctr + 1));
}
constexpr uint64_t kStreamTauRows = 0;
constexpr uint64_t kStreamProjection = 1;
constexpr uint64_t kStreamSamples = 2;  // + heap index (1-based) of the node

__host__ __device__ inline int32_t sample_index(uint64_t seed, int level, int node, int n_keys, int j) {
  const uint64_t stream = kStreamSamples + (1ull << level) + (uint64_t)node;
  const uint64_t hi = rand_u64(seed, stream, (uint64_t)j) >> 32;
  return (int32_t)((hi * (uint64_t)n_keys) >> 32);
}

// ---------------------------------------------------------------------------
// Geometry of one forward call, shared by host validation and kernels.
// Unmasked problem: one level, one node of s = n rows per head.
// Causal problem (Algorithm 4): level l has 2^l nodes of s = n >> (l+1) rows;
// node j takes queries [(2j+1)s, (2j+2)s) and keys [2js, (2j+1)s).
// ---------------------------------------------------------------------------
struct Geometry {
  int32_t BH, n, d, dtype;
  int32_t b, m, r, causal, n_min;
  int32_t levels;       // node levels (0 if causal and n <= n_min)
  int32_t total_nodes;  // per head
  int32_t n_cov;        // rows covered per level per head
  int32_t base_len;     // causal: rows of one exact diagonal block (n if n <= n_min)
};

struct NodeRef {
  int32_t s;        // rows (queries = keys) in the node
  int32_t q_start;  // first query row within the head
  int32_t k_start;  // first key row within the head
  int32_t heap;     // 0-based heap index: (1 << level) - 1 + node
};

__host__ __device__ inline NodeRef node_ref(const Geometry& g, int level, int node) {
  NodeRef nr;
  if (g.causal) {
    nr.s = g.n >> (level + 1);
    nr.q_start = (2 * node + 1) * nr.s;
    nr.k_start = (2 * node) * nr.s;
  } else {
    nr.s = g.n;
    nr.q_start = 0;
    nr.k_start = 0;
  }
  nr.heap = (1 << level) - 1 + node;
  return nr;
}

// ---------------------------------------------------------------------------
// Arguments of the attention kernels (the bf16 and the fp32 kernels share them).
// ---------------------------------------------------------------------------
enum AttnMode : int32_t {
  kModeNode = 0,   // unmasked node(s): block keys by list + kept sampled keys
  kModeExact = 1,  // contiguous keys, optional causal mask (exact attention / causal base case)
  kModeCap = 2,    // node mode with Algorithm 2's cap on every sampled entry and its lower cap
  kModeValue = 3,  // cap mode for the row sums, Lemma 2's rows for the output (fp32)
};

// Division of 0 <= n < 2^31 by a divisor known on the host: two scalar multiplications and a shift, where
// a division by a kernel argument is some thirty vector instructions.  A node workgroup's place took eight of them (and a
// 64-bit one) ahead of its first load.  Measured (MI355X) with one barrier less in the key list: forward + backward,
// 12 heads, n = 16384, d = 64: 234.7 -> 231.8 us; what the forwards gained (up to 1 %) is no more than two runs of one
// build differ.
struct FastDiv {
  uint32_t mul, shift, d;
  __host__ __device__ inline int div(int n) const { return (int)(((uint64_t)(uint32_t)n * mul) >> shift); }
};
inline FastDiv make_fast_div(int64_t divisor) {  // 1 <= divisor < 2^31: mul = ceil(2^shift / divisor) < 2^32, 2^shift >= 2^31 divisor
  FastDiv f;
  f.d = (uint32_t)(divisor < 1 ? 1 : divisor);
  uint32_t log = 0;
  while ((1ull << log) < f.d) ++log;
  f.shift = 31 + log;
  f.mul = (uint32_t)(((1ull << f.shift) + f.d - 1) / f.d);
  return f;
}

struct AttnArgs {
  const void* Q;  // [BH][rows_q][d]
  const void* K;  // [BH][rows_k][d]
  const void* V;
  int64_t q_bh_stride, k_bh_stride;  // elements between heads
  // node mode
  const int32_t* perm_q;   // [levels][BH][n_cov] or null (sorted position == row)
  const int32_t* perm_k;   // same, or null
  const int32_t* pos_k;    // [levels][BH][n_cov]; null => pos == row
  const int32_t* samples;  // [total_nodes][m] node-local key indices; null or m == 0 => none
  const int32_t* samp_blk; // [BH][total_nodes][m] sorted block of each sampled key; null => look up pos_k
  int32_t use_block;       // 0: residual part alone
  // small nodes (node_sort.h): bucket codes [BH][n]; the attention launch sorts by itself and writes the four arrays above
  const uint8_t* codes_q;  // null: they are there
  const uint8_t* codes_k;
  int32_t* perm_q_out;
  int32_t* perm_k_out;
  int32_t* pos_k_out;
  int32_t* samp_blk_out;
  // outputs
  void* out;        // final output in dtype (may be null)
  float* lse;       // final log row sum (may be null)
  float* out_f32;   // optional unrounded copy of the final output (bf16 tensors; may be null)
  void* part_o;     // outputs [levels][BH][n_cov][d] (node mode when non-null; merged in by the base case):
                    // bf16 if part_bf16, else fp32
  float* part_l;
  int32_t part_bf16;
  int64_t out_bh_stride;  // elements between heads of `out` ; lse stride = out_bh_stride / d
  int32_t scatter_out;    // node mode: 1 => write row perm_q[p], 0 => write sorted position p
  Geometry g;
  // node mode, set by the launchers (set_node_divs): tiles per level, heads, tiles per block, blocks of the last level's nodes;
  // exact mode (set_exact_divs): div_tpb tiles per block, div_unit blocks per head, div_tpl blocks of all heads
  FastDiv div_tpl, div_bh, div_tpb, div_unit;
  int32_t wg_first;  // fp32 kernel and cap mode: number of the launch's first workgroup, where a call takes several launches
  // cap mode: log tau of every node [BH][total_nodes], the constant of C_i and kappa (<= 0: that cap is off)
  const float* log_tau;
  float cap_scale, kappa;
  // value mode: every node's rows drawn by value norm and their log weights, [BH][total_nodes][m]
  const int32_t* vsamp;
  const float* vlogw;
  // Algorithm 2, causal: log of the scale that partial rows are taken against, [levels][BH][n_cov] like part_l; null: part_l itself.
  // Uncapped weights can exceed the capped row sum by more than an exponent holds, so a row is normalised by the larger of
  // its sum and its weights' reference, and the merge undoes that.  (Normalised by the sum alone, 71 of 2048 rows of clustered inputs
  // were NaN in fp32, 33 wrong in bf16: d = 64, n_min = 512, b = m = 64, cap 8.  Time: 32 causal heads, n = 32768, d = 128 2146 -> 2163 us, the
  // forward's base case as before.)
  float* part_ref;
  // exact mode
  int32_t exact_rows_q, exact_rows_k;  // rows per head (full problem)
  int32_t exact_block;                 // rows per independent diagonal block (== rows for full attention)
  int32_t exact_causal;
  int32_t exact_lpt;                   // set by the launchers: workgroups that fill a CU each (exact_place)
  int32_t merge_levels;                // exact mode: merge part_o/part_l of this many levels into the result
  // measurement only (null in every product call): kStampWords 64-bit words per workgroup, indexed by the
  // workgroup's logical tile number, written by the instrumented instantiation of the MFMA kernel
  long long* stamps;
};

// Words of a workgroup's stamp record: shader-clock readings at entry, after the key list is built,
// before the tile loop (first scores done), after the loop and at the end; the constant-rate
// counter at entry and at the end; the number of key tiles.
constexpr int kStampWords = HA_STAMP_WORDS;

constexpr int64_t kMaxLaunch = 1 << 23;  // workgroups of 256 threads per launch: the threads of one are counted in 32 bits

// launchers (defined in the .hip files)
int launch_seg_sort_nodes(const uint8_t* codes_q, const uint8_t* codes_k, int32_t* perm_q, int32_t* perm_k,
                          int32_t* pos_k, const int32_t* samples, int32_t* samp_blk, uint32_t* chunk_hist,
                          const Geometry& g, hipStream_t st, int32_t* pos_q = nullptr);  // pos_q: as pos_k, for the queries
int64_t seg_sort_chunks(const Geometry& g);  // rows of 256 counters the chunked sort needs
int launch_seg_sort_flat(const uint8_t* codes, int32_t* perm, int32_t* pos, int n_seg, int seg_len,
                         hipStream_t st);
int launch_attn_mfma(const AttnArgs& a, int mode, hipStream_t st);
int64_t attn_mfma_grid(const AttnArgs& a, int mode);  // workgroups of the four-wave launch of that mode
bool attn_mfma_sorts(const Geometry& g);               // whether the node launch sorts its nodes by itself
int launch_attn_f32(const AttnArgs& a, int mode, hipStream_t st);
bool f32_exact_eight(const AttnArgs& a);  // whether eight waves share 32 rows of an exact fp32 launch
bool attn_f32_sorts(const Geometry& g);               // whether the node launch sorts its nodes by itself
int attn_f32_node_ways(const Geometry& g);            // ways of its workgroups (attn_f32.hip)
int launch_gather_rows(const void* src, const int32_t* idx, void* dst, int groups, int n, int d, int dtype,
                       hipStream_t st);
int launch_merge_unpermute(const float* o_b, const float* lse_b, const float* o_r, const float* lse_r,
                           const int32_t* perm_q, void* out, float* lse, int groups, int n, int d, int dtype,
                           hipStream_t st);

inline int check_launch() { return hipGetLastError() == hipSuccess ? HA_OK : HA_ERR_LAUNCH; }

// Lets kernel `fn` use up to 160 KiB of dynamic LDS on the current device.  The
// attribute is per device; `done` (one per kernel instantiation) remembers the
// devices already set, so concurrent callers and several devices are both fine.
inline int allow_full_lds(const void* fn, std::atomic<uint64_t>& done) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return HA_ERR_LAUNCH;
  const uint64_t bit = 1ull << (dev & 63);
  if (dev < 64 && (done.load(std::memory_order_acquire) & bit)) return HA_OK;
  if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess) {
    (void)hipGetLastError();
    return HA_ERR_LAUNCH;
  }
  if (dev < 64) done.fetch_or(bit, std::memory_order_release);
  return HA_OK;
}

}  // namespace ha
