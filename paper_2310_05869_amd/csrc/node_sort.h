// The sort of a small node inside the attention kernels: every workgroup finds the rows of its own tile from the node's
// bucket codes, instead of reading them from a permutation that a launch ahead of it wrote.
//
// What bounds a small call is the number of dependent launches, each some 1.5 us before its first instruction and 2 us
// until its first data has arrived, so a chain of LDS passes over the node's codes in every workgroup (6 us with the codes' arrival
// at 4096 keys) beats a sorting launch (6.5 to 8 us and the wait for it), though each workgroup counts the whole node.  Cycles of
// that (four waves, 4096 keys, 128 buckets; counters read at these points in a build made for it: the stamped forward keeps the
// sorting launch): 3.7 k until the codes are there, 2.7 k counting (the LDS atomics), 1.1 k positions, 2.2 k keys
// of the range, 1.9 k ranks, 1.9 k samples and the last barriers; 17.5 k before two waves' counts shared a word and every wave
// formed its own positions (forward, 12 heads, n = 4096, d = 64 28.1 -> 26.4 us; fp32, one head, n = 1024 18.5 -> 17.2).  A stable counting sort by bucket, of which
// only what lies in the workgroup's range of sorted positions is carried out: all keys are counted, the range is found in
// the bucket starts, and only keys of buckets that touch it are ranked.
//
// The workgroup also writes its part of perm_q, perm_k, pos_k and samp_blk (the block's first tile: its keys), bit
// for bit what the sorting launches write: the backward and the workspace's readers need them.
#pragma once

#include "attn_common.h"

namespace ha {

typedef uint32_t codes16 __attribute__((ext_vector_type(4)));
typedef uint32_t codes32 __attribute__((ext_vector_type(8)));

// Keys [16 t, 16 t + 16) of a run of s bucket codes, at any address (heads of an odd number of rows): one 16-byte load where the
// run starts at a 16-byte boundary, else the aligned words that hold a key of the run.  Keys past the end are undefined.
__device__ inline codes16 load_16_codes(const uint8_t* codes, int s, int t) {
  const int i0 = 16 * t, left = s - i0 < 16 ? s - i0 : 16;
  codes16 v = {0, 0, 0, 0};
  if (left <= 0) return v;
  const uintptr_t addr = reinterpret_cast<uintptr_t>(codes) + i0;
  if ((reinterpret_cast<uintptr_t>(codes) & 15u) == 0 && left == 16) return *reinterpret_cast<const codes16*>(addr);
  const int skip = (int)(addr & 3u), last = (skip + left - 1) >> 2;
  const uint32_t* words = reinterpret_cast<const uint32_t*>(addr - skip);
  uint32_t raw[5];
#pragma unroll
  for (int k = 0; k < 5; ++k) raw[k] = words[k < last ? k : last];
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = __builtin_amdgcn_alignbyte(raw[k + 1], raw[k], skip);
  return v;
}

// Keys [4 N t, 4 N (t + 1)) of the run, N = 1 or 2, likewise.
template <int N>
__device__ inline codes32 load_few_codes(const uint8_t* codes, int s, int t) {
  codes32 v = {0, 0, 0, 0, 0, 0, 0, 0};
  const int left = s - 4 * N * t;
  if (left > 0) {
    const uintptr_t addr = reinterpret_cast<uintptr_t>(codes) + 4 * N * t;
    const int skip = (int)(addr & 3u), last = (skip + (left < 4 * N ? left : 4 * N) - 1) >> 2;
    const uint32_t* words = reinterpret_cast<const uint32_t*>(addr - skip);
    const uint32_t r0 = words[0], r1 = words[1 < last ? 1 : last], r2 = words[N < last ? N : last];
    v[0] = __builtin_amdgcn_alignbyte(r1, r0, skip);
    if (N == 2) v[1] = __builtin_amdgcn_alignbyte(r2, r1, skip);
  }
  return v;
}

constexpr int kNodeSortMax = 32 * 64 * 4;  // keys of a node: 32 per thread of the smallest form, four waves

__host__ __device__ inline int node_sort_rows(const Geometry& g) { return ((g.causal ? g.n >> 1 : g.n) + 63) & ~63; }

// Workgroups of `lds` bytes that a CU holds, up to `most` by their registers: its 160 KB are dealt in 128 pieces.
inline int64_t lds_workgroups(size_t lds, int most) {
  const int64_t fit = 128 / (int64_t)((lds + 1279) / 1280);
  return fit < most ? fit : most;
}

typedef uint32_t words4 __attribute__((ext_vector_type(4)));
// half of a word of `pos`, which is written as words4: no two accesses of the table may be taken for independent by their types
typedef uint16_t half_word __attribute__((may_alias));

constexpr int kNodeSortBuckets = 256;

struct NodeSortLds {
  uint8_t* codes;              // [2][rows] the keys' buckets (a wave ranks only keys that its own lanes wrote)
  uint16_t* rel;               // [2][rows] keys of the buckets that touch the range, wave by wave: index in the node
  uint32_t* count;             // [2][wave pairs][kNodeSortBuckets] two waves' counts in a word
  uint32_t* pos;               // [waves][kNodeSortBuckets] sorted position of a wave's next key, queries | keys << 16
  unsigned long long* peers;   // [2][waves][buckets]
  uint32_t* member;            // [rows / 32] bits: keys of the workgroup's block
};
template <int NW>  // waves of the workgroup: 4 or 8
__host__ __device__ inline size_t node_sort_lds_bytes(const Geometry& g) {
  const size_t rows = node_sort_rows(g), buckets = (size_t)1 << g.r;
  return 6 * rows + (NW + NW) * kNodeSortBuckets * 4 + 2 * NW * buckets * 8 + rows / 8;
}
template <int NW>
__device__ inline NodeSortLds node_sort_lds(const Geometry& g, unsigned char* sm) {
  const int rows = node_sort_rows(g), buckets = 1 << g.r;
  NodeSortLds l;
  l.codes = sm;
  l.rel = reinterpret_cast<uint16_t*>(sm + 2 * rows);
  l.count = reinterpret_cast<uint32_t*>(sm + 6 * rows);
  l.pos = l.count + NW * kNodeSortBuckets;
  l.peers = reinterpret_cast<unsigned long long*>(l.pos + NW * kNodeSortBuckets);
  l.member = reinterpret_cast<uint32_t*>(l.peers + 2 * NW * buckets);
  return l;
}

// inclusive sums over the wave's lanes
__device__ inline uint32_t wave_scan(uint32_t x) {
  const int lane = threadIdx.x & 63;
  // within rows of 16 lanes, then the last lane of the row before, then of the first half
  x += __builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true);
  const uint32_t r0 = __builtin_amdgcn_readlane(x, 15), r1 = __builtin_amdgcn_readlane(x, 31), r2 = __builtin_amdgcn_readlane(x, 47);
  return x + (lane >= 16 ? r0 : 0u) + (lane >= 32 ? r1 : 0u) + (lane >= 48 ? r2 : 0u);
}

// The tile's query rows to qrows[0 .. rows_valid) and its block's key rows to list[0 .. b), both rows within the head.
// All threads call it; the results are visible on return.
template <int NW>
__device__ inline void sort_node_tile(const AttnArgs& a, const TileWork& w, unsigned char* sm, int32_t* list, int32_t* qrows) {
  constexpr int NT = 64 * NW;
  static_assert(NW == 4 || NW == 8);
  const Geometry& g = a.g;
  const NodeSortLds l = node_sort_lds<NW>(g, sm);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int s = w.nr.s, rows = node_sort_rows(g), buckets = 1 << g.r;
  const int lo[2] = {w.p0, w.t * g.b}, hi[2] = {w.p0 + w.rows_valid, w.t * g.b + g.b};
  const bool first_tile = w.p0 == w.t * g.b;  // of its block: it writes the block's keys

  // a thread's keys are consecutive, 4, 8, 16 or 32 by the node's size, and so are a wave's: with 16 from the smallest nodes on,
  // one wave did the work of all
  const int wpt = s <= 4 * NT ? 1 : s <= 8 * NT ? 2 : s <= 16 * NT ? 4 : 8;  // words of four keys
  const int per = 4 * wpt, i0 = per * tid;
  codes32 v[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const uint8_t* codes = t ? a.codes_k + (int64_t)w.bh * g.n + w.nr.k_start : a.codes_q + (int64_t)w.bh * g.n + w.nr.q_start;
    if (wpt <= 2) {
      v[t] = wpt == 1 ? load_few_codes<1>(codes, s, tid) : load_few_codes<2>(codes, s, tid);
    } else {
      const codes16 lo4 = load_16_codes(codes, s, i0 / 16), hi4 = wpt == 8 ? load_16_codes(codes, s, i0 / 16 + 1) : lo4;
      v[t] = __builtin_shufflevector(lo4, hi4, 0, 1, 2, 3, 4, 5, 6, 7);
    }
  }
  const words4 zero = {0u, 0u, 0u, 0u};
  static_assert(NT * 4 == NW * kNodeSortBuckets);
  reinterpret_cast<words4*>(l.count)[tid] = zero;
  for (int i = tid; i < NW * buckets; i += NT) reinterpret_cast<words4*>(l.peers)[i] = zero;
  for (int i = tid; i < rows / 32; i += NT) l.member[i] = 0u;
  __syncthreads();

  const int left = s - i0;  // the thread's keys
  const uint32_t code_bytes = (uint32_t)(buckets - 1) * 0x01010101u;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
#pragma unroll
    for (int u = 0; u < 8; ++u) v[t][u] &= code_bytes;
    if (left <= 0) continue;
    uint32_t* dst = reinterpret_cast<uint32_t*>(l.codes + t * rows + i0);
    if (wpt <= 2) {
      dst[0] = v[t][0];
      if (wpt == 2) dst[1] = v[t][1];
    } else {
      reinterpret_cast<words4*>(dst)[0] = (words4){v[t][0], v[t][1], v[t][2], v[t][3]};
      if (wpt == 8) reinterpret_cast<words4*>(dst)[1] = (words4){v[t][4], v[t][5], v[t][6], v[t][7]};
    }
  }
  auto each_key = [&](auto&& f) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (u >= wpt) break;
#pragma unroll
      for (int j = 0; j < 4; ++j) f(4 * u + j, (v[0][u] >> (8 * j)) & 255u, (v[1][u] >> (8 * j)) & 255u);
    }
  };
  uint32_t* count_q = l.count + (wave >> 1) * kNodeSortBuckets;
  uint32_t* count_k = count_q + NW / 2 * kNodeSortBuckets;
  const uint32_t one = 1u << (16 * (wave & 1));
  if (64 * per * (wave + 1) <= s) {  // no key of the wave is past the end
    each_key([&](int, uint32_t cq, uint32_t ck) {
      atomicAdd(&count_q[cq], one);
      atomicAdd(&count_k[ck], one);
    });
  } else {
    each_key([&](int j, uint32_t cq, uint32_t ck) {
      if (j < left) {
        atomicAdd(&count_q[cq], one);
        atomicAdd(&count_k[ck], one);
      }
    });
  }
  __syncthreads();

  // Sorted position of the wave's first key of every bucket, queries and keys in the halves of a word (a node has up to 8192), and the
  // first and the last bucket that touch the range.  Every wave forms them for itself: one wave for the queries and one for the keys had
  // the others wait at a further barrier.
  uint32_t b0[2] = {0u, 0u}, b1[2] = {0u, 0u};
  {
    const words4* tab = reinterpret_cast<const words4*>(l.count) + lane;
    auto both_halves = [](uint32_t x) { return (x & 0xffffu) + (x >> 16); };
    words4 of[2] = {zero, zero}, before[2] = {zero, zero};  // counts of all waves and of the earlier ones, two waves to a word
#pragma unroll
    for (int p = 0; p < NW / 2; ++p) {
      const uint32_t earlier = 2 * p + 1 < wave ? ~0u : 2 * p < wave ? 0xffffu : 0u;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const words4 c = tab[(NW / 2 * t + p) * (kNodeSortBuckets / 4)];
        of[t] += c;
        before[t] += c & earlier;
      }
    }
    uint32_t all[4], sum = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      all[j] = both_halves(of[0][j]) | both_halves(of[1][j]) << 16;
      sum += all[j];
    }
    uint32_t at = wave_scan(sum) - sum;
    words4 first;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      first[j] = at + (both_halves(before[0][j]) | both_halves(before[1][j]) << 16);
      at += all[j];
      const uint32_t end[2] = {at & 0xffffu, at >> 16};
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        b0[t] += __popcll(__ballot(end[t] <= (uint32_t)lo[t]));
        b1[t] += __popcll(__ballot(end[t] < (uint32_t)hi[t]));
      }
    }
    reinterpret_cast<words4*>(l.pos)[wave * (kNodeSortBuckets / 4) + lane] = first;
  }

  // the wave's keys of those buckets, in order, to rel
  const uint32_t span[2] = {b1[0] - b0[0], b1[1] - b0[1]};
  uint32_t hit[2] = {0u, 0u};  // bits: the thread's keys
  each_key([&](int j, uint32_t cq, uint32_t ck) {
    hit[0] |= (cq - b0[0] <= span[0] ? 1u : 0u) << j;
    hit[1] |= (ck - b0[1] <= span[1] ? 1u : 0u) << j;
  });
  const uint32_t real = left >= 32 ? ~0u : left > 0 ? (1u << left) - 1u : 0u;
  int n[2];
  {
    uint32_t bits_q = hit[0] & real, bits_k = hit[1] & real;
    const uint32_t mine = __popc(bits_q) | __popc(bits_k) << 16;
    const uint32_t incl = wave_scan(mine), total = __builtin_amdgcn_readlane(incl, 63), at = incl - mine;
    n[0] = (int)(total & 0xffffu);
    n[1] = (int)(total >> 16);
    uint16_t* dst_q = l.rel + min(64 * per * wave, rows) + (at & 0xffffu);
    uint16_t* dst_k = l.rel + rows + min(64 * per * wave, rows) + (at >> 16);
    while (bits_q | bits_k) {
      if (bits_q) *dst_q++ = (uint16_t)(i0 + __builtin_ctz(bits_q));
      if (bits_k) *dst_k++ = (uint16_t)(i0 + __builtin_ctz(bits_k));
      bits_q &= bits_q - 1;
      bits_k &= bits_k - 1;
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

  // sorted positions: a key's place among the equal keys of its 64 from the lanes' bits in a word per bucket
  const unsigned long long lane_bit = 1ull << lane;
  const int most = n[0] > n[1] ? n[0] : n[1];
  half_word* next = reinterpret_cast<half_word*>(l.pos + wave * kNodeSortBuckets);
  for (int k0 = 0; k0 < most; k0 += 64) {
    uint32_t i[2], c[2];
    bool valid[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      valid[t] = k0 + lane < n[t];
      i[t] = valid[t] ? l.rel[t * rows + 64 * per * wave + k0 + lane] : 0u;
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      c[t] = l.codes[t * rows + i[t]];
      if (valid[t]) atomicOr(&l.peers[(t * NW + wave) * buckets + c[t]], lane_bit);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    unsigned long long pm[2];
    uint32_t seen[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      pm[t] = l.peers[(t * NW + wave) * buckets + c[t]];
      seen[t] = next[2 * c[t] + t];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if (!valid[t]) continue;
      const uint32_t rank = __popcll(pm[t] & (lane_bit - 1ull)), cnt = __popcll(pm[t]);
      if (rank == cnt - 1) {  // one lane per distinct key
        l.peers[(t * NW + wave) * buckets + c[t]] = 0ull;
        next[2 * c[t] + t] = (uint16_t)(seen[t] + cnt);
      }
      const int p = (int)(seen[t] + rank);
      if (p < lo[t] || p >= hi[t]) continue;
      if (t == 0) {
        qrows[p - lo[0]] = w.nr.q_start + (int)i[t];
      } else {
        list[p - lo[1]] = w.nr.k_start + (int)i[t];
        atomicOr(&l.member[i[t] >> 5], 1u << (i[t] & 31));
        if (first_tile) a.pos_k_out[w.seg_off + i[t]] = p;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  __syncthreads();
  for (int i = tid; i < w.rows_valid; i += NT) a.perm_q_out[w.seg_off + lo[0] + i] = qrows[i];
  if (first_tile)
    for (int i = tid; i < g.b; i += NT) a.perm_k_out[w.seg_off + lo[1] + i] = list[i];
}

// Appends the kept samples to the block's keys (build_key_list's list): those that are no keys of the block.  All threads call
// it behind sort_node_tile; on return the list is whole and sm is read no more.  `l0` = sample threadIdx.x, fetched ahead.
template <int NW>
__device__ inline int append_node_samples(const AttnArgs& a, const TileWork& w, unsigned char* sm, int32_t* list,
                                          int32_t* scratch, int l0) {
  constexpr int NT = 64 * NW;
  const Geometry& g = a.g;
  const uint32_t* member = node_sort_lds<NW>(g, sm).member;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m = a.samples != nullptr ? g.m : 0;
  const bool first_tile = w.p0 == w.t * g.b;
  int base = g.b;
  for (int j0 = 0; j0 < m; j0 += NT) {
    const int j = j0 + tid;
    int l = l0;
    bool keep = false;
    if (j < m) {
      if (j0 > 0) l = a.samples[(int64_t)w.nr.heap * g.m + j];
      keep = ((member[l >> 5] >> (l & 31)) & 1u) == 0;  // 1 - M_{i, l_j}: same for every row of the block
      if (first_tile && !keep) a.samp_blk_out[((int64_t)w.bh * g.total_nodes + w.nr.heap) * g.m + j] = w.t;
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
  const int pad = (base + 63) & ~63;
  for (int i = base + tid; i < pad; i += NT) list[i] = w.nr.k_start;  // loadable, masked by position
  __syncthreads();
  return base;
}

__device__ inline int first_node_sample(const AttnArgs& a, const TileWork& w) {
  return a.samples != nullptr && (int)threadIdx.x < a.g.m ? a.samples[(int64_t)w.nr.heap * a.g.m + threadIdx.x] : 0;
}

}  // namespace ha
