// fp32 products on the bf16 matrix cores, to the precision of fp32 ones.
//
// A float's 24 significant bits are three bf16 numbers: x = hi + mid + lo, without remainder (hi: x rounded to 8 bits; mid: what is left,
// rounded; lo: what is left then).  Of the nine products of two such numbers six are formed, exactly, and summed in fp32 by
// v_mfma_f32_32x32x16_bf16: six instructions of 32 cycles for 16 terms, where v_mfma_f32_32x32x2_f32 takes eight of 64.  The three left out are at
// most 2^-24.2 of the whole; one product, rounded, is off by at most 2^-23.2, r.m.s. 2^-25.21 over all mantissas (a fused fp32 product 2^-24,
// 2^-25.24).  (hi cut off instead of rounded: 2^-22 and 2^-24.85.  mid lo and lo mid formed as well: 2^-24 and 2^-25.24, for 5 to 20 % of
// the calls' time.)  The sums are rounded once per 16 terms instead of once per two, so that errors fall wherever more than a term or two counts.
// Errors against 64 bits, fp32 instruction -> split (2-norm, relative; exact attention, 2 heads, n = 2048):
//   d = 64: out 4.3e-7 -> 2.9e-7, dQ 5.4e-7 -> 4.3e-7, dK 5.5e-7 -> 4.3e-7, dV 5.7e-7 -> 4.6e-7; causal 2.7e-7 -> 1.5e-7, 3.6e-7 -> 2.5e-7, 5.0e-7 -> 3.6e-7,
//   4.7e-7 -> 3.5e-7; 64 clusters, scores to 250: 2.0e-5 -> 8.6e-6, 2.2e-5 -> 1.3e-5, 1.9e-5 -> 9.3e-6, 2.1e-5 -> 9.9e-6; d = 128 likewise
//   scores to 250 and gradients that one column carries (geometric means of eight shapes): dK 2.6e-7 -> 2.3e-7, dV 2.5e-7 -> 1.9e-7, largest of a log row
//   sum 1.5e-5 both; two of d columns: dQ 9.4e-6 -> 9.1e-6, dK 1.5e-5 -> 1.4e-5, dV 3.1e-6 -> 3.4e-6, log row sum 1.2e-4 -> 8.5e-5
// The matrix cores take parts below 2^-126 as zeros: numbers of the tensors (split at half their value) are taken with an absolute error of up
// to 2^-125, computed ones with 2^-126, so that 24 bits are kept from 2^-101 upwards.  Errors of dQ at values of 2^-100 are
// those of 1 (5.1e-7 against 5.0e-7); fp32 instructions hold theirs down to 2^-116.  2^-100 is what the criterion for
// gradients takes for zero.
//
// What it costs is vector work: 13 instructions per two numbers, 208 for a wave's operand of 32 rows of 64 floats, beside 24 products.  So
// where several waves use a tile it is split once and kept in LDS (SplitTile).
#pragma once

#include "attn_common.h"

namespace ha {

typedef __bf16 split_bf16x8 __attribute__((ext_vector_type(8)));
typedef float split_f32x16 __attribute__((ext_vector_type(16)));
typedef float split_f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t split_u32x4 __attribute__((ext_vector_type(4)));

struct Split8 {  // eight numbers, a lane's share of an operand
  split_bf16x8 hi, mid, lo;
};

// An infinity's hi is infinite and its mid and lo are NaN: of its products only that of hi and hi counts (split_bound).
template <class F>
__device__ inline Split8 split8(F&& x) {
  auto upper = [](uint32_t w) { return __uint_as_float(w & 0xffff0000u); };
  auto lower = [](uint32_t w) { return __uint_as_float(w << 16); };
  split_u32x4 h, m, l;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float a = x(2 * e), b = x(2 * e + 1);
    h[e] = pack_bf16x2(a, b);
    const float ra = a - lower(h[e]), rb = b - upper(h[e]);
    m[e] = pack_bf16x2(ra, rb);
    const float la = ra - lower(m[e]), lb = rb - upper(m[e]);
    l[e] = __builtin_amdgcn_perm(__float_as_uint(lb), __float_as_uint(la), 0x07060302u);
  }
  Split8 s;
  s.hi = __builtin_bit_cast(split_bf16x8, h);
  s.mid = __builtin_bit_cast(split_bf16x8, m);
  s.lo = __builtin_bit_cast(split_bf16x8, l);
  return s;
}

// Numbers of the caller's tensors, at half their value: rounding hi up leaves the largest ones finite.
constexpr float kSplitRaw = 0.5f;
template <class F>
__device__ inline Split8 split8_raw(F&& x) {
  return split8([&](int e) { return x(e) * kSplitRaw; });
}

__device__ inline split_f32x16 split_mfma(split_bf16x8 a, split_bf16x8 b, split_f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// The products of a b but that of hi and hi, smallest first
__device__ inline void split_small(const Split8& a, const Split8& b, split_f32x16& small) {
  small = split_mfma(a.lo, b.hi, small);
  small = split_mfma(a.hi, b.lo, small);
  small = split_mfma(a.mid, b.mid, small);
  small = split_mfma(a.mid, b.hi, small);
  small = split_mfma(a.hi, b.mid, small);
}

// Their sum, or something finite that takes no sum past the largest number.  Where an operand is infinite or a product overflows, hi and hi
// have the result that fp32 has, and what the other products have, an infinity of either sign or NaN, must not be added to it.  (They are at
// most 2^-8 of theirs: 2^126 is none of a sum that is finite.)
__device__ inline float split_bound(float small) {
  return __builtin_amdgcn_fmed3f(small, -0x1p126f, 0x1p126f);
}

// A score's: the small products in a sum of their own, so that its rounding is that of a few additions of 16 terms, and the same whichever
// operand is a.
__device__ inline void split_product(const Split8& a, const Split8& b, split_f32x16& big, split_f32x16& small) {
  split_small(a, b, small);
  big = split_mfma(a.hi, b.hi, big);
}

// c += small, here: behind a branch the compiler (ROCm 7.2) counts the wait states from the last product to its first reader along one
// of the two ways only, and on the other the reader came too early.  Of raw operands the sum is the score times kSplitRaw^2; kSplitScore takes it
// back where its reader has an fma for it.
constexpr float kSplitScore = 1.f / (kSplitRaw * kSplitRaw);
template <bool BOUND>
__device__ inline void split_sum(split_f32x16& c, const split_f32x16& small) {
#pragma unroll
  for (int i = 0; i < 16; ++i) c[i] += BOUND ? split_bound(small[i]) : small[i];
  asm volatile("" : "+v"(c));
}

// acc[k] += a(k, 0) b[0] + a(k, 1) b[1] for N accumulators, 32 rows of a tile.
// kSumTile: a tile's sum is rounded once.  Where one wave's sums run over all tiles of a long row, twelve roundings a tile (kSumEach) are most of
// the result's error (exact attention, n = 4013, one way: out 1.1e-6 -> 2.9e-7).  The sum is added while the next accumulator's
// products run: behind its own the wave waits for the last of them.  kSumSmall, three roundings: for the dK / dV passes of one way at d = 64, which
// have no registers for it (backward, exact, 32 heads, n = 1024 244 -> 226 us, 16 heads, n = 4096 1402 -> 1380).
// BOUND: the small products are bounded before they are added.  A workgroup, or a wave whose tiles are its own, forms its sums without that first; only where they
// hold an infinity or NaN, which a product of parts may have left there, it forms them again with it (split_finite).  (Bounded always, exact passes of one way took
// 8 % longer forward and 15 % backward at d = 128, where a SIMD has one wave; a branch at each tile left the passes 100 to 300 bytes of spills.)
enum SplitSum { kSumEach, kSumSmall, kSumTile };
template <int N, SplitSum SUM, bool BOUND, class A>
__device__ inline void split_tile_products(A&& a, const Split8 (&b)[2], split_f32x16* acc) {
  if constexpr (BOUND || SUM == kSumSmall) {
#pragma unroll
    for (int k = 0; k < N; ++k) {
      split_f32x16 t;
      split_bf16x8 hi[2];
#pragma unroll
      for (int i = 0; i < 16; ++i) t[i] = 0.f;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const Split8 f = a(k, s);
        split_small(f, b[s], t);
        hi[s] = f.hi;
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[k][i] += BOUND ? split_bound(t[i]) : t[i];
#pragma unroll
      for (int s = 0; s < 2; ++s) acc[k] = split_mfma(hi[s], b[s].hi, acc[k]);
      __builtin_amdgcn_sched_barrier(0);
    }
  } else if constexpr (SUM == kSumTile) {
    split_f32x16 t[2];
#pragma unroll
    for (int k = 0; k < N; ++k) {
#pragma unroll
      for (int i = 0; i < 16; ++i) t[k & 1][i] = 0.f;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const Split8 f = a(k, s);
        split_small(f, b[s], t[k & 1]);
        t[k & 1] = split_mfma(f.hi, b[s].hi, t[k & 1]);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (k > 0) acc[k - 1] += t[(k - 1) & 1];
    }
    acc[N - 1] += t[(N - 1) & 1];
  } else {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int k = 0; k < N; ++k) {
        const Split8 f = a(k, s);
        split_small(f, b[s], acc[k]);
        acc[k] = split_mfma(f.hi, b[s].hi, acc[k]);
      }
  }
}

// Behind a loop of products, ahead of what reads its sums: the wait states of the last one whichever way the loop was left (split_sum).
__device__ inline void split_settle() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 15" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Whether a lane's sums are finite
template <int N>
__device__ inline bool split_finite(const split_f32x16 (&acc)[N]) {
  float z[2] = {0.f, 0.f};
#pragma unroll
  for (int k = 0; k < N; ++k)
#pragma unroll
    for (int i = 0; i < 16; i += 4) {  // (maxima that a NaN passes through)
      z[0] = __builtin_elementwise_maximum(__builtin_elementwise_maximum(z[0], __builtin_fabsf(acc[k][i])), __builtin_fabsf(acc[k][i + 1]));
      z[1] = __builtin_elementwise_maximum(__builtin_elementwise_maximum(z[1], __builtin_fabsf(acc[k][i + 2])), __builtin_fabsf(acc[k][i + 3]));
    }
  return __builtin_elementwise_maximum(z[0], z[1]) <= 3.40282347e38f;
}

// The same of a workgroup of NW waves, where their loops have barriers: each wave posts its lanes' ahead of a barrier, all read it behind that.
template <int NW>
struct SplitFinite {
  static constexpr int BYTES = NW * 4;
  int32_t* flags;
  __device__ void post(int wave, bool finite) const {
    const int all = __all(finite);
    if (__lane_id() == 0) flags[wave] = all;
  }
  __device__ bool all() const {
    int f = 1;
#pragma unroll
    for (int w = 0; w < NW; ++w) f &= flags[w];
    return __builtin_amdgcn_readfirstlane(f) != 0;
  }
};

// A tile of 32 rows in LDS: three planes of bf16 rows, unpadded; piece c (16 bytes) of row r sits at place c ^ swz(r), which keeps the
// writes and both readers free of bank conflicts (attn_bwd_mfma.hip's layout).
template <int D>
struct SplitTile {
  static constexpr int ROWB = D * 2, PLANE = 32 * ROWB, BYTES = 3 * PLANE;
  static constexpr int PPR = D / 8;  // pieces per row
  __device__ static int swz(int row) {
    if (D == 128) return ((row & 3) << 2) | ((row >> 2) & 3);
    return ((row & 2) << 1) | ((row >> 2) & 3);
  }
  __device__ static void store(unsigned char* tile, int row, int piece, split_f32x4 x0, split_f32x4 x1) {
    store(tile, row, piece, split8_raw([&](int e) { return e < 4 ? x0[e] : x1[e - 4]; }));
  }
  __device__ static void store(unsigned char* tile, int row, int piece, const Split8& s) {
    unsigned char* at = tile + row * ROWB + ((piece ^ swz(row)) << 4);
    *reinterpret_cast<split_bf16x8*>(at) = s.hi;
    *reinterpret_cast<split_bf16x8*>(at + PLANE) = s.mid;
    *reinterpret_cast<split_bf16x8*>(at + 2 * PLANE) = s.lo;
  }
  // Row lane & 31, columns 16 s + 8 h ... + 7; `at` = row_at(lane).
  __device__ static int row_at(int lane) {
    const int row = lane & 31;
    return row * ROWB + (((lane >> 5) ^ swz(row)) << 4);
  }
  __device__ static Split8 row_frag(const unsigned char* tile, int at, int s) {
    const unsigned char* p = tile + (at ^ (32 * s));
    return Split8{*reinterpret_cast<const split_bf16x8*>(p), *reinterpret_cast<const split_bf16x8*>(p + PLANE),
                  *reinterpret_cast<const split_bf16x8*>(p + 2 * PLANE)};
  }
  // Column 32 dt + (lane & 31) of rows 16 j + 4 h ... + 3 and 16 j + 8 + 4 h ... + 3, the rows of accumulator elements 8 j ... 8 j + 7;
  // `at` = col_at(lane).
  __device__ static int col_at(int lane) {
    const int row = 4 * (lane >> 5) + ((lane & 15) >> 2);
    return row * ROWB + (((((lane >> 4) & 1) * 2 + ((lane & 3) >> 1)) ^ swz(row)) << 4) + (lane & 1) * 8;
  }
  __device__ static Split8 col_frag(const unsigned char* tile, int at, int j, int dt) {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    typedef s16x4 __attribute__((address_space(3))) * lds_s16x4_ptr;
    auto plane = [&](const unsigned char* p) {
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + (at ^ (64 * dt)) + 16 * j * ROWB));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + (at ^ (64 * dt + 32)) + (16 * j + 8) * ROWB));
      return __builtin_bit_cast(split_bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    return Split8{plane(tile), plane(tile + PLANE), plane(tile + 2 * PLANE)};
  }
};

}  // namespace ha
