// sortLSH hashing of bf16 rows (Definition 1; Algorithm 1, "hash rows of Q, K")
// at HBM speed: the r projections of 32 rows are one chain of bf16 MFMAs, and
// only the rare rows whose sign that arithmetic cannot certify are redone in
// exact fp64.
//
//   P   = X R          32 rows x 32 columns (r of them real) per wave and trip
//   P'  = |X| |R|      same shape: sum_c |x_c R_ck|, the scale of the rounding error
//
// A wave reads 32 rows straight from global memory in the MFMA's operand layout
// (lane l: row l%32, 8 consecutive elements starting at 16*ks + 8*(l/32); or, of
// a large problem, as they lie and into that layout through LDS); R
// and |R| sit in registers as the other operand.  The products are formed as
// R^T X^T so that a lane ends up with the projections of ONE row.  bf16 x bf16 products are exact; the
// fp32 accumulation of the d products deviates from the exact sum by far less
// than 2^-14 * P' (d <= 128 terms, fp32 unit roundoff 2^-24 per add, with a 4x
// margin for the matrix core's internal order).  So sign(P) is certified
// wherever |P| > 2^-14 P'; any row with an uncertified projection (a fraction
// of a percent of rows) is recomputed by the whole wave in fp64, whose sum of
// exact products carries a relative error of about d * 2^-53.  The resulting
// codes are those of an fp64 evaluation, bit for bit, except for projections
// that vanish to ~1e-13.
//
// At small sizes the way to the first product counts: the bound is scaled by 2^-14 where it is compared, not in the 2 KS
// operand registers, and R for the fp64 path goes to LDS from the registers that hold it, wave by wave, without a barrier
// (15 heads, n = 6300, d = 128, forward: 52.3 -> 50.5 us; 12 heads, n = 4096, d = 64: 28.9 -> 28.3 us).
//
// If R holds values that are not bf16-representable (caller-supplied
// hyperplanes), every row takes the fp64 path.
#include "hash_common.h"

namespace ha {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// A group of 32 rows in LDS: piece c (16 bytes) of row n at place c ^ swz(n), free of bank conflicts for writes of whole rows
// and for reads of one piece of many rows.
template <int D>
struct HashTile {
  static constexpr int ROWB = D * 2, PPR = D / 8, BYTES = 32 * ROWB;
  __device__ static int at(int row, int piece) { return row * ROWB + ((piece ^ (D == 128 ? row & 15 : (row >> 1) & 7)) << 4); }
};

// ARGS: R comes in the arguments (bf16 values by construction), else from a.R.
// STREAM: rows are read as they lie in memory, 1 KiB per instruction and non-temporally, and take the operand layout through LDS
// (stream_rows).
template <int D, bool ARGS, bool STREAM>
__global__ __launch_bounds__(256) void lsh_hash_mfma_kernel(HashArgs a) {
  constexpr int KS = D / 16;
  constexpr int EL = D / 64;  // elements per lane on the fp64 path
  const int lane = threadIdx.x & 63;
  const int n = lane & 31, h = lane >> 5;
  const int r = a.r;
  const int64_t rows = a.rows;
  // wave-uniform, and known to be: group numbers and row addresses stay in scalar registers
  const int64_t wave = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t nwaves = (int64_t)gridDim.x * 4;
  const int64_t gpt = (rows + 31) / 32;  // groups of 32 rows per tensor
  const int64_t ngroups = a.X[1] ? 2 * gpt : gpt;

  auto load_group = [&](int64_t g, u32x4 (&xa)[KS]) {
    const bool second = g >= gpt;
    const int64_t row0 = (second ? g - gpt : g) * 32;
    const uint16_t* X = reinterpret_cast<const uint16_t*>(second ? a.X[1] : a.X[0]) + row0 * D;
    if constexpr (STREAM) {
      const int pieces = (int)(rows - row0 < 32 ? rows - row0 : 32) * HashTile<D>::PPR;
      const u32x4* xs = reinterpret_cast<const u32x4*>(X);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int i = lane + 64 * ks;
        xa[ks] = __builtin_nontemporal_load(xs + (i < pieces ? i : pieces - 1));
      }
      return;
    }
    const int last = (int)(rows - row0 < 32 ? rows - row0 - 1 : 31);
    const u32x4* xp = reinterpret_cast<const u32x4*>(X + (n < last ? n : last) * D + 8 * h);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) xa[ks] = xp[2 * ks];
  };
  // the rows of the next two trips are in flight while the current one is
  // processed; three register sets rotate so nothing is copied
  u32x4 xa[KS], xb[KS], xc[KS];
  int64_t g = wave;
  if (g < ngroups) {
    load_group(g, xa);
    load_group(g + nwaves < ngroups ? g + nwaves : g, xb);
  }

  // matrix operands R^T and |R|^T as bf16: projection n (zero for n >= r)
  u32x4 rb[KS], rabs[KS];
  bool exact = true;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    if constexpr (ARGS) {
      rb[ks] = (u32x4){0, 0, 0, 0};
      if (n < 8) rb[ks] = *reinterpret_cast<const u32x4*>(&a.Rb[n][16 * ks + 8 * h]);
    } else {
      uint32_t pk[4];
#pragma unroll
      for (int e2 = 0; e2 < 4; ++e2) {
        uint32_t lo = 0, hi = 0;
        if (n < r) {
          lo = __float_as_uint(a.R[(16 * ks + 8 * h + 2 * e2) * r + n]);
          hi = __float_as_uint(a.R[(16 * ks + 8 * h + 2 * e2 + 1) * r + n]);
        }
        exact = exact && ((lo & 0xFFFFu) == 0) && ((hi & 0xFFFFu) == 0);
        pk[e2] = (lo >> 16) | (hi & 0xFFFF0000u);
      }
      rb[ks] = (u32x4){pk[0], pk[1], pk[2], pk[3]};
    }
    rabs[ks] = rb[ks] & 0x7FFF7FFFu;
  }
  const bool all_exact = ARGS || __all(exact);

  // for the fp64 path: R, and one row of X per wave.  ARGS: every wave's own copy of R's bf16 rows, straight from its
  // registers (zero beyond r); else R in fp32, eight columns per row, for the workgroup.
  __shared__ __attribute__((aligned(16))) float Rs[ARGS ? 4 : D * 8];
  __shared__ __attribute__((aligned(16))) uint16_t Rw[ARGS ? 4 : 1][8][ARGS ? D : 1];
  __shared__ __attribute__((aligned(16))) uint16_t xrow[4][D];
  const int wv = threadIdx.x >> 6;
  if constexpr (ARGS) {
    if (n < 8) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) *reinterpret_cast<u32x4*>(&Rw[wv][n][16 * ks + 8 * h]) = rb[ks];
    }
  } else {
    for (int i = threadIdx.x; i < D * 8; i += blockDim.x) Rs[i] = i % 8 < r ? a.R[i / 8 * r + i % 8] : 0.f;
  }
  if (a.store_draws) store_draws(a);
  if constexpr (!ARGS) __syncthreads();

  __shared__ __attribute__((aligned(16))) unsigned char tiles[STREAM ? 4 : 1][STREAM ? HashTile<D>::BYTES : 16];
  const uint32_t mask_r = (1u << r) - 1u;
  auto trip = [&](int64_t g, u32x4 (&xs)[KS], u32x4 (&xn)[KS]) {
    const bool second = g >= gpt;
    const int64_t row0 = (second ? g - gpt : g) * 32;
    // unconditional (past the end: this trip's own rows again, a cache hit), so
    // the count of loads in flight is the same on every path and the waits
    // before the MFMAs below leave the two younger groups in flight
    load_group(g + 2 * nwaves < ngroups ? g + 2 * nwaves : g, xn);

    u32x4 xa[KS];
    if constexpr (STREAM) {  // (LDS serves one wave's requests in order)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int i = lane + 64 * ks;
        *reinterpret_cast<u32x4*>(tiles[wv] + HashTile<D>::at(i / HashTile<D>::PPR, i % HashTile<D>::PPR)) = xs[ks];
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) xa[ks] = *reinterpret_cast<const u32x4*>(tiles[wv] + HashTile<D>::at(n, 2 * ks + h));
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) xa[ks] = xs[ks];
    }

    f32x16 p, pa;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      p[i] = 0.f;
      pa[i] = 0.f;
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      p = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, rb[ks]), __builtin_bit_cast(bf16x8, xa[ks]),
                                                  p, 0, 0, 0);
      const u32x4 ax = xa[ks] & 0x7FFF7FFFu;
      pa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, rabs[ks]), __builtin_bit_cast(bf16x8, ax),
                                                   pa, 0, 0, 0);
    }

    // The product is taken transposed (R^T X^T), so accumulator element i < 4 of
    // lane (n, h) is projection 4 h + i of row n: every lane forms one nibble of
    // its row's sign word, and the two halves of the wave swap nibbles.
    uint32_t nib = 0;
    bool lane_doubt = !all_exact;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool real = 4 * h + i < r;
      nib |= (p[i] > 0.f ? 1u : 0u) << i;
      lane_doubt = lane_doubt || (real && !(fabsf(p[i]) > pa[i] * 0x1.0p-14f));
    }
    nib <<= 4 * h;
    uint32_t my_word = (nib | (uint32_t)__shfl_xor((int)nib, 32)) & mask_r;
    const unsigned long long dbal = __ballot(lane_doubt);
    const uint32_t doubt_rows = (uint32_t)dbal | (uint32_t)(dbal >> 32);
    const int64_t left = rows - row0;
    // a wave-uniform row mask, held in scalar registers
    uint32_t redo = __builtin_amdgcn_readfirstlane(doubt_rows);
    if (left < 32) redo &= (1u << left) - 1u;

    // Exact fp64 evaluation of the doubtful rows, one row at a time by the whole
    // wave: the two lanes that hold row j hand it over through LDS, then lane l
    // multiplies elements EL*l .. EL*l + EL - 1 with their rows of R.
    while (redo) {
      const int j = __builtin_ctz(redo);
      redo &= redo - 1;
      if (n == j) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) *reinterpret_cast<u32x4*>(&xrow[wv][16 * ks + 8 * h]) = xa[ks];
      }
      __builtin_amdgcn_wave_barrier();  // LDS serves one wave's requests in order
      double acc[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) acc[k] = 0.0;
#pragma unroll
      for (int e = 0; e < EL; ++e) {
        const double x = (double)__uint_as_float((uint32_t)xrow[wv][lane * EL + e] << 16);
        f32x4 r0, r1;
        if constexpr (ARGS) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            r0[k] = __uint_as_float((uint32_t)Rw[wv][k][lane * EL + e] << 16);
            r1[k] = __uint_as_float((uint32_t)Rw[wv][4 + k][lane * EL + e] << 16);
          }
        } else {
          r0 = *reinterpret_cast<const f32x4*>(&Rs[(lane * EL + e) * 8]);
          r1 = *reinterpret_cast<const f32x4*>(&Rs[(lane * EL + e) * 8 + 4]);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          acc[k] = __builtin_fma(x, (double)r0[k], acc[k]);
          acc[4 + k] = __builtin_fma(x, (double)r1[k], acc[4 + k]);
        }
      }
      __builtin_amdgcn_wave_barrier();
      // transposing butterfly over the 64 lanes: 8 -> 4 -> 2 -> 1 values, then plain
      const bool u1 = (lane & 32) != 0;
      double w4[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double keep = u1 ? acc[4 + q] : acc[q];
        const double send = u1 ? acc[q] : acc[4 + q];
        w4[q] = keep + __shfl_xor(send, 32);
      }
      const bool u2 = (lane & 16) != 0;
      double w2[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const double keep = u2 ? w4[2 + q] : w4[q];
        const double send = u2 ? w4[q] : w4[2 + q];
        w2[q] = keep + __shfl_xor(send, 16);
      }
      const bool u3 = (lane & 8) != 0;
      double ws = (u3 ? w2[1] : w2[0]) + __shfl_xor(u3 ? w2[0] : w2[1], 8);
      ws += __shfl_xor(ws, 4);
      ws += __shfl_xor(ws, 2);
      ws += __shfl_xor(ws, 1);
      // lane l now holds projection (l >> 3) & 7
      const unsigned long long bal = __ballot(ws > 0.0);
      uint32_t word = 0;
#pragma unroll
      for (int k = 0; k < 8; ++k) word |= (uint32_t)((bal >> (8 * k)) & 1ull) << k;
      if (lane == j) my_word = word & mask_r;
    }

    if (lane < 32 && row0 + lane < rows) {
      // position in the reflected Gray sequence: the i with i ^ (i >> 1) == word
      uint32_t idx = my_word;
      idx ^= idx >> 1;
      idx ^= idx >> 2;
      idx ^= idx >> 4;
      (second ? a.codes[1] : a.codes[0])[row0 + lane] = (uint8_t)idx;
    }
  };
  while (g < ngroups) {
    trip(g, xa, xc);
    g += nwaves;
    if (g >= ngroups) break;
    trip(g, xb, xa);
    g += nwaves;
    if (g >= ngroups) break;
    trip(g, xc, xb);
    g += nwaves;
  }
}

// Workgroups of four waves, at most: one per CU, every wave streaming its 32-row groups with two of them ahead; two for rows of 128 bytes,
// whose groups are half the bytes in flight, past 32 groups per wave.  Forward, 512 -> 256 (MI355X, us; groups per wave of 256 workgroups;
// b = m = 64):
//   d = 64: 8 heads, n = 4096 (2) 18.2 -> 17.5, 12 (3) 20.7 -> 20.6, 16 (4) 27.8 -> 27.0, 32 (8) 38.8 -> 38.6; n = 16384: 24 heads (24) 81.4 -> 81.1,
//     32 (32) 110.1 -> 110.0, 40 (40) 138.5 -> 140.0, 48 (48) 162.3 -> 166.6, 64 (64) 216.4 -> 221.6; 64 heads, n = 65536 (256) 845 -> 865;
//     b = m = 256: n = 16384: 29 heads (29) 125.2 -> 125.8, 32 (32) 136.0 -> 135.9, 48 (48) 201.8 -> 204.6; 64 heads, n = 65536 1044 -> 1066
//   d = 128: 4 heads, n = 4096 (1) 18.9 both, 6 (1.5) 24.1 -> 22.2, 8 (2) 25.6 -> 23.8, 12 (3) 35.6 -> 34.6, 16 (4) 40.2 -> 39.2, 32 (8) 59.2 -> 59.1; 24 heads,
//     n = 16384 (24) 147.7 -> 147.3; 32 heads, n = 32768 (64) 394 -> 391; 64 heads, n = 65536 (256) 1525 -> 1511; 32 causal heads, n = 131072 no difference
// The gain of the small calls does not show in the launch's own time (12 heads, n = 4096, d = 64: 7.0 -> 7.3 us in a kernel trace): where it
// comes from is open.  320 to 448: up to 6 % slower at small sizes, 768: 4 to 6 %.
static int most_hash_blocks(int64_t ngroups, int d) { return d == 64 && ngroups > 32 * 4 * 256 ? 512 : 256; }

// In the operand layout a load takes 32 bytes from each of 32 rows, four loads to a line, which non-temporal loads would fetch four times (a
// plain read of 2 GB: 6.4 TB/s so, 3.85 non-temporally; of whole lines 6.3 and 7.0 to 7.2).  From what the Infinity Cache holds (256 MB) on
// the rows are therefore read as they lie and go through LDS; below, what the launch leaves in the caches serves the attention launch.
// Forward, in the operand layout -> as they lie (MI355X, us; Q and K together):
//   d = 128: 46 MB 52.2 -> 53.0, 64 MB 75.2 -> 78.4, 128 MB 127.3 -> 132.4, 256 MB 247.6 -> 244.5, 512 MB 477.3 -> 467.0, 2 GB 1517 -> 1476
//   d = 64: 256 MB 263.3 -> 260.7, 1 GB 1326 -> 1310
// Three or four groups ahead instead of two: no gain.
static bool stream_rows(int64_t bytes) { return bytes >= 256ll << 20; }

template <int D, bool STREAM>
static void launch_d(const HashArgs& a, dim3 grid, hipStream_t st) {
  if (a.R) hipLaunchKernelGGL((lsh_hash_mfma_kernel<D, false, STREAM>), grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL((lsh_hash_mfma_kernel<D, true, STREAM>), grid, dim3(256), 0, st, a);
}

int launch_lsh_hash_mfma(const HashArgs& a, int d, hipStream_t st) {
  if (a.rows <= 0) return HA_OK;
  const int64_t ngroups = (a.rows + 31) / 32 * (a.X[1] ? 2 : 1);
  int64_t blocks = (ngroups + 3) / 4;
  const bool stream = stream_rows(ngroups * 32 * d * 2);
  if (blocks > most_hash_blocks(ngroups, d)) blocks = most_hash_blocks(ngroups, d);
  const dim3 grid((unsigned)blocks);
  if (d == 128) stream ? launch_d<128, true>(a, grid, st) : launch_d<128, false>(a, grid, st);
  else if (d == 64) stream ? launch_d<64, true>(a, grid, st) : launch_d<64, false>(a, grid, st);
  else return HA_ERR_SHAPE;
  return check_launch();
}

}  // namespace ha
