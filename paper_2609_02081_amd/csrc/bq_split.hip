// Split-precision real GEMM (Ozaki-style) for gfx950.
//
// A real FP64 product T = X Y (X m x k, Y k x n) is computed from
// low-precision slices:
//   * every row i of X gets a power-of-two exponent e_i (the frexp exponent
//     of its largest magnitude, plus h), every column j of Y an exponent f_j;
//   * x_ij 2^-e_i in (-2^-h, 2^-h) is written as S signed digits,
//     q_1 = rint(2^b y), y_1 = y - q_1 2^-b, q_s = rint(2^{bs} y_{s-1}), ...
//     so x = 2^e_i (sum_s q_s 2^{-bs} + remainder), |q_1| <= 2^{b-h},
//     |q_s| <= 2^{b-1}; the digits are small integers, exact in BF16 (b = 7,
//     h = 0), OCP FP8 E4M3 (b = 5, h = 1: every digit within 16) or INT8
//     (b = 7, h = 1: one bit of headroom keeps the leading digit inside a
//     signed byte);
//   * T_ij = 2^{e_i + f_j} sum_{d = 2}^{S+1} 2^{-bd} sum_{s + t = d} (Q_s R_t)_ij
//     (pairs with s + t > S + 1 are dropped).
// Each level d is accumulated by MFMA in FP32 (BF16/FP8) or int32 (INT8)
// over as many k-steps as keep every partial sum an exact integer (the bound
// is in slice_flush_steps), then added, scaled by 2^{-bd}, into FP64
// accumulators.  Only the splitting, the exponent scaling and the level
// accumulation are FP64.
#include <limits.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "bq_split_common.h"

namespace bq {

// Largest magnitude of a set of doubles, kept as the high words of |x| and
// the low words (which count only where every high word is zero): three
// integer operations an element, and exact exponents down to denormals.
struct MaxMagnitude {
  unsigned hi = 0, lo = 0;
  __device__ __forceinline__ void add(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    hi = max(hi, (unsigned)(u >> 32) & 0x7fffffffu);
    lo = max(lo, (unsigned)u);
  }
  __device__ __forceinline__ void merge(unsigned h, unsigned l) {
    hi = max(hi, h);
    lo = max(lo, l);
  }
  // The frexp exponent plus head, or one of the markers.
  __device__ __forceinline__ int exponent(int head) const {
    if (hi >= 0x7ff00000u) return kExpNonFinite;
    if (hi >= 0x00100000u) return (int)(hi >> 20) - 1022 + head;
    if (hi != 0) return 32 - 1073 + 31 - __builtin_clz(hi) + head;
    return lo != 0 ? 31 - __builtin_clz(lo) - 1073 + head : INT_MIN;
  }
};

// Exponents of 16 rows or columns of the wanted values of an operand, 1024
// threads: where the inner dimension is contiguous a wave per row, else 16
// columns (128 bytes of a stored row) by 64 row lanes.  Indices past the end
// are clamped to the last one (a repeated element leaves the maximum), so the
// loads of four steps are in flight together.  One launch per complex product
// reads r and i once for three exponents; no initialisation and no atomics, but
// for a long inner dimension and few blocks (CHUNK): inner elements c0 .. c1 - 1
// only, the exponent joined to the one in memory (which starts at INT_MIN) by an
// atomic maximum; c0 is even.
constexpr int kExpThreads = 1024;
struct ExpLds {
  unsigned hi[3][16][16], lo[3][16][16];  // value, wave, column
};
template <bool CHUNK>
__device__ __forceinline__ void exponent_block(const SplitOperand& a, int64_t b, int64_t c0, int64_t c1, ExpLds& red) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t K = a.along ? a.cols : a.rows;
  const int64_t begin = CHUNK ? c0 : 0, end = CHUNK ? c1 : K;
  const bool want_i = a.e[1] != nullptr || a.e[2] != nullptr;
  MaxMagnitude mx[3];
  auto add = [&](double r, double i) {
    if (a.e[0]) mx[0].add(r);
    if (a.e[1]) mx[1].add(i);
    if (a.e[2]) mx[2].add(__builtin_fma(a.w2, i, r));
  };
  if (a.along) {
    const int64_t v = min(b * 16 + wave, a.dim - 1);
    const double* pr = a.r + v * a.ld;
    const double* pi = want_i ? a.i + v * a.ld : pr;
    if (a.vec && (K & 1) == 0) {
      for (int64_t c = begin + 2 * lane; c < end + 2 * lane; c += 512) {
        double2 x[4], y[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int64_t q = min(c + 128 * u, end - 2);
          x[u] = *reinterpret_cast<const double2*>(pr + q);
          y[u] = want_i ? *reinterpret_cast<const double2*>(pi + q) : x[u];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          add(x[u].x, y[u].x);
          add(x[u].y, y[u].y);
        }
      }
    } else {
      for (int64_t c = begin + lane; c < end + lane; c += 256) {
        double x[4], y[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int64_t q = min(c + 64 * u, end - 1);
          x[u] = pr[q];
          y[u] = want_i ? pi[q] : x[u];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) add(x[u], y[u]);
      }
    }
  } else {
    const int64_t v = min(b * 16 + (t & 15), a.dim - 1);
    const int rl = t >> 4;
    for (int64_t c = begin + rl; c < end + rl; c += 256) {
      double x[4], y[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t q = min(c + 64 * u, end - 1) * a.ld + v;
        x[u] = a.r[q];
        y[u] = want_i ? a.i[q] : x[u];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) add(x[u], y[u]);
    }
  }
  auto put = [&](int* e, int x) {
    if constexpr (CHUNK) {
      if (x != INT_MIN) atomicMax(e, x);
    } else {
      *e = x;
    }
  };
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    if (!a.e[s]) continue;
    for (int o = 32; o >= (a.along ? 1 : 16); o >>= 1)
      mx[s].merge(__shfl_xor(mx[s].hi, o), __shfl_xor(mx[s].lo, o));
    if (a.along) {
      const int64_t v = b * 16 + wave;
      if (lane == 0 && v < a.dim) put(a.e[s] + v, mx[s].exponent(a.head));
    } else if (lane < 16) {
      red.hi[s][wave][lane] = mx[s].hi;
      red.lo[s][wave][lane] = mx[s].lo;
    }
  }
  if (!a.along) {
    __syncthreads();
    const int c = t & 15;
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      if (t >> 4 != s || !a.e[s] || b * 16 + c >= a.dim) continue;
      MaxMagnitude m;
      for (int w = 0; w < 16; ++w) m.merge(red.hi[s][w][c], red.lo[s][w][c]);
      put(a.e[s] + b * 16 + c, m.exponent(a.head));
    }
  }
}

// Both operands of a product in one launch: the blocks of x, then those of y.
__global__ void __launch_bounds__(kExpThreads) operand_exponents(const SplitOperand x, const SplitOperand y, int64_t xblocks) {
  __shared__ ExpLds red;
  const int64_t b = blockIdx.x;
  if (b < xblocks) exponent_block<false>(x, b, 0, 0, red);
  else exponent_block<false>(y, b - xblocks, 0, 0, red);
}

// The same with the inner dimension (of K elements) in chunks, blockIdx.y, and
// the launch before it, which sets the exponents to INT_MIN.
__global__ void __launch_bounds__(kExpThreads) operand_exponents_chunked(const SplitOperand x, const SplitOperand y,
                                                                         int64_t xblocks, int64_t K, int64_t chunk) {
  __shared__ ExpLds red;
  const int64_t b = blockIdx.x, c0 = blockIdx.y * chunk, c1 = min(K, c0 + chunk);
  if (b < xblocks) exponent_block<true>(x, b, c0, c1, red);
  else exponent_block<true>(y, b - xblocks, c0, c1, red);
}
__global__ void __launch_bounds__(256) clear_exponents(const SplitOperand x, const SplitOperand y) {
  const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    if (v < x.dim && x.e[s]) x.e[s][v] = INT_MIN;
    if (v < y.dim && y.e[s]) y.e[s][v] = INT_MIN;
  }
}

// The same over the items of many problems.
__global__ void __launch_bounds__(kExpThreads) operand_exponents_grouped(const SplitOperand* items, const int64_t* prefix,
                                                                int count) {
  __shared__ ExpLds red;
  const int64_t b = blockIdx.x;
  const int i = find_item(prefix, count, b);
  const SplitOperand a = items[i];
  exponent_block<false>(a, b - prefix[i], 0, 0, red);
}

// Digits of one 64 x 64 tile (64 rows of the left factor, or columns of the
// right one, by 64 of the inner dimension) of the wanted value of an operand,
// in the tiled 64-byte layout.  Thread: 16 consecutive inner elements of one
// row or column (one 16-byte chunk of each plane, two for BF16).  With z = x
// 2^(b - e), a digit is rint(z), read off the low bits of z + 1.5 2^52, and
// the next z is the remainder times 2^b: four full-rate FP64 instructions a
// digit, all exact.  The slices run in a loop.  Exponents and digits of all
// operands of a product, n = 2048: INT8 (8 slices) 1.62 ms against 1.96 with
// three launches per operand, an atomic pass and ldexp per digit, FP8 (12) 1.81
// against 3.35; n = 256, launch-bound, 0.35 against 0.81.
template <int ET>
__device__ __forceinline__ void digits_block(const SplitOperand& a, int64_t b) {
  constexpr double kMagic = 6755399441055744.0;  // 1.5 2^52
  const int64_t nkt = a.kp / 64;
  const int64_t rt = b / nkt, kt = b % nkt;
  const int t = threadIdx.x;
  const int64_t v = rt * 64 + (a.along ? t >> 2 : t & 63);
  const int64_t k0 = kt * 64 + (a.along ? t & 3 : t >> 6) * 16;
  const int64_t K = a.along ? a.cols : a.rows;
  const bool in = v < a.dim;
  const int s = a.out[0] ? 0 : (a.out[1] ? 1 : 2);  // the value wanted
  double z[16];
  load_inner16(a, s == 1 ? a.i : a.r, v, k0, K, in, z);
  if (s == 2) {
    double im[16];
    load_inner16(a, a.i, v, k0, K, in, im);
#pragma unroll
    for (int j = 0; j < 16; ++j) z[j] = __builtin_fma(a.w2, im[j], z[j]);
  }
  const int e = in ? a.e[s][v] : INT_MIN;
#pragma unroll
  for (int j = 0; j < 16; ++j) z[j] = exp_special(e) ? 0.0 : ldexp(z[j], a.bits - e);
  const double step = (double)(1 << a.bits);
  constexpr int ES = ET == 0 ? 2 : 1;
  unsigned char* out = static_cast<unsigned char*>(a.out[s]);
  const int64_t o0 = digit_offset(v, k0 * ES, a.kp * ES);
  const int64_t o1 = ET == 0 ? digit_offset(v, k0 * ES + 16, a.kp * ES) : 0;
  for (int i = 0; i < a.count; ++i) {
    int d[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const double m = z[j] + kMagic;
      d[j] = (int)(uint32_t)__builtin_bit_cast(uint64_t, m);
      z[j] = (z[j] - (m - kMagic)) * step;
    }
    i4v q;
    if constexpr (ET == 2) {
#pragma unroll
      for (int g = 0; g < 4; ++g) q[g] = pack_bytes(d[4 * g], d[4 * g + 1], d[4 * g + 2], d[4 * g + 3]);
      *reinterpret_cast<i4v*>(out + o0) = q;
    } else if constexpr (ET == 1) {
      // |digit| <= 16: exact in E4M3.
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        int w = __builtin_amdgcn_cvt_pk_fp8_f32((float)d[4 * g], (float)d[4 * g + 1], 0, false);
        q[g] = __builtin_amdgcn_cvt_pk_fp8_f32((float)d[4 * g + 2], (float)d[4 * g + 3], w, true);
      }
      *reinterpret_cast<i4v*>(out + o0) = q;
    } else {
      // |digit| <= 128: exact in BF16, the upper half of the FP32 number.
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
          q[g] = (int)__builtin_amdgcn_perm(__float_as_uint((float)d[8 * h + 2 * g + 1]),
                                            __float_as_uint((float)d[8 * h + 2 * g]), 0x07060302u);
        *reinterpret_cast<i4v*>(out + (h ? o1 : o0)) = q;
      }
    }
    out += a.plane;
  }
}

template <int ET>
__global__ void __launch_bounds__(256) split_digits(const SplitOperand x, const SplitOperand y, int64_t xblocks) {
  const int64_t b = blockIdx.x;
  if (b < xblocks) digits_block<ET>(x, b);
  else digits_block<ET>(y, b - xblocks);
}

// ---------------------------------------------------------------------------
// Slice GEMM (BF16 and INT8 digits; FP8 digits: bq_split_f8.hip).
//
// MFMA layouts (checked with one-wave probes on gfx950):
//   A: lane l holds row l % 16, k = E (l / 16) .. +E-1   (E elements/lane)
//   B: lane l holds column l % 16, same k
//   D: lane l, element v holds row 4 (l / 16) + v, column l % 16.
// ---------------------------------------------------------------------------
template <int ET>
struct SliceTraits;
template <>
struct SliceTraits<0> {  // BF16 digits, v_mfma_f32_16x16x32_bf16
  static constexpr int ES = 1 * 2, KSTEP = 32, CH = 16, BETA = 7;
  typedef bf16x8 frag_t;
  typedef f4 acc_t;
  __device__ static acc_t mfma(frag_t a, frag_t b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};
template <>
struct SliceTraits<2> {  // INT8 digits, v_mfma_i32_16x16x64_i8 (exact int32 sums)
  static constexpr int ES = 1, KSTEP = 64, CH = 16, BETA = 7;
  typedef i4v frag_t;
  typedef i4v acc_t;
  __device__ static acc_t mfma(frag_t a, frag_t b, acc_t c) {
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
  }
};

// 2^-e for 0 <= e <= 126 (levels reach e = b (S + 1) = 70): two shifts of at
// most 63 bits each, so no shift reaches the width of the operand.
constexpr double pow2neg(int e) {
  return (1.0 / (double)(1ull << (e / 2))) * (1.0 / (double)(1ull << (e - e / 2)));
}

// Output of one wave tile (16 MI x 16 NI at rows r0.., columns c0..):
// exponent scaling, then coef * T into every target block (store_targets).
template <int MI, int NI>
__device__ __forceinline__ void store_tile(const SliceGemmArgs& g, const d4s (&acc)[MI][NI], int64_t r0, int64_t c0,
                                           int fr, int fg) {
  double t[MI * NI * 4];
  int64_t off[MI * NI * 4];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int e = (i * NI + j) * 4 + v;
        const int64_t r = r0 + i * 16 + 4 * fg + v;
        const int64_t c = c0 + j * 16 + fr;
        const bool in = r < g.m && c < g.n;
        off[e] = in ? r * g.ldc + c : -1;
        t[e] = in ? exp_scaled(acc[i][j][v], g.ea[r], g.eb[c], 0) : 0.0;
      }
  store_targets(g, t, off);
}

// ---------------------------------------------------------------------------
// Slice GEMM with direct global -> LDS loads (BF16 and INT8 digits: rows of
// 64 bytes in 16-byte chunks, digits in the tiled layout).  64 x 64 block
// tile, 4 waves of 32 x 32, one wave per SIMD.  Per k-step every thread
// copies 16 bytes of each A and each B slice tile straight into LDS
// (buffer_load_dwordx4 ... lds: lane l of a wave writes bytes 16 l .. 16 l +
// 15 after the wave's LDS base); the tiles are stored in LDS order, so the
// copy is contiguous on both sides.  Two LDS stages: the loads of k-step kt + 1 are issued
// during the MFMAs of k-step kt, one after each slice pair until all are
// out.  Pairs run level by level (d = s + t = 2 .. S + 1); level d needs
// only the new fragments of slice d - 1, read from LDS one level ahead.
// Level sums stay in registers across k-steps and go to FP64 every
// g.kflush k-steps.
// ---------------------------------------------------------------------------
template <int ET, int S>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
slice_gemm_dma(const SliceGemmArgs g) {
  typedef SliceTraits<ET> Tr;
  typedef typename Tr::frag_t frag_t;
  typedef typename Tr::acc_t acc_t;
  constexpr int ES = Tr::ES, BK = Tr::KSTEP, BETA = Tr::BETA;
  static_assert(Tr::CH == 16 && BK * ES == 64, "rows of four 16-byte chunks");
  constexpr int BM = 64, BN = 64, ROWB = 64, MI = 2, NI = 2;
  constexpr int SLICE = BM * ROWB;  // 4 KB per slice tile (A and B alike)
  constexpr int A_BYTES = S * SLICE;
  constexpr int STAGE = 2 * A_BYTES;
  static_assert(2 * STAGE <= 160 * 1024, "two stages must fit LDS");
  __shared__ __attribute__((aligned(16))) unsigned char lds[2 * STAGE];

  const int tiles_m = (int)((g.m + BM - 1) / BM);
  const int tiles_n = (int)((g.n + BN - 1) / BN);
  int tm, tn;
  slice_tile_coords(tiles_m, tiles_n, tm, tn);
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave >> 1) * 32, wn0 = (wave & 1) * 32;
  const int fr = lane & 15, fg = lane >> 4;

  // Loads: the digits are tiled (digit_offset), so the tile of slice s
  // for k-step kt is 4 KB contiguous, already in LDS order; thread tid copies
  // its bytes 16 tid .. 16 tid + 15.  Buffer loads with one resource per
  // slice and block row (column) tile: its nk tiles, so any offset past them
  // would read zeros rather than another tile.
  const int64_t nk = g.kp / BK;
  const unsigned char* ga = static_cast<const unsigned char*>(g.a) + (int64_t)tm * nk * 4096;
  const unsigned char* gb = static_cast<const unsigned char*>(g.b) + (int64_t)tn * nk * 4096;
  const int64_t sa = g.slice_stride_a * ES, sb = g.slice_stride_b * ES;
  const int nrec = (int)(uint32_t)(nk * 4096);  // num_records is unsigned
  const int voff = tid * 16;
  const int wave_lds = wave * 64 * 16;
  // Load number q (0 .. 2S-1) of k-step kt into stage st: A slice q / 2 or
  // B slice q / 2.
  auto dma = [&](int q, int64_t kt, int st) {
    const int sl = q >> 1;
    const unsigned char* base = (q & 1) ? gb + sl * sb : ga + sl * sa;
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, nrec, 0x00020000);
    unsigned char* dst = lds + st * STAGE + ((q & 1) ? A_BYTES : 0) + sl * SLICE + wave_lds;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_ptr)dst, 16, voff, (int)(kt * 4096), 0, 0);
  };
  auto frag = [&](const unsigned char* tile, int row) {
    return *reinterpret_cast<const frag_t*>(tile + row * ROWB + swz_chunk<16>(row, fg) * 16);
  };

  d4s acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = d4s{0.0, 0.0, 0.0, 0.0};

#pragma unroll
  for (int q = 0; q < 2 * S; ++q) dma(q, 0, 0);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  for (int64_t k0 = 0; k0 < nk; k0 += g.kflush) {
    const int64_t k1 = min(nk, k0 + (int64_t)g.kflush);
    acc_t lvl[S][MI][NI];
#pragma unroll
    for (int d = 0; d < S; ++d)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) lvl[d][i][j] = acc_t{0, 0, 0, 0};
    for (int64_t kt = k0; kt < k1; ++kt) {
      const int st = (int)(kt & 1);
      // The last k-step reloads itself into the idle stage (never read), so
      // the loads need no branch.
      const int64_t knext = kt + 1 < nk ? kt + 1 : kt;
      const unsigned char* ta = lds + st * STAGE;
      const unsigned char* tb = ta + A_BYTES;
      frag_t fa[S][MI], fb[S][NI];
#pragma unroll
      for (int i = 0; i < MI; ++i) fa[0][i] = frag(ta, wm0 + i * 16 + fr);
#pragma unroll
      for (int j = 0; j < NI; ++j) fb[0][j] = frag(tb, wn0 + j * 16 + fr);
      int q = 0;  // loads of the next k-step issued so far
#pragma unroll
      for (int d = 2; d <= S + 1; ++d) {
        // Fragments of slice d (needed from level d + 1 on), one level ahead.
        if (d <= S) {
#pragma unroll
          for (int i = 0; i < MI; ++i) fa[d - 1][i] = frag(ta + (d - 1) * SLICE, wm0 + i * 16 + fr);
#pragma unroll
          for (int j = 0; j < NI; ++j) fb[d - 1][j] = frag(tb + (d - 1) * SLICE, wn0 + j * 16 + fr);
        }
#pragma unroll
        for (int s = 1; s < d; ++s) {
          const int t = d - s;
#pragma unroll
          for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
              lvl[d - 2][i][j] = Tr::mfma(fa[s - 1][i], fb[t - 1][j], lvl[d - 2][i][j]);
          if (q < 2 * S) dma(q++, knext, st ^ 1);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (; q < 2 * S; ++q) dma(q, knext, st ^ 1);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
    }
#pragma unroll
    for (int d = 2; d <= S + 1; ++d) {
      const double sc = pow2neg(BETA * d);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[i][j][v] = __builtin_fma((double)lvl[d - 2][i][j][v], sc, acc[i][j][v]);
    }
  }

  store_tile<MI, NI>(g, acc, m0 + wm0, n0 + wn0, fr, fg);
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
// Chunks of the inner dimension (K elements) of an exponent launch of `blocks`
// blocks: one where the blocks occupy the card (512 fit at a time) or K is short,
// else enough to fill it, none below kExpChunkMin elements.  A block alone reads
// about 30 GB/s, 256 elements of the inner dimension in 2.2 us.  Whole calls, one
// chunk against this rule: CRT 16 x 8192 x 16 (m, k, n) 1836 against 1493 us, 256
// x 2048 x 256 (two chunks) 974 against 938, 40 x 78008 x 197 23.5 against 17.4
// ms, 1024 x 4096 x 1024 3.73 against 3.58, 2000 x 5000 x 2000 (two chunks) 12.81
// against 12.76; INT8 digits 256 x 16384 x 256 13.7 against 10.7.  With at least
// 2048 elements a chunk 256 x 4096 x 256 takes 1286 us, 1206 this way.
constexpr int64_t kExpChunkMin = 1024;
int64_t exponent_chunks(int64_t blocks, int64_t K) {
  return std::max<int64_t>(1, std::min<int64_t>(512 / std::max<int64_t>(1, blocks), K / kExpChunkMin));
}

hipError_t launch_exponents(const SplitOperand& x, const SplitOperand& y, hipStream_t st) {
  const int64_t xb = exponent_blocks(x), blocks = xb + exponent_blocks(y);
  if (blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  const int64_t K = x.along ? x.cols : x.rows, chunks = exponent_chunks(blocks, K);
  if (chunks == 1) {
    hipLaunchKernelGGL(operand_exponents, dim3((unsigned)blocks), dim3(kExpThreads), 0, st, x, y, xb);
    return hipGetLastError();
  }
  const int64_t chunk = ((K + chunks - 1) / chunks + 511) / 512 * 512;
  hipLaunchKernelGGL(clear_exponents, dim3((unsigned)((std::max(x.dim, y.dim) + 255) / 256)), dim3(256), 0, st, x, y);
  hipLaunchKernelGGL(operand_exponents_chunked, dim3((unsigned)blocks, (unsigned)((K + chunk - 1) / chunk)),
                     dim3(kExpThreads), 0, st, x, y, xb, K, chunk);
  return hipGetLastError();
}

hipError_t launch_exponents_grouped(const SplitOperand* items, const int64_t* prefix, int count, int64_t blocks,
                                  hipStream_t st) {
  if (count <= 0 || blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL(operand_exponents_grouped, dim3((unsigned)blocks), dim3(kExpThreads), 0, st, items, prefix, count);
  return hipGetLastError();
}

hipError_t launch_digits(int et, const SplitOperand& x, const SplitOperand& y, hipStream_t st) {
  const int64_t xb = split_blocks(x), blocks = xb + split_blocks(y);
  if (blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks), block(256);
  if (et == 0) hipLaunchKernelGGL(split_digits<0>, grid, block, 0, st, x, y, xb);
  else if (et == 1) hipLaunchKernelGGL(split_digits<1>, grid, block, 0, st, x, y, xb);
  else hipLaunchKernelGGL(split_digits<2>, grid, block, 0, st, x, y, xb);
  return hipGetLastError();
}

template <int ET, int S>
static hipError_t launch_slice_s(const SliceGemmArgs& g, hipStream_t st) {
  const int64_t tiles = ((g.m + 63) / 64) * ((g.n + 63) / 64);
  if (tiles <= 0) return hipSuccess;
  if (tiles > 0x7fffffff || g.kflush < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL((slice_gemm_dma<ET, S>), dim3((unsigned)tiles), dim3(256), 0, st, g);
  return hipGetLastError();
}

int slice_block_rows(int et, int S) {
  (void)et;
  (void)S;
  return 128;  // digit rows are padded to 128, a multiple of every block's rows
}

int slice_kstep(int et) {
  return et == 0 ? SliceTraits<0>::KSTEP : (et == 1 ? 64 : SliceTraits<2>::KSTEP);
}
int slice_beta(int et) { return et == 0 ? SliceTraits<0>::BETA : (et == 1 ? f8_beta() : SliceTraits<2>::BETA); }
int slice_head(int et) { return et == 0 ? 0 : (et == 1 ? f8_head() : 1); }

// Level sums stay exact while every partial sum is an integer below 2^24
// (FP32) or 2^31 (int32).  Digit bounds: |q_1| <= 2^{b-h}, |q_s| <= 2^{b-1};
// a level d = s + t has at most d - 1 <= S pairs.  With h = 1 every digit is
// within 2^{b-1}, so per k element |level| <= 2^{2b-2} S; with h = 0 the two
// pairs holding a leading digit count twice: |level| <= 2^{2b-2} (S + 3).
int slice_flush_steps(int et, int S) {
  const int b = slice_beta(et);
  const double per_k = std::ldexp(1.0, 2 * b - 2) * (slice_head(et) ? S : S + 3);
  const double lim = et == 2 ? 2147483647.0 : 16777216.0;
  const int64_t kmax = (int64_t)(lim / per_k);
  const int64_t steps = kmax / slice_kstep(et);
  return (int)std::max<int64_t>(1, std::min<int64_t>(steps, 1 << 20));
}

#define BQ_SPLIT_CASES(ET, X) \
  X(ET, 1) X(ET, 2) X(ET, 3) X(ET, 4) X(ET, 5) X(ET, 6) X(ET, 7) X(ET, 8)

hipError_t launch_slice_gemm(int et, int S, const SliceGemmArgs& g, hipStream_t st) {
  if (et == 1) return launch_slice_gemm_f8(S, g, st);
#define X(E, SS) \
  if (et == E && S == SS) return launch_slice_s<E, SS>(g, st);
  BQ_SPLIT_CASES(0, X)
  BQ_SPLIT_CASES(2, X)
  X(2, 9)
#undef X
  return hipErrorInvalidValue;
}

int max_slices(int et) { return et == 0 ? 8 : (et == 1 ? 13 : 9); }

}  // namespace bq
