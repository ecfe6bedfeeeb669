// One-launch biquaternion product for sizes that leave the per-product
// launches of cgemm_f64 short of blocks (FP64, gfx950).
//
//  bq_fused    C = op(A) op(B): one block per C tile runs all eight products
//              of eq. bilinearH on that tile, one wave per product.  The
//              block stages the raw components of its A and B panels and
//              their Hadamard combinations in LDS (formed from the loaded
//              values, so they never reach HBM), every wave accumulates its
//              product's real GEMMs (three by Gauss, or one for real
//              quaternions), and the post-combination reads the eight P from
//              LDS and writes each C element once.
//
// The per-product path takes ten launches, each of the eight GEMM launches
// holding (m / 64)(n / 64) blocks: 1 block at n = 64, 16 at n = 256, 256 (of
// 512 slots) at n = 1024.  Here every tile of 16 x 16 or 32 x 32 carries
// eight waves.  What bounds it at full size is the staging beside the matrix
// pipe: at m = n = k = 1024 (32 x 32 tiles) 841 us, 61.3 TFLOP/s, and about
// 730 us without the Hadamard sums and their LDS writes (865 us before the LDS
// slots made every access conflict-free and the loads took 64 bytes of a row
// together; with 8-byte loads, n = 1023, 1038 -> 911).
//
// The k order of every product, the order of the Hadamard sums and the order
// of the additions into C are those of the per-product path, so the results
// are the same bit for bit.
//
// Tile base pointers are 64-bit; offsets inside a tile are 32-bit.  Build with
//   -Xclang -target-feature -Xclang -packed-fp32-ops
#include <algorithm>
#include <type_traits>
#include <utility>

#include "bq_tile_order.h"

namespace bq {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

namespace {

__device__ __forceinline__ d4 mfma_f64(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// LDS position of (row or column r, k) in one T-wide plane: fragment (k / 4,
// r / 16) is 64 doubles, 16 per k.  An access serves 16 lanes on 16 bank pairs,
// so the slot among the 16 is chosen to make the 16 lanes of every access
// distinct: a fragment read (16 rows, one k), a staging write of a side stored
// along k (2 rows by 8 pairs of k, 4 by 4 or 1 by 16: the pair's bits are
// folded in) and of a side stored along the rows (the even or the odd rows of
// two k, or of two fragments: even rows take slots 0..7, and bit 3 flips with
// k and the fragment).
__device__ __forceinline__ int row_at(int r) { return ((r & 15) >> 1) | ((r & 1) << 3); }
__device__ __forceinline__ int slot_flip(int r, int k) {
  return ((r >> 1) & 8) ^ ((k & 1) << 3) ^ (k & 6) ^ ((k >> 3) & 1) ^ ((k >> 1) & 8);
}
template <int T>
__device__ __forceinline__ int plane_at(int r, int k) {
  return ((k >> 2) * (T / 16) + (r >> 4)) * 64 + (k & 3) * 16 + (row_at(r) ^ slot_flip(r, k));
}

// sum + coef * P, the product rounded before it is added, as in the per-product
// path (it is exact but for denormals).
__device__ __forceinline__ double add_product(double sum, double coef, double P) {
#pragma clang fp contract(off)
  return sum + coef * P;
}

template <int... I, typename F>
__device__ __forceinline__ void static_for_seq(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_seq(std::make_integer_sequence<int, N>{}, f);
}

// IM: components 4..7 present on both sides (eight complex products by
// Gauss), else real quaternions (eight real products).  T: tile edge.
// Staging: a unit is one pair of adjacent stored elements of four components
// (one side, real or imaginary parts); a wave's units share side and part,
// so its component bases are scalar.  U units per thread and k-step.
// LDS of one block: two stages, each 8 planes per part and side.
template <int IM, int T, int BK>
constexpr int kFusedLds = 2 * 2 * (IM ? 2 : 1) * 8 * T * BK;

// Tile (tm, tn) of C.  Args: FusedArgs as kernel arguments, or in a device
// table read as constant memory.
template <int IM, int T, int BK, typename Args>
__device__ __forceinline__ void fused_block(const Args& g, int tm, int tn, double* lds) {
  constexpr int NPART = IM ? 2 : 1;
  constexpr int PLANE = T * BK;             // doubles per plane
  constexpr int SIDE = NPART * 8 * PLANE;   // 4 raw + 4 combined planes per part
  constexpr int STAGE = 2 * SIDE;
  constexpr int PAIRS = T * BK / 2;
  constexpr int UNITS = 2 * NPART * PAIRS;
  constexpr int U = UNITS / 512;
  static_assert(UNITS % 512 == 0 && PAIRS % 64 == 0, "whole waves per side and part");
  constexpr int NI = T / 16;
  constexpr int NACC = IM ? 3 : 1;
  static_assert(2 * STAGE == kFusedLds<IM, T, BK>, "LDS size");
  static_assert(8 * NPART * T * T <= 2 * STAGE, "P of every product fits the stages");
  const int64_t m0 = (int64_t)tm * T, n0 = (int64_t)tn * T;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // This thread's units.  k-contiguous sides (A for op N, B for op T): pair
  // = (row r, k 2 kp), k fastest; the others: pair = (rows 2 rp, k), rows
  // fastest: 64 bytes or more of each stored row.
  constexpr uint32_t kOut = 0x80000000u;  // past the resource's range: reads zero
  int part[U], side[U], kk[U], lpos[U][2];  // LDS positions of the pair's elements
  uint32_t off[U][2];   // byte offsets of the pair's two elements in the tile at k0 = 0
  bool kc[U];
  const double* base[U][4];
  int64_t kstride[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int unit = u * 512 + wave * 64;  // of lane 0: uniform
    side[u] = unit / (NPART * PAIRS);
    part[u] = unit / PAIRS % NPART;
    const int pair = unit % PAIRS + lane;
    kc[u] = side[u] ? g.tb : !g.ta;
    const int64_t ld = side[u] ? g.ldb : g.lda;
    const int64_t lim = side[u] ? g.n - n0 : g.m - m0;
    const int64_t o0 = side[u] ? n0 : m0;
#pragma unroll
    for (int c = 0; c < 4; ++c)
      base[u][c] = (side[u] ? g.b[4 * part[u] + c] : g.a[4 * part[u] + c]) + (kc[u] ? o0 * ld : o0);
    kstride[u] = kc[u] ? 1 : ld;
    if (kc[u]) {
      const int r = pair / (BK / 2);
      kk[u] = 2 * (pair % (BK / 2));
      off[u][0] = r < lim ? (uint32_t)((r * (uint32_t)ld + kk[u]) * 8u) : kOut;
      off[u][1] = r < lim ? off[u][0] + 8u : kOut;
      lpos[u][0] = plane_at<T>(r, kk[u]);
      lpos[u][1] = plane_at<T>(r, kk[u] + 1);
    } else {
      const int r = 2 * (pair % (T / 2));
      kk[u] = pair / (T / 2);
      const uint32_t o = (uint32_t)((kk[u] * (uint32_t)ld + r) * 8u);
      off[u][0] = r < lim ? o : kOut;
      off[u][1] = r + 1 < lim ? o + 8u : kOut;
      lpos[u][0] = plane_at<T>(r, kk[u]);
      lpos[u][1] = plane_at<T>(r + 1, kk[u]);
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) lpos[u][e] += side[u] * SIDE + part[u] * 8 * PLANE;
  }

  const int nk = (int)((g.k + BK - 1) / BK), nkf = (int)(g.k / BK);
  // Loads of k-step kt.  VEC (16-byte rows): one 16-byte load per pair; a
  // pair that straddles the end of an odd row (or of an odd k) reads 8 bytes
  // more of its own 16-byte chunk, which feed outputs outside C (or are
  // cleared before they are staged).  CHK: k-steps that may reach past k,
  // where such elements get an offset past the resource and read as zero.
  // Every k-step issues the same number of loads, so a wait for one register
  // set leaves the other set's loads in flight.
  auto load = [&](auto vec, auto chk, int kt, d2 (&x)[U][4]) {
    constexpr bool VEC = decltype(vec)::value, CHK = decltype(chk)::value;
    const int kleft = (int)(g.k - (int64_t)kt * BK);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t step = (int64_t)kt * BK * kstride[u];
      const uint32_t o0 = !CHK || kk[u] < kleft ? off[u][0] : kOut;
      const uint32_t o1 = !CHK || kk[u] + (kc[u] ? 1 : 0) < kleft ? off[u][1] : kOut;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const __amdgpu_buffer_rsrc_t r =
            __builtin_amdgcn_make_buffer_rsrc((void*)(base[u][c] + step), (short)0, 0x7fffffff, 0x00020000);
        if constexpr (VEC) {
          x[u][c] = __builtin_bit_cast(d2, __builtin_amdgcn_raw_buffer_load_b128(r, (int)o0, 0, 0));
        } else {
          x[u][c][0] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)o0, 0, 0));
          x[u][c][1] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)o1, 0, 0));
        }
      }
    }
  };
  // Staging of k-step kt's tiles in 4 chunks of two planes per unit: raw planes
  // 0..3, then the Hadamard combinations 4..7 of the pair's part, summed left to right
  // over the units as the pre-combination does.  prepare clears what a
  // 16-byte load read past k.
  auto prepare = [&](auto vec, auto chk, int kt, d2 (&x)[U][4]) {
    if constexpr (decltype(vec)::value && decltype(chk)::value) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool half = kc[u] && kk[u] + 1 >= g.k - (int64_t)kt * BK;
#pragma unroll
        for (int c = 0; c < 4; ++c) x[u][c][1] = half ? 0.0 : x[u][c][1];
      }
    }
  };
  auto chunk = [&](auto J, int kt, const d2 (&x)[U][4]) {
    constexpr int u = J.value / 4, j = J.value % 4;
    const double s1 = side[u] ? g.sb[1] : g.sa[1], s2 = side[u] ? g.sb[2] : g.sa[2], s3 = side[u] ? g.sb[3] : g.sa[3];
    double* d0 = lds + (kt & 1) * STAGE + lpos[u][0] + 2 * j * PLANE;
    double* d1 = lds + (kt & 1) * STAGE + lpos[u][1] + 2 * j * PLANE;
    d2 h0, h1;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      if constexpr (j < 2) {
        h0[e] = x[u][2 * j][e];
        h1[e] = x[u][2 * j + 1][e];
      } else {
        constexpr double f = j == 2 ? 1.0 : -1.0;
        const double p = __builtin_fma(f * s1, x[u][1][e], x[u][0][e]);
        h0[e] = __builtin_fma(f * s3, x[u][3][e], __builtin_fma(s2, x[u][2][e], p));
        h1[e] = __builtin_fma(-f * s3, x[u][3][e], __builtin_fma(-s2, x[u][2][e], p));
      }
    }
    d0[0] = h0[0];
    d0[PLANE] = h1[0];
    d1[0] = h0[1];
    d1[PLANE] = h1[1];
  };
  auto store = [&](auto vec, auto chk, int kt, d2 (&x)[U][4]) {
    prepare(vec, chk, kt, x);
    static_for<4 * U>([&](auto J) { chunk(J, kt, x); });
  };

  // This wave's product: operand planes (direct: raw unit pairs; Hadamard:
  // combination wave - 4 on both sides).
  const int ua = wave < 4 ? g.pair_a[wave & 3] : wave, ub = wave < 4 ? g.pair_b[wave & 3] : wave;
  const double* pa = lds + ua * PLANE;
  const double* pb = lds + SIDE + ub * PLANE;
  // Position of this lane's element of fragment (substep s, i) in a plane.
  auto frag_at = [&](int s, int i) { return plane_at<T>(i * 16 + (lane & 15), 4 * s + (lane >> 4)); };
  const double sL = g.sL, sR = g.sR;

  d4 acc[NACC][NI][NI];
#pragma unroll
  for (int q = 0; q < NACC; ++q)
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[q][i][j] = d4{0.0, 0.0, 0.0, 0.0};

  // Fragments of one half of a k-step (HS substeps of 4), and its MFMAs.
  constexpr int HS = BK / 8;
  constexpr int MH = HS * NACC * NI * NI;  // MFMAs per half
  struct Frags {
    double a[HS][NPART][NI], b[HS][NPART][NI];
  };
  auto read = [&](int buf, int half, Frags& f) {
#pragma unroll
    for (int s = 0; s < HS; ++s)
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int p = 0; p < NPART; ++p) {
          const int o = buf * STAGE + p * 8 * PLANE + frag_at(half * HS + s, i);
          f.a[s][p][i] = pa[o];
          f.b[s][p][i] = pb[o];
        }
  };
  // MFMA number I of a half (its Gauss sums are formed where first needed).
  double as[NI], bs[NI];
  auto mfma = [&](auto I, const Frags& f) {
    constexpr int s = I.value / (NACC * NI * NI), r = I.value % (NACC * NI * NI);
    constexpr int q = r % NACC, j = r / NACC % NI, i = r / NACC / NI;
    if constexpr (q == 2) {
      if constexpr (j == 0) as[i] = __builtin_fma(sL, f.a[s][NPART - 1][i], f.a[s][0][i]);
      if constexpr (i == 0) bs[j] = __builtin_fma(sR, f.b[s][NPART - 1][j], f.b[s][0][j]);
      acc[q][i][j] = mfma_f64(as[i], bs[j], acc[q][i][j]);
    } else {
      constexpr int p = q ? NPART - 1 : 0;
      acc[q][i][j] = mfma_f64(f.a[s][p][i], f.b[s][p][j], acc[q][i][j]);
    }
  };
  auto compute = [&](const Frags& f) { static_for<MH>([&](auto I) { mfma(I, f); }); };

  // Between two barriers: the MFMAs of k-step kt - 1's second half (operands
  // in registers) and of kt's first half (read from LDS behind the former),
  // the read of kt's second half, and, spread over all of them, the staging
  // of kt + 1 (loaded two k-steps ago) into the other buffer, whose last
  // reads ended before the previous barrier; the loads of kt + 3 take its
  // registers.  So neither LDS latency nor the staging stands between two
  // MFMAs.  Past the last k-step zeros are staged that nobody uses.
  //
  // The barrier waits for this wave's LDS accesses only: global loads stay
  // in flight across it.
  auto barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
  auto run = [&](auto vec) {
    constexpr std::integral_constant<bool, false> fast{};
    constexpr std::integral_constant<bool, true> chk{};
    d2 x0[U][4], x1[U][4];
    Frags f1, f2;
    auto step = [&](auto c, int kt, d2 (&x)[U][4]) {
      prepare(vec, c, kt + 1, x);
      __builtin_amdgcn_sched_barrier(0);
      static_for<MH>([&](auto I) {
        mfma(I, f1);
        if constexpr (I.value == 0) read(kt & 1, 1, f2);
        // chunk j after MFMA j (2 MH - 2) / (4 U)
        static_for<4 * U>([&](auto J) {
          if constexpr (J.value * (MH - 1) / (4 * U) == I.value) {
            chunk(J, kt + 1, x);
            if constexpr (J.value == 4 * U - 1) load(vec, c, kt + 3, x);
          }
        });
        __builtin_amdgcn_sched_barrier(0);
      });
      barrier();
      static_for<MH>([&](auto I) {
        mfma(I, f2);
        if constexpr (I.value == 0) read((kt + 1) & 1, 0, f1);
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    load(vec, chk, 0, x0);
    load(vec, chk, 1, x1);
    store(vec, chk, 0, x0);
    load(vec, chk, 2, x0);
    barrier();
    read(0, 0, f1);
    int kt = 0;
    for (; kt + 4 < nkf; kt += 2) {
      step(fast, kt, x1);
      step(fast, kt + 1, x0);
    }
    for (; kt + 1 < nk; kt += 2) {
      step(chk, kt, x1);
      step(chk, kt + 1, x0);
    }
    if (kt < nk) step(chk, kt, x1);
    barrier();
  };
  if (g.vec) run(std::integral_constant<bool, true>{});
  else run(std::integral_constant<bool, false>{});

  // P of every product into LDS (free after the last barrier):
  // [product][part][row][column].
  const double sig = sL * sR;
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        double* d = lds + wave * NPART * T * T + (i * 16 + (lane >> 4) + 4 * v) * T + j * 16 + (lane & 15);
        const double t1 = acc[0][i][j][v];
        if constexpr (IM) {
          const double t2 = acc[1 % NACC][i][j][v], t3 = acc[2 % NACC][i][j][v];
          d[0] = t1 - sig * t2;
          d[T * T] = (t3 - t1) - sig * t2;
        } else {
          d[0] = t1;
        }
      }
  barrier();
  // Post-combination: C of unit w and one part = its direct product, then
  // the four Hadamard products in order.
  constexpr int OUT = 4 * NPART * T * T;
#pragma unroll
  for (int o = 0; o < OUT / 512; ++o) {
    const int e = (o * 512 + tid) % (T * T);
    const int comp = __builtin_amdgcn_readfirstlane((o * 512 + tid) / (T * T));  // w + 4 part
    const int w = comp & 3, pt = comp >> 2;
    const int64_t r = m0 + e / T, c = n0 + e % T;
    const double* s = lds + pt * T * T + e;
    double val = g.cd[w] * s[w * NPART * T * T];
#pragma unroll
    for (int q = 0; q < 4; ++q) val = add_product(val, g.ch[w][q], s[(4 + q) * NPART * T * T]);
    double* dst = g.c[comp];
    if (dst && r < g.m && c < g.n) dst[r * g.ldc + c] = val;
  }
}

// k-steps of the two tile edges, and their LDS (the same for both).
template <int IM>
constexpr int kFusedBk16 = IM ? 16 : 32;
template <int IM>
constexpr int kFusedBk32 = IM ? 8 : 16;

// One product in 16 x 16 tiles.  Contiguous ranges of tiles per XCD (blocks are
// dealt to the 8 XCDs round-robin), walked in groups of 8 tile rows.
template <int IM>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
bq_fused16(const FusedArgs g) {
  __shared__ __attribute__((aligned(16))) double lds[kFusedLds<IM, 16, kFusedBk16<IM>>];
  const int tiles_m = (int)((g.m + 15) / 16), tiles_n = (int)((g.n + 15) / 16);
  int tm, tn;
  grouped_tile((int)xcd_position(blockIdx.x, 0, (int64_t)tiles_m * tiles_n), tiles_m, tiles_n, tm, tn);
  fused_block<IM, 16, kFusedBk16<IM>>(g, tm, tn, lds);
}

// One product: blocks 0 .. full - 1 take 32 x 32 tiles, four blocks each the
// remaining ones in 16 x 16 quarters.
template <int IM>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
bq_fused(const FusedArgs g, int full) {
  static_assert(kFusedLds<IM, 16, kFusedBk16<IM>> == kFusedLds<IM, 32, kFusedBk32<IM>>, "one LDS size");
  __shared__ __attribute__((aligned(16))) double lds[kFusedLds<IM, 32, kFusedBk32<IM>>];
  const int tiles_m = (int)((g.m + 31) / 32), tiles_n = (int)((g.n + 31) / 32);
  const int b = blockIdx.x;
  int tm, tn;
  if (b < full) {
    grouped_tile((int)xcd_position(b, 0, full), tiles_m, tiles_n, tm, tn);
    fused_block<IM, 32, kFusedBk32<IM>>(g, tm, tn, lds);
  } else {
    const int q = (int)xcd_position(b, full, full + 4 * ((int64_t)tiles_m * tiles_n - full));
    grouped_tile(full + (q >> 2), tiles_m, tiles_n, tm, tn);
    tm = 2 * tm + (q >> 1 & 1);
    tn = 2 * tn + (q & 1);
    if ((int64_t)tm * 16 >= g.m || (int64_t)tn * 16 >= g.n) return;
    fused_block<IM, 16, kFusedBk16<IM>>(g, tm, tn, lds);
  }
}

// The same over the tiles of many problems: block b takes item b (problem,
// tile edge, tile), the host having put them in order.
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
grouped_fused(const FusedArgs* probs, const FusedItem* items) {
  __shared__ __attribute__((aligned(16))) double lds[kFusedLds<1, 32, kFusedBk32<1>>];
  typedef const __attribute__((address_space(4))) FusedItem* item_ptr;
  typedef const __attribute__((address_space(4))) FusedArgs table_args;
  const item_ptr w = (item_ptr)items + blockIdx.x;
  table_args& g = *((table_args*)probs + w->prob);
  if (w->tile == 16) fused_block<1, 16, kFusedBk16<1>>(g, w->tm, w->tn, lds);
  else fused_block<1, 32, kFusedBk32<1>>(g, w->tm, w->tn, lds);
}

}  // namespace

// Buffer offsets inside a tile must reach every element (T <= 32, BK <= 32).
bool fused_spans_fit(int64_t lda, int64_t ldb) { return 32 * std::max(lda, ldb) * 8 + 32 * 8 < 0x7fffffff; }

// Which path a product takes: an estimate of both in microseconds, from rates
// measured on an MI355X at m = n = k = 64 .. 4096.  One round is one block on
// each of the 256 CUs (fused) or two (per product).
//   fused   a round of 32 x 32 blocks takes, per unit of k, kRound us: past the
//           cache by how A and B are stored and by their rows (where A or B have
//           odd rows, both are loaded 8 bytes at a time; such loads of an A that is
//           stored along k cost most), else by its first orientation and whether
//           rows are odd.  24 products: past the cache 0.201-0.213 with rows of
//           whole 64-byte lines, 0.216 with other even ones (N N, N T), 0.214-0.276
//           with odd ones; n = 1024 and 1280 0.204-0.208 and 0.210-0.243.  8
//           products: 0.069-0.075, and 0.079-0.089 with odd rows (n = 3008; 0.077-
//           0.082 at 2304, 340 MB).  A round of 16 x 16 blocks takes 0.066 and
//           0.028.  A last round of r tiles runs as 4 r quarters where that takes
//           less, up to half a round: 1000 x 777 x 515 (544 tiles) 478 -> 390 us,
//           n = 800 500 -> 438, n = 2300 10.38 -> 10.05 ms.
//   per     each of 8 launches as tile_launch_cost estimates it for one alone, or
//   product for the 64 x 64 tiles of grids of 1024 of them and more, which follow
//           each other, by their rounds and ends (24 products, op N N: 0.1885 us a
//           round and kEnds24, within 1 % of n = 2048 .. 4096 in steps of 64; with
//           edge tiles 1.05 times that, 1.03 to 1.10 measured; 8 products: kLaunch8
//           and kEnds8, 3 % mostly).
//           Plus the pre-combination (16 blocks read and 16
//           written) and the read-modify-write of C at 4.8 TB/s, the latter
//           0.6 exposed.
// Fused against per product: n = 256 23 us against 365, 1024 841 against 1204,
// 2048 6.67 ms against 7.17, 3000 21.5 against 23.1, 3072 23.6 against 22.6, 3136
// 24.5 against 25.4, 3200 26.4 against 26.0, 3334 31.3 against 30.6, 3392 30.8
// against 30.1 (T N 30.1 against 29.0), 3500 35.4 against 35.5, 4096 53.2 against
// 52.0; odd rows 2301 11.8 against 12.6, 2501 T N 13.7 against 15.3, N T 16.9
// against 16.0, 3001 26.5 against 23.7.
// Real quaternions: 1024 314 us against 514, 3000 7.65 ms against 8.38, 3456 11.5
// against 11.3, 3520 12.1 against 13.9, 4096 18.3 against 17.4, odd rows
// 2301 3.86 against 4.70, 3001 9.37 against 8.77.
int64_t fused_full_tiles(int im, int64_t m, int64_t n, int64_t k, int ta, int tb, int64_t lda, int64_t ldb, int vec) {
  constexpr int64_t kCUs = 256;
  auto tiles = [&](int64_t t) { return ((m + t - 1) / t) * ((n + t - 1) / t); };
  auto rounds = [&](int64_t t, int64_t per) { return (tiles(t) + per - 1) / per; };
  if (!fused_spans_fit(lda, ldb) || tiles(32) > 0x1fffffff) return -1;
  // A and B past the 256 MB cache behind the L2s (24 products slow down around 300
  // MB: n = 1511 N T, 292 MB, 0.237, 1600 0.265; 8 between 340 and 467).
  const bool past_cache = (im ? 64.0 : 32.0) * double(k) * (double(m) + double(n)) > (im ? 1.2 : 1.5) * 268435456.0;
  // Rows: 0 of whole 64-byte lines, 1 16-byte aligned, 2 of A odd, 3 of B, 4 both.
  const bool odd_a = lda % 2 != 0, odd_b = ldb % 2 != 0;
  const int rows = vec ? (lda % 8 != 0 || ldb % 8 != 0 ? 1 : 0) : (odd_a == odd_b ? 4 : (odd_a ? 2 : 3));
  // [A stored k x m][B stored n x k][rows]
  constexpr double kRound24[2][2][5] = {{{0.2075, 0.2165, 0.249, 0.2275, 0.2555}, {0.2095, 0.2165, 0.2665, 0.233, 0.276}},
                                        {{0.202, 0.202, 0.216, 0.2135, 0.2215}, {0.202, 0.2045, 0.228, 0.229, 0.236}}};
  constexpr double kRound8[2][2][5] = {{{0.0735, 0.0755, 0.0865, 0.0795, 0.0885}, {0.0735, 0.0755, 0.0865, 0.0805, 0.088}},
                                       {{0.0735, 0.0755, 0.0795, 0.079, 0.0845}, {0.0735, 0.0755, 0.08, 0.0805, 0.0855}}};
  // In the cache: [A stored k x m][odd rows].
  constexpr double kCached24[2][2] = {{0.207, 0.235}, {0.206, 0.216}};
  // Launches of one product on 1024 64 x 64 tiles and more: a round of 512, and the
  // end of the last whole one, a last one of at most 256 tiles or a longer one.
  constexpr double kEnds24[3] = {0.02, 0.122, 0.213};
  constexpr double kOp24[2][2] = {{1.0, 1.025}, {0.96, 1.01}};
  constexpr double kLaunch8[2][4] = {{0.07, 0.076, 0.072, 0.072}, {0.07, 0.0773, 0.0744, 0.0757}};  // [odd][2 ta + tb]
  constexpr double kEnds8[2][2][3] = {{{0.0, 0.043, 0.1}, {0.02, 0.06, 0.08}},  // [odd][transposed]
                                      {{0.0, 0.063, 0.1}, {0.0225, 0.075, 0.105}}};
  // Odd rows beside rows that are no whole lines: 2878 x 1406 x 3383 0.248.
  const bool lines_beside = rows == 2 ? ldb % 8 == 0 : lda % 8 == 0;
  const double c32 = past_cache ? (im ? kRound24 : kRound8)[ta != 0][tb != 0][rows] +
                                      (!ta && (rows == 2 || rows == 3) && !lines_beside ? (im ? 0.01 : 0.0065) : 0.0)
                                : (im ? kCached24[ta != 0][rows > 1] : (rows > 1 ? 0.0825 : 0.0735));
  // Past the cache 16 x 16 blocks wait for their loads as well (n = 2067 N T 0.076).
  const double c16 = im ? std::max(0.066, c32 / 3.6) : 0.028;
  const int64_t t32 = tiles(32), whole = t32 / kCUs * kCUs;
  // All in 32 x 32 tiles, the last round in quarters (those outside C end at
  // once), or all in 16 x 16 tiles.
  const double cost[3] = {c32 * double(rounds(32, kCUs)),
                          c32 * double(whole / kCUs) + c16 * double((4 * (t32 - whole) + kCUs - 1) / kCUs),
                          c16 * double(rounds(16, kCUs))};
  const int64_t full[3] = {t32, whole, 0};
  const int pick = int(std::min_element(cost, cost + 3) - cost);
  const double fused = double(k) * cost[pick];
  const int kind = im ? KIND_GAUSS : KIND_RR;
  const int cfg = default_tile_config(kind, m, n, k);
  const bool trans = ta || tb, odd = vec == 0, edges = m % 64 != 0 || n % 64 != 0;
  const int64_t t64 = tiles(64), tail = t64 % 512;
  const int end = tail == 0 ? 0 : (tail <= 256 ? 1 : 2);
  // Transposed real products run 64 x 64 tiles with k-steps of 16.
  const int run = !im && trans && cfg == 11 ? 3 : cfg;
  double launch = (!im && trans && run == 3 ? 1.1 : 1.0) * tile_launch_cost(kind, run, m, n);
  if (run == 0) {
    const double op = kOp24[ta != 0][tb != 0];
    launch = t64 >= 1024 ? (0.1885 * op * double(t64 / 512) + kEnds24[end]) * (odd ? 1.03 : 1.0) * (edges ? 1.05 : 1.0)
                         : launch * op * (odd ? (trans ? 1.06 : 1.03) : 1.0);
  } else if (t64 >= 1024 && run == 3) {
    launch = kLaunch8[odd][(ta ? 2 : 0) + (tb ? 1 : 0)] * double(t64 / 512) + kEnds8[odd][trans][end];
    if (trans ? edges && !odd : k < 1024) launch *= trans ? 1.045 : 1.2;  // below 1024 without the two-deep loop
  } else if (run == 11) {
    launch *= odd ? 1.09 : (m % 128 != 0 || n % 128 != 0 ? 1.045 : 1.0);
  }
  const double gb = 1e-6 / 4.8 * (im ? 1.0 : 0.5);  // us per byte of the 24-product form
  const double per_product = 8.0 * double(k) * launch + 128.0 * gb * (double(m) + double(n)) * double(k) +
                             0.6 * 576.0 * gb * double(m) * double(n);
  // Eight products within 1 %: the launches of one each, whose estimate is rougher.
  return (im ? 1.0 : 1.01) * fused <= per_product ? full[pick] : -1;
}

hipError_t launch_grouped_fused(const FusedArgs* probs, const FusedItem* items, int nitems, hipStream_t s) {
  if (nitems <= 0) return hipSuccess;
  hipLaunchKernelGGL(grouped_fused, dim3((unsigned)nitems), dim3(512), 0, s, probs, items);
  return hipGetLastError();
}

hipError_t launch_fused(const FusedArgs& g, int im, int64_t full, hipStream_t s) {
  if (g.m <= 0 || g.n <= 0 || g.k <= 0) return hipErrorInvalidValue;
  const int64_t t32 = ((g.m + 31) / 32) * ((g.n + 31) / 32), blocks = full + 4 * (t32 - full);
  if (full < 0 || full > t32 || blocks > 0x7fffffff) return hipErrorInvalidValue;
  if (full == 0) {
    const dim3 grid((unsigned)(((g.m + 15) / 16) * ((g.n + 15) / 16)));
    if (im) hipLaunchKernelGGL(bq_fused16<1>, grid, dim3(512), 0, s, g);
    else hipLaunchKernelGGL(bq_fused16<0>, grid, dim3(512), 0, s, g);
    return hipGetLastError();
  }
  if (im) hipLaunchKernelGGL(bq_fused<1>, dim3((unsigned)blocks), dim3(512), 0, s, g, (int)full);
  else hipLaunchKernelGGL(bq_fused<0>, dim3((unsigned)blocks), dim3(512), 0, s, g, (int)full);
  return hipGetLastError();
}

}  // namespace bq
