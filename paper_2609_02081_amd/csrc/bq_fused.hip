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
// pipe: at m = n = k = 1024 (32 x 32 tiles) 865 us, 59.6 TFLOP/s, and 731 us
// without the Hadamard sums and their LDS writes.
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

#include "bq_internal.h"

namespace bq {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

namespace {

__device__ __forceinline__ d4 mfma_f64(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// LDS position of (row or column r, k) in one T-wide plane: fragment (k / 4,
// r / 16) is 64 consecutive doubles, 16 per k, even rows before odd ones.  A
// fragment read and a staging write (16 rows at one k, or the even or the odd
// rows of two k) then touch 16 distinct consecutive bank pairs.
__device__ __forceinline__ int row_at(int r) { return ((r & 15) >> 1) | ((r & 1) << 3); }
template <int T>
__device__ __forceinline__ int plane_at(int r, int k) {
  return ((k >> 2) * (T / 16) + (r >> 4)) * 64 + (k & 3) * 16 + row_at(r);
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
template <int IM, int T, int BK>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
bq_fused(const FusedArgs g) {
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
  static_assert(8 * NPART * T * T <= 2 * STAGE, "P of every product fits the stages");
  __shared__ __attribute__((aligned(16))) double lds[2 * STAGE];

  // Tile of this block: contiguous ranges of tiles per XCD (blocks are dealt
  // to the 8 XCDs round-robin), columns fastest inside groups of 8 tile rows.
  const int tiles_m = (int)((g.m + T - 1) / T), tiles_n = (int)((g.n + T - 1) / T);
  int tm, tn;
  {
    const int n_tiles = tiles_m * tiles_n, w = blockIdx.x, x = w % 8, slot = w / 8;
    const int base = n_tiles / 8, rem = n_tiles % 8;
    const int t = x * base + (x < rem ? x : rem) + slot;
    const int per_group = 8 * tiles_n, group = t / per_group, first_m = group * 8;
    const int gm = min(tiles_m - first_m, 8), in_g = t - group * per_group;
    tm = first_m + in_g % gm;
    tn = in_g / gm;
  }
  const int64_t m0 = (int64_t)tm * T, n0 = (int64_t)tn * T;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  // This thread's units.  k-contiguous sides (A for op N, B for op T): pair
  // = (row r, k 2 kp), rows fastest; the others: pair = (rows 2 rp, k).
  constexpr uint32_t kOut = 0x80000000u;  // past the resource's range: reads zero
  int part[U], side[U], kk[U], lpos[U];
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
      const int r = pair % T;
      kk[u] = 2 * (pair / T);
      off[u][0] = r < lim ? (uint32_t)((r * (uint32_t)ld + kk[u]) * 8u) : kOut;
      off[u][1] = r < lim ? off[u][0] + 8u : kOut;
      lpos[u] = plane_at<T>(r, kk[u]);
    } else {
      const int r = 2 * (pair % (T / 2));
      kk[u] = pair / (T / 2);
      const uint32_t o = (uint32_t)((kk[u] * (uint32_t)ld + r) * 8u);
      off[u][0] = r < lim ? o : kOut;
      off[u][1] = r + 1 < lim ? o + 8u : kOut;
      lpos[u] = plane_at<T>(r, kk[u]);
    }
    lpos[u] += side[u] * SIDE + part[u] * 8 * PLANE;
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
    double* d0 = lds + (kt & 1) * STAGE + lpos[u] + 2 * j * PLANE;
    double* d1 = d0 + (kc[u] ? 16 : 8);  // the next k, or the next (odd) row
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
  const int frag = (lane & 48) + row_at(lane);
  const double* pa = lds + ua * PLANE + frag;
  const double* pb = lds + SIDE + ub * PLANE + frag;
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
          const int o = buf * STAGE + p * 8 * PLANE + ((half * HS + s) * NI + i) * 64;
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
    for (int q = 0; q < 4; ++q) val = __builtin_fma(g.ch[w][q], s[(4 + q) * NPART * T * T], val);
    double* dst = g.c[comp];
    if (dst && r < g.m && c < g.n) dst[r * g.ldc + c] = val;
  }
}

template <int IM, int T, int BK>
hipError_t launch_fused_t(const FusedArgs& g, hipStream_t s) {
  const int64_t tiles = ((g.m + T - 1) / T) * ((g.n + T - 1) / T);
  if (tiles > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL((bq_fused<IM, T, BK>), dim3((unsigned)tiles), dim3(512), 0, s, g);
  return hipGetLastError();
}

}  // namespace

// Which path a product takes: an estimate of both in microseconds, from rates
// measured on an MI355X at m = n = k = 64 .. 4096 (each line of the model is
// within 5 % of the measured times from n = 1200 on).  One round is one block
// on each of the 256 CUs (fused) or two (per product).
//   fused   a round of 32 x 32 blocks takes 0.233 us per unit of k (24 real
//           products) or 0.0765 (8); of 16 x 16 blocks a third of that, so
//           they win where three of their rounds replace more than one.
//   per     each of 8 launches: 0.20 us per unit of k and full round of 512
//   product 64 x 64 tiles, 0.14 for a last round of at most 256 tiles (one
//           per CU), 0.22 for a longer one; real products 0.07 per round of
//           512 (0.077 transposed), or 0.125 per round of 256 128 x 128
//           blocks.  Plus the pre-combination (16 blocks read and 16
//           written) and the read-modify-write of C at 4.8 TB/s, the latter
//           0.6 exposed.
// At n = 256 the fused kernel takes 24 us against 365, at 1024 865 us against
// 1204, at 2300 11.3 ms against 12.5; at 2600 it loses (16.3 against 15.5 ms)
// and at 3500 the per-product path is 11 % faster.
int fused_tile(int im, int64_t m, int64_t n, int64_t k, int ta, int tb, int64_t lda, int64_t ldb) {
  constexpr int64_t kCUs = 256;
  auto tiles = [&](int64_t t) { return ((m + t - 1) / t) * ((n + t - 1) / t); };
  auto rounds = [&](int64_t t, int64_t per) { return (tiles(t) + per - 1) / per; };
  // Buffer offsets inside a tile must reach every element (T <= 32, BK <= 32).
  if (32 * std::max(lda, ldb) * 8 + 32 * 8 >= 0x7fffffff) return 0;
  const int64_t r16 = rounds(16, kCUs), r32 = rounds(32, kCUs);
  const int tile = r16 <= 3 * r32 ? 16 : 32;
  const double per_k = im ? 0.233 : 0.0765;
  const double fused = double(k) * per_k * (tile == 16 ? double(r16) / 3.0 : double(r32));
  double launch;
  if (im) {
    const int64_t full = tiles(64) / (2 * kCUs), tail = tiles(64) % (2 * kCUs);
    launch = 0.20 * double(full) + (tail == 0 ? 0.0 : tail <= kCUs ? 0.14 : 0.22);
  } else if (!ta && !tb && default_tile_config(KIND_RR, m, n, k) == 11) {
    launch = 0.125 * double(rounds(128, kCUs));
  } else {
    launch = (ta || tb ? 0.077 : 0.07) * double(rounds(64, 2 * kCUs));
  }
  const double gb = 1e-6 / 4.8 * (im ? 1.0 : 0.5);  // us per byte of the 24-product form
  const double per_product = 8.0 * double(k) * launch + 128.0 * gb * (double(m) + double(n)) * double(k) +
                             0.6 * 576.0 * gb * double(m) * double(n);
  return fused <= per_product ? tile : 0;
}

hipError_t launch_fused(const FusedArgs& g, int im, int tile, hipStream_t s) {
  if (g.m <= 0 || g.n <= 0 || g.k <= 0) return hipErrorInvalidValue;
  if (im) return tile == 16 ? launch_fused_t<1, 16, 16>(g, s) : launch_fused_t<1, 32, 8>(g, s);
  return tile == 16 ? launch_fused_t<0, 16, 32>(g, s) : launch_fused_t<0, 32, 16>(g, s);
}

}  // namespace bq
