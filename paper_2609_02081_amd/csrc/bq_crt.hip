// CRT-based split form of one real product (Ozaki scheme II,
// integer-modular), for gfx950.
//
// A real product T = X Y: every row of X (column of Y) gets its frexp
// exponent e (f), the scaled integers X' = rint(x 2^(b - e)) (|X'| <= 2^b,
// b <= 53, exact in FP64) are written as symmetric residues modulo N odd,
// pairwise coprime moduli p_i <= 255 (one signed byte each), every modulus
// is one exact INT8 GEMM with int32 sums (|sum| <= k 127^2 < 2^31), its
// result reduced to a residue again, and P = X'Y' is recovered from its
// residues r_i by the Chinese remainder theorem: P = sum_i r_i c_i - q M
// with M = p_1 ... p_N, c_i = (M / p_i) ((M / p_i)^-1 mod p_i) and q the
// integer nearest to sum_i r_i (c_i / M).  The bound |P| <= k 2^(2b) <
// 2^127 lets that sum run in 128-bit wraparound integers, so P is exact;
// it is rounded to FP64 once and T = P 2^(e + f - 2b) is the correctly
// rounded product of the scaled integers.  N moduli with M > 2 k 2^(2b)
// carry b bits.
#include <limits.h>
#include <stddef.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>

#include "bq_split_common.h"

namespace bq {

constexpr int kCrtModuli[kMaxCrtModuli] = {255, 253, 251, 247, 241, 239, 233, 229, 227, 223,
                                           211, 199, 197, 193, 191, 181, 179, 173, 167, 163};

// Per modulus p: the symmetric residues of 256^j, j = 0..3 and 4..6, as four
// signed bytes each, and p and 1 / p in FP32.
struct CrtModulus {
  int wlo, whi;
  float p, inv;
};
struct CrtModuli {
  CrtModulus m[kMaxCrtModuli];
};
constexpr CrtModuli make_crt_weights() {
  CrtModuli t{};
  for (int i = 0; i < kMaxCrtModuli; ++i) {
    const int p = kCrtModuli[i];
    unsigned w[2] = {0, 0};
    int r = 1;
    for (int j = 0; j < 7; ++j) {
      const int s = r > (p - 1) / 2 ? r - p : r;
      w[j / 4] |= (unsigned)(s & 255) << (8 * (j % 4));
      r = r * 256 % p;
    }
    t.m[i] = {(int)w[0], (int)w[1], (float)p, 1.0f / (float)p};
  }
  return t;
}
__constant__ constexpr CrtModuli kCrtW = make_crt_weights();

// Symmetric residue of t (|t| < 2^31) modulo an odd p, in [-(p-1)/2, (p-1)/2],
// in the low byte of the result: q = rint(t / p) in FP64 is exact (t / p is
// never within 1 / (2 p) of a half-integer for odd p, far above the rounding
// error), and t - q p is formed exactly by one fma.  t enters FP64 through the
// low word of 2^52 + 2^31 + t and the integers leave it through the low word
// of a sum with 1.5 2^52: six full-rate instructions, no conversions.
__device__ __forceinline__ int sym_mod_rt(int t, double p, double inv_p) {
  constexpr double kMagic = 6755399441055744.0;     // 1.5 2^52
  constexpr double kOffset = 4503601774854144.0;    // 2^52 + 2^31
  const uint64_t u = 0x4330000000000000ull | ((uint32_t)t ^ 0x80000000u);
  const double td = __builtin_bit_cast(double, u) - kOffset;
  const double q = __builtin_fma(td, inv_p, kMagic) - kMagic;
  return (int)(uint32_t)__builtin_bit_cast(uint64_t, __builtin_fma(-q, p, td) + kMagic);
}

// X' = rint(x 2^(b - e)) (|X'| <= 2^53) as seven signed bytes d_j with X' =
// sum_j d_j 256^j: adding 128 in each of the seven places makes every digit
// of the sum d_j + 128, and the top bit of each byte turns it back.
__device__ __forceinline__ void crt_digits(double x, int e, int b, int& lo, int& hi) {
  const double y = exp_special(e) ? 0.0 : rint(ldexp(x, b - e));
  const uint64_t u = (uint64_t)(int64_t)y + 0x0080808080808080ull;
  lo = (int)((uint32_t)u ^ 0x80808080u);
  hi = (int)((uint32_t)(u >> 32) ^ 0x00808080u);
}

// Symmetric residue modulo m.p in the low byte of the result: t = sum_j d_j
// (256^j mod p) by two four-byte dot products (|t| < 2^17, summed onto the
// bits of 1.5 2^23, which makes the sum the FP32 number 1.5 2^23 + t), then t
// - p rint(t / p).  rint is exact: t / p is at least 1 / (2 p) from a
// half-integer and its FP32 error below 1e-4.  8 instructions against 25 for
// 18-bit limbs and an integer division by a constant.
__device__ __forceinline__ int crt_residue(int lo, int hi, const CrtModulus& m) {
  constexpr float kMagic = 12582912.0f;  // 1.5 2^23 = 0x4b400000
  int t = __builtin_amdgcn_sdot4(lo, m.wlo, 0x4b400000, false);
  t = __builtin_amdgcn_sdot4(hi, m.whi, t, false);
  const float tm = __builtin_bit_cast(float, t);
  const float q = __builtin_fmaf(tm - kMagic, m.inv, kMagic) - kMagic;
  return __builtin_bit_cast(int, __builtin_fmaf(-q, m.p, tm));
}

// Residues of one 64 x 64 tile (64 rows of the left factor, or columns of the
// right one, by 64 of the inner dimension) of the wanted values of an operand
// in the tiled 64-byte layout.  Thread: 16 consecutive inner elements (one
// 16-byte chunk of each plane) of one row or column; r and i are read once
// for all their values.  Where the inner dimension is contiguous four lanes
// share a row (512 bytes), else 64 lanes a row of the stored matrix.  The
// moduli run in a loop with their constants in scalar registers.  Traffic
// bound (8 or 16 bytes read and N written per element and value): at n = 4096
// all exponents and residues of a product take 6.8 ms (28 GB, 4.1 TB/s)
// against 9.6 with a launch and an atomic pass per operand; at n = 1024 0.59
// ms against 1.35 (32 launches against 144).  A thread's chain of 16 elements,
// three values and 15 moduli takes 20 us however few blocks there are: small
// launches divide the moduli among the blocks of the grid's y, each of which forms
// the digits again (crt_split_parts).  PARTS is an instance of its own: with the
// range of the moduli known at compile time the other saves 0.2 us a launch (n = 768
// 1079 against 1073 us a product, 8 of 300 in a batch 922 against 916).
template <bool PARTS>
__device__ __forceinline__ void crt_split_block(const SplitOperand& a, int64_t b) {
  const int64_t nkt = a.kp / 64;
  const int64_t rt = b / nkt, kt = b % nkt;
  const int t = threadIdx.x;
  const int64_t v = rt * 64 + (a.along ? t >> 2 : t & 63);
  const int64_t k0 = kt * 64 + (a.along ? t & 3 : t >> 6) * 16;
  const int64_t K = a.along ? a.cols : a.rows;
  const bool in = v < a.dim;
  const bool want_i = a.out[1] != nullptr || a.out[2] != nullptr;
  double r[16], im[16];
  load_inner16(a, a.r, v, k0, K, in, r);
  if (want_i) load_inner16(a, a.i, v, k0, K, in, im);
  const int64_t o = digit_offset(v, k0, a.kp);
  // this part's moduli
  const int i0 = PARTS ? (int)blockIdx.y * a.count / (int)gridDim.y : 0;
  const int i1 = PARTS ? ((int)blockIdx.y + 1) * a.count / (int)gridDim.y : a.count;
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    if (!a.out[s]) continue;
    const int e = in ? a.e[s][v] : INT_MIN;
    int lo[16], hi[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const double x = s == 0 ? r[j] : (s == 1 ? im[j] : __builtin_fma(a.w2, im[j], r[j]));
      crt_digits(x, e, a.bits, lo[j], hi[j]);
    }
    unsigned char* out = static_cast<unsigned char*>(a.out[s]) + o + i0 * a.plane;
    for (int i = i0; i < i1; ++i) {
      const CrtModulus m = kCrtW.m[i];
      i4v q;
#pragma unroll
      for (int g = 0; g < 4; ++g)
        q[g] = pack_bytes(crt_residue(lo[4 * g], hi[4 * g], m), crt_residue(lo[4 * g + 1], hi[4 * g + 1], m),
                          crt_residue(lo[4 * g + 2], hi[4 * g + 2], m), crt_residue(lo[4 * g + 3], hi[4 * g + 3], m));
      *reinterpret_cast<i4v*>(out) = q;
      out += a.plane;
    }
  }
}

// Both operands of a product in one launch: the blocks of x, then those of y;
// blockIdx.y: the part.
template <bool PARTS>
__global__ void __launch_bounds__(256) crt_split(const SplitOperand x, const SplitOperand y, int64_t xblocks) {
  const int64_t b = blockIdx.x;
  if (b < xblocks) crt_split_block<PARTS>(x, b);
  else crt_split_block<PARTS>(y, b - xblocks);
}

// One INT8 GEMM per modulus: residue planes of X (rows padded to 256) and Y
// (columns padded to 256) in the tiled 64-byte layout.  A block of 4 waves
// takes 256 x 128 tiles (128 x 64 a wave, 32 v_mfma_i32_16x16x64_i8 per
// k-step) or 128 x 128 ones (64 x 64, 16), three LDS stages filled straight
// from global memory two k-steps ahead, every wave moving a quarter of each 4
// KB operand tile.  The int32 result is reduced to its symmetric residue and
// stored as a byte plane R[i][row][col].
// What bounds it: the loads into LDS.  A launch that only issues the loads of
// 128 x 128 tiles moves 16-21 TB/s (about 26 bytes a clock and CU) and takes
// 48 of the 64 us of n = 1535, the MFMAs alone 43; the taller tile moves 3/4
// of the bytes per MFMA and reads 3/4 of the LDS bytes.  Two blocks a CU, each
// with tiles in a row, overlap the fill, the epilogue (8 instructions per
// element) and the drain.  Launches, 128 x 128 blocks of one tile against 256
// x 128 tiles in a row: n = 1024 24.2 -> 21.8 us, 1535 64.8 -> 59.3, 2048 132
// -> 124, 3072 (against 256 x 256) 413 -> 407; batches of 64 products of n =
// 64..1536 37.0 -> 35.0 ms.
// Modulus and tile of block b of the blocks [p0, p0 + N T) that run the N
// residue GEMMs of one product (T tiles each).  Small planes: each XCD takes
// a contiguous run over (modulus, tile), so it reads one or two moduli's
// planes once into its 4 MB L2 (a modulus spread over all XCDs is read eight
// times from beyond them).  Traced launches: n = 1024 30.8 -> 24.2 us, n =
// 1536 (4.7 MB per modulus) 82.6 -> 79.2, n = 2048 (8.4 MB) 139 -> 131; at
// n = 3072 (19 MB) no difference.  Larger planes: every modulus is spread over
// the XCDs, a run of tiles each, so that the planes in use at a time stay in
// the 256 MB cache behind the L2s.
constexpr int64_t kCrtXcdPlane = 9 << 20;

template <typename Args>
__device__ __forceinline__ void crt_gemm_tile_of(const Args& g, int64_t b, int64_t p0, int nmod, int tiles_m,
                                                 int tiles_n, int& mod, int& tm, int& tn) {
  const unsigned T = (unsigned)(tiles_m * tiles_n);  // launches hold fewer than 2^31 blocks
  unsigned t;
  if (g.plane_a + g.plane_b <= kCrtXcdPlane) {
    const unsigned pos = (unsigned)xcd_position(b, p0, p0 + (int64_t)T * nmod);
    mod = (int)(pos / T);
    t = pos % T;
  } else {
    mod = (int)((unsigned)(b - p0) / T);
    t = (unsigned)xcd_position(b, p0 + (int64_t)mod * T, p0 + (int64_t)(mod + 1) * T);
  }
  grouped_tile((int)t, tiles_m, tiles_n, tm, tn);
}

// 128 x 128 (WI = 4) or 256 x 128 (WI = 8) tile: 4 waves of WI x 4 MFMA tiles.
template <int WI>
struct CrtShape {
  static constexpr int BM = 32 * WI, BN = 128;
  static constexpr int TA = BM / 64, TB = BN / 64;  // 64-row operand tiles of 4 KB
  static constexpr int NPW = TA + TB;               // 1 KB pieces of a stage per wave
  static constexpr int NST = 3;                     // stages: two blocks fit a CU's LDS
  static constexpr int LDS = NST * NPW * 4096;
};
constexpr int kCrtGemmBlocks = 512;  // two on each of 256 CUs

// One output tile: its operand rows, and where its residues go.
struct CrtTile {
  const unsigned char *a, *b;
  int64_t run;  // bytes of a 64-row operand tile
  int nk, p;
  signed char* out;
  int rows, cols;  // from the tile's origin on: rows of the result, bytes of a residue row
  int64_t ldr;
};

template <int WI, typename Args>
__device__ __forceinline__ CrtTile crt_tile(const Args& g, int64_t v, int64_t p0, int nmod) {
  typedef CrtShape<WI> S;
  int mod, tm, tn;
  crt_gemm_tile_of(g, v, p0, nmod, (int)((g.m + S::BM - 1) / S::BM), (int)((g.n + S::BN - 1) / S::BN), mod, tm, tn);
  const int64_t m0 = (int64_t)tm * S::BM, n0 = (int64_t)tn * S::BN;
  CrtTile t;
  t.run = g.kp * 64;
  t.a = static_cast<const unsigned char*>(g.a) + mod * g.plane_a + m0 * g.kp;
  t.b = static_cast<const unsigned char*>(g.b) + mod * g.plane_b + n0 * g.kp;
  t.nk = (int)(g.kp / 64);
  t.p = kCrtModuli[mod];
  t.out = g.out + mod * g.plane_r + m0 * g.ldr + n0;
  t.rows = (int)(g.m - m0 < S::BM ? g.m - m0 : S::BM);
  t.cols = (int)(g.ldr - n0 < S::BN ? g.ldr - n0 : S::BN);
  t.ldr = g.ldr;
  return t;
}

// The tiles blockIdx.x, blockIdx.x + gridDim.x, ... of the launch's total;
// tile_at(v) is tile v.  The ring of LDS stages runs on over the tiles (each
// has two k-steps or more): the first two k-steps of the next tile arrive
// while the last two of this one and its epilogue run, which uses no LDS.
template <int WI, typename Lookup>
__device__ __forceinline__ void crt_gemm_tiles(const Lookup& tile_at, int64_t total, unsigned char* lds) {
  typedef CrtShape<WI> S;
  constexpr int ROWB = 64, TILE = 64 * ROWB, STAGE = S::NPW * TILE;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int wm0 = (wave >> 1) * (16 * WI), wn0 = (wave & 1) * 64;
  const int fr = lane & 15, fg = lane >> 4;

  // Piece i of the wave: its quarter of operand tile i (those of A first).
  auto dma = [&](const unsigned char* ga, const unsigned char* gb, int64_t run, int i, int kt, int st) {
    const unsigned char* src = i < S::TA ? ga + i * run : gb + (i - S::TA) * run;
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)src, (short)0, (int)run, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_ptr)(lds + st * STAGE + i * TILE + wave * 1024), 16,
                                             wave * 1024 + lane * 16, kt * TILE, 0, 0);
  };
  auto frag = [&](const unsigned char* base, int row) {
    return *reinterpret_cast<const i4v*>(base + row * ROWB + swz_chunk<16>(row & 63, fg) * 16);
  };

  int64_t v = blockIdx.x;
  CrtTile c = tile_at(v);
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int i = 0; i < S::NPW; ++i) dma(c.a, c.b, c.run, i, s, s);
  wait_vm<S::NPW>();
  block_sync();
  int st = 0;
  for (;;) {
    const bool more = v + gridDim.x < total;
    CrtTile n = c;  // after the last tile: loads that nothing reads
    if (more) n = tile_at(v + gridDim.x);
    i4v acc[WI][4];
#pragma unroll
    for (int i = 0; i < WI; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = i4v{0, 0, 0, 0};
    for (int kt = 0; kt < c.nk; ++kt) {
      const int sn = st == 0 ? 2 : st - 1;  // the stage of k-step kt - 1
      const bool over = kt + 2 >= c.nk;
      const unsigned char *ga = over ? n.a : c.a, *gb = over ? n.b : c.b;
      const int64_t run = over ? n.run : c.run;
      const int kn = over ? kt + 2 - c.nk : kt + 2;
      const unsigned char* ta = lds + st * STAGE;
      const unsigned char* tb = ta + S::TA * TILE;
      i4v fa[WI], fb[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) fb[j] = frag(tb, wn0 + j * 16 + fr);
#pragma unroll
      for (int i = 0; i < WI; ++i) fa[i] = frag(ta, wm0 + i * 16 + fr);
#pragma unroll
      for (int i = 0; i < WI; ++i) {
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[j], fa[i], acc[i][j], 0, 0, 0);
        if (i < S::NPW) dma(ga, gb, run, i, kn, sn);
        __builtin_amdgcn_sched_barrier(0);
      }
      // The next stage is complete once at most the loads of this k-step are
      // still out (the stores of an epilogue before them count as well).
      wait_vm<S::NPW>();
      block_sync();
      st = st == 2 ? 0 : st + 1;
    }
    // Residues as 16-byte stores (a residue row has a multiple of 16 bytes).
    // The right operand goes first into the MFMA, so a lane holds four columns
    // of a row per result: word j of lane row fg is columns 16 j + 4 fg.  A 4
    // x 4 transpose over the lane rows makes it word fg of lane row j.
    const double pd = (double)c.p, inv_p = 1.0 / pd;
#pragma unroll
    for (int i = 0; i < WI; ++i) {
      unsigned w[4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        w[j] = (unsigned)pack_bytes(sym_mod_rt(acc[i][j][0], pd, inv_p), sym_mod_rt(acc[i][j][1], pd, inv_p),
                                    sym_mod_rt(acc[i][j][2], pd, inv_p), sym_mod_rt(acc[i][j][3], pd, inv_p));
      const auto x = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
      const auto y = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
      const auto lo = __builtin_amdgcn_permlane16_swap(x[0], y[0], false, false);
      const auto hi = __builtin_amdgcn_permlane16_swap(x[1], y[1], false, false);
      const int r = wm0 + i * 16 + fr, col = wn0 + fg * 16;
      if (r < c.rows && col < c.cols)
        *reinterpret_cast<i4v*>(c.out + r * c.ldr + col) = i4v{(int)lo[0], (int)lo[1], (int)hi[0], (int)hi[1]};
    }
    if (!more) break;
    v += gridDim.x;
    c = n;
  }
  wait_vm<0>();  // no load into LDS outlives the block
}

template <int WI>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
crt_gemm(const CrtGemmArgs g, int nmod, int64_t total) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[CrtShape<WI>::LDS];
  crt_gemm_tiles<WI>([&](int64_t v) { return crt_tile<WI>(g, v, 0, nmod); }, total, lds);
}

// The same GEMM for large products: a 256 x 256 block of 4 waves (128 x 128
// each: 8 x 8 v_mfma_i32_16x16x64_i8 per k-step, accumulators in AGPRs), so
// each k-step moves 32 KB into LDS for 2^23 multiply-adds, half the bytes
// per MFMA of the 128 x 128 block.  Four LDS stages of 32 KB filled straight
// from global memory three k-steps ahead (8 KB per wave per k-step, one 1 KB
// piece after each row of MFMAs); the fragments of k-step kt + 1 are read
// from LDS into a second register set while the MFMAs of k-step kt run.
// The int32 results are reduced to residues, gathered as a 256 x 256 byte
// tile in LDS and stored as 16-byte rows.  The right operand goes first into
// the MFMA, so a lane's four results are four columns of one row and leave as
// one word.  n = 4096: 888 us a launch, 2.48 POP/s (918 with byte stores and
// FP64 conversions), at the 1.9-2.1 GHz the socket's power limit leaves.
template <int NST>  // LDS stages; 4 measured faster than 5
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
crt_gemm_256(const CrtGemmArgs g, int nmod) {
  constexpr int BM = 256, BN = 256, ROWB = 64, TILE = 64 * ROWB;  // 4 KB per 64-row tile
  constexpr int STAGE = 8 * TILE;                                  // four A tiles, four B tiles
  constexpr int NPW = 8;
  static_assert(NST >= 4 && NST * STAGE <= 160 * 1024, "stages fit LDS");
  constexpr int OUT_LD = BN + 16;
  static_assert(BM * OUT_LD <= NST * STAGE, "the residue tile fits the stages");
  __shared__ __attribute__((aligned(16))) unsigned char lds[NST * STAGE];
  int mod, tm, tn;
  crt_gemm_tile_of(g, blockIdx.x, 0, nmod, (int)((g.m + BM - 1) / BM), (int)((g.n + BN - 1) / BN), mod, tm, tn);
  const int p = kCrtModuli[mod];
  const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave >> 1) * 128, wn0 = (wave & 1) * 128;
  const int fr = lane & 15, fg = lane >> 4;

  const int64_t nk = g.kp / ROWB;
  const int64_t run = nk * TILE;
  const unsigned char* ga = static_cast<const unsigned char*>(g.a) + mod * g.plane_a + (int64_t)(4 * tm) * run;
  const unsigned char* gb = static_cast<const unsigned char*>(g.b) + mod * g.plane_b + (int64_t)(4 * tn) * run;
  const int nrec = (int)(uint32_t)(4 * run);
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc((void*)ga, (short)0, nrec, 0x00020000);
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void*)gb, (short)0, nrec, 0x00020000);
  // 1 KB piece q of a stage: q < 16 A (tile q / 4, quarter q % 4), else B.
  auto dma = [&](int q, int64_t kt, int st) {
    const int t = (q >> 2) & 3, quarter = q & 3;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(q >= 16 ? rb : ra, (lds_void_ptr)(lds + st * STAGE + q * 1024), 16,
                                             (int)(t * run) + quarter * 1024 + lane * 16, (int)(kt * TILE), 0, 0);
  };
  auto frag = [&](const unsigned char* base, int row) {
    return *reinterpret_cast<const i4v*>(base + row * ROWB + swz_chunk<16>(row & 63, fg) * 16);
  };
  auto read_frags = [&](int st, i4v(&fa)[8], i4v(&fb)[8]) {
    const unsigned char* ta = lds + st * STAGE;
    const unsigned char* tb = ta + 4 * TILE;
#pragma unroll
    for (int i = 0; i < 8; ++i) fa[i] = frag(ta, wm0 + i * 16 + fr);
#pragma unroll
    for (int j = 0; j < 8; ++j) fb[j] = frag(tb, wn0 + j * 16 + fr);
  };

  i4v acc[8][8];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = i4v{0, 0, 0, 0};

  // One k-step: fa, fb hold its fragments; na, nb receive those of kt + 1
  // (for kt + 1 = nk, stale LDS bytes that are never used).  Stage kt + 1 is
  // complete once only the loads of k-steps kt + 2 .. kt + NST - 2 are out;
  // after the barrier every wave holds the fragments of k-step kt, so stage
  // (kt - 1) % NST is free for k-step kt + NST - 1.
  auto step = [&](int64_t kt, i4v(&fa)[8], i4v(&fb)[8], i4v(&na)[8], i4v(&nb)[8]) {
    wait_vm<(NST - 3) * NPW>();
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): fa, fb have landed
    block_sync();
    read_frags((int)((kt + 1) % NST), na, nb);
    const int64_t knext = kt + NST - 1 < nk ? kt + NST - 1 : nk - 1;
    const int sn = (int)((kt + NST - 1) % NST);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fb[j], fa[i], acc[i][j], 0, 0, 0);
      dma(wave * NPW + i, knext, sn);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // Prologue: k-steps 0..NST-2 (past the end: the last one again); the
  // fragments of k-step 0.
#pragma unroll
  for (int s = 0; s < NST - 1; ++s)
#pragma unroll
    for (int i = 0; i < NPW; ++i) dma(wave * NPW + i, s < nk ? s : nk - 1, s);
  wait_vm<(NST - 2) * NPW>();
  block_sync();
  i4v xa[8], xb[8], ya[8], yb[8];
  read_frags(0, xa, xb);
  // nk is even (k padded to 128).
  for (int64_t kt = 0; kt < nk; kt += 2) {
    step(kt, xa, xb, ya, yb);
    step(kt + 1, ya, yb, xa, xb);
  }
  wait_vm<0>();
  __builtin_amdgcn_s_waitcnt(0xC07F);
  block_sync();

  // Residues into a byte tile (rows of OUT_LD bytes), then 16-byte stores.
  const double pd = (double)p, inv_p = 1.0 / pd;
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j)
      *reinterpret_cast<int*>(lds + (wm0 + i * 16 + fr) * OUT_LD + wn0 + j * 16 + 4 * fg) =
          pack_bytes(sym_mod_rt(acc[i][j][0], pd, inv_p), sym_mod_rt(acc[i][j][1], pd, inv_p),
                     sym_mod_rt(acc[i][j][2], pd, inv_p), sym_mod_rt(acc[i][j][3], pd, inv_p));
  __syncthreads();
  signed char* out = g.out + (int64_t)mod * g.plane_r;
  for (int w = tid; w < BM * (BN / 16); w += 256) {
    const int r = w / (BN / 16), ch = w % (BN / 16);
    const int64_t grow = m0 + r, gcol = n0 + ch * 16;
    if (grow < g.m && gcol < g.ldr)
      *reinterpret_cast<i4v*>(out + grow * g.ldr + gcol) = *reinterpret_cast<const i4v*>(lds + r * OUT_LD + ch * 16);
  }
}

// Reconstruction constants of one modulus count: with M = p_1 ... p_N and c_i
// = M_i (M_i^-1 mod p_i), M_i = M / p_i, taken symmetric (|c_i| < M / 2): c_i
// modulo 2^128 as 16 signed bytes, c[j][i / 4] holding byte j of four moduli;
// rint(2^23 c_i / M) as 3 signed bytes the same way; M modulo 2^128 as eight
// 16-bit limbs.  Moduli past the count have zeros.  Everything is formed
// modulo 2^128, so no wider integer is needed.
constexpr int kCrtGroups = kMaxCrtModuli / 4;
struct alignas(16) CrtConsts {
  int c[16][8];  // kCrtGroups used, rows of 32 bytes
  int f[3][8];
  int m16[8];
};
struct CrtConstTable {
  CrtConsts n[kMaxCrtModuli + 1];
};
constexpr CrtConsts make_crt_consts(int N) {
  CrtConsts t{};
  unsigned __int128 M = 1, each = 0;  // each: 0x80 in every byte
  for (int i = 0; i < N; ++i) M *= (unsigned)kCrtModuli[i];
  for (int j = 0; j < 16; ++j) each |= (unsigned __int128)0x80 << (8 * j);
  for (int h = 0; h < 8; ++h) t.m16[h] = (int)((unsigned)(M >> (16 * h)) & 0xffffu);
  for (int i = 0; i < N; ++i) {
    const int p = kCrtModuli[i];
    unsigned __int128 Mi = 1;
    int a = 1, inv = 1;  // M_i modulo p, and its inverse by search
    for (int j = 0; j < N; ++j)
      if (j != i) {
        Mi *= (unsigned)kCrtModuli[j];
        a = a * kCrtModuli[j] % p;
      }
    while (a * inv % p != 1) ++inv;
    // c_i / M = inv / p, symmetric: inv - p where inv / p > 1 / 2.
    const int num = inv > (p - 1) / 2 ? inv - p : inv;
    unsigned __int128 c = Mi * (unsigned)inv;
    if (num < 0) c -= M;
    c += each;  // bytes d_j + 128 of the signed digits d_j
    for (int j = 0; j < 16; ++j)
      t.c[j][i / 4] |= (int)((((unsigned)(c >> (8 * j)) & 255u) ^ 0x80u) << (8 * (i % 4)));
    const int64_t twice = 2 * (int64_t)num * 8388608 + p;  // rint: floor((2 num 2^23 + p) / (2 p))
    const int64_t q = twice >= 0 ? twice / (2 * p) : -((-twice + 2 * p - 1) / (2 * p));
    const unsigned f = (unsigned)(int)q + 0x808080u;
    for (int j = 0; j < 3; ++j) t.f[j][i / 4] |= (int)((((f >> (8 * j)) & 255u) ^ 0x80u) << (8 * (i % 4)));
  }
  return t;
}
constexpr CrtConstTable make_crt_const_table() {
  CrtConstTable t{};
  for (int N = 1; N <= kMaxCrtModuli; ++N) t.n[N] = make_crt_consts(N);
  return t;
}
__constant__ constexpr CrtConstTable kCrtC = make_crt_const_table();

typedef const __attribute__((address_space(4))) CrtConsts* crt_consts_ptr;
typedef int i16v __attribute__((ext_vector_type(16)));

// |P| 2^shift rounded to FP64 once (to nearest even): the leading 64 bits with
// every lower bit folded into a sticky bit, converted as two exact 32-bit
// halves joined by one fma.
__device__ __forceinline__ double u128_to_double(uint64_t hi, uint64_t lo, int shift) {
  const int nlz = hi ? __builtin_clzll(hi) : 0;
  uint64_t top = (hi << nlz) | ((lo >> 1) >> (63 - nlz));
  const uint64_t rest = lo << nlz;
  top |= (uint64_t)(rest != 0);
  top = hi ? top : lo;
  const double d = __builtin_fma((double)(uint32_t)(top >> 32), 4294967296.0, (double)(uint32_t)top);
  return ldexp(d, hi ? 64 - nlz + shift : shift);
}

// P_p from its residues, T_p = P_p 2^(e + f - 2b) for the np real
// products, sum_p coef[q][p] T_p into every target.  Thread: 4 consecutive
// columns of one row (one 32-bit load per residue plane).  P = sum_i r_i c_i -
// q M modulo 2^128 in integers: the byte places of sum_i r_i c_i are a product
// of the constants' bytes (rows) and the residues (a byte transpose of four
// planes' words puts an element's moduli into one lane's operand), two v_mfma
// for 64 elements; two places share a 32-bit sum (|sum| < 2^28 with q M taken
// off), and one pass of carries leaves the 16-bit limbs.  q is rint(s), s =
// sum_i r_i c_i / M from 23-bit fractions the same way (error below 2^-12): for
// at most 16 moduli P may come near M / 2, so a fraction of s within 2^-11 of
// 1/2 is settled by comparing P with M / 2 (M < 2^125: an estimate one off
// leaves P - M or P + M, both in range); with more moduli |P| < 2^-6 M.
// 76 four-byte dot products an element and real product took the matrix
// products' place before; the rare correction and the special exponents are one
// branch for four elements, the sign none.  Launches: n = 1024 37.4 -> 31.3 us,
// 1535 98 -> 88, 4096 477 -> 416; now near the planes' and the targets' traffic
// (87 us at n = 1535 at the copy rate).  The waves of a block without columns end
// at once: the eight launches of 20000 x 16 outputs 0.66 ms (1.75 with all four
// waves at work), of 4000 x 256 0.26 (0.44).
constexpr int kCombineCols = 4;

// The constants as left operands of v_mfma_i32_32x32x32_i8: a lane holds 16 k
// of row (lane & 31), k being the modulus.  The results of a lane are the rows
// 8 (u / 4) + 4 (lane / 32) + u % 4, u = 0..15, of column (lane & 31), so
// digit 2 u + h (c in 0..15, f in 16..18) is put into the row that result u of
// lane half h holds.  lo[i] has zeros in the other half's k: the product with
// [i] sums the residues of the elements of lane half i alone.  top: moduli 16..19.
struct CrtRows {
  i4v lo[2], top[2];
};

template <int NG>
__device__ __forceinline__ CrtRows crt_rows(int nmod) {
  static_assert(offsetof(CrtConsts, c) == 0 && offsetof(CrtConsts, f) == 16 * 32, "digits in rows of 32 bytes");
  const int lane = threadIdx.x & 63, row = lane & 31;
  const int digit = 8 * (row >> 3) + 2 * (row & 3) + (row >> 2 & 1);
  const int* k = reinterpret_cast<const int*>(&kCrtC.n[nmod]) + 8 * (digit < 19 ? digit : 0);
  CrtRows A;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const bool mine = digit < 19 && (lane >> 5) == i;
    const i4v lo = *reinterpret_cast<const i4v*>(k);
    A.lo[i] = mine ? lo : i4v{0, 0, 0, 0};
    A.top[i] = i4v{NG > 4 && mine ? k[4] : 0, 0, 0, 0};
  }
  return A;
}

template <int NG, typename Args>
__device__ __forceinline__ void crt_values(const Args& g, int nmod, const CrtRows& A, const signed char* res,
                                           int64_t off, const int (&shift)[4], double (&out)[4]) {
  // R[e][G]: residues 4 G .. 4 G + 3 of element e.
  int R[4][NG];
#pragma unroll
  for (int G = 0; G < NG; ++G) {
    unsigned w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      w[i] = 4 * G + i < nmod
                 ? *reinterpret_cast<const uint32_t*>(res + (int64_t)(4 * G + i) * g.plane_r + off)
                 : 0u;
    const unsigned ab0 = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u), ab1 = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);
    const unsigned cd0 = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u), cd1 = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
    R[0][G] = (int)__builtin_amdgcn_perm(cd0, ab0, 0x05040100u);
    R[1][G] = (int)__builtin_amdgcn_perm(cd0, ab0, 0x07060302u);
    R[2][G] = (int)__builtin_amdgcn_perm(cd1, ab1, 0x05040100u);
    R[3][G] = (int)__builtin_amdgcn_perm(cd1, ab1, 0x07060302u);
  }
  const crt_consts_ptr K = (crt_consts_ptr)&kCrtC.n[nmod];
  uint64_t lo[4], hi[4];
  unsigned near[4];  // below 32: the fraction of s within 2^-11 of 1/2
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    i4v x{0, 0, 0, 0};
#pragma unroll
    for (int G = 0; G < (NG < 4 ? NG : 4); ++G) x[G] = R[e][G];
    i16v d[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      i16v z;
#pragma unroll
      for (int u = 0; u < 16; ++u) z[u] = 0;
      d[i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A.lo[i], x, z, 0, 0, 0);
      if constexpr (NG > 4)
        d[i] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A.top[i], i4v{R[e][NG - 1], 0, 0, 0}, d[i], 0, 0, 0);
    }
    // Digits 2 u, 2 u + 1 of this lane's element.
    auto digits = [&](int u) { return __builtin_amdgcn_permlane32_swap((unsigned)d[0][u], (unsigned)d[1][u], false, false); };
    int y[8];
#pragma unroll
    for (int h = 0; h < 8; ++h) {
      const auto t = digits(h);
      y[h] = (int)t[0] + ((int)t[1] << 8);
    }
    const auto f0 = digits(8), f2 = digits(9);
    const int v = ((int)f2[0] << 8) + (int)f0[1] + ((int)f0[0] >> 8);
    const int q = (v + (1 << 14)) >> 15;  // s 2^15 in v
#pragma unroll
    for (int h = 0; h < 8; ++h) {
      y[h] += __mul24(-q, K->m16[h]);
      if (h > 0) y[h] += y[h - 1] >> 16;
    }
    auto limb = [&](int j) {
      return __builtin_amdgcn_perm((unsigned)y[2 * j + 1], (unsigned)y[2 * j], 0x05040100u);
    };
    lo[e] = ((uint64_t)limb(1) << 32) | limb(0);
    hi[e] = ((uint64_t)limb(3) << 32) | limb(2);
    near[e] = (unsigned)(v + (1 << 14) + 16) & 0x7fffu;
  }
  if constexpr (NG <= 4) {
    if (min(min(near[0], near[1]), min(near[2], near[3])) < 32u) {
      unsigned __int128 Mu = 0;
#pragma unroll
      for (int h = 0; h < 8; ++h) Mu |= (unsigned __int128)(unsigned)K->m16[h] << (16 * h);
      const __int128 M = (__int128)Mu, half = (M - 1) >> 1;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        __int128 P = (__int128)(((unsigned __int128)hi[e] << 64) | lo[e]);
        const __int128 d = P > half ? M : (P < -half ? -M : (__int128)0);
        P -= near[e] < 32u ? d : (__int128)0;
        lo[e] = (uint64_t)P;
        hi[e] = (uint64_t)((unsigned __int128)P >> 64);
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    // |P| and the sign without a branch: x ^ s - s over 128 bits.
    const uint64_t sg = (uint64_t)((int64_t)hi[e] >> 63);
    const unsigned __int128 sw = ((unsigned __int128)sg << 64) | sg;
    const unsigned __int128 u = ((((unsigned __int128)hi[e] << 64) | lo[e]) ^ sw) - sw;
    const double a = u128_to_double((uint64_t)(u >> 64), (uint64_t)u, shift[e]);
    out[e] = sg ? -a : a;
  }
}

// Columns c0 .. c0 + 3 of row r of the reconstruction of one complex product.
// Args: CrtCombineArgs as kernel arguments, or in a device table read as
// constant memory (a private copy would sit in scratch, as the loop over the
// targets indexes it dynamically).
template <int NG, typename Args>
__device__ __forceinline__ void crt_combine_at(const Args& g, int nmod, int64_t r, int64_t c0) {
  constexpr int CC = kCombineCols;
  // A wave without columns has nothing to do.  In others a thread without
  // columns takes the first ones and stores nothing: the matrix products need the
  // operand rows of every lane.
  const bool live = r < g.m && c0 < g.n;
  if (__builtin_amdgcn_ballot_w64(live) == 0) return;
  if (!live) r = c0 = 0;
  const int np = g.np;
  const int64_t n = g.n;
  const CrtRows A = crt_rows<NG>(nmod);
  double t[kCrtProducts][CC];
#pragma unroll
  for (int p = 0; p < kCrtProducts; ++p) {
#pragma unroll
    for (int e = 0; e < CC; ++e) t[p][e] = 0.0;
    if (p < np) {
      const int ea = g.ea[p][r];
      int eb[CC], shift[CC];
      bool special = exp_special(ea);
#pragma unroll
      for (int e = 0; e < CC; ++e) {
        eb[e] = g.eb[p][c0 + e < n ? c0 + e : n - 1];
        const bool sp = exp_special(ea) || exp_special(eb[e]);
        special = special || sp;
        shift[e] = sp ? 0 : ea + eb[e] - 2 * g.bits;
      }
      crt_values<NG>(g, nmod, A, g.res[p], r * g.ldr + c0, shift, t[p]);
      if (special) {
#pragma unroll
        for (int e = 0; e < CC; ++e)
          if (exp_special(ea) || exp_special(eb[e])) t[p][e] = exp_scaled(0.0, ea, eb[e], 0);
      }
    }
  }
  if (!live) return;
  // Targets in fours: their old values are loaded together before the first
  // store (the blocks of C do not overlap, which the compiler cannot know).
  // The loop stays a loop, so that the targets' arguments are read as needed.
  const int ntgt = g.ntgt;
  const bool pairs = g.vec && c0 + CC <= n;
#pragma unroll 1
  for (int q0 = 0; q0 < ntgt; q0 += 4) {
    double old[4][CC];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
#pragma unroll
      for (int e = 0; e < CC; ++e) old[u][e] = 0.0;
      if (q0 + u < ntgt && g.mode[q0 + u] == TGT_ACCUM) {
        const double* cq = g.c[q0 + u] + r * g.ldc + c0;
        if (pairs) {
#pragma unroll
          for (int e = 0; e < CC; e += 2) {
            const double2 d = *reinterpret_cast<const double2*>(cq + e);
            old[u][e] = d.x;
            old[u][e + 1] = d.y;
          }
        } else {
#pragma unroll
          for (int e = 0; e < CC; ++e)
            if (c0 + e < n) old[u][e] = cq[e];
        }
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (q0 + u >= ntgt) continue;
      double* cq = g.c[q0 + u] + r * g.ldc + c0;
      // Zero coefficients are skipped, as the products they would scale; the
      // first product is added to -0, which leaves every value as it is.
      double val[CC];
#pragma unroll
      for (int e = 0; e < CC; ++e) val[e] = -0.0;
#pragma unroll
      for (int p = 0; p < kCrtProducts; ++p)
        if (g.nz[q0 + u] >> p & 1) {
          const double w = g.coef[q0 + u][p];
#pragma unroll
          for (int e = 0; e < CC; ++e) val[e] = __builtin_fma(w, t[p][e], val[e]);
        }
      if (g.mode[q0 + u] == TGT_ACCUM) {
#pragma unroll
        for (int e = 0; e < CC; ++e) val[e] += old[u][e];
      }
      if (pairs) {
#pragma unroll
        for (int e = 0; e < CC; e += 2) *reinterpret_cast<double2*>(cq + e) = double2{val[e], val[e + 1]};
      } else {
#pragma unroll
        for (int e = 0; e < CC; ++e)
          if (c0 + e < n) cq[e] = val[e];
      }
    }
  }
}

template <int NG>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3)))
crt_combine(const CrtCombineArgs g, int nmod) {
  const int64_t bpr = (g.n + 256 * kCombineCols - 1) / (256 * kCombineCols);
  crt_combine_at<NG>(g, nmod, blockIdx.x / bpr, (blockIdx.x % bpr) * (256 * kCombineCols) + threadIdx.x * kCombineCols);
}

// ---------------------------------------------------------------------------
// Grouped forms: one launch over the items of many problems.
// ---------------------------------------------------------------------------
// VALUES: blockIdx.z is the one of the up to three values that the block forms.
template <bool PARTS, bool VALUES>
__global__ void __launch_bounds__(256) crt_split_grouped(const SplitOperand* items, const int64_t* prefix, int count) {
  const int64_t b = blockIdx.x;
  const int i = find_item(prefix, count, b);
  SplitOperand a = items[i];
  if constexpr (VALUES) {
#pragma unroll
    for (int s = 0; s < 3; ++s)
      if (s != (int)blockIdx.z) a.out[s] = nullptr;
    if (!a.out[0] && !a.out[1] && !a.out[2]) return;
  }
  crt_split_block<PARTS>(a, b - prefix[i]);
}

// The tables are read through the constant address space, so that the search
// for the next tile is scalar loads: a vector load would wait for the loads
// into LDS that are on their way.
template <int WI>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
crt_gemm_grouped(const CrtGemmItem* items, const int64_t* prefix, int count, int64_t total) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[CrtShape<WI>::LDS];
  typedef const __attribute__((address_space(4))) CrtGemmItem table_item;
  typedef const __attribute__((address_space(4))) int64_t table_prefix;
  table_item* ti = (table_item*)items;
  table_prefix* tp = (table_prefix*)prefix;
  auto tile_at = [&](int64_t v) {
    const int i = find_item(tp, count, v);
    return crt_tile<WI>(ti[i].g, v, tp[i], ti[i].nmod);
  };
  crt_gemm_tiles<WI>(tile_at, total, lds);
}

template <int NG>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3)))
crt_combine_grouped(const CrtCombineArgs* items, const int64_t* prefix, int count, int nmod) {
  const int64_t b = blockIdx.x;
  const int i = find_item(prefix, count, b);
  // thread: four columns; the quads of consecutive rows packed into the block
  typedef const __attribute__((address_space(4))) CrtCombineArgs table_args;
  table_args& g = *(table_args*)(items + __builtin_amdgcn_readfirstlane(i));
  const int64_t qpr = (g.n + kCombineCols - 1) / kCombineCols;
  const int64_t q = (b - prefix[i]) * 256 + threadIdx.x;
  crt_combine_at<NG>(g, nmod, q / qpr, (q % qpr) * kCombineCols);
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
// Parts of a residue launch of `blocks` blocks: the moduli in as many as fill the
// CUs once, none from 256 blocks on.  One part against the rule, 2 and 8: one call
// n = 64 (4 blocks) 444 against 346 us, 372, 348; 256 (32) 487 against 393, 440,
// 393; 300 (60) 544 against 470, 500, 488; 512 (128) 621 against 571, 571, 636;
// 1024 (512) 1303, 1329, 1663.  Batches, op N T: 1 product of 72 314 against 214,
// 8 401 against 323, 64 (512 blocks) 744, 756, 945.
constexpr int kCrtSplitMostParts = 15;
// A batch's launch of so few blocks has its (up to three) values in blocks of
// their own as well, the moduli in as many parts as then fill the CUs.  All
// values in a block against this, whole batches: op N T 1 product of 72 (8
// blocks) 215 against 206 us, 2 of unequal shapes 244 against 231; N N 1 of 72
// 221 against 208; 8 of 72 (64 blocks) 328 against 323, within a run's spread.
constexpr int64_t kCrtSplitValuesMost = 42;
static unsigned crt_split_parts(int64_t blocks) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(kCrtSplitMostParts, 256 / std::max<int64_t>(1, blocks)));
}

hipError_t launch_crt_split(const SplitOperand& x, const SplitOperand& y, hipStream_t st) {
  const int64_t xb = split_blocks(x), blocks = xb + split_blocks(y);
  if (blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffff || x.count > kMaxCrtModuli || y.count > kMaxCrtModuli) return hipErrorInvalidValue;
  const unsigned parts = crt_split_parts(blocks);
  auto* kernel = parts > 1 ? crt_split<true> : crt_split<false>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)blocks, parts), dim3(256), 0, st, x, y, xb);
  return hipGetLastError();
}

// Rows of the 128-column tiles of a launch that would hold `small` tiles of
// 128 rows or `tall` of 256: the tall tile where it leaves 1.5 tiles a CU or
// more and little padding (it takes about 1.6 times as long as the small one).
// Launches, 128 against 256 rows: n = 512 (120 tall tiles) 9.8 against 11.8
// us, 768 (270) 16.7 against 17.3, 1024 (480) 22.8 against 21.8, 1535 62.7
// against 59.3, 1700 95.6 against 88.6; batches: 16 products of 1024 18.0
// against 16.3 ms, 64 of 100 (as many tall as small) 1.02 against 1.12.
int crt_tile_rows(int64_t small, int64_t tall) { return tall >= 384 && 8 * tall <= 5 * small ? 256 : 128; }

// Tile of one product's residue GEMMs: 256 x 256 from 16 of them a CU on (a
// third less to move into LDS, but one block a CU, whose fill and drain
// nothing covers), else by the rule above.  256 x 128 against 256 x 256: n =
// 2048 (1024 large tiles) 124 against 132 us, 3072 (2448) 407 against 410,
// 3328 (2873) 524 against 520, 3584 (3332) 637 against 661, 4096 (4608) 934
// against 918.  BQ_CRT_TILE=128, 256x128 or 256 overrides.
enum class CrtTileShape { k128, k256x128, k256 };
CrtTileShape crt_tile_shape(int64_t small, int64_t tall, int64_t large) {
  if (const char* e = std::getenv("BQ_CRT_TILE")) {
    if (std::strcmp(e, "256x128") == 0) return CrtTileShape::k256x128;
    if (std::atoi(e) == 128) return CrtTileShape::k128;
    if (std::atoi(e) == 256) return CrtTileShape::k256;
  }
  if (large >= 4096) return CrtTileShape::k256;
  return crt_tile_rows(small, tall) == 256 ? CrtTileShape::k256x128 : CrtTileShape::k128;
}

template <int WI>
void launch_crt_tiles(int N, const CrtGemmArgs& g, int64_t total, hipStream_t st) {
  const int64_t grid = total < kCrtGemmBlocks ? total : kCrtGemmBlocks;
  hipLaunchKernelGGL(crt_gemm<WI>, dim3((unsigned)grid), dim3(256), 0, st, g, N, total);
}

hipError_t launch_crt_gemm(int N, const CrtGemmArgs& g, hipStream_t st) {
  if (g.m <= 0 || g.n <= 0 || N <= 0) return hipSuccess;
  if (N > kMaxCrtModuli || (g.ldr & 15) != 0 || g.kp % 128 != 0) return hipErrorInvalidValue;  // two k-steps or more
  const int64_t small = crt_gemm_blocks({g, N, 128}), tall = crt_gemm_blocks({g, N, 256});
  const int64_t large = ((g.m + 255) / 256) * ((g.n + 255) / 256) * N;
  const CrtTileShape shape = crt_tile_shape(small, tall, large);
  const int64_t total = shape == CrtTileShape::k128 ? small : (shape == CrtTileShape::k256 ? large : tall);
  if (total > 0x7fffffff) return hipErrorInvalidValue;
  switch (shape) {
    case CrtTileShape::k128: launch_crt_tiles<4>(N, g, total, st); break;
    case CrtTileShape::k256x128: launch_crt_tiles<8>(N, g, total, st); break;
    case CrtTileShape::k256: hipLaunchKernelGGL(crt_gemm_256<4>, dim3((unsigned)total), dim3(256), 0, st, g, N); break;
  }
  return hipGetLastError();
}

hipError_t launch_crt_combine(int N, const CrtCombineArgs& g, hipStream_t st) {
  const int64_t blocks = g.m * ((g.n + 256 * kCombineCols - 1) / (256 * kCombineCols));
  if (blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffff || (g.ldr % kCombineCols) != 0 || N < 1 || N > kMaxCrtModuli) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks), block(256);
  switch ((N + 3) / 4) {
    case 1: hipLaunchKernelGGL(crt_combine<1>, grid, block, 0, st, g, N); break;
    case 2: hipLaunchKernelGGL(crt_combine<2>, grid, block, 0, st, g, N); break;
    case 3: hipLaunchKernelGGL(crt_combine<3>, grid, block, 0, st, g, N); break;
    case 4: hipLaunchKernelGGL(crt_combine<4>, grid, block, 0, st, g, N); break;
    default: hipLaunchKernelGGL(crt_combine<5>, grid, block, 0, st, g, N); break;
  }
  return hipGetLastError();
}

int crt_modulus(int i) { return (i >= 0 && i < kMaxCrtModuli) ? kCrtModuli[i] : 0; }

int64_t crt_combine_blocks(const CrtCombineArgs& c) {
  return (c.m * ((c.n + kCombineCols - 1) / kCombineCols) + 255) / 256;
}

hipError_t launch_crt_split_grouped(const SplitOperand* items, const int64_t* prefix, int count, int64_t blocks,
                                    hipStream_t st) {
  if (count <= 0 || blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  const unsigned values = blocks <= kCrtSplitValuesMost ? 3 : 1, parts = crt_split_parts(values * blocks);
  auto* kernel = values > 1  ? crt_split_grouped<true, true>
                 : parts > 1 ? crt_split_grouped<true, false>
                             : crt_split_grouped<false, false>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)blocks, parts, values), dim3(256), 0, st, items, prefix, count);
  return hipGetLastError();
}

hipError_t launch_crt_gemm_grouped(const CrtGemmItem* items, const int64_t* prefix, int count, int64_t blocks, int rows,
                                   hipStream_t st) {
  if (count <= 0 || blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffff || (rows != 128 && rows != 256)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(blocks < kCrtGemmBlocks ? blocks : kCrtGemmBlocks)), block(256);
  if (rows == 256) hipLaunchKernelGGL(crt_gemm_grouped<8>, grid, block, 0, st, items, prefix, count, blocks);
  else hipLaunchKernelGGL(crt_gemm_grouped<4>, grid, block, 0, st, items, prefix, count, blocks);
  return hipGetLastError();
}

hipError_t launch_crt_combine_grouped(int N, const CrtCombineArgs* items, const int64_t* prefix, int count,
                                      int64_t blocks, hipStream_t st) {
  if (count <= 0 || blocks <= 0) return hipSuccess;
  if (blocks > 0x7fffffff || N < 1 || N > kMaxCrtModuli) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks), block(256);
  switch ((N + 3) / 4) {
    case 1: hipLaunchKernelGGL(crt_combine_grouped<1>, grid, block, 0, st, items, prefix, count, N); break;
    case 2: hipLaunchKernelGGL(crt_combine_grouped<2>, grid, block, 0, st, items, prefix, count, N); break;
    case 3: hipLaunchKernelGGL(crt_combine_grouped<3>, grid, block, 0, st, items, prefix, count, N); break;
    case 4: hipLaunchKernelGGL(crt_combine_grouped<4>, grid, block, 0, st, items, prefix, count, N); break;
    default: hipLaunchKernelGGL(crt_combine_grouped<5>, grid, block, 0, st, items, prefix, count, N); break;
  }
  return hipGetLastError();
}

}  // namespace bq
