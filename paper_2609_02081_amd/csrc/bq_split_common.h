// Device helpers shared by the split-form kernels (bq_split.hip, bq_crt.hip):
// vector types, the split operand, the tiled digit layout, the XCD-aware
// tile order and the explicit wait / barrier primitives of the pipelined
// kernels.
#pragma once

#include <limits.h>

#include "bq_tile_order.h"

namespace bq {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef double d4s __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef int i4v __attribute__((ext_vector_type(4)));

// Row / column exponent markers: INT_MIN for an all-zero row or column (its
// digits are zero and so is its part of the product), kExpNonFinite for one
// holding a NaN or an infinity (it wins every max; its digits are zero and
// its part of the product is NaN, as in the FP64 path).
constexpr int kExpNonFinite = INT_MAX;

__device__ __forceinline__ bool exp_special(int e) { return e == INT_MIN || e == kExpNonFinite; }

// Scale of a product element with row exponent ea and column exponent eb.
__device__ __forceinline__ double exp_scaled(double v, int ea, int eb, int shift) {
  if (ea == kExpNonFinite || eb == kExpNonFinite) return __builtin_nan("");
  if (ea == INT_MIN || eb == INT_MIN) return 0.0;
  return ldexp(v, ea + eb + shift);
}

// Chunk position of logical chunk ch in tile row r (rows of 4 chunks).
// 16-byte chunks (rows of 64 bytes): a 16-byte LDS access is served 8 lanes
// at a time over 32 banks (128 bytes); a fragment read has 8 lanes on 8
// consecutive rows at one logical chunk, and rows 2j, 2j + 1 share a
// 128-byte bank line offset by 64 bytes, so even rows must take 4 distinct
// positions, and odd rows too: position = ch ^ f(r) with f built from row
// bits 1..3.  8-byte chunks (rows of 32 bytes): 16 lanes per access on 16
// consecutive rows; rows r and r + 4 share banks, so f = bits 2..3.
template <int CH>
__device__ __forceinline__ int swz_chunk(int r, int ch) {
  if constexpr (CH == 16) return ch ^ ((((r >> 1) ^ (r >> 3)) & 1) | ((r >> 1) & 2));
  else return ch ^ ((r >> 2) & 3);
}

// Tiled digit layout (direct-to-LDS slice and residue GEMMs): within one
// slice, the 64 rows x one k-step (64 bytes per row) of row tile rt, k-step
// kt form one 4 KB block at (rt * nk + kt) * 4096, stored in the LDS order
// (row r at r * 64, logical 16-byte chunk ch at the swizzled position), so
// that a straight copy lands the tile ready for fragment reads.  Byte
// offset of the digit at (row r, byte b of the row) in one slice whose rows
// hold row_bytes.
__device__ __forceinline__ int64_t digit_offset(int64_t r, int64_t byte_in_row, int64_t row_bytes) {
  constexpr int RB = 64;
  const int64_t nk = row_bytes / RB, kt = byte_in_row / RB;
  const int rr = (int)(r & 63), b = (int)(byte_in_row % RB);
  return ((r >> 6) * nk + kt) * (64 * RB) + rr * RB + swz_chunk<16>(rr, b >> 4) * 16 + (b & 15);
}

// 16 consecutive inner elements from k0 of row or column v of a block (of a
// SplitOperand; K: the inner dimension, in: v exists), zeros past the end.
__device__ __forceinline__ void load_inner16(const SplitOperand& a, const double* p, int64_t v, int64_t k0, int64_t K,
                                             bool in, double (&x)[16]) {
  if (a.along) {
    const double* q = p + v * a.ld + k0;
    if (a.vec && in && k0 + 16 <= K) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const double2 d = *reinterpret_cast<const double2*>(q + 2 * j);
        x[2 * j] = d.x;
        x[2 * j + 1] = d.y;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 16; ++j) x[j] = in && k0 + j < K ? q[j] : 0.0;
    }
  } else {
    const double* q = p + k0 * a.ld + v;
    if (in && k0 + 16 <= K) {
#pragma unroll
      for (int j = 0; j < 16; ++j) x[j] = q[j * a.ld];
    } else {
#pragma unroll
      for (int j = 0; j < 16; ++j) x[j] = in && k0 + j < K ? q[j * a.ld] : 0.0;
    }
  }
}

// Low bytes of four words, packed.
__device__ __forceinline__ int pack_bytes(int a, int b, int c, int d) {
  const unsigned ab = __builtin_amdgcn_perm((unsigned)b, (unsigned)a, 0x0c0c0400u);
  const unsigned cd = __builtin_amdgcn_perm((unsigned)d, (unsigned)c, 0x04000c0cu);
  return (int)(ab | cd);
}

// Last item whose first block is at or before block b.
template <typename Prefix>
__device__ __forceinline__ int find_item(Prefix* prefix, int count, int64_t b) {
  int lo = 0, hi = count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (prefix[mid] <= b) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Block -> output tile of a one-output launch: each XCD gets a contiguous run
// of tiles.
__device__ __forceinline__ void slice_tile_coords(int tiles_m, int tiles_n, int& tm, int& tn) {
  grouped_tile((int)xcd_position(blockIdx.x, 0, (int64_t)tiles_m * tiles_n), tiles_m, tiles_n, tm, tn);
}

// coef * T into every target block of a slice GEMM, for this lane's NE
// elements (off < 0: outside C).  Targets outside, elements inside, and a
// target's old values all loaded before its first store: the blocks of C do
// not overlap, which the compiler cannot know, so element by element every
// load waited behind the store before it (8 INT8 slices, n = 2048: 391 us per
// real product on average, 302 this way, of which about 235 are the MFMAs; a
// real product of the Hadamard part adds into up to eight blocks).
template <int NE>
__device__ __forceinline__ void store_targets(const SliceGemmArgs& g, const double (&t)[NE], const int64_t (&off)[NE]) {
  // coef * T is rounded before it is added (it is exact but for denormals).
#pragma clang fp contract(off)
  for (int q = 0; q < g.ntgt; ++q) {
    double* c = g.c[q];
    const double w = g.coef[q];
    if (g.mode[q] == TGT_ACCUM) {
      double old[NE];
#pragma unroll
      for (int e = 0; e < NE; ++e) old[e] = off[e] >= 0 ? c[off[e]] : 0.0;
#pragma unroll
      for (int e = 0; e < NE; ++e)
        if (off[e] >= 0) c[off[e]] = w * t[e] + old[e];
    } else {
#pragma unroll
      for (int e = 0; e < NE; ++e)
        if (off[e] >= 0) c[off[e]] = w * t[e];
    }
  }
}

// LDS destination of the direct global -> LDS buffer loads.
typedef __attribute__((address_space(3))) void* lds_void_ptr;

// Workgroup barrier without the memory fence of __syncthreads (which would
// wait for every load in flight, prefetches included): the kernels order
// their LDS traffic themselves (wait_vm before, fragment reads consumed
// before the barrier).
__device__ __forceinline__ void block_sync() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
}

// s_waitcnt vmcnt(N): wait until at most N vector-memory loads are pending.
#define BQ_WAIT_VM_CASE(K) \
  else if constexpr (N == K) asm volatile("s_waitcnt vmcnt(" #K ")" ::: "memory");
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N <= 31, "vmcnt range used here");
  if constexpr (N == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  BQ_WAIT_VM_CASE(1) BQ_WAIT_VM_CASE(2) BQ_WAIT_VM_CASE(3) BQ_WAIT_VM_CASE(4) BQ_WAIT_VM_CASE(5)
  BQ_WAIT_VM_CASE(6) BQ_WAIT_VM_CASE(7) BQ_WAIT_VM_CASE(8) BQ_WAIT_VM_CASE(9) BQ_WAIT_VM_CASE(10)
  BQ_WAIT_VM_CASE(11) BQ_WAIT_VM_CASE(12) BQ_WAIT_VM_CASE(13) BQ_WAIT_VM_CASE(14) BQ_WAIT_VM_CASE(15)
  BQ_WAIT_VM_CASE(16) BQ_WAIT_VM_CASE(17) BQ_WAIT_VM_CASE(18) BQ_WAIT_VM_CASE(19) BQ_WAIT_VM_CASE(20)
  BQ_WAIT_VM_CASE(21) BQ_WAIT_VM_CASE(22) BQ_WAIT_VM_CASE(23) BQ_WAIT_VM_CASE(24) BQ_WAIT_VM_CASE(25)
  BQ_WAIT_VM_CASE(26) BQ_WAIT_VM_CASE(27) BQ_WAIT_VM_CASE(28) BQ_WAIT_VM_CASE(29) BQ_WAIT_VM_CASE(30)
  BQ_WAIT_VM_CASE(31)
}
#undef BQ_WAIT_VM_CASE

}  // namespace bq
