// In-register inverse of a 16 x 16 FP64 pivot block by one wavefront, the
// step of the blocked Gauss-Jordan eliminations that update with FP64
// matrix instructions 16 pivots at a time.
//
// Lane l holds row l % 16 (16 registers), the four 16-lane rows of the wave
// hold the same block, so a pivot row reaches every lane by a row broadcast
// (DPP row_newbcast) that v_fmac_f64 applies to its own operand: one
// instruction per entry and pivot, no LDS and no cross-row exchange.  A
// pivot's own row is left as it is (multiplier zero) and divided by its
// pivot once at the end.  (Pairs of pivots with their 2 x 2 inverse applied
// at the end lose two digits when a pair is nearly singular: interface
// systems at alpha = 1e4, backward error 5e-8 against 1e-9.)
//
// Bound: the 15 multiply-adds of a pivot at 4 cycles each and its
// reciprocal, about 120 cycles per pivot.
#pragma once
#include <hip/hip_runtime.h>

#include "pivot4.h"

namespace mrcm {

typedef double dbl4 __attribute__((ext_vector_type(4)));

// v of lane K of the lane's 16-lane row.  The wait states cover a write of v
// by the instruction before (a DPP operand must not be read within two
// instructions of its write).
template <int K>
__device__ __forceinline__ double row_bcast(double v) {
  double d;
  asm("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "=v"(d) : "v"(v), "n"(K));
  return d;
}

// a[j] += a[j](lane K) n for the columns j = K + J .. K + J + 4 (mod 16).
// Five per asm block, always in this order, keep the same distance between
// the write of a DPP operand and its read: a column is read again at the
// earliest five instructions after its write.
template <int K, int J>
__device__ __forceinline__ void pivot_update5(double a[16], double n) {
#define MRCM_C(i) a[(K + J + i) & 15]
#define MRCM_F(i) "v_fmac_f64_dpp %" #i ", %" #i ", %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
  asm(MRCM_F(0) MRCM_F(1) MRCM_F(2) MRCM_F(3) MRCM_F(4)
      : "+v"(MRCM_C(0)), "+v"(MRCM_C(1)), "+v"(MRCM_C(2)), "+v"(MRCM_C(3)), "+v"(MRCM_C(4))
      : "v"(n), "n"(K));
#undef MRCM_F
#undef MRCM_C
}

template <int K>
__device__ __forceinline__ void inv16_pivots(double a[16], int r16, double& sc) {
  if constexpr (K < 16) {
    const double id = pivot_rcp(row_bcast<K>(a[K]));
    const bool own = r16 == K;
    sc = own ? id : sc;
    const double n = own ? 0.0 : -a[K] * id;  // negated multiplier
    pivot_update5<K, 1>(a, n);
    pivot_update5<K, 6>(a, n);
    pivot_update5<K, 11>(a, n);
    // own ? 1 : n, where the low word of n is that of 1 (zero) in the own row
    a[K] = __hiloint2double(own ? 0x3FF00000 : __double2hiint(n), __double2loint(n));
    inv16_pivots<K + 1>(a, r16, sc);
  }
}

// a (row threadIdx.x % 16 of the block) <- that row of its inverse.  bad: a
// pivot that cannot be divided by (SPD: not positive; otherwise zero,
// infinite or NaN), read from the reciprocals the lanes keep.
template <bool SPD>
__device__ __forceinline__ void inv16(double a[16], bool& bad) {
  double sc = 1.0;
  inv16_pivots<0>(a, threadIdx.x & 15, sc);
  bad |= SPD ? !(sc > 0.0) : !piv_usable(sc);
#pragma unroll
  for (int j = 0; j < 16; ++j) a[j] *= sc;
}

// A 16 x 16 tile in LDS (256 doubles, 16-byte aligned): element (row, col)
// at 16 row + (col ^ (row & 14)), free of bank conflicts in the accumulator
// layout of v_mfma_f64_16x16x4 (register r of lane l: row 4 r + l / 16,
// column l % 16), transposed (operand A: row l % 16, column 4 c + l / 16) and
// by rows in 16-byte pieces.
constexpr int kTile = 256;

__device__ __forceinline__ int tile_at(int row, int col) { return 16 * row + (col ^ (row & 14)); }

__device__ __forceinline__ void tile_put(double* t, const dbl4& v) {
  const int l = threadIdx.x & 63;
#pragma unroll
  for (int r = 0; r < 4; ++r) t[tile_at(4 * r + (l >> 4), l & 15)] = v[r];
}
__device__ __forceinline__ dbl4 tile_get(const double* t) {
  const int l = threadIdx.x & 63;
  dbl4 v;
#pragma unroll
  for (int r = 0; r < 4; ++r) v[r] = t[tile_at(4 * r + (l >> 4), l & 15)];
  return v;
}
__device__ __forceinline__ dbl4 tile_get_t(const double* t) {
  const int l = threadIdx.x & 63;
  dbl4 v;
#pragma unroll
  for (int c = 0; c < 4; ++c) v[c] = t[tile_at(l & 15, 4 * c + (l >> 4))];
  return v;
}
// rows as inv16 takes them
__device__ __forceinline__ void tile_get_rows(const double* t, double a[16]) {
  const int row = threadIdx.x & 15;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const double2 u = *reinterpret_cast<const double2*>(t + tile_at(row, 2 * j));
    a[2 * j] = u.x;
    a[2 * j + 1] = u.y;
  }
}
// rows as inv16 leaves them (the same in every 16-lane row): lane l writes
// columns 4 (l / 16) .. + 3 of row l % 16
__device__ __forceinline__ void tile_put_rows(double* t, const double a[16]) {
  const int l = threadIdx.x & 63, row = l & 15, g = l >> 4;
  double v[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const double lo = g & 1 ? a[4 + j] : a[j], hi = g & 1 ? a[12 + j] : a[8 + j];
    v[j] = g & 2 ? hi : lo;
  }
  *reinterpret_cast<double2*>(t + tile_at(row, 4 * g)) = make_double2(v[0], v[1]);
  *reinterpret_cast<double2*>(t + tile_at(row, 4 * g + 2)) = make_double2(v[2], v[3]);
}

// LDS written by some lanes of a wave, read by others of the same wave
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// acc += A B for 16 x 16 operands in four k-slices
__device__ __forceinline__ dbl4 mfma16(const dbl4& a, const dbl4& b, dbl4 acc) {
#pragma unroll
  for (int c = 0; c < 4; ++c) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[c], b[c], acc, 0, 0, 0);
  return acc;
}

}  // namespace mrcm
