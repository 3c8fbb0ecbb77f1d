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
typedef float flt4 __attribute__((ext_vector_type(4)));

// v of lane K of the lane's 16-lane row.  The wait states cover a write of v
// by the instruction before (a DPP operand must not be read within two
// instructions of its write).
template <int K>
__device__ __forceinline__ double row_bcast(double v) {
  double d;
  asm("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf" : "=v"(d) : "v"(v), "n"(K));
  return d;
}

template <int K>
__device__ __forceinline__ float row_bcast(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x150 + K, 0xF, 0xF, false));
}

// a[j] += a[j](lane K) n for the columns j = K + J .. K + J + 4 (mod 16).
// The first pivot's columns may have been written by the instruction before
// (two wait states); later, five per asm block, always in this order, keep
// the same distance between the write of a DPP operand and its read: a
// column is read again at the earliest five instructions after its write
// (tests/test_dpp_hazards.py checks the built code for it).
template <int K, int J>
__device__ __forceinline__ void pivot_update5(double a[16], double n) {
#define MRCM_C(i) a[(K + J + i) & 15]
#define MRCM_U                                                                                       \
  MRCM_F(0) MRCM_F(1) MRCM_F(2) MRCM_F(3) MRCM_F(4)                                                  \
      : "+v"(MRCM_C(0)), "+v"(MRCM_C(1)), "+v"(MRCM_C(2)), "+v"(MRCM_C(3)), "+v"(MRCM_C(4))          \
      : "v"(n), "n"(K)
#define MRCM_F(i) "v_fmac_f64_dpp %" #i ", %" #i ", %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
  if constexpr (K == 0) asm("s_nop 1\n\t" MRCM_U);
  else asm(MRCM_U);
}
#undef MRCM_F
#define MRCM_F(i) "v_fmac_f32_dpp %" #i ", %" #i ", %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
template <int K, int J>
__device__ __forceinline__ void pivot_update5(float a[16], float n) {
  if constexpr (K == 0) asm("s_nop 1\n\t" MRCM_U);
  else asm(MRCM_U);
}
#undef MRCM_F
#undef MRCM_U
#undef MRCM_C

__device__ __forceinline__ double pivot_inv(double x) { return pivot_rcp(x); }
__device__ __forceinline__ float pivot_inv(float x) {
  // hardware estimate (1 ulp) refined by a Newton step
  const float r = __builtin_amdgcn_rcpf(x);
  return fmaf(r, fmaf(-x, r, 1.0f), r);
}

__device__ __forceinline__ double one_or(bool own, double n) {
  // the low word of n is that of 1 (zero) in the own row
  return __hiloint2double(own ? 0x3FF00000 : __double2hiint(n), __double2loint(n));
}
__device__ __forceinline__ float one_or(bool own, float n) { return own ? 1.0f : n; }

// np: the block is np x np with identity padding (which eight pivots of
// padding leave as it is)
template <int K, typename T>
__device__ __forceinline__ void inv16_pivots(T a[16], int np, int r16, T& sc) {
  if constexpr (K < 16) {
    if (K == 8 && np <= 8) return;
    const T id = pivot_inv(row_bcast<K>(a[K]));
    const bool own = r16 == K;
    sc = own ? id : sc;
    const T n = own ? T(0) : -a[K] * id;  // negated multiplier
    pivot_update5<K, 1>(a, n);
    pivot_update5<K, 6>(a, n);
    pivot_update5<K, 11>(a, n);
    a[K] = one_or(own, n);
    inv16_pivots<K + 1>(a, np, r16, sc);
  }
}

// a (row threadIdx.x % 16 of the block) <- that row of its inverse.  bad: a
// pivot that cannot be divided by (SPD: not positive; otherwise zero,
// infinite or NaN), read from the reciprocals the lanes keep.
template <bool SPD, typename T>
__device__ __forceinline__ void inv16(T a[16], bool& bad, int np = 16) {
  T sc = T(1);
  inv16_pivots<0>(a, np, threadIdx.x & 15, sc);
  bad |= SPD ? !(sc > T(0)) : !piv_usable(sc);
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
    const double a0 = a[j], a1 = a[4 + j], a2 = a[8 + j], a3 = a[12 + j];
    const double lo = g & 1 ? a1 : a0, hi = g & 1 ? a3 : a2;
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

// FP32 tiles: rows of 16 at a stride of 20 entries, register r of lane l of
// v_mfma_f32_16x16x4 holds row 4 (l / 16) + r, column l % 16; the rows 4 c +
// l / 16 of an FP64 operand are 4 (l / 16) + c here (any order of the
// contraction will do, as long as both operands keep it).
constexpr int kTileF = 320;

__device__ __forceinline__ void tile_put(float* t, const flt4& v) {
  const int l = threadIdx.x & 63;
#pragma unroll
  for (int r = 0; r < 4; ++r) t[20 * (4 * (l >> 4) + r) + (l & 15)] = v[r];
}
__device__ __forceinline__ flt4 tile_get(const float* t) {
  const int l = threadIdx.x & 63;
  flt4 v;
#pragma unroll
  for (int r = 0; r < 4; ++r) v[r] = t[20 * (4 * (l >> 4) + r) + (l & 15)];
  return v;
}
__device__ __forceinline__ flt4 tile_get_t(const float* t) {
  const int l = threadIdx.x & 63;
  return *reinterpret_cast<const flt4*>(t + 20 * (l & 15) + 4 * (l >> 4));
}
__device__ __forceinline__ void tile_get_rows(const float* t, float a[16]) {
  const float* r = t + 20 * (threadIdx.x & 15);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const flt4 u = *reinterpret_cast<const flt4*>(r + 4 * j);
#pragma unroll
    for (int e = 0; e < 4; ++e) a[4 * j + e] = u[e];
  }
}
__device__ __forceinline__ void tile_put_rows(float* t, const float a[16]) {
  const int l = threadIdx.x & 63, g = l >> 4;
  flt4 v;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    // (values: a select between entries of the array is one of addresses,
    // and the array then lives in scratch memory)
    const float a0 = a[j], a1 = a[4 + j], a2 = a[8 + j], a3 = a[12 + j];
    const float lo = g & 1 ? a1 : a0, hi = g & 1 ? a3 : a2;
    v[j] = g & 2 ? hi : lo;
  }
  *reinterpret_cast<flt4*>(t + 20 * (l & 15) + 4 * g) = v;
}
// the lane's whole row, and its whole column
__device__ __forceinline__ void tile_put_row(double* t, const double a[16]) {
  const int row = threadIdx.x & 15;
#pragma unroll
  for (int j = 0; j < 8; ++j)
    *reinterpret_cast<double2*>(t + tile_at(row, 2 * j)) = make_double2(a[2 * j], a[2 * j + 1]);
}
__device__ __forceinline__ void tile_put_row(float* t, const float a[16]) {
  float* r = t + 20 * (threadIdx.x & 15);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    flt4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = a[4 * j + e];
    *reinterpret_cast<flt4*>(r + 4 * j) = v;
  }
}
__device__ __forceinline__ void tile_get_column(const double* t, double a[16]) {
#pragma unroll
  for (int j = 0; j < 16; ++j) a[j] = t[tile_at(j, threadIdx.x & 15)];
}
__device__ __forceinline__ void tile_get_column(const float* t, float a[16]) {
#pragma unroll
  for (int j = 0; j < 16; ++j) a[j] = t[20 * j + (threadIdx.x & 15)];
}

// acc += A B for 16 x 16 operands in four k-slices (nk: entries of the
// contraction that are not zero)
__device__ __forceinline__ flt4 mfma16(const flt4& a, const flt4& b, flt4 acc, int = 16) {
#pragma unroll
  for (int c = 0; c < 4; ++c) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[c], b[c], acc, 0, 0, 0);
  return acc;
}
__device__ __forceinline__ dbl4 mfma16(const dbl4& a, const dbl4& b, dbl4 acc, int nk = 16) {
#pragma unroll
  for (int c = 0; c < 4; ++c)
    if (c < 2 || nk > 8) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[c], b[c], acc, 0, 0, 0);
  return acc;
}

}  // namespace mrcm
