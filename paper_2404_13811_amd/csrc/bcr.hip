// Interface system (Algorithm 1, Step 5) by block cyclic reduction.
//
// With the rows of every coarse interface split between its two subdomains
// (flux rows to the lower-indexed one, pressure rows to the higher one),
// each subdomain owns as many equations as it has seed unknowns, and the
// system is block tridiagonal over the layers of subdomains along the last
// axis:  L_k x_{k-1} + D_k x_k + U_k x_{k+1} = r_k.  Odd-even reduction
// eliminates every other layer per level; all blocks of one level are
// independent, so a level is one batched dense inverse, one batch of block
// products for the eliminated layers and one for the kept layers.  No
// pivoting is used, neither across nor inside blocks (Gauss-Jordan
// inverses of the diagonal blocks).
//
// Storage: every block is dense row-major bp x bp (bp = largest layer size,
// padded layers carry the identity in D and zeros elsewhere), in one pool
// of 5M blocks (initially [D | L | U], then the reduced blocks and the
// factors F, G kept for the back substitution in slots the host schedule
// assigns) and a pool of 3M vectors [r | g | x].
#include "mrcm_internal.h"
#include "gj16.h"

#include <type_traits>

namespace mrcm {
namespace {

// ------------------------------------------------------------------ inverse
// In-place Gauss-Jordan inversion of one n x n block (n = 16 NW <= 128) per
// workgroup of NW waves, 16 pivots per step, no pivoting.  Wave v holds rows
// 16 v .. 16 v + 15 as NW 16 x 16 tiles in the accumulator layout of the FP64
// matrix instructions.  Step p, with P the pivot block, R the pivot rows and C a wave's pivot columns:
//   P <- P^{-1},  R <- P^{-1} R,  C <- -C P^{-1},  A <- A - C P^{-1} R.
// The old pivot rows are in LDS in operand B's layout (the accumulators as
// they are), P^{-1} in LDS too, so a wave needs only its own pivot-column
// tile transposed (through LDS, within the wave): -(C P^{-1})^T, formed as
// a product, comes out in operand A's layout.  Look-ahead: the wave that
// holds the next pivot rows updates the next pivot block first, inverts it
// in registers while the other waves update, and publishes it and its rows;
// one barrier per 16 pivots.  The tiles rotate by one slot per step (slot i
// holds column block p + i), so the step is one loop body: a body unrolled
// per step would not stay in the instruction cache.
//
// Bound: FP64 matrix instructions of one CU (2 n^3 flop: 14 us for n = 128
// at 128 flop per cycle; 32 of 64 cycles per wave and step, two waves per
// SIMD) plus, on the SIMD of the wave that looks ahead, the pivot block's
// inversion, which uses the same FP64 units (16 pivots of about 120 cycles),
// and the LDS round trips before and after it: 9,000 cycles per step
// measured, of which the other SIMDs work 4,100.  Measured per launch, against four
// pivots per step on the vector unit with two to one barriers: n = 128
// 50.5 -> 30.9 us, n = 96 with 66 pivots 30.7 -> 16.5 us, n = 32 7.7 ->
// 4.2 us.  Matrix instructions interleaved with the inversion's pivots were
// no faster (34 us): a wave's vector instructions wait for them.
template <int NW>
__global__ void __launch_bounds__(64 * NW) k_bcr_inv(double* __restrict__ pool,
                                                     const long long* __restrict__ offs,
                                                     const int* __restrict__ npiv, int ld, int* flags) {
  __shared__ __align__(16) double rb[2][NW * 256];      // pivot rows, operand B's layout
  __shared__ __align__(16) double pq[2][kTile];      // inverse of the pivot block
  __shared__ __align__(16) double tw[NW][kTile];     // per wave: transposition
  double* A = pool + offs[blockIdx.x];
  const int l = threadIdx.x & 63, lc = l & 15, lg = l >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // pivots beyond the block's own size act on identity padding, which they
  // leave unchanged: skipped
  const int np = min((npiv[blockIdx.x] + 15) / 16, NW);
  dbl4 T[NW];
#pragma unroll
  for (int i = 0; i < NW; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) T[i][r] = A[(long long)(16 * wv + 4 * r + lg) * ld + 16 * i + lc];
  bool bad = false;
  double* mine = tw[wv];
  // inverse of the pivot block in tile t, published for step st
  auto invert = [&](const dbl4& t, int st) {
    double a[16];
    tile_put(mine, t);
    wave_lds_sync();
    tile_get_rows(mine, a);
    inv16<false>(a, bad);
    tile_put_rows(pq[st & 1], a);
  };
  auto publish = [&](int st) {
#pragma unroll
    for (int i = 1; i < NW; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) rb[st & 1][(4 * i + r) * 64 + l] = T[i][r];
  };
  if (np > 0 && wv == 0) {
    invert(T[0], 0);
    publish(0);
  }
  __syncthreads();
#pragma unroll 1
  for (int p = 0; p < np; ++p) {
    const double* R = rb[p & 1];
    const double* P = pq[p & 1];
    const dbl4 zero = {0.0, 0.0, 0.0, 0.0};
    if (wv == p) {
      const dbl4 pa = tile_get_t(P);
#pragma unroll
      for (int i = 1; i < NW; ++i) T[i - 1] = mfma16(pa, T[i], zero);
      T[NW - 1] = tile_get(P);
    } else {
      const bool ahead = wv == p + 1 && p + 1 < np;
      if (ahead) __builtin_amdgcn_s_setprio(2);
      const dbl4 pn = -tile_get(P);
      tile_put(mine, T[0]);
      wave_lds_sync();
      const dbl4 mt = mfma16(pn, tile_get_t(mine), zero);  // -(C P^{-1})^T: operand A
      auto update = [&](int i) {
        dbl4 r;
#pragma unroll
        for (int c = 0; c < 4; ++c) r[c] = R[(4 * i + c) * 64 + l];
        T[i - 1] = mfma16(mt, r, T[i]);
      };
      update(1);
      if (ahead) {
        invert(T[0], p + 1);
        wave_lds_sync();
      }
      tile_put(mine, mt);
#pragma unroll
      for (int i = 2; i < NW; ++i) update(i);
      wave_lds_sync();
      T[NW - 1] = tile_get_t(mine);  // -C P^{-1}
      if (ahead) {
        publish(p + 1);
        __builtin_amdgcn_s_setprio(0);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const int cb = np + i < NW ? np + i : np + i - NW;  // np <= NW, i < NW
#pragma unroll
    for (int r = 0; r < 4; ++r) A[(long long)(16 * wv + 4 * r + lg) * ld + 16 * cb + lc] = T[i][r];
  }
  if (bad) atomicOr(flags, kFlagSingular);
}

// ------------------------------------------------------------------ products
// C = [C0] + al1 A1 B1 + al2 A2 B2 for a batch of tasks; the operands are
// n x n matrices at element offsets in the pool with leading dimension ld
// (whole blocks, or quarters of a block in the two-by-two inverse).  One
// workgroup of 256 threads (four waves) per 32 x 32 output tile.
constexpr int GT = 32;

// One 32 x 32 output tile of a product task (tile = row-major tile index).
// Each of the four waves computes one 16 x 16 quadrant with FP64 matrix
// instructions (16 x 16 x 4 per instruction: lane l supplies A[l % 16][l / 16]
// and B[l / 16][l % 16] of the k-slice and holds D[4r + l / 16][l % 16] in
// accumulator element r); two accumulators alternate over the k-slices so
// that consecutive instructions do not wait on each other.
//
// The k dimension of every product term is cut into chunks of KC: the A
// rows of the tile (32 x KC, row-major with stride KC + 1 so that the
// strip's rows start in different banks) and the B columns (KC x 32) of a
// chunk are staged in LDS, and the global loads of the next chunk (of this
// term or the next) are in flight while the matrix instructions run on the
// current one.  A small KC keeps the LDS of a workgroup small enough for
// several workgroups per CU.
template <int KC>
__host__ __device__ constexpr size_t gemm_lds_doubles() {
  return (size_t)GT * (KC + 1) + (size_t)KC * GT;
}

template <int KC>
__device__ __forceinline__ void gemm_tile(double* pool, const BcrGemm& T, int n, int ld, int tile,
                                          double* smem) {
  constexpr int NA = GT * KC / 256;  // A (and B) elements per thread per chunk
  constexpr int AS = KC + 1;
  double* As = smem;            // GT x (KC + 1)
  double* Bs = smem + GT * AS;  // KC x GT
  const int ntile = n / GT;
  const int tr0 = (tile / ntile) * GT, tc0 = (tile % ntile) * GT;
  const int tid = threadIdx.x;
  const int wv = tid >> 6, ln = tid & 63;
  const int qr = (wv >> 1) * 16, qc = (wv & 1) * 16;  // quadrant of this wave
  const int li = ln & 15, lk = ln >> 4;
  const int t0 = T.a1 >= 0 ? 0 : 1;  // first product term present
  const int nterm = (T.a1 >= 0 ? 1 : 0) + (T.a2 >= 0 ? 1 : 0);
  const int nch = n / KC, total = nterm * nch;
  double va[NA], vb[NA];
  auto load = [&](int c) {
    const int term = c < nch ? t0 : 1;
    const int k0 = (c % nch) * KC;
    const double* A = pool + (term ? T.a2 : T.a1);
    const double* B = pool + (term ? T.b2 : T.b1);
#pragma unroll
    for (int u = 0; u < NA; ++u) {
      const int e = u * 256 + tid;
      const int ra = e / KC, ka = e % KC;  // A row-major: consecutive k
      const int kb = e >> 5, cb = e & 31;  // B: 32 consecutive columns
      va[u] = A[(long long)(tr0 + ra) * ld + k0 + ka];
      vb[u] = B[(long long)(k0 + kb) * ld + tc0 + cb];
    }
  };
  dbl4 acc0 = {0.0, 0.0, 0.0, 0.0}, acc1 = {0.0, 0.0, 0.0, 0.0};
  if (total > 0) load(0);
  for (int c = 0; c < total; ++c) {
    const double al = (c < nch ? t0 : 1) ? T.al2 : T.al1;
    if (c) __syncthreads();  // the previous chunk's operands are read
#pragma unroll
    for (int u = 0; u < NA; ++u) {
      const int e = u * 256 + tid;
      As[(e / KC) * AS + e % KC] = al * va[u];
      Bs[e] = vb[u];
    }
    __syncthreads();
    if (c + 1 < total) load(c + 1);
    const double* ap = As + (qr + li) * AS + lk;
    const double* bq = Bs + lk * GT + qc + li;
#pragma unroll
    for (int k = 0; k < KC; k += 8) {
      acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(ap[k], bq[k * GT], acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(ap[k + 4], bq[(k + 4) * GT], acc1, 0, 0, 0);
    }
  }
  double* C = pool + T.c;
  const double* C0 = T.c0 >= 0 ? pool + T.c0 : nullptr;
  const int col = tc0 + qc + li;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const long long row = tr0 + qr + 4 * r + lk;
    double v = acc0[r] + acc1[r];
    if (C0) v += C0[row * ld + col];
    C[row * ld + col] = v;
  }
}

template <int KC>
__global__ void __launch_bounds__(256) k_bcr_gemm(double* __restrict__ pool,
                                                  const BcrGemm* __restrict__ tasks, int n, int ld) {
  extern __shared__ double smem[];
  const int ntile = n / GT;
  const int task = blockIdx.x / (ntile * ntile);
  gemm_tile<KC>(pool, tasks[task], n, ld, blockIdx.x - task * ntile * ntile, smem);
}

// y = [y0] + al1 A1 x1 + al2 A2 x2.  Workgroup (task, group of 16 rows);
// 16 lanes per row, each with bp/16 independent loads, then a 16-lane sum.
__device__ __forceinline__ void gemv_rows(const double* pool, double* __restrict__ vec, const BcrGemv& T,
                                          int bp, int rg) {
  const long long bs = (long long)bp * bp;
  const int r = rg * 16 + (threadIdx.x >> 4), l = threadIdx.x & 15;
  double acc = 0.0;
#pragma unroll
  for (int term = 0; term < 2; ++term) {
    const int ai = term ? T.a2 : T.a1;
    if (ai < 0) continue;
    const double* A = pool + ai * bs + (long long)r * bp;
    const double* x = vec + (long long)(term ? T.x2 : T.x1) * bp;
    double s = 0.0;
#pragma unroll 4
    for (int c = l; c < bp; c += 16) s = fma(A[c], x[c], s);
    acc = fma(term ? T.al2 : T.al1, s, acc);
  }
  acc += __shfl_xor(acc, 8);
  acc += __shfl_xor(acc, 4);
  acc += __shfl_xor(acc, 2);
  acc += __shfl_xor(acc, 1);
  if (l == 0) {
    double* y = vec + (long long)T.y * bp;
    y[r] = (T.y0 >= 0 ? vec[(long long)T.y0 * bp + r] : 0.0) + acc;
  }
}

__global__ void __launch_bounds__(256) k_bcr_gemv(const double* __restrict__ pool,
                                                  double* __restrict__ vec,
                                                  const BcrGemv* __restrict__ tasks, int bp) {
  gemv_rows(pool, vec, tasks[blockIdx.x], bp, blockIdx.y);
}

// Block products and block-vector products that do not depend on each
// other, in one launch: workgroups [0, ngblk) are product tiles, the rest
// row groups of the vector tasks.  The caller guarantees that no vector
// task reads a block a product task of the same launch writes.
template <int KC>
__global__ void __launch_bounds__(256) k_bcr_gemm_gemv(double* pool, double* __restrict__ vec,
                                                       const BcrGemm* __restrict__ gtasks, int ngblk,
                                                       const BcrGemv* __restrict__ vtasks, int n,
                                                       int ld, int bp) {
  extern __shared__ double smem[];
  const int b = blockIdx.x;
  if (b < ngblk) {
    const int ntile = n / GT;
    const int task = b / (ntile * ntile);
    gemm_tile<KC>(pool, gtasks[task], n, ld, b - task * ntile * ntile, smem);
  } else {
    const int rgs = bp / 16;
    const int i = b - ngblk;
    gemv_rows(pool, vec, vtasks[i / rgs], bp, i - (i / rgs) * rgs);
  }
}

// Initial state of the reduction in one pass: the 3M blocks [D | L | U] of
// the pool zero except the identity on the padded diagonal of every D
// block (rows and columns past the layer's size), and the M right-hand-side
// vectors zero.  The interface moments are then written straight into
// these blocks, none of them in the padding.
__global__ void k_bcr_init(double* __restrict__ pool, double* __restrict__ vec,
                           const int* __restrict__ lsize, int M, int bp) {
  const long long bs = (long long)bp * bp;
  const long long npool = 3LL * M * bs, nvec = (long long)M * bp;
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < npool) {
    const long long k = e / bs, w = e - k * bs;
    const int r = (int)(w / bp), cc = (int)(w - (long long)r * bp);
    pool[e] = (k < M && r == cc && r >= lsize[k]) ? 1.0 : 0.0;
  } else if (e < npool + nvec) {
    vec[e - npool] = 0.0;
  }
}

// x (layer-major, padded) -> X (unknown order).
__global__ void k_bcr_gather(const double* __restrict__ xv, const int* __restrict__ col_lvl,
                             const int* __restrict__ col_loc, int n, int bp, double* __restrict__ X) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c < n) X[c] = xv[(long long)col_lvl[c] * bp + col_loc[c]];
}

}  // namespace

hipError_t launch_bcr_inv(double* pool, const long long* offs, const int* npiv, int nblk, int n,
                          int ld, int* flags,
                          hipStream_t s) {
  if (nblk <= 0) return hipSuccess;
  switch (n) {
#define MRCM_INV(NW)                                                                             \
  case 16 * NW:                                                                                  \
    hipLaunchKernelGGL(k_bcr_inv<NW>, dim3(nblk), dim3(64 * NW), 0, s, pool, offs, npiv, ld, flags); \
    break;
    MRCM_INV(2) MRCM_INV(4) MRCM_INV(6) MRCM_INV(8)
#undef MRCM_INV
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Chunk of the k dimension for products of n x n blocks: whole 128-wide
// operands when n = 128 (the latency-bound case: one round of loads per
// term), 64 for larger blocks (several workgroups per CU), else 32.
template <typename F>
hipError_t with_chunk(int n, F f) {
  if (n == 128) return f(std::integral_constant<int, 128>());
  if (n % 64 == 0) return f(std::integral_constant<int, 64>());
  return f(std::integral_constant<int, 32>());
}

template <typename KF>
hipError_t gemm_lds_attr(KF kern, size_t lds) {
  if (lds > 64 * 1024)
    return hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  return hipSuccess;
}

hipError_t launch_bcr_gemm(double* pool, const BcrGemm* tasks, int ntask, int n, int ld, hipStream_t s) {
  if (ntask <= 0) return hipSuccess;
  if (n % GT || n > kBcrMaxBlock) return hipErrorInvalidValue;
  const int ntile = n / GT;
  return with_chunk(n, [&](auto kc) -> hipError_t {
    constexpr int KC = decltype(kc)::value;
    const size_t lds = sizeof(double) * gemm_lds_doubles<KC>();
    hipError_t e = gemm_lds_attr(k_bcr_gemm<KC>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bcr_gemm<KC>, dim3(ntask * ntile * ntile), dim3(256), lds, s, pool, tasks, n, ld);
    return hipGetLastError();
  });
}

hipError_t launch_bcr_gemm_gemv(double* pool, double* vec, const BcrGemm* gtasks, int ngemm,
                               const BcrGemv* vtasks, int ngemv, int n, int ld, int bp,
                               hipStream_t s) {
  if (ngemm <= 0 && ngemv <= 0) return hipSuccess;
  if (n % GT || n > kBcrMaxBlock || bp % 16) return hipErrorInvalidValue;
  const int ntile = n / GT;
  const int ngblk = ngemm * ntile * ntile;
  return with_chunk(n, [&](auto kc) -> hipError_t {
    constexpr int KC = decltype(kc)::value;
    const size_t lds = sizeof(double) * gemm_lds_doubles<KC>();
    hipError_t e = gemm_lds_attr(k_bcr_gemm_gemv<KC>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bcr_gemm_gemv<KC>, dim3(ngblk + ngemv * (bp / 16)), dim3(256), lds, s, pool,
                       vec, gtasks, ngblk, vtasks, n, ld, bp);
    return hipGetLastError();
  });
}

hipError_t launch_bcr_gemv(const double* pool, double* vec, const BcrGemv* tasks, int ntask, int bp,
                           hipStream_t s) {
  if (ntask <= 0) return hipSuccess;
  if (bp % 16) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_bcr_gemv, dim3(ntask, bp / 16), dim3(256), 0, s, pool, vec, tasks, bp);
  return hipGetLastError();
}

hipError_t launch_bcr_init(double* pool, double* vec, const int* lsize, int M, int bp, hipStream_t s) {
  const long long tot = 3LL * M * bp * bp + (long long)M * bp;
  hipLaunchKernelGGL(k_bcr_init, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, pool, vec, lsize,
                     M, bp);
  return hipGetLastError();
}

hipError_t launch_bcr_gather(const double* xv, const int* col_lvl, const int* col_loc, int n, int bp,
                             double* X, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_bcr_gather, dim3((n + 255) / 256), dim3(256), 0, s, xv, col_lvl, col_loc, n, bp, X);
  return hipGetLastError();
}

}  // namespace mrcm
