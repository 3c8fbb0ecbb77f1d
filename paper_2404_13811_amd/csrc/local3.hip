// Kernels for 3-D local problems whose plane blocks have at most 64 cells
// (boxes of up to 8 x 8 cells per plane): Steps 1-2 (factor of the
// oversampled box with the seed solves fused into its forward sweep, traces
// on Gamma_i, basis functions on Omega_i), Step 4 (particular problems),
// Step 6 (factor only) and one colour phase of the smoothing sweep
// (Steps 6-7).
//
// A box is ordered x fastest; a block is one plane of cells (same z), so
// the matrix is block tridiagonal with dense plane blocks D_j (the x and y
// couplings of the plane) and diagonal couplings between planes.  The
// factor is the sequence of block inverses W_j = S_j^{-1} of the block
// LDL^T recurrence S_j = D_j - t_{j-1} W_{j-1} t_{j-1} (t: plane couplings).
// One workgroup of NW wavefronts works on one box; wave v holds rows 16v ..
// 16v + 15 of the plane block (padded with the identity to 16 NW) as NW
// 16 x 16 tiles in the accumulator layout of the FP64 matrix instructions,
// so a box of 64-cell planes spreads its block over four waves (four SIMDs)
// and smaller planes take one wave per 16 cells.  W_j is computed in place by
// the symmetric sweep of 16 pivots at a time (sweep3); block-vector products
// of the seeds are matrix instructions on the same tiles, of the particular
// problem's one vector dot products.  Solves:
//   forward   z_j = W_j (b_j + t_{j-1} .* z_{j-1})
//   backward  x_j = z_j + W_j (t_j .* x_{j+1}).
// The inverses are stored whole (nb x nb, row-major), the layout the
// smoothing kernel reads back.
#include "gj16.h"
#include "local3_common.h"

namespace mrcm {
namespace {

// LDS of a workgroup beside its box: the three pivot-row tiles and (last)
// the pivot tile of an elimination step; also a tile per wave to transpose
// through, the x and y couplings of a plane while its block is built, and
// the per-wave partial sums of the smoothing sweep's products (NW waves x 64
// lanes).  8 KB: with the box arrays of 8 x 8 x 8 cells and six seeds,
// three boxes fit a CU.
struct __align__(16) Gj3 {
  double buf[4][kTile];
  int flag;
};

__device__ __forceinline__ double* partials3(Gj3& sm) { return &sm.buf[0][0]; }

// T <- S_j = D_j - t_{j-1} W_{j-1} t_{j-1}, T holding -W_{j-1} on entry
// (sweep3) when j > 0; identity outside the nb x nb block.
template <int NW>
__device__ __forceinline__ void build3(const Geo& g, const Box& B, const Box3& s, int j, Gj3& sm,
                                       dbl4 T[NW]) {
  const int nb = s.m0 * s.m1, m0 = s.m0;
  double* tx = sm.buf[0];
  double* ty = sm.buf[1];
  for (int e = threadIdx.x; e < 2 * nb; e += 64 * NW) {
    const int ax = e >= nb, c = e - ax * nb;
    (ax ? ty : tx)[c] = tplane(g, B, s, j, c, ax);
  }
  lsync<NW>();
  const int lc = lane3() & 15, lg = lane3() >> 4, r0 = 16 * wave3() + lg;
  const double* dj = s.Dg + j * nb;
  const double* tp = s.Tz + (j > 0 ? j - 1 : 0) * nb;
  double di[4], txi[4], tyi[4], ti[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = min(r0 + 4 * r, nb - 1);
    di[r] = dj[i];
    txi[r] = tx[i];
    tyi[r] = ty[i];
    ti[r] = j > 0 ? tp[i] : 0.0;
  }
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const int c = 16 * w + lc, cc = min(c, nb - 1);
    if (j > 0) {
      const double tc = tp[cc];
#pragma unroll
      for (int r = 0; r < 4; ++r) T[w][r] *= ti[r] * tc;
    }
    // tiles that hold no diagonal, x or y coupling are left alone (uniform)
    const int dist = 16 * abs(w - wave3());
    if (dist <= 16 || abs(dist - m0) < 16) {
      const double txc = tx[cc], tyc = ty[cc];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = r0 + 4 * r;
        // sums of selects: with one-cell-wide planes (m0 = 1) the x and y
        // neighbours of the block numbering coincide (the couplings across
        // the box sides are zero)
        double v = i == c ? di[r] : 0.0;
        v -= c == i + 1 ? txi[r] : 0.0;
        v -= c + 1 == i ? txc : 0.0;
        v -= c == i + m0 ? tyi[r] : 0.0;
        v -= c + m0 == i ? tyc : 0.0;
        T[w][r] += v;
      }
    }
    if (nb < 16 * NW) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = r0 + 4 * r;
        T[w][r] = i < nb && c < nb ? T[w][r] : i == c ? 1.0 : 0.0;
      }
    }
  }
  lsync<NW>();
}

// Pivot tile -> its inverse, in sm.buf[3], by the wave that holds it; n: the
// block's cells from the tile's first on (eight pivots do for up to eight).
__device__ __forceinline__ void pivot3(Gj3& sm, const dbl4& t, int n, bool& bad) {
  double a[16];
  tile_put(sm.buf[3], t);
  wave_lds_sync();
  tile_get_rows(sm.buf[3], a);
  inv16<true>(a, bad, n);
  wave_lds_sync();
  tile_put_rows(sm.buf[3], a);
}

// The other tiles of the pivot rows, as operand B reads them.
template <int NW, int P>
__device__ __forceinline__ void publish3(Gj3& sm, const dbl4 T[NW]) {
#pragma unroll
  for (int w = 0; w < NW; ++w)
    if (w != P) {
#pragma unroll
      for (int r = 0; r < 4; ++r) sm.buf[w < P ? w : w - 1][64 * r + lane3()] = T[w][r];
    }
}

// T <- -(block)^{-1} by the symmetric sweep operator, 16 pivots per step, no
// pivoting (the Schur complements are SPD).  Step P, with A_PP the pivot
// block and Q its inverse (inv16):
//   A_PP <- -Q,  A_Pw <- Q A_Pw,  A_vP <- A_vP Q,  A_vw <- A_vw - A_vP Q A_Pw,
// which keeps the whole matrix symmetric, so the pivot columns are the
// transposed pivot rows: a wave's operands are the pivot rows in LDS as
// their owner's accumulators hold them (operand B; read as operand A, the
// tile is its transpose), and Q A_Pv comes out of its product as operand A
// of the update.  No transposition, 20 matrix instructions per wave and
// step.  The pivot rows and Q have one buffer each: every wave takes its
// operands into registers, a barrier frees the buffers, and the wave that
// holds the next pivot rows updates its pivot tile first, inverts it and
// publishes while the others update.
//
// Bound (64 x 64 blocks, three boxes per CU): the FP64 units, by the matrix
// instructions (64 cycles each) and the vector work of the pivot inverses
// and of the block set-up, about three quarters of the kernel's time; the
// rest is the chain of four pivot inverses per plane.  Measured against four
// pivots per step on the vector unit (17,920 boxes of 8 x 8 x 8 cells):
// six seeds 5.92 -> 4.79 ms, 18 seeds (4,480 boxes) 2.00 -> 1.41 ms, the
// particular problems of 4 x 4 x 4 cells 0.37 -> 0.22 ms.
template <int NW, int P>
__device__ __forceinline__ void sweep3_step(int nb, Gj3& sm, dbl4 T[NW], bool& bad) {
  if constexpr (P < NW) {
    if (16 * P < nb) {
      const bool more = 16 * (P + 1) < nb;
      // pivots of the step: eight or fewer take half the instructions
      const int nk = P + 1 < NW ? 16 : nb - 16 * P;
      const dbl4 zero = {0.0, 0.0, 0.0, 0.0};
      const int wv = wave3();
      const dbl4 qa = tile_get_t(sm.buf[3]), qb = tile_get(sm.buf[3]);
      if (wv == P) {
        lsync<NW>();
#pragma unroll
        for (int w = 0; w < NW; ++w)
          if (w != P) T[w] = mfma16(qa, T[w], zero, nk);
        T[P] = -qb;
      } else {
        dbl4 rv, r[NW];
        const double* mv = sm.buf[wv < P ? wv : wv - 1];
#pragma unroll
        for (int c = 0; c < 4; ++c) rv[c] = mv[64 * c + lane3()];
#pragma unroll
        for (int w = 0; w < NW; ++w)
          if (w != P) {
#pragma unroll
            for (int c = 0; c < 4; ++c) r[w][c] = sm.buf[w < P ? w : w - 1][64 * c + lane3()];
          }
        lsync<NW>();
        const dbl4 u = -mfma16(qa, rv, zero, nk);
        if constexpr (P + 1 < NW) T[P + 1] = mfma16(u, r[P + 1], T[P + 1]);
        T[P] = mfma16(rv, qb, zero, nk);
        if constexpr (P + 1 < NW) {
          if (wv == P + 1 && more) pivot3(sm, T[P + 1], nb - 16 * (P + 1), bad);
        }
#pragma unroll
        for (int w = 0; w < NW; ++w)
          if (w != P && w != P + 1) T[w] = mfma16(u, r[w], T[w], nk);
        if constexpr (P + 1 < NW) {
          if (wv == P + 1 && more) publish3<NW, P + 1>(sm, T);
        }
      }
      lsync<NW>();
      sweep3_step<NW, P + 1>(nb, sm, T, bad);
    }
  }
}

template <int NW>
__device__ __forceinline__ void sweep3(int nb, Gj3& sm, dbl4 T[NW]) {
  bool bad = false;
  if (wave3() == 0) {
    pivot3(sm, T[0], nb, bad);
    publish3<NW, 0>(sm, T);
  }
  lsync<NW>();
  sweep3_step<NW, 0>(nb, sm, T, bad);
  if (bad) atomicOr(&sm.flag, kFlagNotPD);
}

// Rows 16v .. of W_j as operand A: the transposed tiles of -W_j in T.
template <int NW>
__device__ __forceinline__ void operand3(Gj3& sm, const dbl4 T[NW], dbl4 wa[NW]) {
  double* t = sm.buf[wave3()];
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    tile_put(t, T[w]);
    wave_lds_sync();
    wa[w] = -tile_get_t(t);
    wave_lds_sync();
  }
}

// The same from the stored inverse: column block v of the rows, by symmetry
// (four 128-byte pieces per load).
template <int NW>
__device__ __forceinline__ void load_operand3(const double* Wj, int nb, dbl4 wa[NW]) {
  const int lc = lane3() & 15, lg = lane3() >> 4, c = 16 * wave3() + lc;
#pragma unroll
  for (int w = 0; w < NW; ++w)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = 16 * w + 4 * k + lg;
      wa[w][k] = i < nb && c < nb ? Wj[i * nb + c] : 0.0;
    }
}

__device__ __forceinline__ void store_tiles3(double* Wj, int nb, int w, const dbl4& t) {
  const int lc = lane3() & 15, lg = lane3() >> 4, c = 16 * w + lc;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = 16 * wave3() + 4 * r + lg;
    if (i < nb && c < nb) Wj[i * nb + c] = -t[r];
  }
}

// v summed over the four 16-lane rows of the wave, in every lane.
__device__ __forceinline__ double rows_sum3(double v) {
  {
    const auto a = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
    v = __hiloint2double(b[0], a[0]) + __hiloint2double(b[1], a[1]);
  }
  const auto a = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
  return __hiloint2double(b[0], a[0]) + __hiloint2double(b[1], a[1]);
}

// X_j (+)= W_j Z for the nrhs vectors staged in s.Z (entry i of vector k at
// Z[nrhs i + k]), 16 right-hand sides per pass of matrix instructions.  ONE:
// a single vector, by dot products on the vector unit (16 multiply-adds of 4
// cycles per lane against 16 matrix instructions of 64; particular problems
// of 3072 boxes of 7 x 7 x 4 cells 430 -> 376 us).
template <int NW, bool ACC, bool ONE>
__device__ __forceinline__ void apply3(const Box3& s, int nb, int j, int nrhs, const dbl4 wa[NW]) {
  const int lc = lane3() & 15, lg = lane3() >> 4;
  if constexpr (ONE) {
    double a0 = 0.0, a1 = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w)
#pragma unroll
      for (int c = 0; c < 4; c += 2) {
        a0 = fma(wa[w][c], s.Z[16 * w + 4 * c + lg], a0);
        a1 = fma(wa[w][c + 1], s.Z[16 * w + 4 * c + 4 + lg], a1);
      }
    const double y = rows_sum3(a0 + a1);
    const int i = 16 * wave3() + lc;
    if (lg == 0 && i < nb) {
      double* x = s.X + j * nb + i;
      *x = ACC ? *x + y : y;
    }
    lsync<NW>();
    return;
  }
  for (int k0 = 0; k0 < nrhs; k0 += 16) {
    const int k = k0 + lc, kk = min(k, nrhs - 1);
    dbl4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      dbl4 z;
#pragma unroll
      for (int c = 0; c < 4; ++c) z[c] = s.Z[(16 * w + 4 * c + lg) * nrhs + kk];
      acc = mfma16(wa[w], z, acc);
    }
    if (k < nrhs) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * wave3() + 4 * r + lg;
        if (i < nb) {
          double* x = s.X + k * s.nc + j * nb + i;
          *x = ACC ? *x + acc[r] : acc[r];
        }
      }
    }
  }
  lsync<NW>();
}

// Forward step of block j for all right-hand sides.
template <int NW, bool ONE>
__device__ __forceinline__ void fwd_tiles3(const Box3& s, int nb, int j, int nrhs, const dbl4 wa[NW]) {
  for (int e = threadIdx.x; e < nrhs * 16 * NW; e += 64 * NW) {
    const int k = e / (16 * NW), i = e % (16 * NW);
    double v = 0.0;
    if (i < nb) {
      v = s.X[k * s.nc + j * nb + i];
      if (j > 0) v = fma(s.Tz[(j - 1) * nb + i], s.X[k * s.nc + (j - 1) * nb + i], v);
    }
    s.Z[i * nrhs + k] = v;
  }
  lsync<NW>();
  apply3<NW, false, ONE>(s, nb, j, nrhs, wa);
}

// Backward step of block j: x_j += W_j (t_j .* x_{j+1}).
template <int NW, bool ONE>
__device__ __forceinline__ void bwd_tiles3(const Box3& s, int nb, int j, int nrhs, const dbl4 wa[NW]) {
  for (int e = threadIdx.x; e < nrhs * 16 * NW; e += 64 * NW) {
    const int k = e / (16 * NW), i = e % (16 * NW);
    s.Z[i * nrhs + k] = i < nb ? s.Tz[j * nb + i] * s.X[k * s.nc + (j + 1) * nb + i] : 0.0;
  }
  lsync<NW>();
  apply3<NW, true, ONE>(s, nb, j, nrhs, wa);
}

// The lane's share of y = W z for the staged vector z (64 values in LDS):
// the 16-term partial dot product of its entries of row c with z.
__device__ __forceinline__ double wdot3(const double w[R3], const double* z) {
  const double* zw = z + R3 * wave3();
  double a0 = 0.0, a1 = 0.0;
#pragma unroll
  for (int ii = 0; ii < R3; ii += 2) {
    const double2 zz = *reinterpret_cast<const double2*>(zw + ii);
    a0 = fma(w[ii], zz.x, a0);
    a1 = fma(w[ii + 1], zz.y, a1);
  }
  return a0 + a1;
}

// Y[k][c] (+)= (W Z_k)[c] for the nrhs vectors staged in Z (k-th at Z + 64k),
// Y[k] at Y + k * ystride; the partial sums of the waves are added through
// LDS in a fixed order, four right-hand sides at a time.
template <int NW, bool ACC>
__device__ __forceinline__ void wmul3(const Box3& s, Gj3& sm, int nb, int nrhs, const double w[R3],
                                      double* Y, int ystride) {
  constexpr int NT = 64 * NW;
  const int c = lane3();
  if constexpr (NW == 1) {
    for (int k = 0; k < nrhs; ++k) {
      const double y = wdot3(w, s.Z + k * P3);
      if (c < nb) {
        if (ACC) Y[k * ystride + c] += y;
        else Y[k * ystride + c] = y;
      }
    }
    lsync<NW>();
  } else {
    double* pt = partials3(sm);
    const int wv = wave3();
    for (int k0 = 0; k0 < nrhs; k0 += 4) {
      const int cnt = min(4, nrhs - k0);
      for (int kk = 0; kk < cnt; ++kk) pt[(kk * NW + wv) * P3 + c] = wdot3(w, s.Z + (k0 + kk) * P3);
      lsync<NW>();
      for (int e = threadIdx.x; e < cnt * P3; e += NT) {
        const int kk = e / P3, L = e % P3;
        double y = 0.0;
#pragma unroll
        for (int u = 0; u < NW; ++u) y += pt[(kk * NW + u) * P3 + L];
        if (L < nb) {
          if (ACC) Y[(k0 + kk) * ystride + L] += y;
          else Y[(k0 + kk) * ystride + L] = y;
        }
      }
      lsync<NW>();
    }
  }
}

// Forward step of block j for all right-hand sides (W_j in w).
template <int NW>
__device__ __forceinline__ void fwd3(const Box3& s, Gj3& sm, int nb, int j, int nrhs, const double w[R3]) {
  constexpr int NT = 64 * NW;
  for (int e = threadIdx.x; e < nrhs * P3; e += NT) {
    const int k = e / P3, L = e % P3;
    double v = 0.0;
    if (L < nb) {
      v = s.X[k * s.nc + j * nb + L];
      if (j > 0) v = fma(s.Tz[(j - 1) * nb + L], s.X[k * s.nc + (j - 1) * nb + L], v);
    }
    s.Z[k * P3 + L] = v;
  }
  lsync<NW>();
  wmul3<NW, false>(s, sm, nb, nrhs, w, s.X + j * nb, s.nc);
}

// Backward step of block j (W_j in w): x_j += W_j (t_j .* x_{j+1}).
template <int NW>
__device__ __forceinline__ void bwd3(const Box3& s, Gj3& sm, int nb, int j, int nrhs, const double w[R3]) {
  constexpr int NT = 64 * NW;
  for (int e = threadIdx.x; e < nrhs * P3; e += NT) {
    const int k = e / P3, L = e % P3;
    s.Z[k * P3 + L] = L < nb ? s.Tz[j * nb + L] * s.X[k * s.nc + (j + 1) * nb + L] : 0.0;
  }
  lsync<NW>();
  wmul3<NW, true>(s, sm, nb, nrhs, w, s.X + j * nb, s.nc);
}

// The lane's entries of the cached symmetric inverse W_j (rows 16v .. of
// column c; coalesced along the rows).
__device__ __forceinline__ void load3(const double* Wj, int nb, double w[R3]) {
  const int c = lane3(), r0 = R3 * wave3();
#pragma unroll
  for (int ii = 0; ii < R3; ++ii) {
    const int i = r0 + ii;
    w[ii] = (i < nb && c < nb) ? Wj[i * nb + c] : (i == c ? 1.0 : 0.0);
  }
}

// Factor of the box fused with the forward sweep of nrhs right-hand sides
// already in X (ONE: one); inverses to Wg.
template <int NW, bool ONE>
__device__ __forceinline__ void factor3(const Geo& g, const Box& B, const Box3& s, double* Wg, int nrhs,
                                        Gj3& sm) {
  const int nb = s.m0 * s.m1;
  dbl4 T[NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) T[w] = dbl4{0.0, 0.0, 0.0, 0.0};
  for (int j = 0; j < s.m2; ++j) {
    build3<NW>(g, B, s, j, sm, T);
    sweep3<NW>(nb, sm, T);
#pragma unroll
    for (int w = 0; w < NW; ++w) store_tiles3(Wg + (long long)j * nb * nb, nb, w, T[w]);
    if (nrhs > 0) {
      dbl4 wa[NW];
      operand3<NW>(sm, T, wa);
      fwd_tiles3<NW, ONE>(s, nb, j, nrhs, wa);
    }
  }
}

// Back substitution; the next plane's inverse is loaded while the current
// one is applied.
template <int NW, bool ONE>
__device__ __forceinline__ void backward3(const Box3& s, const double* Wg, int nrhs) {
  const int nb = s.m0 * s.m1;
  // the stored inverses are read back by other lanes than wrote them
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  if constexpr (NW > 1) __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  const long long bs = (long long)nb * nb;
  dbl4 w0[NW], w1[NW];
  int j = s.m2 - 2;
  if (j >= 0) load_operand3<NW>(Wg + j * bs, nb, w0);
  for (; j >= 0; j -= 2) {
    if (j > 0) load_operand3<NW>(Wg + (j - 1) * bs, nb, w1);
    bwd_tiles3<NW, ONE>(s, nb, j, nrhs, w0);
    if (j > 0) {
      if (j > 1) load_operand3<NW>(Wg + (j - 2) * bs, nb, w0);
      bwd_tiles3<NW, ONE>(s, nb, j - 1, nrhs, w1);
    }
  }
}

// Steps 1-2 on an oversampled box (FO: Step 6, the factor alone).
template <int NW, bool FO, bool TS>
__device__ __forceinline__ void basis3(const Geo& g, const Box& B, const Seed* __restrict__ seeds,
                                       const double* __restrict__ logK, double beta,
                                       double* __restrict__ fac, double* __restrict__ Pk,
                                       double* __restrict__ tr_u, double* __restrict__ tr_phi,
                                       double* __restrict__ tr_beta, double* dsm, Gj3& sm) {
  constexpr int NT = 64 * NW;
  const int tid = threadIdx.x;
  const int nrhs = FO ? 0 : B.nrhs;
  Box3 s = carve3<TS>(dsm, B, nrhs, g.kc);
  load_box3<NW, true>(g, B, logK, beta, s);
  for (int e = tid; e < nrhs * s.nc; e += NT) s.X[e] = 0.0;
  bsync<NW>();
  seed_rhs3<NW>(g, B, s, seeds, beta, nrhs, s.X);
  bsync<NW>();
  double* Wg = fac + B.fac;
  factor3<NW, false>(g, B, s, Wg, nrhs, sm);
  if (FO) return;
  backward3<NW, false>(s, Wg, nrhs);
  basis_out3<NW>(g, B, s, seeds, beta, nrhs, Pk, tr_u, tr_phi, tr_beta);
}

// Step 4 on a subdomain: K = exp(log K) of its cells (the subdomains cover
// the grid once; a K that is not finite and positive is flagged).
template <int NW, bool TS>
__device__ __forceinline__ void particular3(const Geo& g, const Box& B,
                                            const double* __restrict__ logK, double* __restrict__ K,
                                            const double* __restrict__ f,
                                            const double* __restrict__ bcv, double beta,
                                            double* __restrict__ fac, double* __restrict__ pbar,
                                            double* __restrict__ ubar, double* __restrict__ pibar,
                                            double* dsm, Gj3& sm) {
  Box3 s = carve3<TS>(dsm, B, 1, g.kc);
  load_box3<NW, true>(g, B, logK, beta, s);
  part_k3<NW, TS>(g, B, s, K, sm.flag);
  physical3<NW>(g, B, s, f, bcv, s.X);
  bsync<NW>();
  double* Wg = fac + B.fac;
  factor3<NW, true>(g, B, s, Wg, 1, sm);
  backward3<NW, true>(s, Wg, 1);
  part_out3<NW>(g, B, s, beta, pbar, ubar, pibar);
}

// Steps 6-7 for one box: right-hand side from the state, solve with the
// cached inverses, p on Omega_i and Omega_i's Gamma fluxes.
template <int NW, bool TS>
__device__ __forceinline__ void smooth3(const Geo& g, const Box& B, const double* __restrict__ K,
                                        const double* __restrict__ f,
                                        const double* __restrict__ bcv, double beta,
                                        const double* __restrict__ fac, double* p, double* gflux,
                                        double* dsm, Gj3& sm) {
  Box3 s = carve3<TS>(dsm, B, 1, g.kc);
  load_box3<NW, false>(g, B, K, beta, s);
  physical3<NW>(g, B, s, f, bcv, s.X);
  bsync<NW>();
  smooth_rhs3<NW>(g, B, s, p, gflux, beta, s.X);
  bsync<NW>();
  const int nb = s.m0 * s.m1;
  const double* Wg = fac + B.fac;
  double w[R3];
  for (int j = 0; j < s.m2; ++j) {
    load3(Wg + (long long)j * nb * nb, nb, w);
    fwd3<NW>(s, sm, nb, j, 1, w);
  }
  for (int j = s.m2 - 2; j >= 0; --j) {
    load3(Wg + (long long)j * nb * nb, nb, w);
    bwd3<NW>(s, sm, nb, j, 1, w);
  }
  smooth_out3<NW>(g, B, s, p, gflux, beta);
}

// Register budget for three resident boxes of four waves per CU (their LDS
// allows no more): at most 168 registers per lane, which costs the kernels of
// four waves 20 to 27 spilled registers and those of three 8 to 12.
template <int NW, bool TS>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(3))) k_basis3(Geo g, const Box* __restrict__ boxes,
                                                    const Seed* __restrict__ seeds,
                                                    const double* __restrict__ logK, double beta,
                                                    double* __restrict__ fac, double* __restrict__ Pk,
                                                    double* __restrict__ tr_u,
                                                    double* __restrict__ tr_phi,
                                                    double* __restrict__ tr_beta, int factor_only,
                                                    int* flags) {
  extern __shared__ __align__(16) double dsm[];
  __shared__ Gj3 sm;
  if (threadIdx.x == 0) sm.flag = 0;
  bsync<NW>();
  const Box B = boxes[blockIdx.x];
  if (factor_only)
    basis3<NW, true, TS>(g, B, seeds, logK, beta, fac, Pk, tr_u, tr_phi, tr_beta, dsm, sm);
  else
    basis3<NW, false, TS>(g, B, seeds, logK, beta, fac, Pk, tr_u, tr_phi, tr_beta, dsm, sm);
  bsync<NW>();
  if (threadIdx.x == 0 && sm.flag) atomicOr(flags, sm.flag);
}

template <int NW, bool TS>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(3))) k_particular3(Geo g, const Box* __restrict__ boxes,
                                                         const double* __restrict__ logK,
                                                         double* __restrict__ K,
                                                         const double* __restrict__ f,
                                                         const double* __restrict__ bcv, double beta,
                                                         double* __restrict__ fac,
                                                         double* __restrict__ pbar,
                                                         double* __restrict__ ubar,
                                                         double* __restrict__ pibar, int* flags) {
  extern __shared__ __align__(16) double dsm[];
  __shared__ Gj3 sm;
  if (threadIdx.x == 0) sm.flag = 0;
  bsync<NW>();
  const Box B = boxes[blockIdx.x];
  particular3<NW, TS>(g, B, logK, K, f, bcv, beta, fac, pbar, ubar, pibar, dsm, sm);
  bsync<NW>();
  if (threadIdx.x == 0 && sm.flag) atomicOr(flags, sm.flag);
}

template <int NW, bool TS>
__global__ void __launch_bounds__(64 * NW) k_smooth3(Geo g, const Box* __restrict__ boxes,
                                                     const double* __restrict__ K,
                                                     const double* __restrict__ f,
                                                     const double* __restrict__ bcv, double beta,
                                                     const double* __restrict__ fac,
                                                     double* __restrict__ p, double* __restrict__ gflux) {
  extern __shared__ __align__(16) double dsm[];
  __shared__ Gj3 sm;
  const Box B = boxes[blockIdx.x];
  smooth3<NW, TS>(g, B, K, f, bcv, beta, fac, p, gflux, dsm, sm);
}

template <typename KF>
hipError_t lds_attr3(KF kern, size_t bytes) {
  if (bytes > 64 * 1024)
    return hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  return hipSuccess;
}

}  // namespace

size_t box3_lds_bytes(int m0, int m1, int m2, int nrhs, int kc) {
  return sizeof(double) * box3_doubles(m0, m1, m2, nrhs, kc);
}

int box3_waves(int nb) { return nb <= R3 ? 1 : nb <= 2 * R3 ? 2 : 4; }
int box3_tile_waves(int nb) { return (nb + 15) / 16; }

// waves per box (F3: three among them), and the scalar or the tensor form
// of K
#define MRCM_NW_CASES(nw, CALL, TS, F3)    \
  switch (nw) {                            \
    case 1: CALL(1, TS); break;            \
    case 2: CALL(2, TS); break;            \
    F3                                     \
    case 4: CALL(4, TS); break;            \
    default: return hipErrorInvalidValue;  \
  }
#define MRCM_NW_SWITCH(nw, CALL)           \
  if (g.kc > 1) {                          \
    MRCM_NW_CASES(nw, CALL, true, )        \
  } else {                                 \
    MRCM_NW_CASES(nw, CALL, false, )       \
  }
#define MRCM_TILE_SWITCH(nw, CALL)                                   \
  if (g.kc > 1) {                                                    \
    MRCM_NW_CASES(nw, CALL, true, case 3: CALL(3, true); break;)     \
  } else {                                                           \
    MRCM_NW_CASES(nw, CALL, false, case 3: CALL(3, false); break;)   \
  }

hipError_t launch_basis3(const Geo& g, const Box* boxes, int nbox, const Seed* seeds,
                         const double* logK, double beta, double* fac, double* Pk, double* tr_u,
                         double* tr_phi, double* tr_beta, int factor_only, int* flags, size_t lds,
                         int nw, hipStream_t s) {
  if (nbox <= 0) return hipSuccess;
  hipError_t e = hipSuccess;
#define MRCM_CALL(NW, TS)                                                                             \
  e = lds_attr3(k_basis3<NW, TS>, lds);                                                               \
  if (e != hipSuccess) return e;                                                                      \
  hipLaunchKernelGGL((k_basis3<NW, TS>), dim3(nbox), dim3(64 * NW), lds, s, g, boxes, seeds, logK, beta, fac, \
                     Pk, tr_u, tr_phi, tr_beta, factor_only, flags)
  MRCM_TILE_SWITCH(nw, MRCM_CALL)
#undef MRCM_CALL
  return hipGetLastError();
}

hipError_t launch_particular3(const Geo& g, const Box* boxes, int nbox, const double* logK, double* K,
                              const double* f, const double* bcv, double beta, double* fac,
                              double* pbar, double* ubar, double* pibar, int* flags, size_t lds, int nw,
                              hipStream_t s) {
  if (nbox <= 0) return hipSuccess;
  hipError_t e = hipSuccess;
#define MRCM_CALL(NW, TS)                                                                            \
  e = lds_attr3(k_particular3<NW, TS>, lds);                                                         \
  if (e != hipSuccess) return e;                                                                     \
  hipLaunchKernelGGL((k_particular3<NW, TS>), dim3(nbox), dim3(64 * NW), lds, s, g, boxes, logK, K, f, bcv, \
                     beta, fac, pbar, ubar, pibar, flags)
  MRCM_TILE_SWITCH(nw, MRCM_CALL)
#undef MRCM_CALL
  return hipGetLastError();
}

hipError_t launch_smooth3(const Geo& g, const Box* boxes, int nmem, const double* K, const double* f,
                          const double* bcv, double beta, const double* fac, double* p, double* gflux,
                          size_t lds, int nw, hipStream_t s) {
  if (nmem <= 0) return hipSuccess;
  hipError_t e = hipSuccess;
#define MRCM_CALL(NW, TS)                                                                               \
  e = lds_attr3(k_smooth3<NW, TS>, lds);                                                                \
  if (e != hipSuccess) return e;                                                                        \
  hipLaunchKernelGGL((k_smooth3<NW, TS>), dim3(nmem), dim3(64 * NW), lds, s, g, boxes, K, f, bcv, beta, fac, p, \
                     gflux)
  MRCM_NW_SWITCH(nw, MRCM_CALL)
#undef MRCM_CALL
  return hipGetLastError();
}

#undef MRCM_TILE_SWITCH
#undef MRCM_NW_SWITCH
#undef MRCM_NW_CASES

}  // namespace mrcm
