// One-wavefront-per-box kernels for the 2-D local problems (dense blocks of
// at most 32 cells): factorisation with the seed solves fused into its
// forward sweep, particular problems, and one color phase of smoothing.
//
// Register layout of a 32 x 32 block (padded with the identity when the box
// line is shorter): lane L holds rows 16h .. 16h+15 of column c, with
// c = L & 31 and h = L >> 5, so all 64 lanes carry work.
//
// The block inverse takes 16 pivots at a time in registers (no pivoting: the
// pivots of an SPD matrix are positive) and joins the two halves of the
// block by FP64 matrix instructions (winv); no barrier beyond the single
// wave.
//
// Solves use the block LDL^T recurrences of the block-tridiagonal matrix
// (see local.hip): forward w_j = W_j (b_j + t_{j-1} .* w_{j-1}), backward
// x_j = w_j + W_j (t_j .* x_{j+1}).  A block product is a 16-term dot
// product per lane, its vector entries taken by row broadcast, followed by
// one exchange between the two half-waves (block_products).
// Measured against products staged through LDS and Schur complements built
// with branches (24 x 24 cells, all of Steps 1-2 and 4): 256 boxes with eight
// seeds 136 -> 111 us, 4096 with four 942 -> 801 us.  What bounds a box now:
// 13 line inverses of 7,700 cycles in a chain, 12,000 cycles per step with
// the products of eight seeds, and 40,000 cycles of back-substitution.
//
// Everything a sweep touches between block steps lives in LDS: the box's
// permeabilities (with a one-cell halo), its diagonal and couplings, and
// the right-hand sides / solutions.  The back-substitution of Steps 1-2 and
// 4 reads the block inverses from memory four blocks ahead of their use;
// smoothing copies them into LDS first, except for boxes that do not fit
// there, which stream them in the same way.
#include "wave_common.h"

#include <hip/hip_cooperative_groups.h>

#include <algorithm>

namespace mrcm {
namespace {

using namespace wave;

// Store the nb x nb block held in the register layout w to Wj.
__device__ __forceinline__ void store_block(int nb, double* Wj, const double w[HB]) {
  // lower triangle, row-major (the layout block_src reads); entries outside
  // it get an offset out of the buffer's range: dropped
  const int L = lane_id(), c = L & 31, h = L >> 5;
  const auto rs = uniform_buffer(Wj, packed_elems(nb) * (int)sizeof(double));
  const int lo = max(c - HB * h, 0), n = nb - HB * h;  // my rows
#pragma unroll
  for (int i = 0; i < HB; ++i) {
    typedef unsigned int u2 __attribute__((ext_vector_type(2)));
    // r (r + 1) / 2 + c for r = 16 h + i
    const int off = 8 * (c + h * (136 + 16 * i) + i * (i + 1) / 2);
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, w[i]), rs, i >= lo && i < n ? off : 1 << 28, 0, 0);
  }
}

// Block j of the cached FP64 factors of a box
__device__ __forceinline__ double* fblock(double* Wg, int nb, int j) {
  return Wg + (long long)j * packed_elems(nb);
}

// Factorisation fused with the forward sweep; inverses to Wg, couplings to Tg.
__device__ __forceinline__ void factor_forward(const Box& B, double* Wg, double* Tg, int nrhs, const BoxLds& s,
                               WaveSmem& sm) {
  const int L = lane_id();
  const int nb = B.nb;
  for (int e = L; e < B.ncell; e += 64) Tg[e] = s.Tn[e];
  double w[HB];
#pragma unroll
  for (int i = 0; i < HB; ++i) w[i] = 0.0;
  for (int j = 0; j < B.nblk; ++j) {
    wbuild(nb, j, s, w);
    winv(nb, sm, w);
    store_block(nb, fblock(Wg, nb, j), w);
    fwd_step_d(nb, B.ncell, j, j - 1, j > 0, nrhs, s, w);
  }
}


// ------------------------------------------------------------------ kernels

// LDS of a basis box: the box arrays with its right-hand sides, then from
// BoxLds::Z on the forward Schur complement of the meeting block (nb x nb,
// nb = m0, row-major).  The size decides which boxes the wave kernels take;
// it counts two vectors of NBW per right-hand side that only products staged
// through LDS need, so that the set of those boxes stays what it was.
__host__ __device__ inline size_t basis_lds_doubles(int m0, int m1, int nrhs, int kc = 1) {
  return box_lds_doubles(m0, m1, nrhs, kc) + (size_t)nrhs * NBW + (size_t)m0 * m0 + 2;
}

// Steps 1-2: factor the oversampled box, solve every seed, extract
// u and phi on Gamma_i and the restriction to Omega_i.  Two waves solve
// the block-tridiagonal system from both ends (meeting block m = nblk / 2):
// wave 0 eliminates blocks 0 .. m-1 (forward inverses W_j into fac), wave 1
// blocks nblk-1 .. m+1 (backward inverses W'_j = (D_j - t_j W'_{j+1} t_j)^{-1}
// into fact), each with the forward sweep of every seed fused in; wave 1
// then inverts Z_m = (S_m - t_m W'_{m+1} t_m)^{-1} (S_m: forward Schur
// complement of block m, from wave 0), stored at block m of fact, and solves
// the meeting block; both back-substitute outwards.  The chain of block
// inverses on one wave is about half as long as a one-ended elimination,
// and fac / fact are exactly the factors of the two-ended smoothing sweep.
// FO (factor only, Algorithm 1 Step 6): the box is factored with the
// smoothing Robin parameter and nothing else is solved or written (the
// block couplings do not depend on beta and are shared with Step 1).
template <bool FO = false>
__device__ __forceinline__ void basis_box(const Geo& g, const Box& B, const Seed* __restrict__ seeds,
                                          const double* __restrict__ logK, double beta,
                                          double* __restrict__ fac, double* __restrict__ fact,
                                          double* __restrict__ tcoup,
                                          double* __restrict__ Pk, double* __restrict__ tr_u,
                                          double* __restrict__ tr_phi,
                                          double* __restrict__ tr_beta,
                                          const double* __restrict__ f,
                                          const double* __restrict__ bcv, const SmoothStatic& st,
                                          double* dsm, WaveSmem* sm) {
  const int L = lane_id();
  const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nrhs = FO ? 0 : B.nrhs;
  BoxLds s = carve(dsm, B, nrhs, g.kc);
  double* Sm = s.Z;
  const int nc = B.ncell;
  // set-up by both waves: box arrays (K from log K), seed right-hand
  // sides, couplings
  load_box<128, true>(g, B, logK, beta, s);
  if (st.b0) smooth_static<128>(g, B, s, f, bcv, beta, st);
  for (int e = tid; e < nrhs * nc; e += 128) s.X[e] = 0.0;
  __syncthreads();
  // T^R times the seed on the cells of its side, all seeds at once
  const int fs = s.m0 > s.m1 ? s.m0 : s.m1;  // faces of the longest side
  #pragma unroll 1
  for (int e = tid; e < nrhs * fs; e += 128) {
    const int k = e / fs, t = e % fs;
    const Seed sd = seeds[B.seed0 + k];
    const int a = sd.side >> 1, so = sd.side & 1;
    const int nf = (a == 0) ? s.m1 : s.m0;
    if (t >= nf) continue;
    int c[3];
    if (a == 0) { c[0] = so ? B.hi[0] - 1 : B.lo[0]; c[1] = B.lo[1] + t; }
    else { c[1] = so ? B.hi[1] - 1 : B.lo[1]; c[0] = B.lo[0] + t; }
    c[2] = 0;
    const int ox = c[0] + (a == 0 ? (so ? 1 : -1) : 0), oy = c[1] + (a == 1 ? (so ? 1 : -1) : 0);
    const double kc = kat(s, B, c[0], c[1], a);
    const double bt = robin_beta(g, a, kc, kat(s, B, ox, oy, a), beta);
    s.X[k * nc + bloc(B, s, c[0], c[1])] = robin_T(g, kc, bt) * seed_value(g, sd, B.lo, B.hi, c);
  }
  if (!FO)
    for (int e = tid; e < nc; e += 128) tcoup[B.scr + e] = s.Tn[e];
  __syncthreads();
  const int nb = B.nb, nblk = B.nblk, m = nblk / 2;
  double* Wf = fac + B.fac;
  double* Wt = fact + B.fac;
  double w[HB];
#pragma unroll
  for (int i = 0; i < HB; ++i) w[i] = 0.0;
  {
    const bool bot = wv == 1;
    const int cnt = bot ? nblk - 1 - m : m;
#pragma unroll 1
    for (int t = 0; t < cnt; ++t) {
      const int j = bot ? nblk - 1 - t : t, jp = bot ? j + 1 : j - 1;
      wbuild_t(nb, j, t > 0 ? (bot ? j : jp) : -1, s, w);
      winv(nb, sm[wv], w);
      store_block(nb, fblock(bot ? Wt : Wf, nb, j), w);
      fwd_step_d(nb, nc, j, jp, t > 0, nrhs, s, w);
    }
  }
  if (wv == 0) {
    wbuild(nb, m, s, w);  // S_m
    const int c = L & 31, h = L >> 5;
#pragma unroll
    for (int i = 0; i < HB; ++i) {
      const int r = HB * h + i;
      if (r < nb && c < nb) Sm[r * nb + c] = w[i];
    }
  }
  __syncthreads();
  if (wv == 1) {
    // Z_m = (S_m - t_m W'_{m+1} t_m)^{-1}, identity padding kept; w holds
    // W'_{m+1} when the bottom half is not empty
    const int c = L & 31, h = L >> 5;
    const double* Tm = s.Tn + m * nb;
    const double tc = (m < nblk - 1 && c < nb) ? Tm[c] : 0.0;
#pragma unroll
    for (int i = 0; i < HB; ++i) {
      const int r = HB * h + i;
      // identity padding outside the nb x nb block, as wbuild leaves it
      const double smi = (r < nb && c < nb) ? Sm[r * nb + c] : (r == c ? 1.0 : 0.0);
      const double tr = (m < nblk - 1 && r < nb) ? Tm[r] : 0.0;
      w[i] = (m < nblk - 1 && r < nb && c < nb) ? fma(-tr * tc, w[i], smi) : smi;
    }
    winv(nb, sm[1], w);
    store_block(nb, fblock(Wt, nb, m), w);
    if (!FO) mid_step(nb, nc, m, nblk, nrhs, s, w);
  }
  if (FO) return;
  __syncthreads();
  if (wv == 0) twist_back_cached(B, Wf, nrhs, s, false);
  else twist_back_cached(B, Wt, nrhs, s, true);
  __syncthreads();
  int olo[3], ohi[3];
  womega(g, B.sub, olo, ohi);
  const int ncell_o = g.S[0] * g.S[1];
  #pragma unroll 1
  for (int e = tid; e < nrhs * ncell_o; e += 128) {
    const int k = e / ncell_o, t = e % ncell_o;
    Pk[(long long)(B.seed0 + k) * ncell_o + t] =
        s.X[k * nc + bloc(B, s, olo[0] + t % g.S[0], olo[1] + t / g.S[0])];
  }
  for (int q = 0; q < 4; ++q) {
    const int nf = (q >> 1) == 0 ? g.S[1] : g.S[0];
    const bool has = wneighbor(g, B.sub, q) >= 0;
    const int a = q >> 1, so = q & 1;
    #pragma unroll 1
    for (int e = tid; e < nrhs * nf; e += 128) {
      const int k = e / nf, t = e % nf;
      const long long oidx = (long long)(B.seed0 + k) * g.gstride + g.gside_off[q] + t;
      if (!has) {
        tr_u[oidx] = 0.0;
        tr_phi[oidx] = 0.0;
        continue;
      }
      int x, y;
      wgface(olo, ohi, q, t, x, y);
      const int ox = x + (a == 0 ? (so ? 1 : -1) : 0), oy = y + (a == 1 ? (so ? 1 : -1) : 0);
      const double kc = kat(s, B, x, y, a), ko = kat(s, B, ox, oy, a);
      const double Pc = s.X[k * nc + bloc(B, s, x, y)];
      const double bt = robin_beta(g, a, kc, ko, beta);
      double u;
      if (win_box(B, ox, oy)) {
        u = g.area * kharm(kc, ko) / g.h * (Pc - s.X[k * nc + bloc(B, s, ox, oy)]) / g.area;
      } else {
        const Seed sd = seeds[B.seed0 + k];
        const int c[3] = {x, y, 0};
        const double lam = (sd.side == q) ? seed_value(g, sd, B.lo, B.hi, c) : 0.0;
        u = robin_T(g, kc, bt) * (Pc - lam) / g.area;
      }
      const double pi = Pc - u * g.h / (2.0 * kc);
      tr_u[oidx] = u;
      tr_phi[oidx] = -bt * u + pi;
      if (k == 0) tr_beta[(long long)B.sub * g.gstride + g.gside_off[q] + t] = bt;
    }
  }
}

// Step 4: particular problem on Omega_i with zero Robin data on Gamma_i.
// The box is Omega_i itself: it also writes K = exp(log K) of its cells
// (the subdomains cover the grid once) and flags a K that is not finite
// and positive.
__device__ __forceinline__ void particular_box(const Geo& g, const Box& B,
                                               const double* __restrict__ logK,
                                               double* __restrict__ K,
                                               const double* __restrict__ f,
                                               const double* __restrict__ bcv, double beta,
                                               double* __restrict__ fac, double* __restrict__ tcoup,
                                               double* __restrict__ pbar, double* __restrict__ ubar,
                                               double* __restrict__ pibar, double* dsm, WaveSmem& sm) {
  const int L = lane_id();
  BoxLds s = carve(dsm, B, 1, g.kc);
  load_box<64, true>(g, B, logK, beta, s);
  for (int t = L; t < B.ncell; t += 64) {
    const int x = B.lo[0] + t % s.m0, y = B.lo[1] + t / s.m0;
    for (int a = 0; a < g.kc; ++a) {
      const double k = kat(s, B, x, y, a);
      if (!(k > 0.0) || !isfinite(k)) atomicOr(&sm.flag, kFlagBadK);
      K[kaxis(g, a) + x + g.n[0] * y] = k;
    }
  }
  physical_rhs(g, B, s, f, bcv, s.X);
  wsync();
  double* Wg = fac + B.fac;
  factor_forward(B, Wg, tcoup + B.scr, 1, s, sm);
  backward_cached(B, Wg, 1, s);
  for (int t = L; t < B.ncell; t += 64) pbar[(long long)B.sub * B.ncell + t] = s.X[t];
  for (int q = 0; q < 4; ++q) {
    const int nf = (q >> 1) == 0 ? g.S[1] : g.S[0];
    const bool has = wneighbor(g, B.sub, q) >= 0;
    const int a = q >> 1, so = q & 1;
    #pragma unroll 1
    for (int t = L; t < nf; t += 64) {
      const long long oidx = (long long)B.sub * g.gstride + g.gside_off[q] + t;
      if (!has) {
        ubar[oidx] = 0.0;
        pibar[oidx] = 0.0;
        continue;
      }
      int x, y;
      wgface(B.lo, B.hi, q, t, x, y);
      const int ox = x + (a == 0 ? (so ? 1 : -1) : 0), oy = y + (a == 1 ? (so ? 1 : -1) : 0);
      const double kc = kat(s, B, x, y, a);
      const double bt = robin_beta(g, a, kc, kat(s, B, ox, oy, a), beta);
      const double u = robin_T(g, kc, bt) * s.X[bloc(B, s, x, y)] / g.area;
      ubar[oidx] = u;
      pibar[oidx] = bt * u;
    }
  }
}

// Steps 1-2 and 4 in one launch of two-wave workgroups.  Workgroups
// [0, nbox) handle the oversampled boxes (factors of both ends, seeds,
// traces); in the workgroups after them each of the first npart waves
// solves the particular problem of one subdomain (one-ended factorisation
// of Omega_i), in its own part_ld doubles of LDS.  The two sets share nothing, so their waves run side
// by side instead of one launch after the other.
__global__ void __launch_bounds__(128) k_local_w(Geo g, const Box* __restrict__ obox,
                                                 const Box* __restrict__ pbox, int nbox,
                                                 const Seed* __restrict__ seeds,
                                                 const double* __restrict__ logK,
                                                 double* __restrict__ K,
                                                 const double* __restrict__ f,
                                                 const double* __restrict__ bcv, double beta,
                                                 double* __restrict__ fac,
                                                 double* __restrict__ tcoup,
                                                 double* __restrict__ facp,
                                                 double* __restrict__ tcp,
                                                 double* __restrict__ Pk,
                                                 double* __restrict__ tr_u,
                                                 double* __restrict__ tr_phi,
                                                 double* __restrict__ tr_beta,
                                                 double* __restrict__ pbar,
                                                 double* __restrict__ ubar,
                                                 double* __restrict__ pibar,
                                                 double* __restrict__ fact, SmoothStatic st,
                                                 int npart, int part_ld, int* flags) {
  extern __shared__ __align__(16) double dsm[];
  __shared__ WaveSmem sm[2];
  const int L = lane_id(), wv = threadIdx.x >> 6;
  if (L == 0) sm[wv].flag = 0;
  const int b = blockIdx.x;
  if (b < nbox) {
    const Box B = obox[b];
    basis_box(g, B, seeds, logK, beta, fac, fact, tcoup, Pk, tr_u, tr_phi, tr_beta, f, bcv, st, dsm, sm);
  } else {
    // npart (1 or 2) subdomains per workgroup, one per wave, each in its own
    // part_ld doubles of LDS
    const int pi = npart * (b - nbox) + wv;
    if (wv < npart && pi < nbox) {
      const Box B = pbox[pi];
      particular_box(g, B, logK, K, f, bcv, beta, facp, tcp, pbar, ubar, pibar,
                     dsm + (size_t)wv * part_ld, sm[wv]);
    }
  }
  __syncthreads();
  if (threadIdx.x == 0 && (sm[0].flag | sm[1].flag)) atomicOr(flags, sm[0].flag | sm[1].flag);
}

// Algorithm 1, Step 6: the oversampled boxes factored again with the
// smoothing Robin parameter (when it differs from the basis one), two waves
// per box as in k_local_w, into their own forward / backward inverses.
__global__ void __launch_bounds__(128) k_factor_w(Geo g, const Box* __restrict__ obox,
                                                  const double* __restrict__ logK, double beta,
                                                  const double* __restrict__ f,
                                                  const double* __restrict__ bcv,
                                                  double* __restrict__ fac,
                                                  double* __restrict__ fact, SmoothStatic st,
                                                  int* flags) {
  extern __shared__ __align__(16) double dsm[];
  __shared__ WaveSmem sm[2];
  const int L = lane_id(), wv = threadIdx.x >> 6;
  if (L == 0) sm[wv].flag = 0;
  const Box B = obox[blockIdx.x];
  basis_box<true>(g, B, nullptr, logK, beta, fac, fact, nullptr, nullptr, nullptr, nullptr,
                  nullptr, f, bcv, st, dsm, sm);
  __syncthreads();
  if (threadIdx.x == 0 && (sm[0].flag | sm[1].flag)) atomicOr(flags, sm[0].flag | sm[1].flag);
}

// Factor blocks a box's smoothing solve needs first (the first ring slots of
// both halves on waves 0 and 1, the meeting block on wave 0): constant data,
// loaded early so that their memory latency overlaps other work.
template <int NT>
__device__ __forceinline__ void smooth_preload(const Box& B, const double* Wf, const double* Wt,
                                               double w[RING][HB], double zm[HB]) {
  const int wv = threadIdx.x >> 6;
  if (NT > 64 && wv < 2) twist_preload(twist_half(B, wv == 0 ? Wf : Wt, B.nblk / 2, wv == 1), w);
  if (threadIdx.x < 64) wload_block(block_src(Wt, B.nb, B.nblk), B.nblk / 2, zm);
}

// Steps 6-7 for one box: stage the box's data, build the right-hand side,
// solve with the two-ended block sweep (its halves on the first two waves
// when NT >= 128) and write p on Omega_i and Omega_i's Gamma fluxes.
template <int NT>
__device__ __forceinline__ void smooth_box(const Geo& g, const Box& B, const double* __restrict__ K,
                                           const double* __restrict__ f,
                                           const double* __restrict__ bcv, double beta,
                                           const double* Wf, const double* Wt,
                                           const double* __restrict__ tcoup, double* p,
                                           double* gflux, double w[RING][HB], const double zm[HB],
                                           double* dsm) {
  SmoothLds r = carve_smooth(dsm, B, g.kc);
  stage_smooth<NT>(g, B, r, K, p, f, gflux, bcv, tcoup);
  bsync<NT>();
  smooth_rhs<NT>(g, B, r, beta, r.b.X);
  bsync<NT>();
  sweep_twisted<NT>(B, Wf, Wt, r.b, r.b.Z, w, zm);
  smooth_out<NT>(g, B, r, r.b.X, beta, p, gflux);
}

// The fields of Geo a smoothing box uses, as scalars: every inlined use of
// the kernel argument itself counts against the compiler's limit for
// reading it in place, beyond which it is copied to scratch memory.
struct Geo2 {
  int n0, n1, cut, l, S0, S1, M0, M1, mcut, gstride, go0, go1, go2, go3;
  double area;
};
__device__ __forceinline__ Geo2 geo2(const Geo& g) {
  return Geo2{g.n[0], g.n[1], g.cut, g.l, g.S[0], g.S[1], g.M[0], g.M[1], g.mcut, g.gstride,
              g.gside_off[0], g.gside_off[1], g.gside_off[2], g.gside_off[3], g.area};
}
__device__ __forceinline__ int gside2(const Geo2& g, int q) {
  return q == 0 ? g.go0 : q == 1 ? g.go1 : q == 2 ? g.go2 : g.go3;
}
// moving from `from` to `to` along an axis of n entries (cut: batch members)
__device__ __forceinline__ bool off2(int n, int cut, int from, int to) {
  return to < 0 || to >= n || (cut > 0 && to / cut != from / cut);
}

// What the Robin term of box-side face u reads: its two coefficients, the
// state on this side (va; without overlap the neighbour's flux at the face)
// and beyond the face (vb).  Zero on the domain boundary.
struct FaceIn {
  double c0, c1, va, vb;
};
__device__ __forceinline__ FaceIn face_in(const Geo2& g, int lo0, int lo1, int hi0, int hi1, int sub, int u,
                                          const double* __restrict__ fc, const double* p,
                                          const double* gflux) {
  FaceIn r{0.0, 0.0, 0.0, 0.0};
  int t, x, y, ox, oy;
  const int q = face_side(hi0 - lo0, hi1 - lo1, u, t), a = q >> 1, sd = q & 1, n0 = g.n0;
  face_cells(lo0, lo1, hi0, hi1, q, t, x, y, ox, oy);
  const bool dom = off2(a == 0 ? g.n0 : g.n1, a == 0 ? 0 : g.cut, a == 0 ? x : y, a == 0 ? ox : oy);
  if (dom) return r;
  r.c0 = fc[2 * u];
  r.c1 = fc[2 * u + 1];
  r.vb = p[ox + n0 * oy];
  if (g.l > 0) {
    r.va = p[x + n0 * y];
  } else {
    // the face's place on the neighbour's opposite side
    const int isub = sub % g.M0, jsub = sub / g.M0;
    const int j = sub + (a == 0 ? (sd ? 1 : -1) : (sd ? g.M0 : -g.M0));
    const int tj = a == 0 ? y - jsub * g.S1 : x - isub * g.S0;
    r.va = gflux[(long long)j * g.gstride + gside2(g, q ^ 1) + tj];
  }
  return r;
}
// T^R lambda of that face
__device__ __forceinline__ double face_add(bool overlap, const FaceIn& r) {
  return overlap ? fma(r.c0, r.va, -r.c1 * (r.va - r.vb)) : fma(r.c0, r.vb, r.c1 * r.va);
}

// Gamma face u of a subdomain (side by side): side q, position t, and its
// index in the subdomain's Gamma fluxes
__device__ __forceinline__ int gamma_face(const Geo2& g, int u, int& q, int& t) {
  q = face_side(g.S0, g.S1, u, t);
  return gside2(g, q) + t;
}

// The same with the box's factors resident in LDS and what does not change
// between phases read from the smooth_static arrays (see lds_sweep): the
// form of every box whose LDS fits a workgroup.  Ends with a barrier.
//
// Bound: latency, one box per CU or two.  Of 20,000 cycles of a 24 x 24 box,
// 12,000 are the 25 block steps, 3,500 the staging, 1,600 the outputs.
template <int NT>
__device__ __forceinline__ void smooth_box_res(const Geo2& g, const Box& B, const SmoothStatic& st,
                                               const double* Wf, const double* Wt,
                                               const double* __restrict__ tcoup, double* p,
                                               double* gflux, double* dsm) {
  const int tid = threadIdx.x % NT;
  const int lo0 = B.lo[0], lo1 = B.lo[1], hi0 = B.hi[0], hi1 = B.hi[1], sub = B.sub;
  const int m0 = hi0 - lo0, m1 = hi1 - lo1, nc = m0 * m1, nce = (nc + 1) / 2 * 2;
  const int n0 = g.n0, ns = 2 * (m0 + m1), ng = 2 * (g.S0 + g.S1);
  double* img = dsm;
  double* X = img + factor_image_doubles(m0, m1);
  double* Tn = X + nce;
  double* AF = Tn + nce;  // T^R lambda of the box sides
  const double* fc = st.fc + (long long)sub * st.fstride;
  const double* gc = st.gc + (long long)sub * g.gstride;
  // the first faces' loads are in flight before the staging is issued
  FaceIn first{0.0, 0.0, 0.0, 0.0};
  if (tid < ns) first = face_in(g, lo0, lo1, hi0, hi1, sub, tid, fc, p, gflux);
  stage_factors<NT>(B, Wf, Wt, img);
  stage_lds<NT>(st.b0 + B.scr, X, nc);
  stage_lds<NT>(tcoup + B.scr, Tn, nc);
  if (tid < ns) AF[tid] = face_add(g.l > 0, first);
#pragma unroll 1
  for (int u = tid + NT; u < ns; u += NT)
    AF[u] = face_add(g.l > 0, face_in(g, lo0, lo1, hi0, hi1, sub, u, fc, p, gflux));
  staged_wait<NT>();
  // both sides of an axis in one pass, except in a box one cell thick along
  // it, where they add to the same cells
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const int nf = a == 0 ? m1 : m0, st0 = a == 0 ? 1 : m0;  // faces per side, step along a side's normal
    const int base = a == 0 ? 0 : 2 * m1, ma = a == 0 ? m0 : m1, stf = a == 0 ? m0 : 1;
    if (ma > 1) {
      for (int u = tid; u < 2 * nf; u += NT) {
        const int hiq = u >= nf, t = u - (hiq ? nf : 0);
        X[t * stf + (hiq ? (ma - 1) * st0 : 0)] += AF[base + u];
      }
    } else {
      for (int t = tid; t < nf; t += NT) X[t * stf] += AF[base + t] + AF[base + nf + t];
    }
    bsync<NT>();
  }
  int q0, t0;
  const double gc0 = tid < ng ? gc[gamma_face(g, tid, q0, t0)] : 0.0;  // in flight during the sweep
  lds_sweep<NT>(B, img, Tn, X);
  // Omega_i's Gamma fluxes and p on Omega_i
  const int ix = sub % g.M0, iy = sub / g.M0, w0 = ix * g.S0, w1 = iy * g.S1;
#pragma unroll 1
  for (int u = tid; u < ng; u += NT) {
    int q, t;
    const int at = gamma_face(g, u, q, t), a = q >> 1, so = q & 1;
    const int nj = (a == 0 ? ix : iy) + (so ? 1 : -1);
    if (off2(a == 0 ? g.M0 : g.M1, a == 0 ? 0 : g.mcut, a == 0 ? ix : iy, nj)) continue;
    const int cx = a == 0 ? (so ? w0 + g.S0 - 1 : w0) : w0 + t, cy = a == 1 ? (so ? w1 + g.S1 - 1 : w1) : w1 + t;
    const double* x = X + (cx - lo0) + m0 * (cy - lo1);
    double v;
    if (g.l > 0) {
      v = (u == tid ? gc0 : gc[at]) * (*x - x[a == 0 ? (so ? 1 : -1) : (so ? m0 : -m0)]);
    } else {
      // the box is Omega_i: T^R (x_c - lambda) / |e|
      const int uf = face_off(m0, m1, q) + t;
      v = (fc[2 * uf] * *x - AF[uf]) * rcp_d(g.area);
    }
    gflux[(long long)sub * g.gstride + at] = v;
  }
  const int ncell_o = g.S0 * g.S1;
#pragma unroll 1
  for (int t = tid; t < ncell_o; t += NT) {
    const int cx = w0 + t % g.S0, cy = w1 + t / g.S0;
    p[cx + n0 * cy] = X[(cx - lo0) + m0 * (cy - lo1)];
  }
  bsync<NT>();
}

// Steps 6-7: one color phase of the smoothing sweep, one workgroup of NT
// threads (64, 128 or 256, chosen by the autotuner) per box.  The result
// does not depend on NT.  RES: factors resident in LDS.
template <int NT, bool RES>
__global__ void __launch_bounds__(NT) k_smooth_w(Geo g, const Box* __restrict__ boxes,
                                                 const double* __restrict__ K,
                                                 const double* __restrict__ f,
                                                 const double* __restrict__ bcv, double beta,
                                                 const double* __restrict__ fac,
                                                 const double* __restrict__ fact,
                                                 const double* __restrict__ tcoup, SmoothStatic st,
                                                 double* __restrict__ p,
                                                 double* __restrict__ gflux) {
  extern __shared__ __align__(16) double dsm[];
  const Box B = boxes[blockIdx.x];
  if constexpr (RES) {
    smooth_box_res<NT>(geo2(g), B, st, fac + B.fac, fact + B.fac, tcoup, p, gflux, dsm);
  } else {
    double w[RING][HB], zm[HB];
    smooth_preload<NT>(B, fac + B.fac, fact + B.fac, w, zm);
    smooth_box<NT>(g, B, K, f, bcv, beta, fac + B.fac, fact + B.fac, tcoup, p, gflux, w, zm, dsm);
  }
}

// All colour phases of nphase / ncol smoothing steps in one cooperative
// launch.  In phase k (colour k % ncol) workgroup b takes boxes b, b + G,
// b + 2G, ... of that colour (G workgroups, all resident at once), and a
// grid-wide barrier separates the phases, so that a phase reads the state
// its predecessors wrote.  Without resident factors (RES) a workgroup loads
// the first factor blocks of its next box already after each box, also
// across the barrier (factors do not change during smoothing).  Every
// workgroup passes every barrier.
template <int NT, bool RES>
__global__ void __launch_bounds__(NT) k_smooth_grid(Geo g, const Box* __restrict__ boxes,
                                                    SmoothPhases ph, int nphase,
                                                    const double* __restrict__ K,
                                                    const double* __restrict__ f,
                                                    const double* __restrict__ bcv, double beta,
                                                    const double* __restrict__ fac,
                                                    const double* __restrict__ fact,
                                                    const double* __restrict__ tcoup,
                                                    SmoothStatic st, double* p, double* gflux) {
  extern __shared__ __align__(16) double dsm[];
  cooperative_groups::grid_group grid = cooperative_groups::this_grid();
  const int G = gridDim.x, b0 = blockIdx.x;
  auto count = [&](int k) { return ph.off[k % ph.ncol + 1] - ph.off[k % ph.ncol]; };
  auto box_at = [&](int k, int j) { return ph.off[k % ph.ncol] + j; };
  if constexpr (RES) {
    for (int k = 0; k < nphase; ++k) {
      for (int j = b0; j < count(k); j += G) {
        const Box B = boxes[box_at(k, j)];
        smooth_box_res<NT>(geo2(g), B, st, fac + B.fac, fact + B.fac, tcoup, p, gflux, dsm);
      }
      grid.sync();
    }
  } else {
    auto preload = [&](int bi, double w[RING][HB], double zm[HB]) {
      const Box B = boxes[bi];
      smooth_preload<NT>(B, fac + B.fac, fact + B.fac, w, zm);
    };
    double w[RING][HB], zm[HB];
    int bi = b0 < count(0) ? box_at(0, b0) : -1;
    if (bi >= 0) preload(bi, w, zm);
    for (int k = 0; k < nphase; ++k) {
      const int n = count(k);
      const int n1 = k + 1 < nphase ? count(k + 1) : 0;
      for (int j = b0; j < n; j += G) {
        const Box B = boxes[bi];
        smooth_box<NT>(g, B, K, f, bcv, beta, fac + B.fac, fact + B.fac, tcoup, p, gflux, w, zm, dsm);
        bsync<NT>();  // the next box stages over what its outputs read
        bi = j + G < n ? box_at(k, j + G) : (b0 < n1 ? box_at(k + 1, b0) : -1);
        if (bi >= 0) preload(bi, w, zm);
      }
      if (b0 >= n && b0 < n1) {
        bi = box_at(k + 1, b0);
        preload(bi, w, zm);
      }
      grid.sync();
    }
  }
}

template <typename KF>
hipError_t set_lds(KF kern, size_t bytes) {
  if (bytes > 64 * 1024)
    return hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)bytes);
  return hipSuccess;
}

SmoothStatic statics(const SmoothArrays& a) { return SmoothStatic{a.b0, a.fc, a.gc, a.fstride}; }

}  // namespace

size_t wave_basis_lds_bytes(int m0, int m1, int nrhs, int kc) {
  return sizeof(double) * basis_lds_doubles(m0, m1, nrhs, kc);
}

size_t wave_lds_bytes(int m0, int m1, int nrhs, int kc) {
  return sizeof(double) * box_lds_doubles(m0, m1, nrhs, kc);
}

size_t wave_smooth_lds_bytes(int m0, int m1, int kc) { return sizeof(double) * smooth_lds_doubles(m0, m1, kc); }

size_t wave_smooth_res_lds_bytes(int m0, int m1) { return sizeof(double) * smooth_res_doubles(m0, m1); }

long long wave_packed_elems(int nb) { return packed_elems(nb); }

hipError_t launch_local_w(const Geo& g, const Box* obox, const Box* pbox, int nbox,
                          const Seed* seeds, const double* logK, double* K, const double* f,
                          const double* bcv,
                          double beta, double* fac, double* tcoup, double* facp, double* tcp,
                          double* Pk, double* tr_u, double* tr_phi, double* tr_beta, double* pbar,
                          double* ubar, double* pibar, double* fact, const SmoothArrays& sa,
                          int* flags, size_t lds, size_t lds_part, hipStream_t s) {
  if (nbox <= 0) return hipSuccess;
  hipError_t e = set_lds(k_local_w, lds);
  if (e != hipSuccess) return e;
  if (!fact) return hipErrorInvalidValue;
  // Two subdomains per workgroup when the boxes outnumber the CUs several
  // times over (the launch is throughput-bound and a second wave per
  // workgroup costs no LDS); one when every box has a CU of its own and
  // the basis workgroups' latency decides.
  int dev = 0, ncu = 0;
  e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  const int part_ld = (int)((lds_part / sizeof(double) + 1) / 2 * 2);  // 16-byte aligned waves
  const int npart = (nbox > 2 * ncu && (size_t)2 * part_ld * sizeof(double) <= lds) ? 2 : 1;
  if ((size_t)part_ld * sizeof(double) > lds) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_local_w, dim3(nbox + (nbox + npart - 1) / npart), dim3(128), lds, s, g, obox,
                     pbox, nbox, seeds, logK, K, f, bcv, beta, fac, tcoup, facp, tcp, Pk, tr_u,
                     tr_phi, tr_beta, pbar, ubar, pibar, fact, statics(sa), npart, part_ld, flags);
  return hipGetLastError();
}

hipError_t launch_factor_w(const Geo& g, const Box* obox, int nbox, const double* logK,
                           double beta, const double* f, const double* bcv, double* fac, double* fact,
                           const SmoothArrays& sa, int* flags, size_t lds, hipStream_t s) {
  if (nbox <= 0) return hipSuccess;
  if (!fac || !fact) return hipErrorInvalidValue;
  hipError_t e = set_lds(k_factor_w, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_factor_w, dim3(nbox), dim3(128), lds, s, g, obox, logK, beta, f, bcv, fac, fact,
                     statics(sa), flags);
  return hipGetLastError();
}

hipError_t launch_smooth_w(const Geo& g, const Box* boxes, int nmem,
                           const double* K, const double* f, const double* bcv, double beta,
                           const double* fac, const double* fact, const double* tcoup,
                           const SmoothArrays& sa, double* p, double* gflux, size_t lds, size_t lds_res,
                           int nt, hipStream_t s) {
  if (nmem <= 0) return hipSuccess;
  if (!fact) return hipErrorInvalidValue;
  hipError_t e;
#define MRCM_SMOOTH_NT(N)                                                                     \
  if (lds_res) {                                                                              \
    e = set_lds(k_smooth_w<N, true>, lds_res);                                                \
    if (e != hipSuccess) return e;                                                            \
    hipLaunchKernelGGL((k_smooth_w<N, true>), dim3(nmem), dim3(N), lds_res, s, g, boxes, K, f, bcv, \
                       beta, fac, fact, tcoup, statics(sa), p, gflux);                        \
  } else {                                                                                    \
    e = set_lds(k_smooth_w<N, false>, lds);                                                   \
    if (e != hipSuccess) return e;                                                            \
    hipLaunchKernelGGL((k_smooth_w<N, false>), dim3(nmem), dim3(N), lds, s, g, boxes, K, f, bcv, \
                       beta, fac, fact, tcoup, statics(sa), p, gflux);                        \
  }
  if (nt == 64) {
    MRCM_SMOOTH_NT(64)
  } else if (nt == 128) {
    MRCM_SMOOTH_NT(128)
  } else if (nt == 256) {
    MRCM_SMOOTH_NT(256)
  } else {
    return hipErrorInvalidValue;
  }
#undef MRCM_SMOOTH_NT
  return hipGetLastError();
}

hipError_t launch_smooth_grid(const Geo& g, const Box* boxes, const SmoothPhases& ph, int nphase, const double* K, const double* f,
                              const double* bcv, double beta, const double* fac, const double* fact,
                              const double* tcoup, const SmoothArrays& sa, double* p, double* gflux,
                              size_t lds_ring, size_t lds_res, int nt, int max_groups, hipStream_t s) {
  if (nphase <= 0) return hipSuccess;
  if (!fact || ph.ncol <= 0 || ph.ncol > 8 || max_groups < 0) return hipErrorInvalidValue;
  int nbox = 0;
  for (int c = 0; c < ph.ncol; ++c) nbox = std::max(nbox, ph.off[c + 1] - ph.off[c]);
  if (nbox <= 0) return hipSuccess;
  int dev = 0, ncu = 0, coop = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  if (!coop) return hipErrorNotSupported;
  Geo gg = g;
  SmoothPhases pp = ph;
  SmoothStatic st = statics(sa);
  const size_t lds = lds_res ? lds_res : lds_ring;
  void* args[] = {&gg, &boxes, &pp, &nphase, &K, &f, &bcv, &beta, &fac, &fact, &tcoup, &st, &p, &gflux};
  auto go = [&](auto kern, int N) -> hipError_t {
    hipError_t r = set_lds(kern, lds);
    if (r != hipSuccess) return r;
    int per_cu = 0;
    r = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, N, lds);
    if (r != hipSuccess) return r;
    long long grid = std::min<long long>(nbox, (long long)per_cu * ncu);
    if (max_groups > 0) grid = std::min<long long>(grid, max_groups);
    if (grid <= 0) return hipErrorCooperativeLaunchTooLarge;
    return hipLaunchCooperativeKernel((const void*)kern, dim3((unsigned)grid), dim3(N), args, lds, s);
  };
  if (nt == 64) return lds_res ? go(k_smooth_grid<64, true>, 64) : go(k_smooth_grid<64, false>, 64);
  if (nt == 128) return lds_res ? go(k_smooth_grid<128, true>, 128) : go(k_smooth_grid<128, false>, 128);
  if (nt == 256) return lds_res ? go(k_smooth_grid<256, true>, 256) : go(k_smooth_grid<256, false>, 256);
  return hipErrorInvalidValue;
}

}  // namespace mrcm
