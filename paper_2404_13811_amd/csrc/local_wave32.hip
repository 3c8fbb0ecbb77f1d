// FP32 local factorisations and solves with FP64 iterative refinement, for
// the 2-D boxes of lines of at most 32 cells.
//
// The block-tridiagonal factorisation of local_wave.hip is applied in FP32
// to the symmetrically scaled matrix  A^ = D^-1/2 A D^-1/2  (D = diag A,
// which removes the permeability contrast from the diagonal), and stored
// as FP32 block inverses (half the bytes of the FP64 form).  Every local
// solve is then refined in FP64:
//     x = 0;  repeat  r = b - A x (FP64, two-point stencil from K in LDS);
//                     x += D^-1/2 solve32(D^-1/2 r)
// until the componentwise backward error
//     max_c |r_c| / (|A| |x| + |b|)_c  <=  tol
// or max_refine corrections have been applied (flag MRCM_ENOCONV).  The
// interface system and every reduction stay in FP64.
//
// A box is solved by four waves (Steps 1-2, 4; two where many boxes wait,
// see two_waves32), two (Step 6) or one to four (smoothing):
// the factor and every sweep from both ends on a pair of waves, residuals
// and updates on all threads.  The kernels come in classes by the largest
// box (wave32_form): <KN, NBK> with KN products per block step (half a line)
// and the inverses of up to NBK blocks per half held in registers over all
// refinement sweeps.
// Bound: Steps 1-2 the block inversions, 13 of them in a chain at 24 lines
// (a third of a box's time) and the FP64 residuals (a quarter); smoothing the
// chain of 2 (nblk + 1) / 2 block steps of about 270 cycles per FP32 solve.
// Measured against one wave per box eliminated from one end (24 x 24 cells,
// three FP32 solves): Steps 1-2 and 4 of 256 boxes with eight seeds 690 ->
// 164 us, of 4096 with four 3776 -> 1182 us; smoothing per phase 65 -> 28 us
// (64 boxes), 140 -> 66 us (1024 boxes).
#include "wave32_common.h"

#include <algorithm>

namespace mrcm {
namespace {

using namespace wave;

// ------------------------------------------------------------------ kernels

// Steps 1-2 on an oversampled box by NT threads: FP32 factor, seeds refined
// to tol (TAB: the seeds' T^R from a table, see kSeedTable).
template <int NT, int KN, int NBK, bool TAB>
__device__ __forceinline__ void basis32_box(const Geo& g, const Box& B, const Seed* __restrict__ seeds,
                                            const double* __restrict__ K, double beta,
                                            float* __restrict__ fac32, double* __restrict__ Pk,
                                            double* __restrict__ tr_u, double* __restrict__ tr_phi,
                                            double* __restrict__ tr_beta, double tol, int max_refine,
                                            int* iters, unsigned long long* resid, double* dsm,
                                            WaveSmemF* sm) {
  const int L = threadIdx.x;
  const int nrhs = B.nrhs;
  BoxR R = carve_r(dsm, B, max(nrhs, 1), 0, g.kc);
  load_box<NT>(g, B, K, beta, R.b);
  scale_box<NT>(B, R);
  if (TAB && nrhs > 0) seed_faces<NT>(g, B, R, beta);
  float* Wg = fac32 + B.fac;
  factor32<NT>(B, Wg, R, sm);
  double omega = 0.0;
  int it = 0;
  if (nrhs > 0) {
    const Lane32<KN> f = lane32<KN>(B, Wg);
    Rows32<KN, NBK> rw;
    rows32<KN, NBK>(f, (threadIdx.x >> 6) & 1, rw);
    it = refine<NT, KN, NBK, 4, true, TAB>(g, B, R, f, rw, nrhs, seeds, beta, tol, max_refine, omega, sm[0].flag);
  }
  if (L < 64) record_refine(it, omega, iters, resid);
  const BoxLds& s = R.b;
  const int nc = B.ncell;
  int olo[3], ohi[3];
  womega(g, B.sub, olo, ohi);
  const int ncell_o = g.S[0] * g.S[1];
  #pragma unroll 1
  for (int e = L; e < nrhs * ncell_o; e += NT) {
    const int k = e / ncell_o, t = e % ncell_o;
    Pk[(long long)(B.seed0 + k) * ncell_o + t] =
        s.X[k * nc + bloc(B, s, olo[0] + t % g.S[0], olo[1] + t / g.S[0])];
  }
  for (int q = 0; q < 4; ++q) {
    const int nf = (q >> 1) == 0 ? g.S[1] : g.S[0];
    const bool has = wneighbor(g, B.sub, q) >= 0;
    const int a = q >> 1, so = q & 1;
    #pragma unroll 1
    for (int e = L; e < nrhs * nf; e += NT) {
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

// Step 4 on a subdomain: FP32 factor, particular solution refined to tol.
template <int NT, int KN, int NBK>
__device__ __forceinline__ void particular32_box(const Geo& g, const Box& B, const double* __restrict__ K,
                                                 const double* __restrict__ f,
                                                 const double* __restrict__ bcv, double beta,
                                                 float* __restrict__ fac32, double* __restrict__ pbar,
                                                 double* __restrict__ ubar, double* __restrict__ pibar,
                                                 double tol, int max_refine, int* iters,
                                                 unsigned long long* resid, double* dsm,
                                                 WaveSmemF* sm) {
  const int L = threadIdx.x;
  BoxR R = carve_r(dsm, B, 1, 1, g.kc);
  load_box<NT>(g, B, K, beta, R.b);
  scale_box<NT>(B, R);
  physical_rhs<NT>(g, B, R.b, f, bcv, R.Bv);
  bsync<NT>();
  float* Wg = fac32 + B.fac;
  factor32<NT>(B, Wg, R, sm);
  double omega = 0.0;
  const Lane32<KN> fl = lane32<KN>(B, Wg);
  Rows32<KN, NBK> rw;
  rows32<KN, NBK>(fl, (threadIdx.x >> 6) & 1, rw);
  const int it = refine<NT, KN, NBK, 1>(g, B, R, fl, rw, 1, nullptr, beta, tol, max_refine, omega, sm[0].flag);
  if (L < 64) record_refine(it, omega, iters, resid);
  const BoxLds& s = R.b;
  for (int t = L; t < B.ncell; t += NT) pbar[(long long)B.sub * B.ncell + t] = s.X[t];
  for (int q = 0; q < 4; ++q) {
    const int nf = (q >> 1) == 0 ? g.S[1] : g.S[0];
    const bool has = wneighbor(g, B.sub, q) >= 0;
    const int a = q >> 1, so = q & 1;
    #pragma unroll 1
    for (int t = L; t < nf; t += NT) {
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

// Steps 1-2 and 4 in one launch: workgroups [0, nbox) take the oversampled
// boxes, workgroups [nbox, 2 nbox) the particular problems.  The two sets are
// independent and run side by side.
template <int NT, int KN, int NBK, bool TAB>
__global__ void __launch_bounds__(NT, NT == 128 ? 4 : KN == 12 ? 2 : 1) k_local32(Geo g, const Box* __restrict__ obox,
                                                const Box* __restrict__ pbox, int nbox,
                                                const Seed* __restrict__ seeds,
                                                const double* __restrict__ K,
                                                const double* __restrict__ f,
                                                const double* __restrict__ bcv, double beta,
                                                float* __restrict__ fac32,
                                                float* __restrict__ facp32,
                                                double* __restrict__ Pk,
                                                double* __restrict__ tr_u,
                                                double* __restrict__ tr_phi,
                                                double* __restrict__ tr_beta,
                                                double* __restrict__ pbar,
                                                double* __restrict__ ubar,
                                                double* __restrict__ pibar, double tol,
                                                int max_refine, int* iters,
                                                unsigned long long* resid, int* flags) {
  extern __shared__ __align__(16) double dsm[];
  __shared__ WaveSmemF sm[2];
  if (threadIdx.x < 2) sm[threadIdx.x].flag = 0;
  __syncthreads();
  const int b = blockIdx.x;
  if (b < nbox) {
    const Box B = obox[b];
    basis32_box<NT, KN, NBK, TAB>(g, B, seeds, K, beta, fac32, Pk, tr_u, tr_phi, tr_beta, tol, max_refine, iters,
                resid, dsm, sm);
  } else {
    const Box B = pbox[b - nbox];
    particular32_box<NT, KN, NBK>(g, B, K, f, bcv, beta, facp32, pbar, ubar, pibar, tol, max_refine, iters,
                     resid, dsm, sm);
  }
  __syncthreads();
  if (threadIdx.x == 0 && (sm[0].flag | sm[1].flag)) atomicOr(flags, sm[0].flag | sm[1].flag);
}

// Algorithm 1, Step 6 in the FP32 form: the oversampled boxes factored
// again (FP32, diagonally scaled) with the smoothing Robin parameter; no
// right-hand side is solved, so a wave per half is all it takes.
constexpr int kFactor32NT = 128;
__global__ void __launch_bounds__(kFactor32NT) k_factor32(Geo g, const Box* __restrict__ obox,
                                                 const double* __restrict__ K, double beta,
                                                 float* __restrict__ fac32, int* iters,
                                                 unsigned long long* resid, int* flags) {
  extern __shared__ __align__(16) double dsm[];
  __shared__ WaveSmemF sm[2];
  if (threadIdx.x < 2) sm[threadIdx.x].flag = 0;
  __syncthreads();
  Box B = obox[blockIdx.x];
  B.nrhs = 0;
  basis32_box<kFactor32NT, 16, 0, false>(g, B, nullptr, K, beta, fac32, nullptr, nullptr, nullptr, nullptr, 1.0, 0, iters,
              resid, dsm, sm);
  __syncthreads();
  if (threadIdx.x == 0 && (sm[0].flag | sm[1].flag)) atomicOr(flags, sm[0].flag | sm[1].flag);
}

template <int NT, int KN, int NBK>
__global__ void __launch_bounds__(NT) k_smooth32(Geo g, const Box* __restrict__ boxes,
                                                 const double* __restrict__ K,
                                                 const double* __restrict__ f,
                                                 const double* __restrict__ bcv, double beta,
                                                 const float* __restrict__ fac32,
                                                 double* __restrict__ p,
                                                 double* __restrict__ gflux, double tol,
                                                 int max_refine, int* iters,
                                                 unsigned long long* resid, int* flags) {
  extern __shared__ __align__(16) double dsm[];
  __shared__ int flag;
  const Box B = boxes[blockIdx.x];
  if (threadIdx.x == 0) flag = 0;
  // the inverses of this wave's half, in flight during the set-up
  const Lane32<KN> fl = lane32<KN>(B, fac32 + B.fac);
  Rows32<KN, NBK> rw;
  if (NBK > 0 && threadIdx.x < 128) rows32<KN, NBK>(fl, (threadIdx.x >> 6) & 1, rw);
  SmoothLds r = carve_smooth(dsm, B, g.kc);
  BoxR R = carve_smooth_r(dsm, r);
  stage_smooth<NT>(g, B, r, K, p, f, gflux, bcv, nullptr);
  __syncthreads();
  smooth_rhs<NT>(g, B, r, beta, R.Bv);
  coef_box<NT>(g, B, beta, R.b);
  scale_box<NT>(B, R);
  double omega = 0.0;
  const int it = refine<NT, KN, NBK, 1>(g, B, R, fl, rw, 1, nullptr, beta, tol, max_refine, omega, flag);
  if (threadIdx.x < 64) record_refine(it, omega, iters, resid);
  __syncthreads();
  smooth_out<NT>(g, B, r, R.b.X, beta, p, gflux);
  if (threadIdx.x == 0 && flag) atomicOr(flags, flag);
}

template <typename KF>
hipError_t set_lds(KF kern, size_t bytes) {
  if (bytes > 64 * 1024)
    return hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)bytes);
  return hipSuccess;
}

}  // namespace

size_t wave32_lds_bytes(int m0, int m1, int nrhs, int nbrhs, int kc) {
  return boxr_bytes(m0, m1, nrhs, nbrhs, kc);
}

// Registers draw the lines: <12, 12> keeps 156 entries of inverses per lane
// and fits two waves per SIMD (12 x 12 exactly covers lines of 24 cells and
// 25 blocks), <16, 16> keeps 272 of the 512 that one wave can have; longer
// boxes stream their blocks.  Where the inverses fit, holding them is the
// faster: a 256 x 256 solve of 256 boxes 1.10 ms, 1.29 ms streamed.
int wave32_form(int nb, int nblk) { return nblk > 33 ? 2 : nb <= 24 && nblk <= 25 ? 0 : 1; }

size_t wave32_smooth_lds_bytes(int m0, int m1, int kc) { return smooth32_lds_bytes(m0, m1, kc); }

// Steps 1-2 and 4 by two waves per box that stream the inverses (128
// registers, up to eight boxes per CU) instead of four that hold them (form
// 0: two boxes per CU, form 1: one)?  A box alone takes 1.15 times as long
// with up to four seeds, 1.5 times with more (they go four at a time to a
// pair of waves), so two waves pay where enough boxes wait and LDS lets more
// of them share a CU.  Measured, four waves against two, all of Steps 1-2
// and 4: 4096 boxes of 6 x 6 cells and four seeds 410 and 162 us, 14 x 14
// 617 and 322 us, 20 x 20 991 and 811 us, 24 x 24 1395 and 1585 us; 1024
// boxes of 10 x 10 with eight seeds 180 and 124 us, 16 x 16 234 and 258 us;
// 256 boxes of 14 x 14 with four seeds 61 and 67 us.
static bool two_waves32(int form, int nbox, int nrhs, size_t lds, int ncu) {
  const size_t box = lds + 2 * sizeof(WaveSmemF);
  const double fit = std::max<double>(1.0, (double)(size_t)(160 * 1024 / box));
  auto rounds = [&](double per_cu) { return std::max(1.0, nbox / (std::min(per_cu, fit) * ncu)); };
  return rounds(8.0) * (nrhs <= 4 ? 1.15 : 1.5) < rounds(form == 0 ? 2.0 : 1.0);
}

hipError_t launch_local32_w(const Geo& g, const Box* obox, const Box* pbox, int nbox,
                            const Seed* seeds, const double* K, const double* f, const double* bcv,
                            double beta, float* fac32, float* facp32, double* Pk, double* tr_u,
                            double* tr_phi, double* tr_beta, double* pbar, double* ubar,
                            double* pibar, double tol, int max_refine, int* iters,
                            unsigned long long* resid, int* flags, int form, int nrhs, size_t lds,
                            hipStream_t s) {
  if (nbox <= 0) return hipSuccess;
  if (form < 2) lds += kSeedTable;
  int dev = 0, ncu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  auto go = [&](auto kern, int nt) -> hipError_t {
    const hipError_t er = set_lds(kern, lds);
    if (er != hipSuccess) return er;
    hipLaunchKernelGGL(kern, dim3(2 * nbox), dim3(nt), lds, s, g, obox, pbox, nbox, seeds, K, f, bcv,
                       beta, fac32, facp32, Pk, tr_u, tr_phi, tr_beta, pbar, ubar, pibar, tol, max_refine,
                       iters, resid, flags);
    return hipGetLastError();
  };
  if (form == 2) return go(k_local32<256, 16, 0, false>, 256);
  if (two_waves32(form, nbox, nrhs, lds, ncu)) return go(k_local32<128, 16, 0, true>, 128);
  return form == 0 ? go(k_local32<256, 12, 12, true>, 256) : go(k_local32<256, 16, 16, true>, 256);
}

hipError_t launch_factor32_w(const Geo& g, const Box* obox, int nbox, const double* K, double beta,
                             float* fac32, int* iters, unsigned long long* resid, int* flags,
                             size_t lds, hipStream_t s) {
  if (nbox <= 0) return hipSuccess;
  hipError_t e = set_lds(k_factor32, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_factor32, dim3(nbox), dim3(kFactor32NT), lds, s, g, obox, K, beta, fac32, iters,
                     resid, flags);
  return hipGetLastError();
}

hipError_t launch_smooth32_w(const Geo& g, const Box* boxes, int nmem,
                             const double* K, const double* f, const double* bcv, double beta,
                             const float* fac32, double* p, double* gflux, double tol,
                             int max_refine, int* iters, unsigned long long* resid, int* flags,
                             int form, size_t lds, int nt, hipStream_t s) {
  if (nmem <= 0) return hipSuccess;
  auto go = [&](auto kern, int N) -> hipError_t {
    const hipError_t e = set_lds(kern, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(nmem), dim3(N), lds, s, g, boxes, K, f, bcv, beta, fac32, p, gflux, tol,
                       max_refine, iters, resid, flags);
    return hipGetLastError();
  };
  // one wave per box holds no inverses in registers (both halves are its own)
  if (nt == 64) return go(k_smooth32<64, 16, 0>, 64);
  if (nt == 128)
    return form == 0 ? go(k_smooth32<128, 12, 12>, 128)
                     : form == 1 ? go(k_smooth32<128, 16, 16>, 128) : go(k_smooth32<128, 16, 0>, 128);
  if (nt == 256)
    return form == 0 ? go(k_smooth32<256, 12, 12>, 256)
                     : form == 1 ? go(k_smooth32<256, 16, 16>, 256) : go(k_smooth32<256, 16, 0>, 256);
  return hipErrorInvalidValue;
}

}  // namespace mrcm
