// FP32 solves with FP64 iterative refinement on the wavefront-per-half 2-D
// layout, shared by the FP32 local kernels (local_wave32.hip) and the FP32
// form of the adjoint (adjoint.hip): LDS carve-up of a box with its diagonal
// scaling, the FP32 block-tridiagonal factor of the scaled matrix
// A^ = D^-1/2 A D^-1/2 as explicit block inverses, its sweeps, and the
// refinement loop
//     x = 0;  repeat  r = b - A x (FP64);  x += D^-1/2 solve32(D^-1/2 r)
// until the componentwise backward error max_c |r_c| / (|A| |x| + |b|)_c
// is at most tol.
//
// The factor is two-ended, as the FP64 one: forward inverses W_j of the
// blocks below the meeting block m = nblk / 2, backward inverses above it,
// Z_m at m, all in one array (nblk blocks, nb x nb row-major).  A solve runs
// its halves on two waves, each holding the inverses of its half in
// registers across all refinement sweeps where they fit (Rows32), and the
// residuals and updates run on all threads of the box.
#pragma once
#include <type_traits>

#include "wave_common.h"

namespace mrcm {
namespace wave {

using WaveSmemF = InvSmem<float>;

// LDS of one box for the refinement kernels.
struct BoxR {
  BoxLds b;     // Kt, Dg, Tx, Tn (FP64); b.X = solution x (nrhs x ncell)
  double* sd;   // ncell, 1 / sqrt(diag)
  double* Bv;   // nb_rhs x ncell right-hand sides (not stored for seeds)
  float* Wf;    // nrhs x ncell FP32 work vectors
  float* Txf;   // ncell scaled x couplings
  float* Tnf;   // ncell scaled block couplings
  double* red;  // the reductions' scratch (one value per wave), then T^R of
                // the box-side faces where a kernel tables them (kSeedTable)
};

__host__ __device__ inline size_t boxr_bytes(int m0, int m1, int nrhs, int nbrhs, int kc = 1) {
  const size_t nc = (size_t)m0 * m1;
  const size_t d = kx_doubles(kc, m0, m1) + (size_t)(m0 + 2) * (m1 + 2) + 3 * nc + nrhs * nc + nc + nbrhs * nc;
  const size_t f = nrhs * nc + 2 * nc + (size_t)(nrhs < 2 ? 2 : nrhs) * NBW + 4;
  return d * sizeof(double) + f * sizeof(float);
}

__device__ __forceinline__ BoxR carve_r(double* base, const Box& B, int nrhs, int nbrhs, int kc = 1) {
  BoxR r;
  r.b.m0 = B.hi[0] - B.lo[0];
  r.b.m1 = B.hi[1] - B.lo[1];
  const int nc = r.b.m0 * r.b.m1;
  base = attach_kx(r.b, base, kc);
  r.b.Kt = base;
  attach_ky(r.b);
  r.b.Dg = r.b.Kt + (r.b.m0 + 2) * (r.b.m1 + 2);
  r.b.Tx = r.b.Dg + nc;
  r.b.Tn = r.b.Tx + nc;
  r.b.X = r.b.Tn + nc;
  r.sd = r.b.X + (size_t)nrhs * nc;
  r.Bv = r.sd + nc;
  r.b.Z = nullptr;
  float* fb = reinterpret_cast<float*>(r.Bv + (size_t)nbrhs * nc);
  r.Wf = fb;
  r.Txf = r.Wf + (size_t)nrhs * nc;
  r.Tnf = r.Txf + nc;
  r.red = reinterpret_cast<double*>(align16(base, r.Tnf + nc));
  return r;
}

// Scale factors and scaled couplings (after load_box).
template <int NT = 64>
__device__ __forceinline__ void scale_box(const Box& B, BoxR& R) {
  const int nc = B.ncell, nb = B.nb;
  const int tid = threadIdx.x % NT;
#pragma unroll 1
  for (int e = tid; e < nc; e += NT) R.sd[e] = rcp_d(sqrt(R.b.Dg[e]));
  bsync<NT>();
#pragma unroll 1
  for (int e = tid; e < nc; e += NT) {
    const int xl = e % R.b.m0;
    R.Txf[e] = (xl + 1 < R.b.m0) ? (float)(R.b.Tx[e] * R.sd[e] * R.sd[e + 1]) : 0.0f;
    R.Tnf[e] = (e + nb < nc) ? (float)(R.b.Tn[e] * R.sd[e] * R.sd[e + nb]) : 0.0f;
  }
  bsync<NT>();
}

// Scaled Schur complement of block j, see wbuild_t.
__device__ __forceinline__ void wbuild32(int nb, int j, int tpi, const BoxR& R, float w[HB]) {
  schur_block<float>(nb, nullptr, R.Txf + j * nb, R.Tnf + max(tpi, 0) * nb, tpi >= 0, w);
}

// Entries outside the block get an offset out of the buffer's range: dropped.
__device__ __forceinline__ void store32(int nb, float* Wj, const float w[HB]) {
  const int L = lane_id(), c = L & 31, h = L >> 5;
  const auto rs = uniform_buffer(Wj, nb * nb * (int)sizeof(float));
  const int n = c < nb ? nb - HB * h : 0;  // my rows
  int off = (HB * h * nb + c) * (int)sizeof(float);
#pragma unroll
  for (int i = 0; i < HB; ++i) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(w[i]), rs, i < n ? off : 1 << 28, 0, 0);
    off += nb * (int)sizeof(float);
  }
}

// Two-ended factor of the box by NT threads, the halves on waves 0 and 1;
// the forward Schur complement of
// the meeting block passes through that block's slot of Wg.  sm: one per
// wave that factors.
template <int NT>
__device__ __forceinline__ void factor32(const Box& B, float* Wg, const BoxR& R, WaveSmemF* sm) {
  const int L = lane_id(), wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x % NT) >> 6);
  const int c = L & 31, h = L >> 5;
  const int nb = B.nb, nblk = B.nblk, m = nblk / 2;
  // blocks written by one wave and read by another
  auto handover = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  };
  const long long bs = (long long)nb * nb;
  float w[HB];
#pragma unroll
  for (int i = 0; i < HB; ++i) w[i] = 0.0f;
  static_assert(NT >= 128, "a wave per half");
  constexpr int BW = 1;  // the wave of the bottom half
  if (wv < 2) {
    const bool bot = wv == BW;
    const int cnt = bot ? nblk - 1 - m : m;
#pragma unroll 1
    for (int t = 0; t < cnt; ++t) {
      const int j = bot ? nblk - 1 - t : t;
      wbuild32(nb, j, t > 0 ? (bot ? j : j - 1) : -1, R, w);
      winv(nb, sm[wv], w);
      store32(nb, Wg + j * bs, w);
    }
    if (!bot) {
      wbuild32(nb, m, m - 1, R, w);
      store32(nb, Wg + m * bs, w);
    }
  }
  handover();
  if (wv == BW) {
    // Z_m = (S_m - t_m W'_{m+1} t_m)^{-1}; w holds W'_{m+1} when the bottom
    // half is not empty
    const float* Tm = R.Tnf + m * nb;
    const bool low = m < nblk - 1;
    const float tc = low && c < nb ? Tm[c] : 0.0f;
#pragma unroll
    for (int i = 0; i < HB; ++i) {
      const int r = HB * h + i;
      const bool in = r < nb && c < nb;
      const float smi = in ? Wg[m * bs + r * nb + c] : (r == c ? 1.0f : 0.0f);
      const float tr = low && r < nb ? Tm[r] : 0.0f;
      w[i] = low && in ? fmaf(-tr * tc, w[i], smi) : smi;
    }
    winv(nb, sm[BW], w);
    store32(nb, Wg + m * bs, w);
  }
  handover();  // the sweeps read every block
}

// ------------------------------------------------------------- FP32 sweeps
// Lanes of a block step, as LdsFac: lines in two parts of nh = (nb + 1) / 2
// <= KN entries; lane (g, i) holds row nh (g % 2) + i and the columns of part
// g / 2 of a block, and of a vector entry nh (g / 2) + i.
template <int KN>
struct Lane32 {
  __amdgpu_buffer_rsrc_t rs;
  int off[KN], bbytes;
  int nb, nblk, zi, ci;
  bool zv, cv, zo;
};
template <int KN>
__device__ __forceinline__ Lane32<KN> lane32(const Box& B, const float* Wg) {
  Lane32<KN> f;
  const int nb = B.nb, nh = (nb + 1) / 2, L = lane_id(), i = L & 15, g = L >> 4;
  const int bytes = __builtin_amdgcn_readfirstlane(B.nblk * nb * nb * (int)sizeof(float));
  f.rs = uniform_buffer(Wg, bytes);
  f.bbytes = __builtin_amdgcn_readfirstlane(nb * nb * (int)sizeof(float));
  f.nb = nb;
  f.nblk = B.nblk;
  const int rr = nh * (g & 1) + i, zz = nh * (g >> 1) + i;
  const bool in = i < nh;
  f.cv = in && rr < nb && g < 2;
  f.zv = in && zz < nb;
  f.zo = f.zv && !(g & 1);
  f.ci = min(rr, nb - 1);
  f.zi = min(zz, nb - 1);
#pragma unroll
  for (int k = 0; k < KN; ++k) {
    // by symmetry the column of the lane's row: consecutive lanes read
    // consecutive entries; an offset out of range reads zero
    const int r = nh * (g >> 1) + k;
    f.off[k] = (k < nh && r < nb && in && rr < nb) ? (r * nb + rr) * (int)sizeof(float) : bytes;
  }
  return f;
}
template <int KN>
__device__ __forceinline__ void load32(const Lane32<KN>& f, int j, float w[KN]) {
#pragma unroll
  for (int k = 0; k < KN; ++k)
    w[k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
        f.rs, f.off[k], __builtin_amdgcn_readfirstlane(j * f.bbytes), 0));
}

// y of the lane's row (wgemv_rows in FP32 over KN columns)
template <int KN>
__device__ __forceinline__ float gemv32(const float w[KN], float z) {
  float a0 = 0.0f, a1 = 0.0f;
#define MRCM_P(I0, K0, I1, K1)                                                                     \
  "v_fmac_f32_dpp %0, %2, %" #I0 " row_newbcast:" #K0 " row_mask:0xf bank_mask:0xf\n\t"            \
  "v_fmac_f32_dpp %1, %2, %" #I1 " row_newbcast:" #K1 " row_mask:0xf bank_mask:0xf\n\t"
#define MRCM_S12                                                                                   \
  "s_nop 1\n\t" MRCM_P(3, 0, 4, 1) MRCM_P(5, 2, 6, 3) MRCM_P(7, 4, 8, 5) MRCM_P(9, 6, 10, 7)       \
      MRCM_P(11, 8, 12, 9) MRCM_P(13, 10, 14, 11)
#define MRCM_S16 MRCM_S12 MRCM_P(15, 12, 16, 13) MRCM_P(17, 14, 18, 15)
#define MRCM_W12                                                                                   \
  "v"(z), "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]), "v"(w[4]), "v"(w[5]), "v"(w[6]), "v"(w[7]),    \
      "v"(w[8]), "v"(w[9]), "v"(w[10]), "v"(w[11])
  static_assert(KN == 12 || KN == 16, "products per block step");
  if constexpr (KN == 12) asm(MRCM_S12 : "+v"(a0), "+v"(a1) : MRCM_W12);
  if constexpr (KN == 16)
    asm(MRCM_S16 : "+v"(a0), "+v"(a1) : MRCM_W12, "v"(w[12]), "v"(w[13]), "v"(w[14]), "v"(w[15]));
#undef MRCM_P
#undef MRCM_S12
#undef MRCM_S16
#undef MRCM_W12
  return half_sum_f(a0 + a1);
}
__device__ __forceinline__ float to_rows_f(float y) {
  const int u = __float_as_int(y);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return __int_as_float(lane_id() >= 32 ? a[1] : a[0]);
}

// The inverses of one half of a box in registers (block b away from its end
// of the box in w[b], b < NBK) and, on the top half, Z_m; NBK = 0: none held,
// blocks are loaded as the sweeps reach them.
template <int KN, int NBK>
struct Rows32 {
  float w[NBK > 0 ? NBK : 1][KN], zm[KN];
};
template <int KN, int NBK>
__device__ __forceinline__ void rows32(const Lane32<KN>& f, bool bottom, Rows32<KN, NBK>& r) {
  const int m = f.nblk / 2, cnt = bottom ? f.nblk - 1 - m : m;
#pragma unroll
  for (int b = 0; b < NBK; ++b)
    if (b < cnt) load32(f, bottom ? f.nblk - 1 - b : b, r.w[b]);
  if (NBK > 0 && !bottom) load32(f, m, r.zm);
}

// Forward and back halves of the two-ended sweep of NR vectors (X + q nc).
template <int KN, int NBK, int NR>
__device__ __forceinline__ void fwd32(const Lane32<KN>& f, const Rows32<KN, NBK>& rw, const float* Tn,
                                      float* X, int nc, bool bottom) {
  const int nb = f.nb, m = f.nblk / 2, cnt = bottom ? f.nblk - 1 - m : m;
  const int dj = bottom ? -1 : 1, j0 = bottom ? f.nblk - 1 : 0;
  float yz[NR], tp = 0.0f;
#pragma unroll
  for (int q = 0; q < NR; ++q) yz[q] = 0.0f;
  const int dt = bottom ? -nb : 0, dc = f.ci - f.zi;
  // my entry of the step's block (kept as one running index: the addresses
  // of all steps, hoisted out of the refinement loop, would take the
  // registers of the inverses)
  int e = j0 * nb + f.zi;
  float xv[NR];            // and its value, read a step ahead
#pragma unroll
  for (int q = 0; q < NR; ++q) xv[q] = X[q * nc + e];
  auto step = [&](const float* w) {
    keep_here(e);
    float z[NR], y[NR];
#pragma unroll
    for (int q = 0; q < NR; ++q) z[q] = f.zv ? fmaf(tp, yz[q], xv[q]) : 0.0f;
    tp = Tn[max(e + dt, 0)];
    // the half's last step reads the meeting block, which is in range
#pragma unroll
    for (int q = 0; q < NR; ++q) xv[q] = X[q * nc + e + dj * nb];
#pragma unroll
    for (int q = 0; q < NR; ++q) y[q] = gemv32<KN>(w, z[q]);
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      yz[q] = to_rows_f(y[q]);
      if (f.cv) X[q * nc + e + dc] = y[q];
    }
    e += dj * nb;
  };
  if constexpr (NBK > 0) {
#pragma unroll
    for (int t = 0; t < NBK; ++t)
      if (t < cnt) step(rw.w[t]);
  } else {
    float wa[KN], wb[KN];
    if (cnt > 0) load32(f, j0, wa);
    for (int t = 0; t < cnt; t += 2) {
      load32(f, j0 + dj * min(t + 1, cnt - 1), wb);
      step(wa);
      if (t + 1 < cnt) {
        load32(f, j0 + dj * min(t + 2, cnt - 1), wa);
        step(wb);
      }
    }
  }
}

template <int KN, int NBK, int NR>
__device__ __forceinline__ void mid32(const Lane32<KN>& f, const Rows32<KN, NBK>& rw, const float* Tn,
                                      float* X, int nc) {
  const int nb = f.nb, m = f.nblk / 2;
  int em = m * nb + f.zi;
  keep_here(em);
  float zl[KN];
  if constexpr (NBK == 0) load32(f, m, zl);
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    const float* Xq = X + q * nc;
    float v = Xq[em];
    if (m > 0) v = fmaf(Tn[em - nb], Xq[em - nb], v);
    if (m + 1 < f.nblk) v = fmaf(Tn[em], Xq[em + nb], v);
    const float y = gemv32<KN>(NBK > 0 ? rw.zm : zl, f.zv ? v : 0.0f);
    if (f.cv) X[q * nc + em - f.zi + f.ci] = y;
  }
}

template <int KN, int NBK, int NR>
__device__ __forceinline__ void bwd32(const Lane32<KN>& f, const Rows32<KN, NBK>& rw, const float* Tn,
                                      float* X, int nc, bool bottom) {
  const int nb = f.nb, m = f.nblk / 2, cnt = bottom ? f.nblk - 1 - m : m;
  const int dj = bottom ? -1 : 1, j0 = bottom ? f.nblk - 1 : 0;
  float xn[NR];
#pragma unroll
  for (int q = 0; q < NR; ++q) xn[q] = f.zv ? X[q * nc + m * nb + f.zi] : 0.0f;
  // from the block beside the meeting one outwards
  int e = (j0 + dj * (cnt - 1)) * nb + f.zi;
  const int dt = bottom ? -nb : 0, nlast = (f.nblk - 1) * nb + f.zi;
  float xv[NR], tv = 0.0f;  // the step's entries, read a step ahead
  if (cnt > 0) tv = Tn[e + dt];
#pragma unroll
  for (int q = 0; q < NR; ++q) xv[q] = cnt > 0 ? X[q * nc + e] : 0.0f;
  auto step = [&](const float* w) {
    keep_here(e);
    const float t = f.zv ? tv : 0.0f;
    float y[NR], xc[NR];
    const int en = min(max(e - dj * nb, f.zi), nlast);  // clamped after the last step
    tv = Tn[max(en + dt, 0)];
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      xc[q] = xv[q];
      xv[q] = X[q * nc + en];
    }
#pragma unroll
    for (int q = 0; q < NR; ++q) y[q] = gemv32<KN>(w, t * xn[q]);
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      xn[q] = xc[q] + to_rows_f(y[q]);
      xn[q] = f.zv ? xn[q] : 0.0f;
      if (f.zo) X[q * nc + e] = xn[q];
    }
    e -= dj * nb;
  };
  if constexpr (NBK > 0) {
#pragma unroll
    for (int b = NBK - 1; b >= 0; --b)
      if (b < cnt) step(rw.w[b]);
  } else {
    float wa[KN], wb[KN];
    if (cnt > 0) load32(f, j0 + dj * (cnt - 1), wa);
    for (int b = cnt - 1; b >= 0; b -= 2) {
      load32(f, j0 + dj * max(b - 1, 0), wb);
      step(wa);
      if (b > 0) {
        load32(f, j0 + dj * max(b - 2, 0), wa);
        step(wb);
      }
    }
  }
}

// FP32 solve of the scaled system on the nrhs work vectors in R.Wf by the NT
// threads of a box: the halves of a vector on the two waves of a pair (one
// after the other when NT = 64), the vectors NR at a time dealt to the
// pairs.  Ends with a barrier of the box.
template <int NT, int KN, int NBK, int NR>
__device__ __forceinline__ void solve32(const Lane32<KN>& f, const Rows32<KN, NBK>& rw, int nc, int nrhs,
                                        const BoxR& R) {
  constexpr int NP = NT >= 128 ? NT / 128 : 1;  // pairs
  static_assert(NBK == 0 || NT >= 128, "one wave cannot hold both halves");
  const int wv = (int)(threadIdx.x % NT) >> 6;
  const int pair = NT >= 128 ? wv >> 1 : 0;
  const bool top = NT < 128 || !(wv & 1), bot = NT < 128 || (wv & 1);
  const float* Tn = R.Tnf;
  // vectors [k0, k0 + NR) of this pair, the last group one by one
  auto each = [&](auto&& go) {
    int k = pair * NR;
    for (; k + NR <= nrhs; k += NP * NR) go(k, std::integral_constant<int, NR>());
    const int end = min(nrhs, k + NR);
    for (; NR > 2 && k + 2 <= end; k += 2) go(k, std::integral_constant<int, 2>());
    for (; k < end; ++k) go(k, std::integral_constant<int, 1>());
  };
  each([&](int k, auto n) {
    constexpr int N = decltype(n)::value;
    if (top) fwd32<KN, NBK, N>(f, rw, Tn, R.Wf + (size_t)k * nc, nc, false);
    if (bot) fwd32<KN, NBK, N>(f, rw, Tn, R.Wf + (size_t)k * nc, nc, true);
  });
  bsync<NT>();
  if (top)
    each([&](int k, auto n) {
      mid32<KN, NBK, decltype(n)::value>(f, rw, Tn, R.Wf + (size_t)k * nc, nc);
    });
  bsync<NT>();
  each([&](int k, auto n) {
    constexpr int N = decltype(n)::value;
    if (top) bwd32<KN, NBK, N>(f, rw, Tn, R.Wf + (size_t)k * nc, nc, false);
    if (bot) bwd32<KN, NBK, N>(f, rw, Tn, R.Wf + (size_t)k * nc, nc, true);
  });
  bsync<NT>();
}

template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}

// Maximum over the wave of non-negative values: quad and row steps by DPP,
// then the row pairs and the half-waves by lane swaps (no LDS).
__device__ __forceinline__ double wave_max(double v) {
  v = fmax(v, dpp_d<0xB1>(v));   // quad_perm(1,0,3,2)
  v = fmax(v, dpp_d<0x4E>(v));   // quad_perm(2,3,0,1)
  v = fmax(v, dpp_d<0x124>(v));  // row_ror:4
  v = fmax(v, dpp_d<0x128>(v));  // row_ror:8
  {
    const int lo = __double2loint(v), hi = __double2hiint(v);
    const auto l2 = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h2 = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    v = fmax(__hiloint2double(h2[0], l2[0]), __hiloint2double(h2[1], l2[1]));
  }
  {
    const int lo = __double2loint(v), hi = __double2hiint(v);
    const auto l2 = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h2 = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    v = fmax(__hiloint2double(h2[0], l2[0]), __hiloint2double(h2[1], l2[1]));
  }
  return v;
}

// The largest v over the NT threads of the box (red: NT / 64 doubles of LDS);
// a barrier of the box as well.
template <int NT>
__device__ __forceinline__ double box_max(double v, double* red) {
  v = wave_max(v);
  if constexpr (NT == 64) {
    bsync<NT>();
    return v;
  }
  if (lane_id() == 0) red[(int)(threadIdx.x % NT) >> 6] = v;
  bsync<NT>();
#pragma unroll
  for (int u = 0; u < NT / 64; ++u) v = fmax(v, red[u]);
  bsync<NT>();
  return v;
}

// T^R of box-side face u (side_off order), zero on the domain's boundary.
__device__ __forceinline__ double seed_face(const Geo& g, const Box& B, const BoxR& R, double beta, int u) {
  int t, x, y, ox, oy;
  const int q = face_side(R.b.m0, R.b.m1, u, t), a = q >> 1;
  face_cells(B.lo[0], B.lo[1], B.hi[0], B.hi[1], q, t, x, y, ox, oy);
  if (off_domain(g, a, a == 0 ? x : y, a == 0 ? ox : oy)) return 0.0;
  // the tile by value: a select between fields of R is one of addresses, and
  // R then lives in scratch memory
  const double *kx = R.b.Kt, *ky = R.b.Ky, *K = a == 0 ? kx : ky;
  const double kc = K[tile_at(R.b, B, x, y)];
  return robin_T(g, kc, robin_beta(g, a, kc, K[tile_at(R.b, B, ox, oy)], beta));
}
// The faces' T^R tabled in R.red + NT / 64 by kernels whose boxes have at
// most 33 lines (LDS reserved by the host: kSeedTable bytes); longer boxes
// compute it where it is needed, their table would grow with the box.
constexpr int kSeedTable = (2 * (32 + 33) + 4) * (int)sizeof(double);
template <int NT>
__device__ __forceinline__ void seed_faces(const Geo& g, const Box& B, const BoxR& R, double beta) {
#pragma unroll 1
  for (int u = threadIdx.x % NT; u < 2 * (R.b.m0 + R.b.m1); u += NT)
    R.red[NT / 64 + u] = seed_face(g, B, R, beta, u);
}
// Right-hand side of a seed at box cell (xl, yl): T^R times the seed on its
// side (TRs: the table, or null).
__device__ __forceinline__ double seed_rhs(const Geo& g, const Box& B, const BoxR& R, const Seed& sd,
                                           const double* TRs, double beta, int xl, int yl) {
  const int a = sd.side >> 1, so = sd.side & 1;
  const bool on = a == 0 ? xl == (so ? R.b.m0 - 1 : 0) : yl == (so ? R.b.m1 - 1 : 0);
  if (!on) return 0.0;
  const int c[3] = {B.lo[0] + xl, B.lo[1] + yl, 0};
  const int u = side_off(R.b, sd.side) + (a == 0 ? yl : xl);
  return (TRs ? TRs[u] : seed_face(g, B, R, beta, u)) * seed_value(g, sd, B.lo, B.hi, c);
}

// Iterative refinement of nrhs systems A x_k = b_k by the NT threads of a
// box; b from seeds (SEEDS; TAB: after seed_faces) or from R.Bv (nrhs x
// ncell).  Returns the number of FP32 solves.
template <int NT, int KN, int NBK, int NR, bool SEEDS = false, bool TAB = (NBK > 0)>
__device__ __forceinline__ int refine(const Geo& g, const Box& B, const BoxR& R, const Lane32<KN>& f,
                                      const Rows32<KN, NBK>& rw, int nrhs, const Seed* seeds,
                                      double beta, double tol, int max_refine, double& omega_out,
                                      int& flag) {
  const int tid = threadIdx.x % NT;
  const int nc = B.ncell, m0 = R.b.m0, nb = B.nb;
#pragma unroll 1
  for (int e = tid; e < nrhs * nc; e += NT) R.b.X[e] = 0.0;
  bsync<NT>();
  int it = 0;
  double omega = 0.0;
  while (true) {
    // r = b - A x, scaled into the FP32 work vectors; componentwise backward
    // error.  A cell's couplings are read once for all vectors.
    double om = 0.0;
#pragma unroll 1
    for (int loc = tid; loc < nc; loc += NT) {
      const int yl = loc / m0, xl = loc - yl * m0;
      const double dg = R.b.Dg[loc], sc = R.sd[loc];
      const double txm = xl > 0 ? R.b.Tx[loc - 1] : 0.0, txp = xl + 1 < m0 ? R.b.Tx[loc] : 0.0;
      const double tnm = loc >= nb ? R.b.Tn[loc - nb] : 0.0, tnp = loc + nb < nc ? R.b.Tn[loc] : 0.0;
      const int im = xl > 0 ? loc - 1 : loc, ip = xl + 1 < m0 ? loc + 1 : loc;
      const int jm = loc >= nb ? loc - nb : loc, jp = loc + nb < nc ? loc + nb : loc;
#pragma unroll 1
      for (int k = 0; k < nrhs; ++k) {
        const double* x = R.b.X + (size_t)k * nc;
        const double bv = SEEDS ? seed_rhs(g, B, R, seeds[B.seed0 + k], TAB ? R.red + NT / 64 : nullptr, beta, xl, yl)
                                : R.Bv[(size_t)k * nc + loc];
        const double d = dg * x[loc];
        const double t0 = txm * x[im], t1 = txp * x[ip], t2 = tnm * x[jm], t3 = tnp * x[jp];
        const double ax = (((d - t0) - t1) - t2) - t3;
        const double aa = (((fabs(d) + fabs(t0)) + fabs(t1)) + fabs(t2)) + fabs(t3);
        const double r = bv - ax;
        const double den = aa + fabs(bv);
        // a non-finite residual or iterate never counts as converged (fmax
        // would drop a NaN ratio)
        if (!(r - r == 0.0 && den - den == 0.0)) om = INFINITY;
        else if (den > 0.0) om = fmax(om, fabs(r) / den);
        R.Wf[(size_t)k * nc + loc] = (float)(sc * r);
      }
    }
    omega = box_max<NT>(om, R.red);
    if (it > 0 && omega <= tol) break;
    if (it > max_refine || !(omega <= 1e300)) {
      if (tid == 0) flag |= kFlagNoConv;
      break;
    }
    solve32<NT, KN, NBK, NR>(f, rw, nc, nrhs, R);
#pragma unroll 1
    for (int loc = tid; loc < nc; loc += NT) {
      const double sc = R.sd[loc];
      for (int k = 0; k < nrhs; ++k) R.b.X[(size_t)k * nc + loc] += sc * (double)R.Wf[(size_t)k * nc + loc];
    }
    bsync<NT>();
    ++it;
  }
  omega_out = omega;
  return it;
}

__device__ __forceinline__ void record_refine(int it, double omega, int* iters,
                                              unsigned long long* resid) {
  if (lane_id() == 0) {
    atomicMax(iters, it);
    atomicMax(resid, (unsigned long long)__double_as_longlong(omega));
  }
}

// The refinement arrays of a smoothing box, after its carve_smooth layout
// (smooth32_lds_bytes in all).
__device__ __forceinline__ BoxR carve_smooth_r(double* base, const SmoothLds& r) {
  const int nc = r.b.m0 * r.b.m1;
  BoxR R;
  R.b = r.b;
  R.sd = r.b.Z + 2 * NBW;
  R.Bv = R.sd + nc;
  float* fb = reinterpret_cast<float*>(R.Bv + nc);
  R.Wf = fb;
  R.Txf = R.Wf + nc;
  R.Tnf = R.Txf + nc;
  R.red = reinterpret_cast<double*>(align16(base, R.Tnf + nc));
  return R;
}

__host__ __device__ inline size_t smooth32_lds_bytes(int m0, int m1, int kc = 1) {
  const size_t nc = (size_t)m0 * m1;
  return sizeof(double) * (smooth_lds_doubles(m0, m1, kc) + 2 * nc) + sizeof(float) * (3 * nc + 2 * NBW + 4);
}

}  // namespace wave
}  // namespace mrcm
