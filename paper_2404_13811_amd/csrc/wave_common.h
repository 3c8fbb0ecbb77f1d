// Shared pieces of the 2-D local kernels, a wave per half of a box (FP64 and
// FP32-with-refinement forms): LDS layout of a box, coefficient loading,
// the block inverse in the two-half-wave register layout, and
// geometry helpers.  See local_wave.hip for the algorithm.
#pragma once
#include "local_common.h"
#include "gj16.h"

namespace mrcm {
namespace wave {

constexpr int NBW = 32;
constexpr int HB = 16;
constexpr int RING = 4;

// Two tiles of the block inverse (winv) and the kernel's error flags.
template <typename T>
struct InvSmem;
template <>
struct __align__(16) InvSmem<double> {
  using V = dbl4;
  double t[2][kTile];
  int flag;
};
template <>
struct __align__(16) InvSmem<float> {
  using V = flt4;
  float t[2][kTileF];
  int flag;
};
using WaveSmem = InvSmem<double>;

// Dynamic LDS carve-up of one box.
struct BoxLds {
  double* Kt;   // (m0 + 2) x (m1 + 2) permeabilities, one-cell halo
  double* Dg;   // ncell diagonal of A
  double* Tx;   // ncell coupling to the x+1 neighbour (0 at the box edge)
  double* Tn;   // ncell coupling to the next block (y+1)
  double* X;    // nrhs x ncell right-hand sides / solutions
  double* Z;    // nrhs x NBW staging of one block
  int m0, m1;
  // diagonal permeability tensor: the halo tiles of the entries of axes
  // 1.., ktn doubles apart (ktn = 0: scalar K), and the tile axis 1 reads
  // (Kt with scalar K)
  double* Kx;
  int ktn;
  const double* Ky;
};

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

// p rounded up to a 16-byte boundary (for 128-bit LDS accesses), measured
// from a 16-byte aligned base of the same array, so that the pointer keeps
// its address space.
template <typename T, typename B>
__device__ __forceinline__ T* align16(B* base, T* p) {
  constexpr int q = 16 / sizeof(T);
  const char* b = reinterpret_cast<const char*>(base);
  const long long off = (reinterpret_cast<const char*>(p) - b) / (long long)sizeof(T);
  return reinterpret_cast<T*>(const_cast<char*>(b)) + ((off + q - 1) / q) * q;
}

// Single-wave synchronisation through LDS: wait for this wave's LDS
// operations; the wave barrier keeps the compiler from moving memory
// operations across it.
__device__ __forceinline__ void wsync() {
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0) only
  __builtin_amdgcn_wave_barrier();
}

// Synchronisation of the NT threads working on one box (NT = 64: one wave).
template <int NT>
__device__ __forceinline__ void bsync() {
  if (NT == 64) wsync();
  else __syncthreads();
}

// v(lane c) + v(lane c + 32) in every lane of column c, by two half-wave
// swaps of the 32-bit words (no LDS); both halves add in the same order.
__device__ __forceinline__ double half_sum(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  return __hiloint2double(b[0], a[0]) + __hiloint2double(b[1], a[1]);
}

__device__ __forceinline__ float half_sum_f(float v) {
  const int u = __float_as_int(v);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __int_as_float(a[0]) + __int_as_float(a[1]);
}

// Cached block inverses of one box read through a buffer resource: per lane
// the byte offsets of its 16 entries (row 16h + i, column c) within a block,
// and the buffer size for the padding entries, which the range check turns
// into zeros; the block index goes into the scalar offset.  The blocks are
// the inverses of symmetric Schur complements and are stored as their lower
// triangle, row-major (entry (r, c), r >= c, at r (r + 1) / 2 + c; both
// (r, c) and (c, r) read it): half the bytes of a full block, padded to an
// even number so that every block starts at a 16-byte boundary.  (The FP32
// form's blocks are stored whole, see Lane32.)
__host__ __device__ inline int packed_elems(int nb) { return (nb * (nb + 1) / 2 + 1) / 2 * 2; }

struct BlockSrc {
  __amdgpu_buffer_rsrc_t rs;
  int off[HB];
  int bbytes;
};

// Buffer of a wave-uniform base and size, kept in scalar registers so that
// accesses need no per-lane resource; offsets past it read zero and store
// nothing.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_buffer(const void* p, int bytes) {
  const unsigned long long pa = reinterpret_cast<unsigned long long>(p);
  const unsigned plo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)pa);
  const unsigned phi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(pa >> 32));
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<char*>(((unsigned long long)phi << 32) | plo), (short)0,
                                           __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

__device__ __forceinline__ BlockSrc block_src(const double* Wg, int nb, int nblk) {
  BlockSrc b;
  const int bsz = packed_elems(nb);
  const int bytes = nblk * bsz * (int)sizeof(double);
  b.rs = uniform_buffer(Wg, bytes);
  const int c = threadIdx.x & 31, h = (threadIdx.x >> 5) & 1;
#pragma unroll
  for (int i = 0; i < HB; ++i) {
    const int r = HB * h + i;
    const int hi = r > c ? r : c, lo = r > c ? c : r;
    const int idx = hi * (hi + 1) / 2 + lo;
    b.off[i] = (r < nb && c < nb) ? idx * (int)sizeof(double) : bytes;
  }
  b.bbytes = __builtin_amdgcn_readfirstlane(bsz * (int)sizeof(double));
  return b;
}

__device__ __forceinline__ void wload_block(const BlockSrc& b, int j, double w[HB]) {
#pragma unroll
  for (int i = 0; i < HB; ++i)
    w[i] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(
        b.rs, b.off[i], __builtin_amdgcn_readfirstlane(j * b.bbytes), 0));
}

// dst[e] = *addr(e, fill) for e < n (or `fill` where addr returns nullptr),
// by NT threads with CH loads each in flight before any of them is waited for.
template <int CH, int NT = 64, typename AddrFn>
__device__ __forceinline__ void gather(double* dst, int n, AddrFn addr) {
  const int L = threadIdx.x % NT;
#pragma unroll 1
  for (int e0 = 0; e0 < n; e0 += NT * CH) {
    double v[CH];
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int e = e0 + u * NT + L;
      double fill = 0.0;
      const double* a = (e < n) ? addr(e, fill) : nullptr;
      v[u] = a ? *a : fill;
    }
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int e = e0 + u * NT + L;
      if (e < n) dst[e] = v[u];
    }
  }
}

// 1/x from the hardware estimate refined by two Newton steps (x normal).
__device__ __forceinline__ double rcp_d(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  e = fma(-x, r, 1.0);
  return fma(r, e, r);
}

// Robin coefficients of the face between box cell c (K = kc) and the
// outside cell o (K = ko): beta (paper: alpha H / K_H, or a constant) and
// T^R = |e| / (h / (2 K_c) + beta), with reciprocals in place of divisions.
__device__ __forceinline__ void robin_face(const Geo& g, int a, double kc, double ko, double beta,
                                           double& bt, double& TR) {
  const double Ha = (a == 0 ? g.S[0] : g.S[1]) * g.h;
  bt = g.beta_mode == 1 ? beta : beta * Ha * (kc + ko) * rcp_d(2.0 * kc * ko);
  TR = g.area * 2.0 * kc * rcp_d(g.h + 2.0 * kc * bt);
}

// LDS of the extra permeability tiles of a diagonal tensor with kc entries
// per cell (axes 1.., one halo tile each), placed ahead of a box's other
// arrays; 0 for scalar K.  Even, so that what follows keeps its alignment.
__host__ __device__ inline size_t kx_doubles(int kc, int m0, int m1) {
  return kc > 1 ? ((size_t)(kc - 1) * (m0 + 2) * (m1 + 2) + 1) / 2 * 2 : 0;
}

// The extra tiles at base; returns where the box's own arrays start.
__device__ __forceinline__ double* attach_kx(BoxLds& s, double* base, int kc) {
  s.Kx = base;
  s.ktn = kc > 1 ? (s.m0 + 2) * (s.m1 + 2) : 0;
  return base + kx_doubles(kc, s.m0, s.m1);
}

// After Kt is set: the tile axis 1 reads.
__device__ __forceinline__ void attach_ky(BoxLds& s) { s.Ky = s.ktn ? s.Kx : s.Kt; }

__host__ __device__ inline size_t box_lds_doubles(int m0, int m1, int nrhs, int kc = 1) {
  const int nc = m0 * m1;
  return kx_doubles(kc, m0, m1) + (size_t)(m0 + 2) * (m1 + 2) + 3 * (size_t)nc + (size_t)nrhs * nc +
         (size_t)nrhs * NBW + 2;
}

__device__ __forceinline__ BoxLds carve(double* base, const Box& B, int nrhs, int kc = 1) {
  BoxLds s;
  s.m0 = B.hi[0] - B.lo[0];
  s.m1 = B.hi[1] - B.lo[1];
  const int nc = s.m0 * s.m1;
  base = attach_kx(s, base, kc);
  s.Kt = base;
  attach_ky(s);
  s.Dg = s.Kt + (s.m0 + 2) * (s.m1 + 2);
  s.Tx = s.Dg + nc;
  s.Tn = s.Tx + nc;
  s.X = s.Tn + nc;
  s.Z = align16(base, s.X + (size_t)nrhs * nc);
  return s;
}

// The halo tile of axis a's permeability entries.
__device__ __forceinline__ const double* ktile(const BoxLds& s, int a) { return a == 0 ? s.Kt : s.Ky; }

// K along axis a at global cell (x, y), which must lie in the box or its
// halo.
__device__ __forceinline__ double kat(const BoxLds& s, const Box& B, int x, int y, int a) {
  return ktile(s, a)[(y - B.lo[1] + 1) * (s.m0 + 2) + (x - B.lo[0] + 1)];
}

template <int NT = 64>
__device__ __forceinline__ void coef_box(const Geo& g, const Box& B, double beta, BoxLds& s);

// The tiles of the permeability entries of axes 1.. (diagonal tensor), as
// the Kt tile (LOG: exponentiated here).
template <int NT, bool LOG>
__device__ __forceinline__ void load_kx(const Geo& g, const Box& B, const double* K, const BoxLds& s) {
  if (!s.ktn) return;
  const int W2 = s.m0 + 2, nt = s.ktn;
  gather<1024 / NT, NT>(s.Kx, (g.kc - 1) * nt, [&](int e, double& fill) -> const double* {
    const int a = 1 + e / nt, u = e - (a - 1) * nt;
    const int x = B.lo[0] - 1 + u % W2, y = B.lo[1] - 1 + u / W2;
    fill = LOG ? 0.0 : 1.0;
    return (x >= 0 && x < g.n[0] && !off_domain(g, 1, B.lo[1], y)) ? K + kaxis(g, a) + x + g.n[0] * y
                                                                   : nullptr;
  });
  if (LOG) {
    bsync<NT>();
    for (int e = threadIdx.x % NT; e < (g.kc - 1) * nt; e += NT) s.Kx[e] = exp(s.Kx[e]);
  }
}

// Load the K tile and the matrix coefficients of the box into LDS.
// With LOG, K points to log K and the tile is exponentiated in LDS (cells
// outside the domain read log K = 0, i.e. K = 1, as without).
template <int NT = 64, bool LOG = false>
__device__ __forceinline__ void load_box(const Geo& g, const Box& B, const double* K, double beta, BoxLds& s) {
  const int W2 = s.m0 + 2, H2 = s.m1 + 2;
  gather<1024 / NT, NT>(s.Kt, W2 * H2, [&](int e, double& fill) -> const double* {
    const int x = B.lo[0] - 1 + e % W2, y = B.lo[1] - 1 + e / W2;
    fill = LOG ? 0.0 : 1.0;
    return (x >= 0 && x < g.n[0] && !off_domain(g, 1, B.lo[1], y)) ? K + x + g.n[0] * y : nullptr;
  });
  load_kx<NT, LOG>(g, B, K, s);
  if (LOG) {
    bsync<NT>();
    for (int e = threadIdx.x % NT; e < W2 * H2; e += NT) s.Kt[e] = exp(s.Kt[e]);
  }
  bsync<NT>();
  coef_box<NT>(g, B, beta, s);
}

// Diagonal and couplings of the box matrix from the K tile in LDS.
template <int NT>
__device__ __forceinline__ void coef_box(const Geo& g, const Box& B, double beta, BoxLds& s) {
  const int nc = s.m0 * s.m1;
  const double ih = rcp_d(g.h);
#pragma unroll 1
  for (int loc = threadIdx.x % NT; loc < nc; loc += NT) {
    const int x = B.lo[0] + loc % s.m0, y = B.lo[1] + loc / s.m0;
    double diag = 0.0, tx = 0.0, tn = 0.0;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const double kc = kat(s, B, x, y, a);
#pragma unroll
      for (int sd = 0; sd < 2; ++sd) {
        const int ox = x + (a == 0 ? (sd ? 1 : -1) : 0);
        const int oy = y + (a == 1 ? (sd ? 1 : -1) : 0);
        const int t = a == 0 ? ox : oy;
        if (off_domain(g, a, a == 0 ? x : y, t)) {
          if (g.bc_type[2 * a + sd]) diag += 2.0 * kc * g.area * ih;
          continue;
        }
        const double ko = kat(s, B, ox, oy, a);
        const bool inside = ox >= B.lo[0] && ox < B.hi[0] && oy >= B.lo[1] && oy < B.hi[1];
        if (inside) {
          const double T = g.area * 2.0 * kc * ko * rcp_d(kc + ko) * ih;
          diag += T;
          if (sd) {
            if (a == 0) tx = T;
            else tn = T;
          }
        } else {
          double bt, TR;
          robin_face(g, a, kc, ko, beta, bt, TR);
          diag += TR;
        }
      }
    }
    s.Dg[loc] = diag;
    s.Tx[loc] = tx;
    s.Tn[loc] = tn;
  }
  bsync<NT>();
}

// An index the compiler recomputes where it is used instead of keeping what
// it derives from it in registers over unrolled steps and loops.
__device__ __forceinline__ void keep_here(int& e) { asm volatile("" : "+v"(e)); }

// d += a(lane K of the row) b
template <int K>
__device__ __forceinline__ void fmac_bcast(double& d, double a, double b) {
  asm("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(d) : "v"(a), "v"(b), "n"(K));
}
template <int K>
__device__ __forceinline__ void fmac_bcast(float& d, float a, float b) {
  asm("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf" : "+v"(d) : "v"(a), "v"(b), "n"(K));
}
// row entries of the Schur complement: w <- band entry - th(row) (tc w)
template <int I, typename T>
__device__ __forceinline__ void schur_rows(T w[HB], int ic, T dc, T xl, T xr, T th, T ntc) {
  if constexpr (I < HB) {
    keep_here(ic);  // (the comparisons of all rows at once spill to branches)
    T e = ic == I ? dc : T(0);
    e = ic == I + 1 ? xl : e;
    e = ic == I - 1 ? xr : e;
    fmac_bcast<I>(e, th, ntc * w[I]);
    w[I] = e;
    schur_rows<I + 1>(w, ic, dc, xl, xr, th, ntc);
  }
}
// Schur complement (column c, my half) into w: the tridiagonal line with
// diagonal D (null: ones, FP32) and couplings Tx, less t W t with the coupling t =
// Tp (lower; else any line that can be read) to the block eliminated before,
// whose inverse W w holds on entry.  A lane reads the entries of its own column and one of
// t, which the others of its 16-lane row take by row broadcast.
template <typename T>
__device__ __forceinline__ void schur_block(int nb, const T* D, const T* Tx, const T* Tp, bool lower, T w[HB]) {
  const int L = lane_id(), c = L & 31, h = L >> 5;
  const int r = HB * h + (L & 15);
  const bool in = c < nb;
  const int cc = in ? c : 0, rc = r < nb ? r : 0;
  const T dv = D ? D[cc] : T(1), x0 = Tx[cc > 0 ? cc - 1 : 0], x1 = Tx[cc], t0 = Tp[cc], t1 = Tp[rc];
  const T dc = in ? dv : T(1);
  const T xl = in && c > 0 ? -x0 : T(0), xr = in && c + 1 < nb ? -x1 : T(0);
  const T ntc = in && lower ? -t0 : T(0);
  T th = r < nb ? t1 : T(0);
  asm("s_nop 1" : "+v"(th));  // a DPP operand: two wait states after its write
  schur_rows<0>(w, c - HB * h, dc, xl, xr, th, ntc);
}
// Block j of a box; tpi: line of Tn that couples it to the block eliminated
// before (forward elimination j - 1, backward j), negative: none.
__device__ __forceinline__ void wbuild_t(int nb, int j, int tpi, const BoxLds& s, double w[HB]) {
  schur_block<double>(nb, s.Dg + j * nb, s.Tx + j * nb, s.Tn + max(tpi, 0) * nb, tpi >= 0, w);
}

// S_j of the forward elimination; w holds W_{j-1} on entry when j > 0.
__device__ __forceinline__ void wbuild(int nb, int j, const BoxLds& s, double w[HB]) {
  wbuild_t(nb, j, j - 1, s, w);
}

// In-place inverse of the block held in w (symmetric, identity padding
// outside nb x nb), 16 pivots at a time.  The 16-lane rows of the wave hold
// the quarters of the block as the rows of 00, 10, 01 and 11, so 00 is ready
// for the in-register inverse P; with U = block 01 and Z = P U follow
//   S = A11 - U^T Z,  Q = S^{-1},  W10 = -Q Z^T,  W00 = P - Z W10,  W11 = Q
// on the matrix instructions, the operands through two tiles of LDS (X^T Y
// of accumulator layouts needs no transposition, Z^T takes one).
// Bound: the two chains of pivots (16, then 8 or 16, about 120 cycles each
// in FP64) and the LDS round trips between them, 7,300 cycles at 24 cells.
// Measured against four pivots per step on the vector unit with an LDS round
// trip each (boxes of 24 x 24 cells, all of Steps 1-2 and 4): 256 boxes with
// eight seeds 155 -> 136 us, 4096 with four 1226 -> 942 us; FP32 222 ->
// 206 us and 1643 -> 1506 us.
template <typename T>
__device__ __forceinline__ void winv(int nb, InvSmem<T>& sm, T w[HB]) {
  using V = typename InvSmem<T>::V;
  const int rho = lane_id() >> 4;
  bool bad = false;
  T a[HB];
#pragma unroll
  for (int i = 0; i < HB; ++i) a[i] = w[i];
  V u, d;
  if (nb > 16) {
    if (rho & 1) tile_put_row(sm.t[rho >> 1], w);
    wave_lds_sync();
    u = tile_get_t(sm.t[0]);
    d = tile_get(sm.t[1]);
  }
  inv16<true>(a, bad, nb);
  bad = bad && rho == 0;  // the other rows invert what they hold
  if (nb <= 16) {
    if (rho == 0) {
#pragma unroll
      for (int i = 0; i < HB; ++i) w[i] = a[i];
    }
  } else {
    const V zero = {T(0), T(0), T(0), T(0)};
    wave_lds_sync();
    if (rho == 0) tile_put_row(sm.t[0], a);
    wave_lds_sync();
    const V p = tile_get(sm.t[0]);
    const V z = mfma16(p, u, zero);
    const V s = mfma16(-u, z, d);
    wave_lds_sync();
    tile_put(sm.t[0], z);
    tile_put(sm.t[1], s);
    wave_lds_sync();
    const V zt = tile_get_t(sm.t[0]);
    tile_get_rows(sm.t[1], a);
    inv16<true>(a, bad, nb - 16);
    wave_lds_sync();
    tile_put_rows(sm.t[1], a);
    wave_lds_sync();
    const V q = tile_get(sm.t[1]);
    const V w10 = mfma16(-q, zt, zero, nb - 16);
    const V w00 = mfma16(-zt, w10, p, nb - 16);
    wave_lds_sync();
    tile_put(sm.t[0], w00);
    tile_put(sm.t[1], w10);
    wave_lds_sync();
    if (rho < 2) tile_get_rows(sm.t[rho], w);
    else if (rho == 2) tile_get_column(sm.t[1], w);
    else {
#pragma unroll
      for (int i = 0; i < HB; ++i) w[i] = a[i];
    }
    wave_lds_sync();
  }
  if (bad) atomicOr(&sm.flag, kFlagNotPD);
}

__device__ __forceinline__ void womega(const Geo& g, int sub, int lo[3], int hi[3]) {
  const int ix = sub % g.M[0], iy = sub / g.M[0];
  lo[0] = ix * g.S[0];
  hi[0] = lo[0] + g.S[0];
  lo[1] = iy * g.S[1];
  hi[1] = lo[1] + g.S[1];
  lo[2] = 0;
  hi[2] = 1;
}

__device__ __forceinline__ bool win_box(const Box& B, int x, int y) {
  return x >= B.lo[0] && x < B.hi[0] && y >= B.lo[1] && y < B.hi[1];
}

__device__ __forceinline__ int wneighbor(const Geo& g, int sub, int q) {
  const int a = q >> 1, sd = q & 1;
  const int ia = (a == 0) ? sub % g.M[0] : sub / g.M[0];
  const int t = ia + (sd ? 1 : -1);
  if (off_subgrid(g, a, ia, t)) return -1;
  const int stride = (a == 0) ? 1 : g.M[0];
  return sub + (sd ? stride : -stride);
}

// Inner cell of face t on side q of [lo, hi) (2-D).
__device__ __forceinline__ void wgface(const int lo[3], const int hi[3], int q, int t, int& x, int& y) {
  const int a = q >> 1, sd = q & 1;
  const int xe = sd ? hi[0] - 1 : lo[0], ye = sd ? hi[1] - 1 : lo[1];
  x = a == 0 ? xe : lo[0] + t;
  y = a == 0 ? lo[1] + t : ye;
}

__device__ __forceinline__ int bloc(const Box& B, const BoxLds& s, int x, int y) {
  return (x - B.lo[0]) + s.m0 * (y - B.lo[1]);
}

// Physical right-hand side (source, boundary data) of box B into out.
template <int NT = 64>
__device__ __forceinline__ void physical_rhs(const Geo& g, const Box& B, const BoxLds& s, const double* f,
                             const double* bcv, double* out) {
  const int nc = s.m0 * s.m1;
  #pragma unroll 1
  for (int loc = threadIdx.x % NT; loc < nc; loc += NT) {
    const int x = B.lo[0] + loc % s.m0, y = B.lo[1] + loc / s.m0;
    const int ci = x + g.n[0] * y;
    double b = f[ci] * g.vol;
    const int c[3] = {x, y, 0};
    for (int a = 0; a < 2; ++a)
      for (int sd = 0; sd < 2; ++sd) {
        const int t = c[a] + (sd ? 1 : -1);
        if (!off_domain(g, a, c[a], t)) continue;
        const int side = 2 * a + sd;
        const double val = bcv[g.bc_off[side] + bface_index(g, c, a)];
        if (g.bc_type[side]) b += 2.0 * kat(s, B, x, y, a) * g.area / g.h * val;
        else b -= g.area * val;
      }
    out[loc] = b;
  }
}

// lambda = -beta u.n + pi on the Robin face of box B at inside cell (x, y),
// normal along a, side sd, from the current global state (Section 3).
__device__ __forceinline__ double wlambda(const Geo& g, const Box& B, const BoxLds& s,
                                          const double* p, const double* gflux, double beta,
                                          int x, int y, int a, int sd) {
  const int ox = x + (a == 0 ? (sd ? 1 : -1) : 0), oy = y + (a == 1 ? (sd ? 1 : -1) : 0);
  const int ci = x + g.n[0] * y, oi = ox + g.n[0] * oy;
  const double kc = kat(s, B, x, y, a), ko = kat(s, B, ox, oy, a);
  const double bt = robin_beta(g, a, kc, ko, beta);
  if (g.l > 0) {
    const double u = g.area * kharm(kc, ko) / g.h * (p[ci] - p[oi]) / g.area;
    const double pi = p[ci] - u * g.h / (2.0 * kc);
    return -bt * u + pi;
  }
  const int q = 2 * a + sd;
  const int j = wneighbor(g, B.sub, q);
  int jlo[3], jhi[3];
  womega(g, j, jlo, jhi);
  const int t = (a == 0) ? oy - jlo[1] : ox - jlo[0];
  const double uj = gflux[(long long)j * g.gstride + g.gside_off[q ^ 1] + t];
  const double pij = p[oi] - uj * g.h / (2.0 * ko);
  return bt * uj + pij;
}


// ----------------------------------------------------------------- smoothing
// LDS of a smoothing box: the K and p tiles with a one-cell halo, the source,
// the block couplings, the neighbours' Gamma fluxes on the box sides (used
// when the boxes do not overlap) and the boundary data of the box sides on
// the domain boundary, all gathered in one pass; then the matrix
// coefficients, the solution vector and the block staging.
struct SmoothLds {
  BoxLds b;    // Kt, Dg, Tx, Tn, X, Z (Z: 2 x NBW)
  double* P;   // (m0 + 2) x (m1 + 2) pressure tile
  double* F;   // ncell source density
  double* GF;  // 2 (m0 + m1): neighbour flux per face of each box side
  double* BC;  // 2 (m0 + m1): boundary value per face of each box side
};

__host__ __device__ inline size_t smooth_lds_doubles(int m0, int m1, int kc = 1) {
  const size_t nc = (size_t)m0 * m1, nt = (size_t)(m0 + 2) * (m1 + 2);
  return kx_doubles(kc, m0, m1) + 2 * nt + 5 * nc + 4 * (size_t)(m0 + m1) + 4 * NBW + 2;
}

__device__ __forceinline__ int side_off(const BoxLds& s, int q) {
  // faces of side q are numbered along the tangential axis
  return q == 0 ? 0 : q == 1 ? s.m1 : q == 2 ? 2 * s.m1 : 2 * s.m1 + s.m0;
}

// Gather order: [Kt | P | F | Tn | GF | BC] contiguous (after the extra
// permeability tiles of a tensor).
__device__ __forceinline__ SmoothLds carve_smooth(double* base, const Box& B, int kc = 1) {
  SmoothLds r;
  BoxLds& s = r.b;
  s.m0 = B.hi[0] - B.lo[0];
  s.m1 = B.hi[1] - B.lo[1];
  const int nc = s.m0 * s.m1, nt = (s.m0 + 2) * (s.m1 + 2), ns = 2 * (s.m0 + s.m1);
  base = attach_kx(s, base, kc);
  s.Kt = base;
  attach_ky(s);
  r.P = s.Kt + nt;
  r.F = r.P + nt;
  s.Tn = r.F + nc;
  r.GF = s.Tn + nc;
  r.BC = r.GF + ns;
  s.Dg = r.BC + ns;
  s.Tx = s.Dg + nc;
  s.X = s.Tx + nc;
  s.Z = align16(base, s.X + nc);
  return r;
}

// One gather for everything the smoothing solve of box B reads from memory.
// The block couplings come from tcoup (cached by the factorisation) unless
// it is null (then they are left to coef_box).
template <int NT>
__device__ __forceinline__ void stage_smooth(const Geo& g, const Box& B, const SmoothLds& r,
                                             const double* K, const double* p, const double* f,
                                             const double* gflux, const double* bcv,
                                             const double* tcoup) {
  const BoxLds& s = r.b;
  const int m0 = s.m0, m1 = s.m1, W2 = m0 + 2;
  const int nc = m0 * m1, nt = W2 * (m1 + 2), ns = 2 * (m0 + m1);
  const int n0 = g.n[0];
  const int lo0 = B.lo[0], lo1 = B.lo[1];
  const double* tg = tcoup ? tcoup + B.scr : nullptr;
  // per side q: a box side on the domain boundary reads its boundary values;
  // with non-overlapping boxes an interior side reads the neighbour's flux
  const int Mx = g.M[0];
  const int isub = B.sub % Mx, jsub = B.sub / Mx;
  // one gather over the contiguous LDS arrays Kt, P, F, Tn, GF, BC, with
  // about 12 loads per thread in flight (a 24 x 24 box needs one round)
  gather<64 * 48 / NT, NT>(s.Kt, 2 * nt + 2 * nc + 2 * ns, [&](int e, double& fill) -> const double* {
    if (e < 2 * nt) {
      const bool isk = e < nt;
      const int u = isk ? e : e - nt;
      const int y = lo1 - 1 + u / W2, x = lo0 - 1 + (u - (u / W2) * W2);
      fill = isk ? 1.0 : 0.0;
      if (x < 0 || x >= n0 || off_domain(g, 1, lo1, y)) return nullptr;
      return (isk ? K : p) + x + n0 * y;
    }
    e -= 2 * nt;
    if (e < nc) return f + (lo0 + e % m0) + n0 * (lo1 + e / m0);
    e -= nc;
    if (e < nc) return tg ? tg + e : nullptr;
    e -= nc;
    fill = 0.0;
    const bool isgf = e < ns;
    const int u = isgf ? e : e - ns;
    const int q = u < 2 * m1 ? (u < m1 ? 0 : 1) : (u < 2 * m1 + m0 ? 2 : 3);
    const int t = u - (q == 0 ? 0 : q == 1 ? m1 : q == 2 ? 2 * m1 : 2 * m1 + m0);
    const int a = q >> 1, sd = q & 1;
    const int x = a == 0 ? (sd ? B.hi[0] - 1 : lo0) : lo0 + t;
    const int y = a == 1 ? (sd ? B.hi[1] - 1 : lo1) : lo1 + t;
    const int o = (a == 0 ? x : y) + (sd ? 1 : -1);
    const bool dom = off_domain(g, a, a == 0 ? x : y, o);
    if (!isgf) {
      if (!dom) return nullptr;
      const int off = q == 0 ? g.bc_off[0] : q == 1 ? g.bc_off[1] : q == 2 ? g.bc_off[2] : g.bc_off[3];
      const int c3[3] = {x, y, 0};
      return bcv + off + bface_index(g, c3, a);
    }
    if (dom || g.l > 0) return nullptr;
    // neighbour across side q and the face's position on its opposite side
    const int j = B.sub + (a == 0 ? (sd ? 1 : -1) : (sd ? Mx : -Mx));
    const int go = q == 0 ? g.gside_off[1] : q == 1 ? g.gside_off[0] : q == 2 ? g.gside_off[3] : g.gside_off[2];
    const int tj = a == 0 ? y - jsub * g.S[1] : x - isub * g.S[0];
    return gflux + (long long)j * g.gstride + go + tj;
  });
  load_kx<NT, false>(g, B, K, s);
}

// K and p at a cell of the box or its halo.
__device__ __forceinline__ int tile_at(const BoxLds& s, const Box& B, int x, int y) {
  return (y - B.lo[1] + 1) * (s.m0 + 2) + (x - B.lo[0] + 1);
}

// lambda on the face of box cell (x, y) normal to a on side sd of the box,
// from the staged state (Section 3; the neighbour's flux and trace when the
// boxes do not overlap).  bt is the face's beta.
__device__ __forceinline__ double lambda_s(const Geo& g, const Box& B, const SmoothLds& r,
                                           double bt, int x, int y, int a, int sd) {
  const BoxLds& s = r.b;
  const int ox = x + (a == 0 ? (sd ? 1 : -1) : 0), oy = y + (a == 1 ? (sd ? 1 : -1) : 0);
  const int ti = tile_at(s, B, x, y), to = tile_at(s, B, ox, oy);
  const double kc = ktile(s, a)[ti], ko = ktile(s, a)[to];
  if (g.l > 0) {
    // u = K_H (p_c - p_o) / h, pi = p_c - u h / (2 K_c)
    const double u = 2.0 * kc * ko * rcp_d(kc + ko) * (r.P[ti] - r.P[to]) * rcp_d(g.h);
    const double pi = r.P[ti] - u * g.h * 0.5 * rcp_d(kc);
    return -bt * u + pi;
  }
  const int q = 2 * a + sd;
  const double uj = r.GF[side_off(s, q) + (a == 0 ? y - B.lo[1] : x - B.lo[0])];
  const double pij = r.P[to] - uj * g.h * 0.5 * rcp_d(ko);
  return bt * uj + pij;
}

// Right-hand side of the smoothing problem of box B into out (LDS), by NT
// threads: the source on every cell, then the faces of the box sides (x
// sides, then y sides, so that no cell is updated twice at once).
template <int NT>
__device__ __forceinline__ void smooth_rhs(const Geo& g, const Box& B, const SmoothLds& r,
                                           double beta, double* out) {
  const BoxLds& s = r.b;
  const int nc = s.m0 * s.m1;
  const int tid = threadIdx.x % NT;
#pragma unroll 1
  for (int loc = tid; loc < nc; loc += NT) out[loc] = r.F[loc] * g.vol;
  bsync<NT>();
  // both sides of an axis in one pass, except in a box one cell thick
  // along that axis, where they add to the same cells: then one pass each
  auto face = [&](int a, int sd, int t) {
    const int x = a == 0 ? (sd ? B.hi[0] - 1 : B.lo[0]) : B.lo[0] + t;
    const int y = a == 1 ? (sd ? B.hi[1] - 1 : B.lo[1]) : B.lo[1] + t;
    const int c[3] = {x, y, 0};
    const int kind = face_kind(g, B, c, a, sd);
    const double* Ka = ktile(s, a);
    const double kc = Ka[tile_at(s, B, x, y)];
    double add;
    if (kind == kFaceRobin) {
      const int ox = x + (a == 0 ? (sd ? 1 : -1) : 0), oy = y + (a == 1 ? (sd ? 1 : -1) : 0);
      double bt, TR;
      robin_face(g, a, kc, Ka[tile_at(s, B, ox, oy)], beta, bt, TR);
      add = TR * lambda_s(g, B, r, bt, x, y, a, sd);
    } else {
      const double val = r.BC[side_off(s, 2 * a + sd) + t];
      add = kind == kFaceDir ? 2.0 * kc * g.area / g.h * val : -g.area * val;
    }
    out[bloc(B, s, x, y)] += add;
  };
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const int nf = a == 0 ? s.m1 : s.m0;
    const int ma = a == 0 ? s.m0 : s.m1;
    if (ma > 1) {
#pragma unroll 1
      for (int u = tid; u < 2 * nf; u += NT) face(a, u >= nf, u - (u >= nf ? nf : 0));
    } else {
#pragma unroll 1
      for (int t = tid; t < nf; t += NT) face(a, 0, t);
      bsync<NT>();
#pragma unroll 1
      for (int t = tid; t < nf; t += NT) face(a, 1, t);
    }
    bsync<NT>();
  }
}

// Smoothing outputs of box B from its solution x (LDS), by NT threads: p on
// Omega_i and Omega_i's own Gamma fluxes (TPFA of the new pressure; the
// Robin formula with the staged lambda when the boxes do not overlap).
template <int NT, typename T>
__device__ __forceinline__ void smooth_out(const Geo& g, const Box& B, const SmoothLds& r, const T* x,
                                           double beta, double* p, double* gflux) {
  const BoxLds& s = r.b;
  const int tid = threadIdx.x % NT;
  int olo[3], ohi[3];
  womega(g, B.sub, olo, ohi);
  const int nfx = g.S[1], nfy = g.S[0];
#pragma unroll 1
  for (int u = tid; u < 2 * (nfx + nfy); u += NT) {
    const int q = u < 2 * nfx ? (u < nfx ? 0 : 1) : (u < 2 * nfx + nfy ? 2 : 3);
    const int t = u - (q == 0 ? 0 : q == 1 ? nfx : q == 2 ? 2 * nfx : 2 * nfx + nfy);
    if (wneighbor(g, B.sub, q) < 0) continue;
    const int a = q >> 1, so = q & 1;
    int cx, cy;
    wgface(olo, ohi, q, t, cx, cy);
    const int ox = cx + (a == 0 ? (so ? 1 : -1) : 0), oy = cy + (a == 1 ? (so ? 1 : -1) : 0);
    const double kc = ktile(s, a)[tile_at(s, B, cx, cy)], ko = ktile(s, a)[tile_at(s, B, ox, oy)];
    const double xc = x[bloc(B, s, cx, cy)];
    double v;
    if (win_box(B, ox, oy)) {
      v = 2.0 * kc * ko * rcp_d(kc + ko) * (xc - x[bloc(B, s, ox, oy)]) * rcp_d(g.h);
    } else {
      double bt, TR;
      robin_face(g, a, kc, ko, beta, bt, TR);
      const double lam = lambda_s(g, B, r, bt, cx, cy, a, so);
      v = TR * (xc - lam) * rcp_d(g.area);
    }
    const int go = q == 0 ? g.gside_off[0] : q == 1 ? g.gside_off[1] : q == 2 ? g.gside_off[2] : g.gside_off[3];
    gflux[(long long)B.sub * g.gstride + go + t] = v;
  }
  const int ncell_o = g.S[0] * g.S[1];
#pragma unroll 1
  for (int t = tid; t < ncell_o; t += NT) {
    const int cx = olo[0] + t % g.S[0], cy = olo[1] + t / g.S[0];
    p[cx + g.n[0] * cy] = x[bloc(B, s, cx, cy)];
  }
}

// ------------------------------------------------------------- block sweeps
// W_j z for the block staged in z (LDS): lane (c, h) sums its 16 rows with
// two accumulators; half_sum completes the column.
__device__ __forceinline__ double wgemv2(const double w[HB], const double* z) {
  const int h = lane_id() >> 5;
  const double2* z2 = reinterpret_cast<const double2*>(z + HB * h);
  double a0 = 0.0, a1 = 0.0;
#pragma unroll
  for (int i = 0; i < HB / 2; ++i) {
    const double2 v = z2[i];
    a0 = fma(w[2 * i], v.x, a0);
    a1 = fma(w[2 * i + 1], v.y, a1);
  }
  return half_sum(a0 + a1);
}

// W_j z without LDS, for the single-vector sweeps: the lane holds z[zi],
// zi = 16 h + lane % 16 (the index its half of the columns needs), and a row
// broadcast hands z[16 h + k] to the 16 lanes of its row inside the
// multiply-add (v_fmac_f64 with row_newbcast), so a block step is 16
// instructions in four chains, the sum of the halves and one exchange of
// 16-lane rows.  The leading wait states cover the write of z.
__device__ __forceinline__ double wgemv_rows(const double w[HB], double z) {
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
#define MRCM_F(A, I, K) "v_fmac_f64_dpp %" #A ", %4, %" #I " row_newbcast:" #K " row_mask:0xf bank_mask:0xf\n\t"
  asm("s_nop 1\n\t" MRCM_F(0, 5, 0) MRCM_F(1, 6, 1) MRCM_F(2, 7, 2) MRCM_F(3, 8, 3) MRCM_F(0, 9, 4)
          MRCM_F(1, 10, 5) MRCM_F(2, 11, 6) MRCM_F(3, 12, 7) MRCM_F(0, 13, 8) MRCM_F(1, 14, 9)
              MRCM_F(2, 15, 10) MRCM_F(3, 16, 11) MRCM_F(0, 17, 12) MRCM_F(1, 18, 13) MRCM_F(2, 19, 14)
                  MRCM_F(3, 20, 15)
      : "+v"(a0), "+v"(a1), "+v"(a2), "+v"(a3)
      : "v"(z), "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]), "v"(w[4]), "v"(w[5]), "v"(w[6]), "v"(w[7]),
        "v"(w[8]), "v"(w[9]), "v"(w[10]), "v"(w[11]), "v"(w[12]), "v"(w[13]), "v"(w[14]), "v"(w[15]));
#undef MRCM_F
  return half_sum((a0 + a1) + (a2 + a3));
}

// y of column c = lane % 32 -> y of index zi, by a swap of 16-lane rows
__device__ __forceinline__ double to_rows(double y) {
  const int lo = __double2loint(y), hi = __double2hiint(y);
  const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  const bool h = lane_id() >= 32;
  return __hiloint2double(h ? b[1] : b[0], h ? a[1] : a[0]);
}

// Products of the block in w with a vector per right-hand side, four at a
// time so that their chains overlap: zf(k) gives the lane's entry zi = 16 h +
// lane % 16 of vector k (zero past nb), of(k, y) takes entry lane % 32 of the
// product.  Entries and results live in LDS, no staging between them.
template <typename Zf, typename Of>
__device__ __forceinline__ void block_products(int nrhs, const double w[HB], Zf&& zf, Of&& of) {
  wsync();
  int k = 0;
#pragma unroll 1
  for (; k + 4 <= nrhs; k += 4) {
    double z[4], y[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) z[q] = zf(k + q);
#pragma unroll
    for (int q = 0; q < 4; ++q) y[q] = wgemv_rows(w, z[q]);
#pragma unroll
    for (int q = 0; q < 4; ++q) of(k + q, y[q]);
  }
#pragma unroll 1
  for (; k < nrhs; ++k) of(k, wgemv_rows(w, zf(k)));
  wsync();
}

// Forward step of block j for all right-hand sides, inverse in w, with jp
// the block eliminated just before j (j - 1 going down the box, j + 1 going
// up; has_prev false for the first block of a chain):
// X_j <- W (X_j + t .* X_jp), t the coupling of j and jp (Tn row min(j, jp)).
__device__ __forceinline__ void fwd_step_d(int nb, int ncell, int j, int jp, bool has_prev,
                                           int nrhs, const BoxLds& s, const double w[HB]) {
  const int L = lane_id(), c = L & 31, zi = HB * (L >> 5) + (L & 15);
  const bool zv = zi < nb, cv = L < 32 && c < nb;
  const int zc = zv ? zi : 0;
  const double t = has_prev ? s.Tn[min(j, jp) * nb + zc] : 0.0;
  const double* Xj = s.X + j * nb + zc;
  const double* Xp = s.X + (has_prev ? jp : j) * nb + zc;
  double* Xo = s.X + j * nb + c;
  block_products(
      nrhs, w, [&](int k) { return zv ? fma(t, Xp[k * ncell], Xj[k * ncell]) : 0.0; },
      [&](int k, double y) {
        if (cv) Xo[k * ncell] = y;
      });
}

// Back-substitution step of block j towards block jn (the block solved just
// before it): X_j <- X_j + W (t .* X_jn), t the coupling of j and jn.
__device__ __forceinline__ void bwd_step_d(int nb, int ncell, int j, int jn, int nrhs,
                                           const BoxLds& s, const double w[HB]) {
  const int L = lane_id(), c = L & 31, zi = HB * (L >> 5) + (L & 15);
  const bool zv = zi < nb, cv = L < 32 && c < nb;
  const int zc = zv ? zi : 0;
  const double t = s.Tn[min(j, jn) * nb + zc];
  const double* Xn = s.X + jn * nb + zc;
  double* Xo = s.X + j * nb + c;
  block_products(
      nrhs, w, [&](int k) { return zv ? t * Xn[k * ncell] : 0.0; },
      [&](int k, double y) {
        if (cv) Xo[k * ncell] += y;
      });
}

// Meeting block of the two-ended solve, all right-hand sides, Z_m in w:
// X_m <- Z_m (X_m + t_{m-1} .* X_{m-1} + t_m .* X_{m+1}).
__device__ __forceinline__ void mid_step(int nb, int ncell, int m, int nblk, int nrhs,
                                         const BoxLds& s, const double w[HB]) {
  const int L = lane_id(), c = L & 31, zi = HB * (L >> 5) + (L & 15);
  const bool zv = zi < nb, cv = L < 32 && c < nb;
  const int e = m * nb + (zv ? zi : 0), up = m > 0 ? nb : 0, dn = m + 1 < nblk ? nb : 0;
  const double tu = up ? s.Tn[e - up] : 0.0, td = dn ? s.Tn[e] : 0.0;
  double* Xo = s.X + m * nb + c;
  block_products(
      nrhs, w,
      [&](int k) {
        const double* X = s.X + k * ncell + e;
        const double v = fma(td, X[dn], fma(tu, X[-up], X[0]));
        return zv ? v : 0.0;
      },
      [&](int k, double y) {
        if (cv) Xo[k * ncell] = y;
      });
}

// Back-substitution of the one-ended solve, X_j <- X_j + W_j (t_j .*
// X_{j+1}), with the cached inverses streamed from memory, RING blocks ahead.
__device__ __forceinline__ void backward_cached(const Box& B, const double* Wg, int nrhs, const BoxLds& s) {
  const int nb = B.nb, nblk = B.nblk;
  const BlockSrc src = block_src(Wg, nb, nblk);
  double w[RING][HB];
  // block j = nblk - 2 - t uses ring slot t % RING
#pragma unroll
  for (int q = 0; q < RING; ++q)
    if (nblk - 2 - q >= 0) wload_block(src, (nblk - 2 - q), w[q]);
  for (int t0 = 0; t0 <= nblk - 2; t0 += RING) {
#pragma unroll
    for (int q = 0; q < RING; ++q) {
      const int j = nblk - 2 - (t0 + q);
      if (j >= 0) {
        bwd_step_d(nb, B.ncell, j, j + 1, nrhs, s, w[q]);
        if (j - RING >= 0) wload_block(src, (j - RING), w[q]);
      }
    }
  }
}

// Halves of the two-ended solve of all right-hand sides with cached inverses
// (meeting block m = nblk / 2).  Top: blocks 0 .. m-1 with the forward
// inverses W_j; bottom: blocks nblk-1 .. m+1 with the backward inverses
// W'_j = (D_j - t_j W'_{j+1} t_j)^{-1}.  The forward pass of a half runs
// from its end of the box towards m; the back-substitution from m outwards.
// The inverses stream from memory RING blocks ahead of their use.
__device__ __forceinline__ void twist_fwd_cached(const Box& B, const double* Wg, int nrhs,
                                                 const BoxLds& s, bool bottom) {
  const int nb = B.nb, nblk = B.nblk, m = nblk / 2;
  const int cnt = bottom ? nblk - 1 - m : m;
  const int j0 = bottom ? nblk - 1 : 0, dj = bottom ? -1 : 1;
  if (cnt <= 0) return;
  const BlockSrc src = block_src(Wg, nb, nblk);
  double w[RING][HB];
#pragma unroll
  for (int q = 0; q < RING; ++q)
    if (q < cnt) wload_block(src, j0 + dj * q, w[q]);
  for (int t0 = 0; t0 < cnt; t0 += RING) {
#pragma unroll
    for (int q = 0; q < RING; ++q) {
      const int t = t0 + q;
      if (t < cnt) {
        const int j = j0 + dj * t;
        fwd_step_d(nb, B.ncell, j, j - dj, t > 0, nrhs, s, w[q]);
        if (t + RING < cnt) wload_block(src, j0 + dj * (t + RING), w[q]);
      }
    }
  }
}

__device__ __forceinline__ void twist_back_cached(const Box& B, const double* Wg, int nrhs,
                                                  const BoxLds& s, bool bottom) {
  const int nb = B.nb, nblk = B.nblk, m = nblk / 2;
  const int cnt = bottom ? nblk - 1 - m : m;
  const int dj = bottom ? 1 : -1;  // direction away from m
  if (cnt <= 0) return;
  const BlockSrc src = block_src(Wg, nb, nblk);
  double w[RING][HB];
#pragma unroll
  for (int q = 0; q < RING; ++q)
    if (q < cnt) wload_block(src, m + dj * (q + 1), w[q]);
  for (int t0 = 0; t0 < cnt; t0 += RING) {
#pragma unroll
    for (int q = 0; q < RING; ++q) {
      const int t = t0 + q;
      if (t < cnt) {
        const int j = m + dj * (t + 1);
        bwd_step_d(nb, B.ncell, j, j - dj, nrhs, s, w[q]);
        if (t + RING < cnt) wload_block(src, m + dj * (t + RING + 1), w[q]);
      }
    }
  }
}

// The whole two-ended solve of all right-hand sides in s.X by one wave:
// Wf holds the forward inverses (blocks < m), Wt the backward inverses
// (blocks > m) and Z_m at block m.
__device__ __forceinline__ void twisted_cached(const Box& B, const double* Wf, const double* Wt,
                                               int nrhs, const BoxLds& s) {
  const int m = B.nblk / 2;
  twist_fwd_cached(B, Wf, nrhs, s, false);
  twist_fwd_cached(B, Wt, nrhs, s, true);
  double zm[HB];
  wload_block(block_src(Wt, B.nb, B.nblk), m, zm);
  mid_step(B.nb, B.ncell, m, B.nblk, nrhs, s, zm);
  twist_back_cached(B, Wf, nrhs, s, false);
  twist_back_cached(B, Wt, nrhs, s, true);
}

// Forward and backward sweeps of one right-hand side in s.X with the cached
// inverses.  The value of the previous block stays in registers (every lane
// of column c holds it), so a block step is one LDS write of the staged
// vector, the 16-term products and one half-wave exchange.  z points to
// 2 x NBW doubles of LDS (alternating buffers).
__device__ __forceinline__ void sweep1(const Box& B, const double* Wg, const BoxLds& s, double* z) {
  const int L = lane_id();
  const int c = L & 31, h = L >> 5;
  const int nb = B.nb, nblk = B.nblk;
  const bool cv = c < nb;
  const BlockSrc src = block_src(Wg, nb, nblk);
  {
    double w[RING][HB];
#pragma unroll
    for (int q = 0; q < RING; ++q)
      if (q < nblk) wload_block(src, q, w[q]);
    double y = 0.0;
    double xn = cv ? s.X[c] : 0.0, tp = 0.0;
    for (int j0 = 0; j0 < nblk; j0 += RING) {
#pragma unroll
      for (int q = 0; q < RING; ++q) {
        const int j = j0 + q;
        if (j < nblk) {
          double* zb = z + (j & 1) * NBW;
          if (h == 0) zb[c] = cv ? fma(tp, y, xn) : 0.0;
          __builtin_amdgcn_wave_barrier();
          const bool more = j + 1 < nblk;
          xn = (more && cv) ? s.X[(j + 1) * nb + c] : 0.0;
          tp = (more && cv) ? s.Tn[j * nb + c] : 0.0;
          y = wgemv2(w[q], zb);
          if (h == 0 && cv) s.X[j * nb + c] = y;
          if (j + RING < nblk) wload_block(src, (j + RING), w[q]);
        }
      }
    }
  }
  {
    double w[RING][HB];
#pragma unroll
    for (int q = 0; q < RING; ++q)
      if (nblk - 2 - q >= 0) wload_block(src, (nblk - 2 - q), w[q]);
    // x_{nblk-1} = w_{nblk-1} is final; every lane of column c reads it
    __builtin_amdgcn_wave_barrier();
    double xnext = cv ? s.X[(nblk - 1) * nb + c] : 0.0;
    double tj = (nblk >= 2 && cv) ? s.Tn[(nblk - 2) * nb + c] : 0.0;
    double wj = (nblk >= 2 && cv) ? s.X[(nblk - 2) * nb + c] : 0.0;
    for (int t0 = 0; t0 <= nblk - 2; t0 += RING) {
#pragma unroll
      for (int q = 0; q < RING; ++q) {
        const int j = nblk - 2 - (t0 + q);
        if (j >= 0) {
          double* zb = z + (j & 1) * NBW;
          if (h == 0) zb[c] = cv ? tj * xnext : 0.0;
          __builtin_amdgcn_wave_barrier();
          const double wcur = wj;
          tj = (j >= 1 && cv) ? s.Tn[(j - 1) * nb + c] : 0.0;
          wj = (j >= 1 && cv) ? s.X[(j - 1) * nb + c] : 0.0;
          xnext = wcur + wgemv2(w[q], zb);
          if (h == 0 && cv) s.X[j * nb + c] = xnext;
          if (j - RING >= 0) wload_block(src, (j - RING), w[q]);
        }
      }
    }
  }
  wsync();
}

// ---------------------------------------------------------- twisted sweep
// The block-tridiagonal box system solved from both ends towards the
// meeting block m = nblk / 2 (a twisted block factorisation):
//   top:     z_j = W_j (b_j + t_{j-1} z_{j-1}),    j = 0 .. m-1
//   bottom:  z_j = W'_j (b_j + t_j z_{j+1}),       j = nblk-1 .. m+1
//   meet:    x_m = Z_m (b_m + t_{m-1} z_{m-1} + t_m z_{m+1})
//   top:     x_j = z_j + W_j (t_j x_{j+1}),        j = m-1 .. 0
//   bottom:  x_j = z_j + W'_j (t_{j-1} x_{j-1}),   j = m+1 .. nblk-1
// with the forward inverses W_j, the backward inverses W'_j =
// (D_j - t_j W'_{j+1} t_j)^{-1} and Z_m = (S_m - t_m W'_{m+1} t_m)^{-1}, S_m
// the forward Schur complement of block m.  All of them are symmetric, so
// the column-per-lane products of sweep1 apply.  The two halves touch
// disjoint blocks of s.X and may run on two waves at once; each half needs
// its own 2 x NBW doubles of LDS staging z.

// One half of the twisted sweep: block j = j0 + dj * b for the b-th block
// away from the end (b = 0 .. cnt-1).  The register ring holds block b in
// slot (b + o) % RING, with o chosen so that the last block of the forward
// pass sits in slot RING-1: the back pass then finds its first RING blocks
// in place (slot RING-1-q for its q-th block) and the slot of every block
// stays a compile-time index.
struct TwistHalf {
  BlockSrc src;
  int cnt, j0, dj, o;
};

__device__ __forceinline__ TwistHalf twist_half(const Box& B, const double* Wg, int m, bool bottom) {
  TwistHalf hf;
  hf.src = block_src(Wg, B.nb, B.nblk);
  hf.cnt = bottom ? B.nblk - 1 - m : m;
  hf.j0 = bottom ? B.nblk - 1 : 0;
  hf.dj = bottom ? -1 : 1;
  hf.o = hf.cnt > 0 ? (RING - hf.cnt % RING) % RING : 0;
  return hf;
}

// First RING blocks of the forward pass into the ring (block b in slot
// (b + o) % RING).
__device__ __forceinline__ void twist_preload(const TwistHalf& hf, double w[RING][HB]) {
#pragma unroll
  for (int q = 0; q < RING; ++q) {
    const int b = (q - hf.o + RING) % RING;
    if (b < hf.cnt) wload_block(hf.src, hf.j0 + hf.dj * b, w[q]);
  }
}

// Forward half (ring preloaded); z_j replaces b_j in s.X.
__device__ __forceinline__ void twist_fwd(const Box& B, const TwistHalf& hf, const BoxLds& s,
                                          double* z, bool bottom, double w[RING][HB]) {
  const int L = lane_id();
  const int c = L & 31, h = L >> 5;
  const int nb = B.nb;
  const bool cv = c < nb;
  const int cnt = hf.cnt;
  if (cnt <= 0) return;
  double y = 0.0, tp = 0.0;
  double xn = cv ? s.X[hf.j0 * nb + c] : 0.0;
  for (int v0 = 0; v0 < cnt + hf.o; v0 += RING) {
#pragma unroll
    for (int q = 0; q < RING; ++q) {
      const int t = v0 + q - hf.o;
      if (t >= 0 && t < cnt) {
        const int j = hf.j0 + hf.dj * t;
        double* zb = z + (t & 1) * NBW;
        if (h == 0) zb[c] = cv ? fma(tp, y, xn) : 0.0;
        __builtin_amdgcn_wave_barrier();
        const bool more = t + 1 < cnt;
        const int jn = j + hf.dj;             // next block of this half
        const int ti = bottom ? jn : j;       // coupling between j and jn
        xn = (more && cv) ? s.X[jn * nb + c] : 0.0;
        tp = (more && cv) ? s.Tn[ti * nb + c] : 0.0;
        y = wgemv2(w[q], zb);
        if (h == 0 && cv) s.X[j * nb + c] = y;
        if (t + RING < cnt) wload_block(hf.src, hf.j0 + hf.dj * (t + RING), w[q]);
      }
    }
  }
}

// Meeting block: x_m from b_m and the neighbouring z of both halves; zm
// holds Z_m in the block register layout.
__device__ __forceinline__ void twist_mid(const Box& B, const double zm[HB], const BoxLds& s,
                                          double* z, int m) {
  const int L = lane_id();
  const int c = L & 31, h = L >> 5;
  const int nb = B.nb, nblk = B.nblk;
  const bool cv = c < nb;
  double v = 0.0;
  if (cv) {
    v = s.X[m * nb + c];
    if (m > 0) v = fma(s.Tn[(m - 1) * nb + c], s.X[(m - 1) * nb + c], v);
    if (m + 1 < nblk) v = fma(s.Tn[m * nb + c], s.X[(m + 1) * nb + c], v);
  }
  if (h == 0) z[c] = v;
  __builtin_amdgcn_wave_barrier();
  const double y = wgemv2(zm, z);
  if (h == 0 && cv) s.X[m * nb + c] = y;
}

// Back-substitution half, outwards from the meeting block.  With
// have_ring the ring is the one the forward pass of this half left behind.
__device__ __forceinline__ void twist_back(const Box& B, const TwistHalf& hf, const BoxLds& s,
                                           double* z, int m, bool bottom, bool have_ring,
                                           double w[RING][HB]) {
  const int L = lane_id();
  const int c = L & 31, h = L >> 5;
  const int nb = B.nb;
  const bool cv = c < nb;
  const int cnt = hf.cnt;
  if (cnt <= 0) return;
  if (!have_ring) {
#pragma unroll
    for (int q = 0; q < RING; ++q) {
      const int b = cnt - 1 - q;
      if (b >= 0) wload_block(hf.src, hf.j0 + hf.dj * b, w[RING - 1 - q]);
    }
  }
  const int jf = hf.j0 + hf.dj * (cnt - 1);  // first block of the back pass (next to m)
  double xnext = cv ? s.X[m * nb + c] : 0.0;
  double tj = cv ? s.Tn[(bottom ? jf - 1 : jf) * nb + c] : 0.0;
  double wj = cv ? s.X[jf * nb + c] : 0.0;
  for (int v0 = 0; v0 < cnt; v0 += RING) {
#pragma unroll
    for (int q = 0; q < RING; ++q) {
      const int t = v0 + q;
      if (t < cnt) {
        const int b = cnt - 1 - t;
        const int j = hf.j0 + hf.dj * b;
        double* zb = z + (t & 1) * NBW;
        if (h == 0) zb[c] = cv ? tj * xnext : 0.0;
        __builtin_amdgcn_wave_barrier();
        const double wcur = wj;
        const bool more = t + 1 < cnt;
        const int jn = j - hf.dj;             // next block, away from m
        tj = (more && cv) ? s.Tn[(bottom ? jn - 1 : jn) * nb + c] : 0.0;
        wj = (more && cv) ? s.X[jn * nb + c] : 0.0;
        xnext = wcur + wgemv2(w[RING - 1 - q], zb);
        if (h == 0 && cv) s.X[j * nb + c] = xnext;
        if (b - RING >= 0) wload_block(hf.src, hf.j0 + hf.dj * (b - RING), w[RING - 1 - q]);
      }
    }
  }
}

// The whole twisted sweep of one right-hand side by the NT threads of a
// box.  With NT >= 128 the two halves run on waves 0 and 1 at once, each
// keeping its ring from the forward into the back pass; the caller has
// preloaded the ring of its half (twist_preload) and wave 0 the meeting
// block (zm), before staging, so that their memory latency is hidden.  With
// NT = 64 one wave runs the halves one after the other and loads as it
// goes.  The arithmetic is the same in both cases, and so is the result.
// Wf: forward inverses, Wt: backward inverses and Z_m; z: 4 x NBW doubles.
template <int NT>
__device__ __forceinline__ void sweep_twisted(const Box& B, const double* Wf, const double* Wt,
                                              const BoxLds& s, double* z, double w[RING][HB],
                                              const double zm[HB]) {
  const int wv = threadIdx.x >> 6;
  const int m = B.nblk / 2;
  double* za = z;
  double* zb = z + 2 * NBW;
  const TwistHalf top = twist_half(B, Wf, m, false);
  const TwistHalf bot = twist_half(B, Wt, m, true);
  if (NT == 64) {
    twist_preload(top, w);
    twist_fwd(B, top, s, za, false, w);
    twist_preload(bot, w);
    twist_fwd(B, bot, s, zb, true, w);
  } else if (wv == 0) {
    twist_fwd(B, top, s, za, false, w);
  } else if (wv == 1) {
    twist_fwd(B, bot, s, zb, true, w);
  }
  bsync<NT>();
  if (wv == 0) twist_mid(B, zm, s, za, m);
  bsync<NT>();
  if (NT == 64) {
    twist_back(B, top, s, za, m, false, false, w);
    twist_back(B, bot, s, zb, m, true, false, w);
  } else if (wv == 0) {
    twist_back(B, top, s, za, m, false, true, w);
  } else if (wv == 1) {
    twist_back(B, bot, s, zb, m, true, true, w);
  }
  bsync<NT>();
}

// ------------------------------------------------- factors resident in LDS
// The two-ended sweep with all block inverses of the box in LDS: an image of
// the packed blocks 0 .. m-1 (forward) and m .. nblk-1 (meeting block and
// backward), copied there once by the whole workgroup in 16-byte pieces
// (global_load_lds: no registers, every piece in flight at once).
// Why: read per lane from memory, a block is 16 gathers of 64 scattered
// 8-byte entries, and their address processing, not the dependency chain,
// set the time of a block step (760 cycles on lines of 24 cells, the same
// with the products' operands through LDS or by row broadcasts, in the
// forward pass from memory and in the back pass from L2).  From LDS the
// gathers are nearly free of bank conflicts (triangular numbers modulo 32
// are a permutation) and each block crosses the memory bus once instead of
// twice.  A block step takes 480 cycles: 192 of dependency chain, the rest
// the issue of its reads and their addresses by the one wave.
// Measured per colour phase, with smooth_static: 64 boxes of 24 x 24 cells
// 17.4 -> 10.2 us, 4 boxes of 20 x 20 15.6 -> 8.2 us, 1024 boxes of 24 x 24
// (two per CU) 39 -> 27 us.
__host__ __device__ inline size_t factor_image_doubles(int nb, int nblk) {
  return (size_t)nblk * packed_elems(nb);
}

// n doubles (rounded up to even) from src to LDS, both 16-byte aligned, by
// the NT threads of the box; complete after staged_wait.
template <int NT>
__device__ __forceinline__ void stage_lds(const double* src, double* dst, int n) {
  const int n2 = (n + 1) / 2, l = lane_id();
  const int w0 = __builtin_amdgcn_readfirstlane((int)(threadIdx.x % NT) & ~63);
  for (int e = w0; e < n2; e += NT) {
    auto* d = (__attribute__((address_space(3))) void*)(unsigned)(uintptr_t)(dst + 2 * e);
    auto* a = (__attribute__((address_space(1))) void*)(uintptr_t)(src + 2 * (e + l));
    if (e + l < n2) __builtin_amdgcn_global_load_lds(a, d, 16, 0, 0);
  }
}
template <int NT>
__device__ __forceinline__ void staged_wait() {
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  bsync<NT>();
}

template <int NT>
__device__ __forceinline__ void stage_factors(const Box& B, const double* Wf, const double* Wt, double* img) {
  const int m = B.nblk / 2, be = packed_elems(B.nb);
  stage_lds<NT>(Wf, img, m * be);
  stage_lds<NT>(Wt + (long long)m * be, img + m * be, (B.nblk - m) * be);
}

// Lanes of a block step with resident factors: the lines are cut into two
// parts of nh = (nb + 1) / 2 <= KN entries; lane (g, i) (g = lane / 16,
// i = lane % 16) holds row nh (g % 2) + i and the columns of part g / 2, and
// of a vector entry nh (g / 2) + i.  The exchange of 16-lane rows (to_rows)
// then turns products into vector entries as before, and a step takes KN
// products and reads instead of 16.  Entries outside the block read a valid
// one instead: rows beyond give results nobody reads, columns beyond meet a
// zero.
template <int KN>
struct LdsFac {
  const double* img;
  int off[KN], be, nb, nblk;
  int zi, ci;     // vector entry and row of the lane
  bool zv, cv;    // valid; cv: in one lane per row
  bool zo;        // valid in one lane per entry
};
template <int KN>
__device__ __forceinline__ LdsFac<KN> lds_fac(const Box& B, const double* img) {
  LdsFac<KN> f;
  f.img = img;
  f.nb = B.nb;
  f.nblk = B.nblk;
  f.be = packed_elems(B.nb);
  const int nb = B.nb, nh = (nb + 1) / 2, L = lane_id(), i = L & 15, g = L >> 4;
  const int rr = nh * (g & 1) + i, zz = nh * (g >> 1) + i;
  const bool in = i < nh;
  f.cv = in && rr < nb && g < 2;
  f.zv = in && zz < nb;
  f.zo = f.zv && !(g & 1);
  f.ci = min(rr, nb - 1);
  f.zi = min(zz, nb - 1);
  const int c = f.ci;
#pragma unroll
  for (int k = 0; k < KN; ++k) {
    const int r = min(nh * (g >> 1) + k, nb - 1);
    const int hi = r > c ? r : c, lo = r > c ? c : r;
    f.off[k] = hi * (hi + 1) / 2 + lo;
  }
  return f;
}
template <int KN, int K0 = 0, int K1 = KN>
__device__ __forceinline__ void lds_block(const LdsFac<KN>& f, int j, double w[KN]) {
  const double* b = f.img + j * f.be;
#pragma unroll
  for (int k = K0; k < K1; ++k) w[k] = b[f.off[k]];
}
// reads issued before the current block's products: at most 15 LDS
// operations can be told apart by a wait, and more would make it wait for
// some of the new ones
constexpr int kAhead = 8;

// y of the lane's row: wgemv_rows over KN columns
template <int KN>
__device__ __forceinline__ double lds_gemv(const double w[KN], double z) {
  double a0 = 0.0, a1 = 0.0;
#define MRCM_P(I0, K0, I1, K1)                                                                     \
  "v_fmac_f64_dpp %0, %2, %" #I0 " row_newbcast:" #K0 " row_mask:0xf bank_mask:0xf\n\t"            \
  "v_fmac_f64_dpp %1, %2, %" #I1 " row_newbcast:" #K1 " row_mask:0xf bank_mask:0xf\n\t"
#define MRCM_S10                                                                                   \
  "s_nop 1\n\t" MRCM_P(3, 0, 4, 1) MRCM_P(5, 2, 6, 3) MRCM_P(7, 4, 8, 5) MRCM_P(9, 6, 10, 7)       \
      MRCM_P(11, 8, 12, 9)
#define MRCM_S12 MRCM_S10 MRCM_P(13, 10, 14, 11)
#define MRCM_S14 MRCM_S12 MRCM_P(15, 12, 16, 13)
#define MRCM_S16 MRCM_S14 MRCM_P(17, 14, 18, 15)
#define MRCM_W10                                                                                   \
  "v"(z), "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]), "v"(w[4]), "v"(w[5]), "v"(w[6]), "v"(w[7]),    \
      "v"(w[8]), "v"(w[9])
  static_assert(KN == 10 || KN == 12 || KN == 14 || KN == 16, "products per block step");
  if constexpr (KN == 10) asm(MRCM_S10 : "+v"(a0), "+v"(a1) : MRCM_W10);
  if constexpr (KN == 12) asm(MRCM_S12 : "+v"(a0), "+v"(a1) : MRCM_W10, "v"(w[10]), "v"(w[11]));
  if constexpr (KN == 14)
    asm(MRCM_S14 : "+v"(a0), "+v"(a1) : MRCM_W10, "v"(w[10]), "v"(w[11]), "v"(w[12]), "v"(w[13]));
  if constexpr (KN == 16)
    asm(MRCM_S16
        : "+v"(a0), "+v"(a1)
        : MRCM_W10, "v"(w[10]), "v"(w[11]), "v"(w[12]), "v"(w[13]), "v"(w[14]), "v"(w[15]));
#undef MRCM_P
#undef MRCM_S10
#undef MRCM_S12
#undef MRCM_S14
#undef MRCM_S16
#undef MRCM_W10
  return half_sum(a0 + a1);
}

// One half of the two-ended sweep (see twist_fwd and twist_back), the next
// block's entries and the next line's vector entries read before the current
// block's products are issued.
template <int KN>
__device__ __forceinline__ void lds_fwd(const LdsFac<KN>& f, const double* Tn, double* X, int m, bool bottom) {
  const int nb = f.nb, cnt = bottom ? f.nblk - 1 - m : m;
  if (cnt <= 0) return;
  const int dj = bottom ? -1 : 1;
  int j = bottom ? f.nblk - 1 : 0;
  double yz = 0.0, tp = 0.0;
  double xn = X[j * nb + f.zi];
  xn = f.zv ? xn : 0.0;
  double wa[KN], wb[KN];
  lds_block(f, j, wa);
  auto step = [&](const double* w, double* wn, bool more) {
    const double z = fma(tp, yz, xn);
    const int jn = more ? j + dj : j;
    xn = X[jn * nb + f.zi];
    tp = Tn[(bottom ? jn : j) * nb + f.zi];
    lds_block<KN, 0, kAhead>(f, jn, wn);
    __builtin_amdgcn_sched_barrier(0);
    const double y = lds_gemv<KN>(w, z);
    lds_block<KN, kAhead>(f, jn, wn);
    yz = to_rows(y);
    if (f.cv) X[j * nb + f.ci] = y;
    xn = f.zv ? xn : 0.0;
    tp = f.zv ? tp : 0.0;
    j = jn;
  };
  int t = 0;
  for (; t + 1 < cnt; t += 2) {
    step(wa, wb, true);
    step(wb, wa, t + 2 < cnt);
  }
  if (t < cnt) step(wa, wb, false);
}

template <int KN>
__device__ __forceinline__ void lds_mid(const LdsFac<KN>& f, const double* Tn, double* X, int m) {
  const int nb = f.nb;
  double w[KN];
  lds_block(f, m, w);
  double v = X[m * nb + f.zi];
  if (m > 0) v = fma(Tn[(m - 1) * nb + f.zi], X[(m - 1) * nb + f.zi], v);
  if (m + 1 < f.nblk) v = fma(Tn[m * nb + f.zi], X[(m + 1) * nb + f.zi], v);
  const double y = lds_gemv<KN>(w, f.zv ? v : 0.0);
  if (f.cv) X[m * nb + f.ci] = y;
}

template <int KN>
__device__ __forceinline__ void lds_back(const LdsFac<KN>& f, const double* Tn, double* X, int m, bool bottom) {
  const int nb = f.nb, cnt = bottom ? f.nblk - 1 - m : m;
  if (cnt <= 0) return;
  const int dj = bottom ? 1 : -1;
  int j = m + dj;
  double xnext = X[m * nb + f.zi];
  double tj = Tn[(bottom ? j - 1 : j) * nb + f.zi];
  tj = f.zv ? tj : 0.0;
  double wj = X[j * nb + f.zi];
  double wa[KN], wb[KN];
  lds_block(f, j, wa);
  auto step = [&](const double* w, double* wn, bool more) {
    const double z = tj * xnext, wcur = wj;
    const int jn = more ? j + dj : j;
    tj = Tn[(bottom ? jn - 1 : jn) * nb + f.zi];
    wj = X[jn * nb + f.zi];
    lds_block<KN, 0, kAhead>(f, jn, wn);
    __builtin_amdgcn_sched_barrier(0);
    const double y = lds_gemv<KN>(w, z);
    lds_block<KN, kAhead>(f, jn, wn);
    xnext = wcur + to_rows(y);
    if (f.zo) X[j * nb + f.zi] = xnext;
    tj = f.zv ? tj : 0.0;
    j = jn;
  };
  int t = 0;
  for (; t + 1 < cnt; t += 2) {
    step(wa, wb, true);
    step(wb, wa, t + 2 < cnt);
  }
  if (t < cnt) step(wa, wb, false);
}

template <int NT, int KN>
__device__ __forceinline__ void lds_sweep_k(const Box& B, const double* img, const double* Tn, double* X) {
  const int wv = (int)(threadIdx.x % NT) >> 6, m = B.nblk / 2;
  const LdsFac<KN> f = lds_fac<KN>(B, img);
  if (wv < 2) {
    if (NT == 64 || wv == 0) lds_fwd(f, Tn, X, m, false);
    if (NT == 64 || wv == 1) lds_fwd(f, Tn, X, m, true);
  }
  bsync<NT>();
  if (wv == 0) lds_mid(f, Tn, X, m);
  bsync<NT>();
  if (wv < 2) {
    if (NT == 64 || wv == 0) lds_back(f, Tn, X, m, false);
    if (NT == 64 || wv == 1) lds_back(f, Tn, X, m, true);
  }
  bsync<NT>();
}

// The whole two-ended sweep of one right-hand side in X (LDS; couplings to
// the next line in Tn) by the NT threads of a box: the halves on waves 0
// and 1 when NT >= 128, else one after the other.  The result does not
// depend on NT.  Ends with a barrier of the box.
template <int NT>
__device__ __forceinline__ void lds_sweep(const Box& B, const double* img, const double* Tn, double* X) {
  if (B.nb <= 20) lds_sweep_k<NT, 10>(B, img, Tn, X);
  else if (B.nb <= 24) lds_sweep_k<NT, 12>(B, img, Tn, X);
  else if (B.nb <= 28) lds_sweep_k<NT, 14>(B, img, Tn, X);
  else lds_sweep_k<NT, 16>(B, img, Tn, X);
}

// ------------------------------------------------ what smoothing keeps per box
// Everything of a box's smoothing problem that does not change between
// colour phases is written once with the factors (smooth_static):
//   b0   its right-hand side of the source and the boundary data,
//   fc   two coefficients per face of the box sides (side_off order): with
//        overlap T^R and T = |e| K_H / h, so that T^R lambda =
//        T^R p_c - T (p_c - p_o); without, T^R and T^R (beta - h / (2 K_o))
//        of lambda = p_o + (beta - h / (2 K_o)) u_j; zero on the domain
//        boundary,
//   gc   K_H / h of every Gamma face (the layout of gflux).
// A phase then reads the factors, b0, the couplings, these coefficients and
// the pressures on both sides of the box sides, and no permeability.
struct SmoothStatic {
  double *b0, *fc, *gc;
  int fstride;  // doubles of fc per box
};

__device__ __forceinline__ int face_off(int m0, int m1, int q) {
  return q == 0 ? 0 : q == 1 ? m1 : q == 2 ? 2 * m1 : 2 * m1 + m0;
}
// side of face u (side_off order) and its position on it
__device__ __forceinline__ int face_side(int m0, int m1, int u, int& t) {
  const int q = u < 2 * m1 ? (u < m1 ? 0 : 1) : (u < 2 * m1 + m0 ? 2 : 3);
  t = u - face_off(m0, m1, q);
  return q;
}
// its cell in the box [lo0, hi0) x [lo1, hi1) and the one across (by value:
// a select between fields of a Box held by reference is one of addresses)
__device__ __forceinline__ void face_cells(int lo0, int lo1, int hi0, int hi1, int q, int t, int& x, int& y,
                                           int& ox, int& oy) {
  const int a = q >> 1, sd = q & 1;
  x = a == 0 ? (sd ? hi0 - 1 : lo0) : lo0 + t;
  y = a == 1 ? (sd ? hi1 - 1 : lo1) : lo1 + t;
  ox = x + (a == 0 ? (sd ? 1 : -1) : 0);
  oy = y + (a == 1 ? (sd ? 1 : -1) : 0);
}

// from the K tile of the box in LDS, by NT threads
template <int NT>
__device__ __forceinline__ void smooth_static(const Geo& g, const Box& B, const BoxLds& s,
                                              const double* __restrict__ f,
                                              const double* __restrict__ bcv, double beta,
                                              const SmoothStatic& st) {
  const int tid = threadIdx.x % NT, m0 = s.m0, m1 = s.m1;
  physical_rhs<NT>(g, B, s, f, bcv, st.b0 + B.scr);
  double* fc = st.fc + (long long)B.sub * st.fstride;
#pragma unroll 1
  for (int u = tid; u < 2 * (m0 + m1); u += NT) {
    int t, x, y, ox, oy;
    const int q = face_side(m0, m1, u, t), a = q >> 1;
    face_cells(B.lo[0], B.lo[1], B.hi[0], B.hi[1], q, t, x, y, ox, oy);
    double c0 = 0.0, c1 = 0.0;
    if (!off_domain(g, a, a == 0 ? x : y, a == 0 ? ox : oy)) {
      const double kc = kat(s, B, x, y, a), ko = kat(s, B, ox, oy, a);
      double bt;
      robin_face(g, a, kc, ko, beta, bt, c0);
      c1 = g.l > 0 ? g.area * 2.0 * kc * ko * rcp_d(kc + ko) * rcp_d(g.h)
                   : c0 * (bt - g.h * 0.5 * rcp_d(ko));
    }
    fc[2 * u] = c0;
    fc[2 * u + 1] = c1;
  }
  int olo[3], ohi[3];
  womega(g, B.sub, olo, ohi);
#pragma unroll 1
  for (int u = tid; u < 2 * (g.S[0] + g.S[1]); u += NT) {
    int t;
    const int q = face_side(g.S[0], g.S[1], u, t), a = q >> 1, so = q & 1;
    int x, y;
    wgface(olo, ohi, q, t, x, y);
    const int ox = x + (a == 0 ? (so ? 1 : -1) : 0), oy = y + (a == 1 ? (so ? 1 : -1) : 0);
    const double kc = kat(s, B, x, y, a), ko = kat(s, B, ox, oy, a);
    const int go = q == 0 ? g.gside_off[0] : q == 1 ? g.gside_off[1] : q == 2 ? g.gside_off[2] : g.gside_off[3];
    st.gc[(long long)B.sub * g.gstride + go + t] = 2.0 * kc * ko * rcp_d(kc + ko) * rcp_d(g.h);
  }
}

// LDS of a smoothing box with resident factors: the image, the solution
// vector, the couplings, the Robin terms of the box sides.
__host__ __device__ inline size_t smooth_res_doubles(int m0, int m1) {
  const size_t nc = ((size_t)m0 * m1 + 1) / 2 * 2;
  return factor_image_doubles(m0, m1) + 2 * nc + 2 * (size_t)(m0 + m1) + 2;
}

}  // namespace wave
}  // namespace mrcm
