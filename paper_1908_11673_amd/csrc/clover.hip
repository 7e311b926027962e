// SW (clover) term and its odd-site inverse (Sec. 2.3 of arXiv:1908.11673).
//
// On every extended site the site-diagonal part of D is
//   1/(2 kappa) + sum_{mu<nu} (i/2) sigma_{mu nu} E_{mu nu},
//   E = su3csw F + u1csw qhat (i a) 1,  F = (Q - Q^+)/8 (four SU(3) clover leaves),
//   a = (1/4) sum of sin(plaquette angle) over the four U(1) plaquettes at x,
//       x-mu, x-nu, x-mu-nu (unit charge: the 1/q_el of the U(1) tensor cancels
//       against q = qhat q_el).
// In the chiral basis sigma_{0k} = diag(s_k, -s_k), sigma_{jk} = -eps_{jkl} diag(s_l, s_l),
// so the term is block diagonal: H_pm = 1/(2 kappa) + sum_l s_l (x) X_l^pm with
// X_l^pm = (i/2)(pm E_{0l} - E_{B_l}), B = ((2,3), (3,1), (1,2)).
#include <algorithm>

#include "qxd_internal.hpp"

struct PhysExt2 {
  int L[4];
  int64_t Vphys;
};

__device__ inline void step_coords(const Geo& g, int x[4], int mu, int dir) {
  x[mu] += dir;
  int Le = mu == 0 ? g.Le0 : mu == 1 ? g.Le1 : mu == 2 ? g.Le2 : g.Le3;
  if (x[mu] < 0 || x[mu] >= Le) {
    x[mu] = x[mu] < 0 ? x[mu] + Le : x[mu] - Le;
    if (mu >= 2 && mu <= g.cstar) x[1] = geo_mirror_x1(g, x[1]);
  }
}

__device__ inline int64_t phys_of(const PhysExt2& pe, const int x[4], bool& mirror) {
  mirror = x[1] >= pe.L[1];
  int x1 = mirror ? x[1] - pe.L[1] : x[1];
  return (int64_t)x[3] + (int64_t)pe.L[3] * ((int64_t)x[2] + (int64_t)pe.L[2] * ((int64_t)x1 + (int64_t)pe.L[1] * x[0]));
}

struct M3 {
  cx<double> m[9];
};

// U is component-major: [mu][9][Vphys]
__device__ inline M3 load_u(const PhysExt2& pe, const double2* __restrict__ U, const int x[4], int mu) {
  bool mir;
  const int64_t s = phys_of(pe, x, mir);
  const double2* u = U + (int64_t)mu * 9 * pe.Vphys + s;
  const double sg = mir ? -1.0 : 1.0;
  M3 r;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const double2 v = u[k * pe.Vphys];
    r.m[k] = mk(v.x, sg * v.y);
  }
  return r;
}

__device__ inline double load_a(const PhysExt2& pe, const double* __restrict__ A, const int x[4], int mu) {
  bool mir;
  int64_t s = phys_of(pe, x, mir);
  double a = A[mu * pe.Vphys + s];
  return mir ? -a : a;
}

// acc += a b, acc += conj(a) b as fused multiply-adds
__device__ __forceinline__ void cmac(cx<double>& acc, cx<double> a, cx<double> b) {
  acc.re = fma(a.re, b.re, acc.re);
  acc.re = fma(-a.im, b.im, acc.re);
  acc.im = fma(a.re, b.im, acc.im);
  acc.im = fma(a.im, b.re, acc.im);
}
__device__ __forceinline__ void cmac_conj(cx<double>& acc, cx<double> a, cx<double> b) {
  acc.re = fma(a.re, b.re, acc.re);
  acc.re = fma(a.im, b.im, acc.re);
  acc.im = fma(a.re, b.im, acc.im);
  acc.im = fma(-a.im, b.re, acc.im);
}

// a b, a^+ b, a b^+
__device__ inline M3 mm(const M3& a, const M3& b) {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      cx<double> s = a.m[3 * i] * b.m[j];
      cmac(s, a.m[3 * i + 1], b.m[3 + j]);
      cmac(s, a.m[3 * i + 2], b.m[6 + j]);
      r.m[3 * i + j] = s;
    }
  return r;
}
__device__ inline M3 mdm(const M3& a, const M3& b) {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      cx<double> s = cmul_conj(a.m[i], b.m[j]);
      cmac_conj(s, a.m[3 + i], b.m[3 + j]);
      cmac_conj(s, a.m[6 + i], b.m[6 + j]);
      r.m[3 * i + j] = s;
    }
  return r;
}
__device__ inline M3 mmd(const M3& a, const M3& b) {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      cx<double> s = cmul_conj(b.m[3 * j], a.m[3 * i]);
      cmac_conj(s, b.m[3 * j + 1], a.m[3 * i + 1]);
      cmac_conj(s, b.m[3 * j + 2], a.m[3 * i + 2]);
      r.m[3 * i + j] = s;
    }
  return r;
}

// The six planes 01 02 03 12 13 23 and where their tensors stand.
enum { E01 = 0, E02, E03, E12, E13, E23 };

// E_{mu nu}(x) = csw F + cu1 qhat (i a) 1 for one plane: anti-Hermitian, kept
// as nine reals, the imaginary diagonal and the entries (0,1), (0,2), (1,2).
// With W = U_mu(x) (X1 - X4^+) + U_mu(x-mu)^+ (X3 - X2^+), the X's the open
// staples of the four leaves, Q - Q^+ = W - W^+: ten products and fourteen link
// loads where the four closed leaves take twelve and sixteen.
__device__ inline void plane_tensor(const Geo& g, const PhysExt2& pe, const double2* __restrict__ U,
                                    const double* __restrict__ A, const int x[4], int mu, int nu, double csw,
                                    double cq, double e[9]) {
  int xpm[4], xpn[4], xmm[4], xmn[4], xmmpn[4], xmmmn[4], xmnpm[4];
  for (int i = 0; i < 4; ++i) xpm[i] = xpn[i] = xmm[i] = xmn[i] = x[i];
  step_coords(g, xpm, mu, +1);
  step_coords(g, xpn, nu, +1);
  step_coords(g, xmm, mu, -1);
  step_coords(g, xmn, nu, -1);
  for (int i = 0; i < 4; ++i) xmmpn[i] = xmmmn[i] = xmm[i];
  step_coords(g, xmmpn, nu, +1);
  step_coords(g, xmmmn, nu, -1);
  for (int i = 0; i < 4; ++i) xmnpm[i] = xmn[i];
  step_coords(g, xmnpm, mu, +1);

  // U(1): plaquette angles at the four corners
  auto angle = [&](const int y[4]) {
    int ym[4], yn[4];
    for (int i = 0; i < 4; ++i) ym[i] = yn[i] = y[i];
    step_coords(g, ym, mu, +1);
    step_coords(g, yn, nu, +1);
    return load_a(pe, A, y, mu) + load_a(pe, A, ym, nu) - load_a(pe, A, yn, mu) - load_a(pe, A, y, nu);
  };
  const double a4 = 0.25 * (sin(angle(x)) + sin(angle(xmm)) + sin(angle(xmn)) + sin(angle(xmmmn)));

  // X1 = U_nu(x+mu) U_mu(x+nu)^+ U_nu(x)^+;  X4^+ = U_nu(x+mu-nu)^+ U_mu(x-nu)^+ U_nu(x-nu)
  M3 T = mmd(mmd(load_u(pe, U, xpm, nu), load_u(pe, U, xpn, mu)), load_u(pe, U, x, nu));
  {
    const M3 t = mdm(load_u(pe, U, xmn, mu), load_u(pe, U, xmn, nu));
    const M3 s = mdm(load_u(pe, U, xmnpm, nu), t);
#pragma unroll
    for (int k = 0; k < 9; ++k) T.m[k] = T.m[k] - s.m[k];
  }
  M3 W = mm(load_u(pe, U, x, mu), T);
  // X3 = U_nu(x-mu-nu)^+ U_mu(x-mu-nu) U_nu(x-nu);  X2^+ = U_nu(x-mu) U_mu(x-mu+nu) U_nu(x)^+
  T = mm(mdm(load_u(pe, U, xmmmn, nu), load_u(pe, U, xmmmn, mu)), load_u(pe, U, xmn, nu));
  {
    const M3 t = mm(load_u(pe, U, xmm, nu), load_u(pe, U, xmmpn, mu));
    const M3 s = mmd(t, load_u(pe, U, x, nu));
#pragma unroll
    for (int k = 0; k < 9; ++k) T.m[k] = T.m[k] - s.m[k];
  }
  T = mdm(load_u(pe, U, xmm, mu), T);
#pragma unroll
  for (int k = 0; k < 9; ++k) W.m[k] = W.m[k] + T.m[k];

#pragma unroll
  for (int i = 0; i < 3; ++i) e[i] = csw * (0.125 * (W.m[4 * i].im + W.m[4 * i].im)) + cq * a4;
  const cx<double> o01 = csw * (0.125 * (W.m[1] - conj(W.m[3]))), o02 = csw * (0.125 * (W.m[2] - conj(W.m[6]))),
                   o12 = csw * (0.125 * (W.m[5] - conj(W.m[7])));
  e[3] = o01.re, e[4] = o01.im, e[5] = o02.re, e[6] = o02.im, e[7] = o12.re, e[8] = o12.im;
}

// X = (i/2) (s a + t b) of two anti-Hermitian tensors (entries `stride` apart)
// at colour (i, j); sc = -1 conjugates both (the mirror half).
template <int I, int J>
__device__ __forceinline__ cx<double> half_i(const double* a, const double* b, int stride, double s, double t,
                                             double sc) {
  if (I == J) return mk(-0.5 * sc * (s * a[I * stride] + t * b[I * stride]), 0.0);
  constexpr int lo = I < J ? I : J, hi = I < J ? J : I, k = lo == 0 ? (hi == 1 ? 3 : 5) : 7;
  const double re = s * a[k * stride] + t * b[k * stride];
  const double im = sc * (s * a[(k + 1) * stride] + t * b[(k + 1) * stride]);
  // (i/2)(re + i im); the entry (j, i) is its conjugate
  return mk(-0.5 * im, (I < J ? 0.5 : -0.5) * re);
}

// entry (I, J) of the 6 x 6 block of chirality sg: 1/(2 kappa) + sum_l s_l (x) X_l,
// X_l = (i/2)(sg E_0l - E_Bl), E_B2 = E_31 = -E_13.  E: [6 planes][9][64 sites].
template <int I, int J>
__device__ __forceinline__ cx<double> block_entry(const double* E, double sg, double sc, double diag) {
  constexpr int P = 9 * 64, ai = I % 3, aj = J % 3;
  if (I / 3 == J / 3) {
    const cx<double> v = half_i<ai, aj>(E + E03 * P, E + E12 * P, 64, sg, -1.0, sc);
    const double f = I < 3 ? 1.0 : -1.0;
    return mk(f * v.re + (I == J ? diag : 0.0), f * v.im);
  }
  const cx<double> v1 = half_i<ai, aj>(E + E01 * P, E + E23 * P, 64, sg, -1.0, sc);
  const cx<double> v2 = half_i<ai, aj>(E + E02 * P, E + E13 * P, 64, sg, 1.0, sc);
  return v1 - ti(v2);
}

// the word K of a packed block (0..2: two diagonal entries, 3..17: the entries
// (0,1), (0,2), .., (4,5))
template <int K>
__device__ __forceinline__ double2 block_word(const double* E, double sg, double sc, double diag) {
  if constexpr (K < 3) {
    return make_double2(block_entry<2 * K, 2 * K>(E, sg, sc, diag).re,
                        block_entry<2 * K + 1, 2 * K + 1>(E, sg, sc, diag).re);
  } else {
    constexpr int n = K - 3, i = n < 5 ? 0 : n < 9 ? 1 : n < 12 ? 2 : n < 14 ? 3 : 4;
    constexpr int j = n - (i == 0 ? 0 : i == 1 ? 5 : i == 2 ? 9 : i == 3 ? 12 : 14) + i + 1;
    const cx<double> v = block_entry<i, j>(E, sg, sc, diag);
    return make_double2(v.re, v.im);
  }
}

template <int K0>
__device__ __forceinline__ void block_store(const double* E, double sg, double sc, double diag, size_t Ve,
                                            double2* __restrict__ out) {
  out[(K0 + 0) * Ve] = block_word<K0 + 0>(E, sg, sc, diag);
  out[(K0 + 1) * Ve] = block_word<K0 + 1>(E, sg, sc, diag);
  out[(K0 + 2) * Ve] = block_word<K0 + 2>(E, sg, sc, diag);
  out[(K0 + 3) * Ve] = block_word<K0 + 3>(E, sg, sc, diag);
  out[(K0 + 4) * Ve] = block_word<K0 + 4>(E, sg, sc, diag);
  out[(K0 + 5) * Ve] = block_word<K0 + 5>(E, sg, sc, diag);
}

constexpr int kClW = 2;  // waves of a workgroup
// A workgroup takes 64 consecutive physical sites: its waves share the six
// planes (tensors kept in LDS), then the words of the two blocks, on the site
// and, with C*, on its mirror image, whose tensors are the complex conjugates:
// half the products of one work-item per extended site.  One work-item for all
// six planes of a site needed 9.4 kB of scratch; one plane at a time fits the
// registers.
// 64 x 32^3: 36.6 -> 2.04 ms (a wave a plane, six waves: 2.39 ms, one workgroup
// a CU; two waves of three planes each: two wavefronts a SIMD).  Now bound by
// the 84 link loads a site (25 GB through the L2) and the FP64 products.
__global__ __launch_bounds__(64 * kClW, 2) void k_clover_build(Geo g, PhysExt2 pe, const double2* __restrict__ U,
                                                         const double* __restrict__ A, double csw, double cq,
                                                         double diag, double2* __restrict__ He,
                                                         double2* __restrict__ Ho) {
  __shared__ double E[6 * 9 * 64];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t s = site_tile(blockIdx.x, gridDim.x, 16) * 64 + lane;  // Vphys < 2^31
  const bool in = s < pe.Vphys;
  int x[4];
  {
    uint32_t r = in ? s : (uint32_t)pe.Vphys - 1;  // work-items past the end repeat the last site and store nothing
    x[3] = r % (uint32_t)pe.L[3];
    r /= (uint32_t)pe.L[3];
    x[2] = r % (uint32_t)pe.L[2];
    r /= (uint32_t)pe.L[2];
    x[1] = r % (uint32_t)pe.L[1];
    x[0] = r / (uint32_t)pe.L[1];
  }
#pragma unroll 1
  for (int pl = w; pl < 6; pl += kClW) {
    const int mu = pl < 3 ? 0 : pl < 5 ? 1 : 2, nu = pl < 3 ? pl + 1 : pl < 5 ? pl - 1 : 3;
    double e[9];
    plane_tensor(g, pe, U, A, x, mu, nu, csw, cq, e);
#pragma unroll
    for (int k = 0; k < 9; ++k) E[(pl * 9 + k) * 64 + lane] = e[k];
  }
  __syncthreads();
  if (!in) return;
  const size_t Ve = g.Ve;
#pragma unroll 1
  for (int part = w; part < 6; part += kClW) {  // chirality part / 3, words 6 (part % 3) ..
    const double sg = part < 3 ? 1.0 : -1.0;
    double2* H = (((x[0] + x[1] + x[2] + x[3]) & 1) ? Ho : He) + (size_t)(part < 3 ? 0 : 18) * Ve;
    for (int m = 0; m < (g.cstar >= 1 ? 2 : 1); ++m) {
      double2* out = H + geo_half(g, x[0], x[1] + m * pe.L[1], x[2], x[3]);
      const double sc = m ? -1.0 : 1.0;
      switch (part % 3) {
        case 0: block_store<0>(E + lane, sg, sc, diag, Ve, out); break;
        case 1: block_store<6>(E + lane, sg, sc, diag, Ve, out); break;
        default: block_store<12>(E + lane, sg, sc, diag, Ve, out); break;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// 6x6 inversion by Gauss-Jordan elimination with partial pivoting (largest
// |a|, lowest row on ties), fully unrolled so that row swaps are selects.

struct InvStats {
  unsigned long long* min_pivot_bits;  // positive doubles order as their bit patterns
  unsigned long long* max_norm_bits;
  unsigned long long* n_singular;
};

// Inverse of one packed block, in place: the eliminated columns of A hold the
// columns of the inverse as they arise, and the row swaps are undone as column
// swaps at the end.
__device__ inline void invert6(double r[36], double& minpiv, double& maxabs) {
  cx<double> A[6][6];
  maxabs = 0.0;
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    A[i][i] = mk(r[i], 0.0);
    maxabs = fmax(maxabs, fabs(r[i]));
#pragma unroll
    for (int j = i + 1; j < 6; ++j) {
      int o = herm6_off(i, j);
      A[i][j] = mk(r[o], r[o + 1]);
      A[j][i] = mk(r[o], -r[o + 1]);
      maxabs = fmax(maxabs, sqrt(r[o] * r[o] + r[o + 1] * r[o + 1]));
    }
  }
  minpiv = 1e300;
  int prow[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    int p = k;
    double best = norm2(A[k][k]);
#pragma unroll
    for (int i = k + 1; i < 6; ++i) {
      double v = norm2(A[i][k]);
      if (v > best) { best = v; p = i; }
    }
    prow[k] = p;
#pragma unroll
    for (int i = k + 1; i < 6; ++i) {
      bool sw = (p == i);
#pragma unroll
      for (int j = 0; j < 6; ++j) {
        cx<double> a = A[k][j], b = A[i][j];
        A[k][j] = sw ? b : a;
        A[i][j] = sw ? a : b;
      }
    }
    minpiv = fmin(minpiv, sqrt(best));
    cx<double> piv = A[k][k];
    double den = 1.0 / norm2(piv);
    cx<double> inv = mk(piv.re * den, -piv.im * den);
#pragma unroll
    for (int j = 0; j < 6; ++j) A[k][j] = j == k ? inv : inv * A[k][j];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      if (i == k) continue;
      cx<double> f = A[i][k];
#pragma unroll
      for (int j = 0; j < 6; ++j) A[i][j] = j == k ? -(f * inv) : A[i][j] - f * A[k][j];
    }
  }
#pragma unroll
  for (int k = 5; k >= 0; --k)
#pragma unroll
    for (int j = k + 1; j < 6; ++j) {
      bool sw = (prow[k] == j);
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        cx<double> a = A[i][k], b = A[i][j];
        A[i][k] = sw ? b : a;
        A[i][j] = sw ? a : b;
      }
    }
  // pack the (Hermitian) inverse, symmetrised
#pragma unroll
  for (int i = 0; i < 6; ++i) r[i] = A[i][i].re;
#pragma unroll
  for (int i = 0; i < 6; ++i)
#pragma unroll
    for (int j = i + 1; j < 6; ++j) {
      int o = herm6_off(i, j);
      r[o] = 0.5 * (A[i][j].re + A[j][i].re);
      r[o + 1] = 0.5 * (A[i][j].im - A[j][i].im);
    }
}

__device__ inline double wave_min(double v) {
  for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off));
  return v;
}
__device__ inline double wave_max(double v) {
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off));
  return v;
}

// HBM bound (2.4 GB at 64 x 32^3: 0.56 ms, 4.3 TB/s).  One work-item per block
// of a site (grid.y: chirality), in place, so that two waves share a SIMD (a
// work-item per site with a separate inverse held 372 registers, one wave a
// SIMD: 1.02 ms); a fixed number of
// wavefronts walk the sites, so that only those update the shared statistics.
__global__ __launch_bounds__(64, 2) void k_clover_invert(int Ve, const double2* __restrict__ Ho,
                                                         double2* __restrict__ Hi, InvStats st) {
  double mp = 1e300, mx = 0.0;
  unsigned long long nsing = 0;
  const size_t sVe = Ve, off = (size_t)18 * blockIdx.y * sVe;
  for (int64_t h = (int64_t)blockIdx.x * 64 + threadIdx.x; h < Ve; h += (int64_t)gridDim.x * 64) {
    double r[36];
#pragma unroll
    for (int k = 0; k < 18; ++k) {
      double2 v = ld_stream(&Ho[off + k * sVe + h]);
      r[2 * k] = v.x;
      r[2 * k + 1] = v.y;
    }
    double piv, nrm;
    invert6(r, piv, nrm);
    mp = fmin(mp, piv);
    mx = fmax(mx, nrm);
    if (!(piv >= 1e-14 * nrm)) ++nsing;  // also counts NaN
#pragma unroll
    for (int k = 0; k < 18; ++k) st_stream(&Hi[off + k * sVe + h], make_double2(r[2 * k], r[2 * k + 1]));
  }
  mp = wave_min(mp);
  mx = wave_max(mx);
  for (int o = 32; o > 0; o >>= 1) nsing += __shfl_xor(nsing, o);
  if (threadIdx.x == 0) {
    atomicMin(st.min_pivot_bits, (unsigned long long)__double_as_longlong(mp));
    atomicMax(st.max_norm_bits, (unsigned long long)__double_as_longlong(mx));
    if (nsing) atomicAdd(st.n_singular, nsing);
  }
}

// FP64 [36][Ve] double2 -> FP32 [18][Ve] float4
__global__ __launch_bounds__(QXD_BLOCK) void k_clover_cast(int Ve, const double2* __restrict__ in,
                                                           float4* __restrict__ out) {
  int64_t t = (int64_t)blockIdx.x * QXD_BLOCK + threadIdx.x;
  if (t >= (int64_t)18 * Ve) return;
  int k = (int)(t / Ve), h = (int)(t % Ve);
  size_t sVe = Ve;
  double2 a = in[(2 * k) * sVe + h], b = in[(2 * k + 1) * sVe + h];
  out[k * sVe + h] = make_float4((float)a.x, (float)a.y, (float)b.x, (float)b.y);
}

static qxd_status alloc_clover(qxd_handle* h) {
  if (h->He64) return QXD_OK;
  size_t n64 = (size_t)36 * h->Ve * sizeof(double2);
  if (!dev_alloc(&h->He64, n64) || !dev_alloc(&h->Ho64, n64) || !dev_alloc(&h->Hi64, n64)) {
    for (double2** p : {&h->He64, &h->Ho64, &h->Hi64}) {  // all or none, so that the next call allocates again
      if (*p) (void)hipFree(*p);
      *p = nullptr;
    }
    return QXD_ENOMEM;
  }
  return QXD_OK;
}

qxd_status ensure_link_copies(qxd_handle* h, unsigned which, hipStream_t s);  // gauge.hip

qxd_status ensure_copies(qxd_handle* h, unsigned which, hipStream_t s) {
  QXD_TRY(ensure_link_copies(h, which, s));
  const size_t n32 = (size_t)18 * h->Ve * sizeof(float4);
  const int g18 = div_up(18 * h->Ve, QXD_BLOCK);
  struct {
    unsigned bit;
    bool ready;
    double2* src;
    float4** dst;
  } cl[3] = {{CP_HE32, h->has_clover, h->He64, &h->He32},
             {CP_HO32, h->has_clover, h->Ho64, &h->Ho32},
             {CP_HI32, h->has_inverse, h->Hi64, &h->Hi32}};
  for (auto& c : cl) {
    if (!(which & c.bit) || (h->copies & c.bit)) continue;
    if (!c.ready) return QXD_ESTATE;
    if (!*c.dst && !dev_alloc(c.dst, n32)) return QXD_ENOMEM;
    hipLaunchKernelGGL(k_clover_cast, dim3(g18), dim3(QXD_BLOCK), 0, s, (int)h->Ve, c.src, *c.dst);
    QXD_HIP(hipGetLastError());
    h->copies |= c.bit;
  }
  return QXD_OK;
}

extern "C" qxd_status qxd_clover_build(qxd_handle* h, void* stream) {
  if (!h) return QXD_EINVAL;
  if (!h->has_flavour || !h->Uphys) return QXD_ESTATE;
  QXD_TRY(alloc_clover(h));
  hipStream_t s = as_stream(stream);
  PhysExt2 pe;
  for (int m = 0; m < 4; ++m) pe.L[m] = h->g.L[m];
  pe.Vphys = h->Vphys;
  double cq = h->fl.u1csw * (double)h->fl.qhat;
  double diag = 1.0 / (2.0 * h->fl.kappa);
  hipLaunchKernelGGL(k_clover_build, dim3(div_up(h->Vphys, 64)), dim3(64 * kClW), 0, s, h->geo, pe,
                     reinterpret_cast<const double2*>(h->Uphys), h->Aphys, h->fl.su3csw, cq, diag, h->He64,
                     h->Ho64);
  QXD_HIP(hipGetLastError());
  h->has_clover = true;
  h->has_inverse = false;
  h->copies &= ~(CP_HE32 | CP_HO32 | CP_HI32);
  return QXD_OK;
}

extern "C" qxd_status qxd_clover_invert(qxd_handle* h, qxd_clover_stats* stats, void* stream) {
  if (!h) return QXD_EINVAL;
  if (!h->has_clover) return QXD_ESTATE;
  hipStream_t s = as_stream(stream);
  unsigned long long* d = reinterpret_cast<unsigned long long*>(h->scal + QXD_NSCAL - 8);
  unsigned long long init[3] = {(unsigned long long)__builtin_bit_cast(long long, 1e300), 0ull, 0ull};
  QXD_HIP(hipMemcpyAsync(d, init, sizeof(init), hipMemcpyHostToDevice, s));
  InvStats st{d, d + 1, d + 2};
  hipLaunchKernelGGL(k_clover_invert, dim3(std::min(div_up(h->Ve, 64), 1024), 2), dim3(64), 0, s, (int)h->Ve, h->Ho64, h->Hi64, st);
  QXD_HIP(hipGetLastError());
  h->copies &= ~CP_HI32;
  unsigned long long res[3];
  QXD_HIP(hipMemcpyAsync(res, d, sizeof(res), hipMemcpyDeviceToHost, s));
  QXD_HIP(hipStreamSynchronize(s));
  double mp = __builtin_bit_cast(double, (long long)res[0]);
  double mx = __builtin_bit_cast(double, (long long)res[1]);
  if (stats) {
    stats->min_pivot = mp;
    stats->max_norm = mx;
    stats->n_singular = (int64_t)res[2];
  }
  if (res[2] != 0) return QXD_ESINGULAR;
  h->has_inverse = true;
  ++h->setup_gen;
  return QXD_OK;
}
