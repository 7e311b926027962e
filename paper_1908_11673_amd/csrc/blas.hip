// BLAS-1 kernels and deterministic reductions for the Krylov solvers.
//
// Vectors are half fields viewed as flat arrays of 16-byte words: double2 (one
// complex128) or float4 (two complex64).  Reductions are two-pass: each of a
// fixed number of workgroups reduces its grid-stride share (wave64 shuffles,
// then LDS) into one partial, and a single-workgroup kernel sums the partials in
// a fixed order, so results are bitwise reproducible run to run.  Scalars such as
// CG's alpha and beta are read by the update kernels straight from device
// memory; the host never waits inside an iteration.
#include <algorithm>
#include <type_traits>

#include "blas.hpp"

__device__ inline double red_block(double v, double* sh) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) s += sh[i];
  return s;
}

// Sums of several values over a wavefront at once.  With C > 1 values left, the
// two halves of the lanes (by bit M) exchange the half of the values that the
// other one keeps, so the C values cost C - 1 exchanges in all instead of C
// log2(64) ; then the one left is summed over the remaining bits.  Returns the
// total of value wave_sums_index(lane).
template <int C, int M>
__device__ __forceinline__ double wave_sums(double* v) {
  const bool up = (threadIdx.x & M) != 0;
  if constexpr (C > 1) {
#pragma unroll
    for (int i = 0; i < C / 2; ++i) {
      const double keep = up ? v[i + C / 2] : v[i], send = up ? v[i] : v[i + C / 2];
      v[i] = keep + __shfl_xor(send, M);
    }
    if constexpr (M > 1) return wave_sums<C / 2, M / 2>(v);
  } else {
    v[0] += __shfl_xor(v[0], M);
    if constexpr (M > 1) return wave_sums<1, M / 2>(v);
  }
  return v[0];
}
constexpr int pow2_from(int n) { return n <= 1 ? 1 : 2 * pow2_from((n + 1) / 2); }

// partial[j gridDim.x + blockIdx.x] = the workgroup's sum of a[j], j < NV: one
// barrier.  (A block reduction per value, two barriers each, took 15 us of a
// launch for the 30 values of 15 dots.)
template <int NV>
__device__ __forceinline__ void block_sums(const double* a, double* __restrict__ partial) {
  constexpr int P = pow2_from(NV), W = QXD_BLOCK / 64;
  static_assert(P <= 64, "values of a wave reduction");
  __shared__ double sh[W][P];
  double v[P];
#pragma unroll
  for (int j = 0; j < P; ++j) v[j] = j < NV ? a[j] : 0.0;
  const double t = wave_sums<P, 32>(v);
  const int lane = threadIdx.x & 63;
  if ((lane & (64 / P - 1)) == 0) sh[threadIdx.x >> 6][lane / (64 / P)] = t;
  __syncthreads();
  if (threadIdx.x < NV) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) s += sh[w][threadIdx.x];
    partial[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = s;
  }
}

// Workgroups of a streaming kernel over n elements: at most QXD_NRED, and no
// more than have an element (the others' sums would be zeros).
static int nred(size_t n) { return (int)std::max<size_t>(1, std::min<size_t>(QXD_NRED, (n + QXD_BLOCK - 1) / QXD_BLOCK)); }

// ---- word helpers ---------------------------------------------------------

__device__ inline double wnorm2(double2 a) { return a.x * a.x + a.y * a.y; }
__device__ inline double wnorm2(float4 a) { return (double)(a.x * a.x + a.y * a.y) + (double)(a.z * a.z + a.w * a.w); }
// conj(a) b
__device__ inline void wcdot(double2 a, double2 b, double& re, double& im) {
  re += a.x * b.x + a.y * b.y;
  im += a.x * b.y - a.y * b.x;
}
__device__ inline void wcdot(float4 a, float4 b, double& re, double& im) {
  re += (double)(a.x * b.x + a.y * b.y) + (double)(a.z * b.z + a.w * b.w);
  im += (double)(a.x * b.y - a.y * b.x) + (double)(a.z * b.w - a.w * b.z);
}
// y + (cr + i ci) x
__device__ inline double2 wcaxpy(double2 y, double cr, double ci, double2 x) {
  return make_double2(y.x + cr * x.x - ci * x.y, y.y + cr * x.y + ci * x.x);
}
__device__ inline float4 wcaxpy(float4 y, double crd, double cid, float4 x) {
  float cr = (float)crd, ci = (float)cid;
  return make_float4(y.x + cr * x.x - ci * x.y, y.y + cr * x.y + ci * x.x, y.z + cr * x.z - ci * x.w,
                     y.w + cr * x.w + ci * x.z);
}
__device__ inline double2 wscale(double2 x, double s) { return make_double2(s * x.x, s * x.y); }
__device__ inline float4 wscale(float4 x, double sd) {
  float s = (float)sd;
  return make_float4(s * x.x, s * x.y, s * x.z, s * x.w);
}
__device__ inline double2 wadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ inline float4 wadd(float4 a, float4 b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); }
__device__ inline double2 wsub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ inline float4 wsub(float4 a, float4 b) { return make_float4(a.x - b.x, a.y - b.y, a.z - b.z, a.w - b.w); }
__device__ inline bool wfinite(double2 a) { return isfinite(a.x) && isfinite(a.y); }

// Solver vectors are streamed once per kernel: loads and stores carry the
// non-temporal hint (ld_stream, st_stream).
#define GRID_STRIDE(i, n) for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < (n); i += (size_t)gridDim.x * blockDim.x)

// Traversal in rounds with QXD_UNR elements in flight per thread: in a round
// workgroup b takes the QXD_UNR * blockDim contiguous elements that start at
// round_start + b QXD_UNR blockDim, thread t the elements t, t + blockDim, ...
// of them, and all loads of the round (load(i) returns an element's words) are
// issued before the first element is used (use(i, words)).  The elements after
// the last full round go one at a time in a plain grid-stride loop.  (With a
// plain grid-stride loop, even unrolled, the compiler waits for an element's
// loads before issuing the next element's; with the elements of a round a grid
// apart, each wave reads several distant regions at once, which measured
// slower than contiguous rounds.)  The order is fixed, so the reductions stay
// reproducible.
#define QXD_UNR 4
template <class Load, class Use>
__device__ __forceinline__ void stream_for(size_t n, Load load, Use use) {
  const size_t B = blockDim.x, span = (size_t)gridDim.x * QXD_UNR * B;  // elements per round
  size_t start = 0;
  for (; start + span <= n; start += span) {
    const size_t i0 = start + (size_t)blockIdx.x * QXD_UNR * B + threadIdx.x;
    decltype(load(i0)) w[QXD_UNR];
#pragma unroll
    for (int u = 0; u < QXD_UNR; ++u) w[u] = load(i0 + u * B);
#pragma unroll
    for (int u = 0; u < QXD_UNR; ++u) use(i0 + u * B, w[u]);
  }
  for (size_t i = start + (size_t)blockIdx.x * B + threadIdx.x; i < n; i += (size_t)gridDim.x * B) use(i, load(i));
}
template <class VT>
struct W2 {
  VT a, b;
};

// ---- kernels ---------------------------------------------------------------

// One workgroup per value.  Latency bound (a few loads a work-item and one
// block reduction): about 3 us whatever nvals, where one workgroup taking the
// values in turn needed 45 us for the 30 values of 15 dots.
// host: also written there (pinned memory), unless null.
__global__ __launch_bounds__(QXD_BLOCK) void k_final_sum(const double* __restrict__ partial, int n, int stride,
                                                         double* __restrict__ out, double* __restrict__ host) {
  __shared__ double sh[QXD_BLOCK / 64];
  const int v = blockIdx.x;
  double s = red_block(partial_share(partial + (size_t)v * stride, n), sh);
  if (threadIdx.x == 0) {
    out[v] = s;
    if (host) host[v] = s;
  }
}

template <class VT>
__global__ __launch_bounds__(QXD_BLOCK) void k_norm2(const VT* __restrict__ x, size_t n, double* __restrict__ partial) {
  __shared__ double sh[QXD_BLOCK / 64];
  double a = 0.0;
  stream_for(n, [&](size_t i) { return ld_stream(&x[i]); }, [&](size_t, VT v) { a += wnorm2(v); });
  double s = red_block(a, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

template <class VT>
__global__ __launch_bounds__(QXD_BLOCK) void k_cdot(const VT* __restrict__ x, const VT* __restrict__ y, size_t n,
                                                    double* __restrict__ partial) {
  double a[2] = {0.0, 0.0};
  stream_for(n, [&](size_t i) { return W2<VT>{ld_stream(&x[i]), ld_stream(&y[i])}; },
             [&](size_t, W2<VT> v) { wcdot(v.a, v.b, a[0], a[1]); });
  block_sums<2>(a, partial);
}

// sum.n partials added up as k_final_sum does, for the whole workgroup; slot's value
// if there are none
__device__ inline double sum_here(PartSum sum, const double* __restrict__ slot, double* sh, double* bc) {
  if (sum.n == 0) return *slot;
  const double s = red_block(partial_share(sum.part, sum.n), sh);
  if (threadIdx.x == 0) *bc = s;
  __syncthreads();
  return *bc;
}

// CG: alpha = zz / ww; x += alpha p; r -= alpha w; partial |r|^2
template <class VT>
__global__ __launch_bounds__(QXD_BLOCK) void k_cg_xr(VT* __restrict__ x, VT* __restrict__ r, const VT* __restrict__ p,
                                                     const VT* __restrict__ w, size_t n, const double* __restrict__ scal,
                                                     int i_zz, int i_ww, PartSum ww, double* __restrict__ partial) {
  __shared__ double sh[QXD_BLOCK / 64], bc;
  double alpha = scal[i_zz] / sum_here(ww, &scal[i_ww], sh, &bc);
  double a = 0.0;
  struct W4 {
    VT x, p, r, w;
  };
  stream_for(
      n, [&](size_t i) { return W4{ld_stream(&x[i]), ld_stream(&p[i]), ld_stream(&r[i]), ld_stream(&w[i])}; },
      [&](size_t i, W4 v) {
        st_stream(&x[i], wcaxpy(v.x, alpha, 0.0, v.p));
        VT rr = wcaxpy(v.r, -alpha, 0.0, v.w);
        st_stream(&r[i], rr);
        a += wnorm2(rr);
      });
  double s = red_block(a, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// CG: beta = zz_new / zz_old; p = z + beta p; zz_new to its slot
template <class VT>
__global__ __launch_bounds__(QXD_BLOCK) void k_cg_p(VT* __restrict__ p, const VT* __restrict__ z, size_t n,
                                                    double* __restrict__ scal, int i_new, int i_old, PartSum zz) {
  __shared__ double sh[QXD_BLOCK / 64], bc;
  const double zn = sum_here(zz, &scal[i_new], sh, &bc);
  double beta = zn / scal[i_old];
  if (zz.n && blockIdx.x == 0 && threadIdx.x == 0) scal[i_new] = zn;
  stream_for(n, [&](size_t i) { return W2<VT>{ld_stream(&z[i]), ld_stream(&p[i])}; },
             [&](size_t i, W2<VT> v) { st_stream(&p[i], wcaxpy(v.a, beta, 0.0, v.b)); });
}

// r = b - w; partial |r|^2
template <class VT>
__global__ __launch_bounds__(QXD_BLOCK) void k_sub_norm(VT* __restrict__ r, const VT* __restrict__ b,
                                                        const VT* __restrict__ w, size_t n,
                                                        double* __restrict__ partial) {
  __shared__ double sh[QXD_BLOCK / 64];
  double a = 0.0;
  stream_for(n, [&](size_t i) { return W2<VT>{ld_stream(&b[i]), ld_stream(&w[i])}; },
             [&](size_t i, W2<VT> bw) {
               VT v = wsub(bw.a, bw.b);
               if (r) st_stream(&r[i], v);  // r = nullptr: the norm only
               a += wnorm2(v);
             });
  double s = red_block(a, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// The multi-vector kernels below are instantiated for every basis size K (0 ..
// QXD_MAXKV): with the count fixed at compile time all loads of an element
// (in groups of QXD_KGROUP) are issued before the first one is used, where a
// run-time count left the compiler waiting for each load in turn.  The
// arithmetic and its order are those of a plain loop over j.
#define QXD_KGROUP 16

// dots (basis_j, v) for j < K: partial[(2j) G + b] = Re, [(2j+1) G + b] = Im
template <class VT, int K>
__global__ __launch_bounds__(QXD_BLOCK) void k_mdot(Ptrs basis, const VT* __restrict__ v, size_t n,
                                                    double* __restrict__ partial) {
  double d[2 * K];
#pragma unroll
  for (int j = 0; j < 2 * K; ++j) d[j] = 0.0;
  GRID_STRIDE(i, n) {
    VT vi = ld_stream(&v[i]);
#pragma unroll
    for (int j0 = 0; j0 < K; j0 += QXD_KGROUP) {
      VT bj[QXD_KGROUP];
#pragma unroll
      for (int j = 0; j < QXD_KGROUP; ++j)
        if (j0 + j < K) bj[j] = ld_stream(&((const VT*)basis.p[j0 + j])[i]);
#pragma unroll
      for (int j = 0; j < QXD_KGROUP; ++j)
        if (j0 + j < K) wcdot(bj[j], vi, d[2 * (j0 + j)], d[2 * (j0 + j) + 1]);
    }
  }
  block_sums<2 * K>(d, partial);
}

// One Gram-Schmidt update of GCR: v -= sum_{j < K} c_j basis_j (c complex at
// coef[2j], coef[2j+1]), and with Z also z -= sum_j c_j zbasis_j; partials of
// |v|^2 and (v, r), so that the normalisation and the residual update that
// follow (k_gcr_step) need no pass of their own over v and r.
template <class VT, int K, bool Z>
__global__ __launch_bounds__(QXD_BLOCK) void k_gcr_update(VT* __restrict__ v, Ptrs basis, VT* __restrict__ z,
                                                          Ptrs zbasis, const double* __restrict__ coef,
                                                          const VT* __restrict__ r, size_t n,
                                                          double* __restrict__ partial) {
  double a[3] = {0.0, 0.0, 0.0};
  GRID_STRIDE(i, n) {
    VT vi = ld_stream(&v[i]);
    const VT ri = ld_stream(&r[i]);
    VT zi;
    if (Z) zi = ld_stream(&z[i]);
#pragma unroll
    for (int j0 = 0; j0 < K; j0 += QXD_KGROUP) {
      VT bj[QXD_KGROUP], zj[QXD_KGROUP];
#pragma unroll
      for (int j = 0; j < QXD_KGROUP; ++j)
        if (j0 + j < K) {
          bj[j] = ld_stream(&((const VT*)basis.p[j0 + j])[i]);
          if (Z) zj[j] = ld_stream(&((const VT*)zbasis.p[j0 + j])[i]);
        }
      if (Z) __builtin_amdgcn_sched_barrier(0);  // else the loads are issued one by one, each next to its use
#pragma unroll
      for (int j = 0; j < QXD_KGROUP; ++j)
        if (j0 + j < K) {
          const double cr = -coef[2 * (j0 + j)], ci = -coef[2 * (j0 + j) + 1];
          vi = wcaxpy(vi, cr, ci, bj[j]);
          if (Z) zi = wcaxpy(zi, cr, ci, zj[j]);
        }
    }
    if (K > 0) {
      st_stream(&v[i], vi);
      if (Z) st_stream(&z[i], zi);
    }
    a[0] += wnorm2(vi);
    wcdot(vi, ri, a[1], a[2]);
  }
  block_sums<3>(a, partial);
}

// The rest of a GCR step, from |v|^2 and (v, r) at dots: v /= |v|, r -= (v, r) v,
// the new r also to r_copy unless that is null; with z: z /= |v|, x += (v, r) z.
// Partial |r|^2.  A norm that is zero or not finite (a Krylov breakdown, e.g. on
// a vanishing source) sets v (and z) to zero instead, which leaves r (and x)
// unchanged.
template <class VT>
__global__ __launch_bounds__(QXD_BLOCK) void k_gcr_step(VT* __restrict__ v, VT* __restrict__ r, size_t n,
                                                        const double* __restrict__ dots, double* __restrict__ partial,
                                                        VT* __restrict__ r_copy, VT* __restrict__ z,
                                                        VT* __restrict__ x) {
  __shared__ double sh[QXD_BLOCK / 64];
  const double n2 = dots[0];
  const bool ok = n2 > 0.0 && n2 < INFINITY;
  const double sc = ok ? 1.0 / sqrt(n2) : 0.0;
  const double cr = ok ? sc * dots[1] : 0.0, ci = ok ? sc * dots[2] : 0.0;
  double a = 0.0;
  stream_for(n, [&](size_t i) { return W2<VT>{ld_stream(&r[i]), ld_stream(&v[i])}; },
             [&](size_t i, W2<VT> w) {
               const VT vi = ok ? wscale(w.b, sc) : VT{};
               st_stream(&v[i], vi);
               const VT ri = wcaxpy(w.a, -cr, -ci, vi);
               st_stream(&r[i], ri);
               if (r_copy) st_stream(&r_copy[i], ri);
               if (z) {
                 const VT zi = ok ? wscale(ld_stream(&z[i]), sc) : VT{};
                 st_stream(&z[i], zi);
                 st_stream(&x[i], wcaxpy(ld_stream(&x[i]), cr, ci, zi));
               }
               a += wnorm2(ri);
             });
  double s = red_block(a, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// x += sum_{j < K} c_j basis_j
template <class VT, int K>
__global__ __launch_bounds__(QXD_BLOCK) void k_multi_axpy(VT* __restrict__ x, Ptrs basis,
                                                          const double* __restrict__ coef, size_t n) {
  GRID_STRIDE(i, n) {
    VT xi = ld_stream(&x[i]);
#pragma unroll
    for (int j0 = 0; j0 < K; j0 += QXD_KGROUP) {
      VT bj[QXD_KGROUP];
#pragma unroll
      for (int j = 0; j < QXD_KGROUP; ++j)
        if (j0 + j < K) bj[j] = ld_stream(&((const VT*)basis.p[j0 + j])[i]);
#pragma unroll
      for (int j = 0; j < QXD_KGROUP; ++j)
        if (j0 + j < K) xi = wcaxpy(xi, coef[2 * (j0 + j)], coef[2 * (j0 + j) + 1], bj[j]);
    }
    st_stream(&x[i], xi);
  }
}

template <class VT>
__global__ __launch_bounds__(QXD_BLOCK) void k_zero(VT* __restrict__ x, size_t n) {
  GRID_STRIDE(i, n) x[i] = VT{};
}

// FP64 half field [12][Ve] double2 -> FP32 half field [6][Ve] float4: word
// j Ve + h holds components 2j and 2j+1 of site h.
// d = s / sqrt(scal[i_n2])
__global__ __launch_bounds__(QXD_BLOCK) void k_down(float4* __restrict__ d, const double2* __restrict__ s, size_t Ve,
                                                    const double* __restrict__ scal, int i_n2) {
  double sc = 1.0 / sqrt(scal[i_n2]);
  stream_for(
      6 * Ve,
      [&](size_t i) {
        size_t j = i / Ve, h = i - j * Ve;
        return W2<double2>{s[(2 * j) * Ve + h], s[(2 * j + 1) * Ve + h]};
      },
      [&](size_t i, W2<double2> w) {
        d[i] = make_float4((float)(sc * w.a.x), (float)(sc * w.a.y), (float)(sc * w.b.x), (float)(sc * w.b.y));
      });
}

// x (FP64) += sqrt(scal[i]) e (FP32), same component map as k_down
__global__ __launch_bounds__(QXD_BLOCK) void k_up_acc(double2* __restrict__ x, const float4* __restrict__ e, size_t Ve,
                                                      const double* __restrict__ scal, int i_n2) {
  double sc = sqrt(scal[i_n2]);
  // the elements of a round touch distinct words of x, so their loads may all
  // precede the stores
  struct W3 {
    float4 v;
    double2 a, b;
  };
  stream_for(
      6 * Ve,
      [&](size_t i) {
        size_t j = i / Ve, h = i - j * Ve;
        return W3{e[i], x[(2 * j) * Ve + h], x[(2 * j + 1) * Ve + h]};
      },
      [&](size_t i, W3 w) {
        size_t j = i / Ve, h = i - j * Ve;
        x[(2 * j) * Ve + h] = make_double2(w.a.x + sc * (double)w.v.x, w.a.y + sc * (double)w.v.y);
        x[(2 * j + 1) * Ve + h] = make_double2(w.b.x + sc * (double)w.v.z, w.b.y + sc * (double)w.v.w);
      });
}

// ---- host launchers -------------------------------------------------------

void launch_final_sum(const double* partial, int n, int nvals, int stride, double* out, hipStream_t s, double* host) {
  hipLaunchKernelGGL(k_final_sum, dim3(nvals), dim3(QXD_BLOCK), 0, s, partial, n, stride, out, host);
}

template <class VT>
void blas_norm2(qxd_handle* h, const VT* x, size_t n, double* slot, hipStream_t s) {
  hipLaunchKernelGGL(k_norm2<VT>, dim3(nred(n)), dim3(QXD_BLOCK), 0, s, x, n, h->partial);
  launch_final_sum(h->partial, nred(n), 1, nred(n), slot, s);
}
template <class VT>
void blas_cdot(qxd_handle* h, const VT* x, const VT* y, size_t n, double* slot, hipStream_t s) {
  hipLaunchKernelGGL(k_cdot<VT>, dim3(nred(n)), dim3(QXD_BLOCK), 0, s, x, y, n, h->partial);
  launch_final_sum(h->partial, nred(n), 2, nred(n), slot, s);
}
template <class VT>
PartSum blas_cg_xr(qxd_handle* h, VT* x, VT* r, const VT* p, const VT* w, size_t n, int i_zz, int i_ww, PartSum ww,
                   hipStream_t s) {
  static_assert(QXD_NRED <= QXD_PARTIAL_B, "partials of the residual");
  hipLaunchKernelGGL(k_cg_xr<VT>, dim3(nred(n)), dim3(QXD_BLOCK), 0, s, x, r, p, w, n, h->scal, i_zz, i_ww, ww,
                     h->partial_b);
  return PartSum{h->partial_b, nred(n)};
}
template <class VT>
void blas_cg_p(qxd_handle* h, VT* p, const VT* z, size_t n, int i_new, int i_old, PartSum zz, hipStream_t s) {
  hipLaunchKernelGGL(k_cg_p<VT>, dim3(nred(n)), dim3(QXD_BLOCK), 0, s, p, z, n, h->scal, i_new, i_old, zz);
}
template <class VT>
void blas_sub_norm(qxd_handle* h, VT* r, const VT* b, const VT* w, size_t n, double* slot, hipStream_t s) {
  hipLaunchKernelGGL(k_sub_norm<VT>, dim3(nred(n)), dim3(QXD_BLOCK), 0, s, r, b, w, n, h->partial);
  launch_final_sum(h->partial, nred(n), 1, nred(n), slot, s);
}
// one case per basis size 0 .. QXD_MAXKV
#define QXD_K_CASES(X)                                                                                         \
  X(0) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16) X(17) X(18) X(19) \
  X(20) X(21) X(22) X(23) X(24) X(25) X(26) X(27) X(28) X(29) X(30) X(31) X(32)
static_assert(QXD_MAXKV == 32, "QXD_K_CASES lists the basis sizes 0 .. QXD_MAXKV");

template <class VT>
void blas_mdot(qxd_handle* h, const Ptrs& basis, int k, const VT* v, size_t n, double* slots, hipStream_t s,
               double* host) {
  if (k < 1 || k > QXD_MAXKV) return;  // no dots
  const int G = nred(n);
  switch (k) {
#define QXD_CASE(K)                                                                                             \
  case K:                                                                                                     \
    if constexpr (K > 0)                                                                                      \
      hipLaunchKernelGGL((k_mdot<VT, K>), dim3(G), dim3(QXD_BLOCK), 0, s, basis, v, n, h->partial);           \
    break;
    QXD_K_CASES(QXD_CASE)
#undef QXD_CASE
  }
  launch_final_sum(h->partial, G, 2 * k, G, slots, s, host);
}
template <class VT>
void blas_gcr_update(qxd_handle* h, VT* v, const Ptrs& basis, VT* z, const Ptrs& zbasis, int k, const double* coef,
                     const VT* r, size_t n, double* slots, hipStream_t s, double* host) {
  const int G = nred(n);
  auto go = [&](auto kc) {
    constexpr int K = decltype(kc)::value;
    if (z) {
      // the coarse solver's vectors are float4 pairs
      if constexpr (std::is_same_v<VT, float4>)
        hipLaunchKernelGGL((k_gcr_update<VT, K, true>), dim3(G), dim3(QXD_BLOCK), 0, s, v, basis, z, zbasis, coef, r,
                           n, h->partial);
    } else {
      hipLaunchKernelGGL((k_gcr_update<VT, K, false>), dim3(G), dim3(QXD_BLOCK), 0, s, v, basis, z, zbasis, coef, r, n,
                         h->partial);
    }
  };
  switch (k) {
#define QXD_CASE(K)                           \
  case K:                                   \
    go(std::integral_constant<int, K>{});   \
    break;
    QXD_K_CASES(QXD_CASE)
#undef QXD_CASE
    default: return;  // callers keep 0 <= k <= QXD_MAXKV
  }
  launch_final_sum(h->partial, G, 3, G, slots, s, host);
}
template <class VT>
void blas_gcr_step(qxd_handle* h, VT* v, VT* r, size_t n, const double* dots, double* slot, hipStream_t s, double* host,
                   VT* r_copy, VT* z, VT* x) {
  hipLaunchKernelGGL(k_gcr_step<VT>, dim3(nred(n)), dim3(QXD_BLOCK), 0, s, v, r, n, dots, h->partial, r_copy, z, x);
  if (slot) launch_final_sum(h->partial, nred(n), 1, nred(n), slot, s, host);
}
template <class VT>
void blas_multi_axpy(qxd_handle* h, VT* x, const Ptrs& basis, int k, const double* coef, size_t n, hipStream_t s) {
  if (k == 0) return;  // x unchanged
  switch (k) {
#define QXD_CASE(K)                                                                                             \
  case K:                                                                                                     \
    hipLaunchKernelGGL((k_multi_axpy<VT, K>), dim3(nred(n)), dim3(QXD_BLOCK), 0, s, x, basis, coef, n);       \
    break;
    QXD_K_CASES(QXD_CASE)
#undef QXD_CASE
    default: return;
  }
}
template <class VT>
void blas_zero(VT* x, size_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_zero<VT>, dim3(nred(n)), dim3(QXD_BLOCK), 0, s, x, n);
}
void blas_down(qxd_handle* h, float4* d, const double2* src, int i_n2, hipStream_t s) {
  hipLaunchKernelGGL(k_down, dim3(nred(6 * (size_t)h->Ve)), dim3(QXD_BLOCK), 0, s, d, src, (size_t)h->Ve, h->scal, i_n2);
}
void blas_up_acc(qxd_handle* h, double2* x, const float4* e, int i_n2, hipStream_t s) {
  hipLaunchKernelGGL(k_up_acc, dim3(nred(6 * (size_t)h->Ve)), dim3(QXD_BLOCK), 0, s, x, e, (size_t)h->Ve, h->scal, i_n2);
}

#define INST(VT)                                                                                        \
  template void blas_norm2<VT>(qxd_handle*, const VT*, size_t, double*, hipStream_t);                  \
  template void blas_cdot<VT>(qxd_handle*, const VT*, const VT*, size_t, double*, hipStream_t);        \
  template PartSum blas_cg_xr<VT>(qxd_handle*, VT*, VT*, const VT*, const VT*, size_t, int, int, PartSum, \
                               hipStream_t);                                                            \
  template void blas_cg_p<VT>(qxd_handle*, VT*, const VT*, size_t, int, int, PartSum, hipStream_t);       \
  template void blas_sub_norm<VT>(qxd_handle*, VT*, const VT*, const VT*, size_t, double*, hipStream_t); \
  template void blas_mdot<VT>(qxd_handle*, const Ptrs&, int, const VT*, size_t, double*, hipStream_t,   \
                              double*);                                                                 \
  template void blas_gcr_update<VT>(qxd_handle*, VT*, const Ptrs&, VT*, const Ptrs&, int, const double*, \
                                    const VT*, size_t, double*, hipStream_t, double*);                  \
  template void blas_gcr_step<VT>(qxd_handle*, VT*, VT*, size_t, const double*, double*, hipStream_t,   \
                                  double*, VT*, VT*, VT*);                                              \
  template void blas_multi_axpy<VT>(qxd_handle*, VT*, const Ptrs&, int, const double*, size_t,          \
                                    hipStream_t);                                                       \
  template void blas_zero<VT>(VT*, size_t, hipStream_t);

INST(double2)
INST(float4)
