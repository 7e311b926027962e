// BLAS-1 launchers for the solvers (see blas.hip).
#pragma once

#include "qxd_internal.hpp"

#define QXD_NRED 1024   // workgroups of a reduction kernel (fixed: results are reproducible)

// This work-item's share of the sum of n workgroup partials: every QXD_BLOCK-th,
// in order, eight loads at a time (one after another they cost a trip to the
// last-level cache each: multi-shift CG 11.7 -> 11.3 ms at 16 x 8^3, FP32 CG 24.8
// -> 24.0 at 32 x 16^3, where a norm of D_hat leaves 2048 partials).
__device__ __forceinline__ double partial_share(const double* __restrict__ p, int n) {
  double a = 0.0;
  for (int i = threadIdx.x; i < n; i += 8 * QXD_BLOCK) {
    double v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = p[min(i + k * QXD_BLOCK, n - 1)];
#pragma unroll
    for (int k = 0; k < 8; ++k) a += i + k * QXD_BLOCK < n ? v[k] : 0.0;
  }
  return a;
}
#define QXD_MAXKV 32    // largest Krylov basis the fused multi-dot kernels take

struct Ptrs {
  const void* p[QXD_MAXKV];
};

template <class VT> void blas_norm2(qxd_handle* h, const VT* x, size_t n, double* slot, hipStream_t s);
template <class VT> void blas_cdot(qxd_handle* h, const VT* x, const VT* y, size_t n, double* slot, hipStream_t s);
template <class VT>
PartSum blas_cg_xr(qxd_handle* h, VT* x, VT* r, const VT* p, const VT* w, size_t n, int i_zz, int i_ww, PartSum ww,
                hipStream_t s);
template <class VT> void blas_cg_p(qxd_handle* h, VT* p, const VT* z, size_t n, int i_new, int i_old, PartSum zz, hipStream_t s);
template <class VT>
void blas_sub_norm(qxd_handle* h, VT* r, const VT* b, const VT* w, size_t n, double* slot, hipStream_t s);
// host (below): pinned memory that the sums are written to as well, or null
template <class VT>
void blas_mdot(qxd_handle* h, const Ptrs& basis, int k, const VT* v, size_t n, double* slots, hipStream_t s,
               double* host = nullptr);
// v -= sum_j c_j basis_j and, unless z is null (float4 only), z -= sum_j c_j zbasis_j;
// slots: |v|^2 and (v, r)
template <class VT>
void blas_gcr_update(qxd_handle* h, VT* v, const Ptrs& basis, VT* z, const Ptrs& zbasis, int k, const double* coef,
                     const VT* r, size_t n, double* slots, hipStream_t s, double* host = nullptr);
// from dots = |v|^2, (v, r): v /= |v|, r -= (v, r) v (also to r_copy), slot = |r|^2;
// unless z is null z /= |v|, x += (v, r) z
template <class VT>
void blas_gcr_step(qxd_handle* h, VT* v, VT* r, size_t n, const double* dots, double* slot, hipStream_t s,
                   double* host = nullptr, VT* r_copy = nullptr, VT* z = nullptr, VT* x = nullptr);
template <class VT>
void blas_multi_axpy(qxd_handle* h, VT* x, const Ptrs& basis, int k, const double* coef, size_t n, hipStream_t s);
template <class VT> void blas_zero(VT* x, size_t n, hipStream_t s);
// FP64 half field <-> FP32 half field (the layouts interleave components differently)
void blas_down(qxd_handle* h, float4* d, const double2* src, int i_n2, hipStream_t s);
void blas_up_acc(qxd_handle* h, double2* x, const float4* e, int i_n2, hipStream_t s);
