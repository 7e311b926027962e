// Gauge preparation on the extended lattice (Sec. 2.1 and 2.3 of arXiv:1908.11673):
// the mirror half U(x + L1 e1) = U(x)*, A(x + L1 e1) = -A(x) is filled from the
// physical half on the fly, and the combined links V(x,mu) = U(x,mu) z(x,mu)^qhat
// with z = exp(i A) are written in the even-odd SoA layout in FP64; the FP32 and
// bf16 copies are made from them when first needed.
#include <algorithm>

#include "qxd_internal.hpp"

struct PhysExt {
  int L[4];
  int64_t Vphys;
};

// The library's copy of the gauge field is component-major, [mu][9][Vphys]
// complex128, so that the kernels that walk it read contiguous words (the
// caller's order puts the nine entries of a link side by side: a wave's loads
// of one entry then touch every line of its 64 links).  Links s0 .. s0 + n of
// one direction, read as doubles (a caller's array need be no more aligned
// than that), transposed through LDS, entry k of site s at lds[9 s + k].
// HBM bound: read and written once, 0.56 ms at 64 x 32^3 (4.3 TB/s) where the
// plain device copy it replaces took 0.47 ms.
__global__ __launch_bounds__(QXD_BLOCK) void k_gauge_soa(int64_t n, const double* __restrict__ in,
                                                         double2* __restrict__ out, int64_t stride) {
  __shared__ double2 lds[9 * QXD_BLOCK];
  const int64_t s0 = (int64_t)blockIdx.x * QXD_BLOCK;
  const int m = (int)(n - s0 < QXD_BLOCK ? n - s0 : QXD_BLOCK);
  double* l = reinterpret_cast<double*>(lds);
  for (int i = threadIdx.x; i < 18 * m; i += QXD_BLOCK) l[i] = in[18 * s0 + i];
  __syncthreads();
  const int t = threadIdx.x;
  if (t < m) {
#pragma unroll
    for (int k = 0; k < 9; ++k) out[k * stride + s0 + t] = lds[9 * t + k];
  }
}

// V = U z^qhat on one physical link and, with C*, its mirror image V* (x1 +
// L1): one read of the gauge field writes both halves of the extended lattice.
// HBM bound (gauge field in, FP64 links out): 64 x 32^3 1.25 -> 0.67 ms against
// one work-item per extended link and the caller's order.
__global__ __launch_bounds__(QXD_BLOCK) void k_make_links(Geo g, PhysExt pe, const double2* __restrict__ U,
                                                           const double* __restrict__ A, int qhat,
                                                           double2* __restrict__ V64) {
  const uint32_t s = blockIdx.x * QXD_BLOCK + threadIdx.x;  // Vphys < 2^31
  const int mu = blockIdx.y;
  if (s >= pe.Vphys) return;
  const int x3 = s % (uint32_t)pe.L[3];
  uint32_t r = s / (uint32_t)pe.L[3];
  const int x2 = r % (uint32_t)pe.L[2];
  r /= (uint32_t)pe.L[2];
  const int x1 = r % (uint32_t)pe.L[1], x0 = r / (uint32_t)pe.L[1];
  const double a = A[mu * pe.Vphys + s];
  double sn, cs;
  sincos((double)qhat * a, &sn, &cs);
  const cx<double> z = mk(cs, sn);
  const size_t Ve = g.Ve;
  // the mirror site has the same parity: L1 is even
  const int p = (x0 + x1 + x2 + x3) & 1;
  double2* V = V64 + (size_t)(p * 4 + mu) * 9 * Ve;
  const int h = geo_half(g, x0, x1, x2, x3);
  const int hm = geo_half(g, x0, x1 + pe.L[1], x2, x3);
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const double2 u = U[(mu * 9 + k) * pe.Vphys + s];
    const cx<double> v = mk(u.x, u.y) * z;
    V[k * Ve + h] = make_double2(v.re, v.im);
    if (g.cstar >= 1) V[k * Ve + hm] = make_double2(v.re, -v.im);
  }
}

// FP32 and bf16 copies of the links (each entry rounded to FP32, then to bf16),
// regrouped so that a site's entries form 16-byte words; these stay aligned
// because Ve is a multiple of 8 (every extent of the lattice is even).  HBM
// bound; one work-item per link writes whole words (64 x 32^3, FP32: 0.68 ms,
// 5.3 TB/s, against 0.88 ms with one work-item per entry).
// entry k of link (parity, mu, h) goes to float2 lk32_index(Ve, k, h) of the
// 9 Ve of (parity, mu)
__global__ __launch_bounds__(QXD_BLOCK) void k_link_cast32(int Ve, const double2* __restrict__ V64,
                                                            float2* __restrict__ V32) {
  const int h = blockIdx.x * QXD_BLOCK + threadIdx.x;
  if (h >= Ve) return;
  const size_t sVe = Ve, pm = blockIdx.y;
  const double2* in = V64 + pm * 9 * sVe + h;
  float2* out = V32 + pm * 9 * sVe;
  double2 v[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) v[k] = ld_stream(&in[k * sVe]);
#pragma unroll
  for (int j = 0; j < 4; ++j)
    reinterpret_cast<float4*>(out + lk32_index(sVe, 2 * j, h))[0] =
        make_float4((float)v[2 * j].x, (float)v[2 * j].y, (float)v[2 * j + 1].x, (float)v[2 * j + 1].y);
  out[lk32_index(sVe, 8, h)] = make_float2((float)v[8].x, (float)v[8].y);
}
// entry k of link (parity, mu, h) goes to word 4 h + k (k < 4), 4 Ve + 4 h + k - 4
// (k < 8) or 8 Ve + h (k = 8) of the 9 Ve words of (parity, mu)
__global__ __launch_bounds__(QXD_BLOCK) void k_link_cast16(int Ve, const double2* __restrict__ V64,
                                                            uint32_t* __restrict__ V16) {
  const int h = blockIdx.x * QXD_BLOCK + threadIdx.x;
  if (h >= Ve) return;
  const size_t sVe = Ve, pm = blockIdx.y;
  const double2* in = V64 + pm * 9 * sVe + h;
  uint32_t* out = V16 + pm * 9 * sVe;
  uint32_t w[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const double2 v = ld_stream(&in[k * sVe]);
    w[k] = pack_bf16x2((float)v.x, (float)v.y);
  }
  reinterpret_cast<uint4*>(out)[h] = make_uint4(w[0], w[1], w[2], w[3]);
  reinterpret_cast<uint4*>(out + 4 * sVe)[h] = make_uint4(w[4], w[5], w[6], w[7]);
  out[8 * sVe + h] = w[8];
}

qxd_status ensure_link_copies(qxd_handle* h, unsigned which, hipStream_t s) {
  const int64_t n = (int64_t)2 * 4 * 9 * h->Ve;
  if ((which & CP_V32) && !(h->copies & CP_V32)) {
    if (!h->has_flavour) return QXD_ESTATE;
    if (!h->V32 && !dev_alloc(&h->V32, n * sizeof(float2))) return QXD_ENOMEM;
    hipLaunchKernelGGL(k_link_cast32, dim3(div_up(h->Ve, QXD_BLOCK), 8), dim3(QXD_BLOCK), 0, s, (int)h->Ve, h->V64,
                       h->V32);
    QXD_HIP(hipGetLastError());
    h->copies |= CP_V32;
  }
  if ((which & CP_V16) && !(h->copies & CP_V16)) {
    if (!h->has_flavour) return QXD_ESTATE;
    if (!h->V16 && !dev_alloc(&h->V16, n * sizeof(uint32_t))) return QXD_ENOMEM;
    hipLaunchKernelGGL(k_link_cast16, dim3(div_up(h->Ve, QXD_BLOCK), 8), dim3(QXD_BLOCK), 0, s, (int)h->Ve, h->V64,
                       h->V16);
    QXD_HIP(hipGetLastError());
    h->copies |= CP_V16;
  }
  return QXD_OK;
}

extern "C" qxd_status qxd_set_gauge(qxd_handle* h, const double* U_phys, const double* A_phys, int on_device,
                                    void* stream) {
  if (!h || !U_phys || !A_phys) return QXD_EINVAL;
  hipStream_t s = as_stream(stream);
  size_t nU = (size_t)4 * h->Vphys * 18 * sizeof(double);
  size_t nA = (size_t)4 * h->Vphys * sizeof(double);
  if (!h->Uphys) {
    if (!dev_alloc(&h->Uphys, nU)) return QXD_ENOMEM;
    if (!dev_alloc(&h->Aphys, nA)) {
      (void)hipFree(h->Uphys);  // both or neither
      h->Uphys = nullptr;
      return QXD_ENOMEM;
    }
  }
  double2* U = reinterpret_cast<double2*>(h->Uphys);
  const int64_t V = h->Vphys;
  if (on_device) {
    for (int mu = 0; mu < 4; ++mu)
      hipLaunchKernelGGL(k_gauge_soa, dim3(div_up(V, QXD_BLOCK)), dim3(QXD_BLOCK), 0, s, V, U_phys + mu * V * 18,
                         U + mu * 9 * V, V);
    QXD_HIP(hipGetLastError());
    QXD_HIP(hipMemcpyAsync(h->Aphys, A_phys, nA, hipMemcpyDeviceToDevice, s));
  } else {
    // in parts through the room of the angles, which are copied last: no device
    // memory beyond what is kept
    const int64_t part = (int64_t)(nA / (18 * sizeof(double)));  // 2 V / 9 links, V >= 16
    double* stage = h->Aphys;
    QXD_HIP(hipStreamSynchronize(s));
    for (int mu = 0; mu < 4; ++mu)
      for (int64_t s0 = 0; s0 < V; s0 += part) {
        const int64_t n = std::min(part, V - s0);
        QXD_HIP(hipMemcpy(stage, U_phys + (mu * V + s0) * 18, (size_t)n * 18 * sizeof(double), hipMemcpyHostToDevice));
        hipLaunchKernelGGL(k_gauge_soa, dim3(div_up(n, QXD_BLOCK)), dim3(QXD_BLOCK), 0, s, n, stage,
                           U + mu * 9 * V + s0, V);
        QXD_HIP(hipGetLastError());
        QXD_HIP(hipStreamSynchronize(s));  // the next part takes the same room
      }
    QXD_HIP(hipMemcpy(h->Aphys, A_phys, nA, hipMemcpyHostToDevice));
  }
  h->has_gauge = true;
  h->has_flavour = h->has_clover = h->has_inverse = false;
  return QXD_OK;
}

extern "C" qxd_status qxd_set_flavour(qxd_handle* h, const qxd_flavour* f, void* stream) {
  if (!h || !f) return QXD_EINVAL;
  if (!h->has_gauge) return QXD_ESTATE;
  if (!(f->kappa > 0.0) || !(f->invqel > 0.0)) return QXD_EINVAL;
  hipStream_t s = as_stream(stream);
  size_t nl = (size_t)2 * 4 * 9 * h->Ve;
  if (!h->V64 && !dev_alloc(&h->V64, nl * sizeof(double2))) return QXD_ENOMEM;
  h->copies = 0;
  PhysExt pe;
  for (int m = 0; m < 4; ++m) pe.L[m] = h->g.L[m];
  pe.Vphys = h->Vphys;
  hipLaunchKernelGGL(k_make_links, dim3(div_up(h->Vphys, QXD_BLOCK), 4), dim3(QXD_BLOCK), 0, s, h->geo, pe,
                     reinterpret_cast<const double2*>(h->Uphys), h->Aphys, f->qhat, h->V64);
  QXD_HIP(hipGetLastError());
  h->fl = *f;
  h->has_flavour = true;
  h->has_clover = h->has_inverse = false;
  return QXD_OK;
}
