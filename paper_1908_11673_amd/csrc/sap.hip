// Schwarz alternating procedure (SAP): the paper's domain-decomposition
// preconditioner for GCR (Sec. 4.4, SAP+GCR), on the full Wilson-clover
// operator in FP32.
//
// The extended lattice is cut into 4^4 blocks coloured by the parity of their
// block coordinates.  A half cycle on colour c: on every block B of colour c,
// r_B = (eta - D x)_B, then nmr minimal-residual steps on the block operator D_B
// (D restricted to B, hops leaving B dropped) from e = 0, and x_B += e.  Blocks
// of one colour are never neighbours, so a half cycle is one launch with one
// workgroup per block and no races: x is read outside the block (other colour)
// and written inside it.  ncy cycles (colour 0 then 1) from x = 0 give M eta.
//
// Block solver.  The paper's SAP solves the blocks by minimal-residual steps
// on the block's even-odd Schur complement D_hat_B = H_ee - D_eo H_oo^-1 D_oe,
// from the source r_e - D_eo H_oo^-1 r_o, and back-substitutes
// e_o = H_oo^-1 (r_o - D_oe e_e) (eo = 1); eo = 0 runs the steps on D_B itself.
//
// Block layout.  The even-odd half fields keep x3 fastest, so the 256 sites of
// a block sit in runs of two consecutive half indices, and a workgroup reading
// them would use a fraction of every cache line it pulls.  SAP therefore works
// on copies in block order: component k of the site in slot t of block B at
// (B * ncomp + k) * 256 + t, blocks numbered colour-major (B = colour * nhalf +
// j, j the workgroup of that colour's launch).  The plain solver keeps the
// local index s = 64 l0 + 16 l1 + 4 l2 + l3 as the slot; the even-odd one sorts
// a block's sites by parity, the site of parity q in slot 128 q + s / 2, so
// that each wavefront holds sites of one parity.  The
// links (36 float2 a site, forward links of both parities), the clover blocks
// (18 float4) and, on odd sites, their inverses are copied once per gauge field
// and flavour; the iterate x and the source eta (6 float4) live in block order
// for the whole application: the first half cycle reads the source, and each
// block's last one writes x to the half fields of the output.
//
// A workgroup of 256 threads owns one block, one thread per site; a site keeps
// its four forward links in registers.  A hop exchange publishes the spinor of
// the sending sites (24.6 kB of LDS for all 256) and, for each direction, the
// backward hop each owes its forward neighbour, (1 + g_mu) U^+ rho as two
// colour vectors (49.2 kB): 75 kB of LDS per block, so two blocks share a CU.
// Hops that leave the block read a slot of zeros, so an exchange has no branch.
// With eo = 1 the even wavefronts send while the odd ones receive and the other
// way round; senders and receivers touch disjoint slots, so one barrier per
// exchange suffices.  The block reductions of the minimal-residual step go
// through LDS.
//
// The residual of a block is formed from x at every visit, through the same
// exchange for the hops inside the block; the hops across its faces run a wave a
// direction on full waves.  FP32 rounding of earlier solves is then part of what
// the next one corrects.  Sums of hops start at zero and the clover product,
// which is larger, is added to them last.  Relative error against complex128 at
// 32 x 16^3, 2 cycles of 8 steps: 1.14e-7 plain, 1.16e-7 even-odd; with the
// residual carried over from the last solve and the hops added to the clover
// product 1.45e-7 and 1.67e-7, growing with the cycles.  (Carried, a plain
// application at 64 x 32^3 took 3035 us where it takes 3110, an even-odd one of
// 5 cycles at 32 x 16^3 655 where it takes 711.)
//
// What bounds it: vector instruction issue with plain blocks (95 % of the cycles
// of the first half cycle, 87 % of those that form a residual; 1400 instructions
// a site and step, of which the products, projections and sums of the method
// are 1350).  64 x 32^3, 8 steps: the first half cycle 715 us, the first on the
// other colour 767, later ones 880 to 895 (825, 954, 954 and 1068 with branches in
// the exchange and face hops in the site's own work-item).  The even-odd blocks
// wait at three exchanges a step (39 % issue): 5 steps at 32 x 16^3, 512 blocks, 72
// us (114), 24 less by the exchange without branches and 17 by separate code for
// the waves of either parity (their registers do not add up) that loads while
// the other parity works.
#include "blas.hpp"
#include "sap_blocks.hpp"

namespace {

// Block-order copies of the links, the clover blocks and, for EO, the inverses
// on odd sites (one thread per site; CIb holds 128 odd slots a block).  The
// blocks are stored as -2 H and H_oo^-1 / 2 (exact), so that the hops add to
// their products without a factor: -2 D_B f = -2 H f + hops(f).
template <bool EO>
__global__ __launch_bounds__(kSapSites) void k_sap_pack(Geo g, SapGeo sb, const float2* __restrict__ V32,
                                                        const float4* __restrict__ He,
                                                        const float4* __restrict__ Ho,
                                                        const float4* __restrict__ Hi, float2* __restrict__ Vb,
                                                        float4* __restrict__ Cb, float4* __restrict__ CIb) {
  const int B = blockIdx.x, colour = B >= sb.nhalf ? 1 : 0;
  int c0, c1, c2, c3;
  sap_block_coords(sb, colour, B - colour * sb.nhalf, c0, c1, c2, c3);
  const int t = threadIdx.x;
  int l0, l1, l2, l3;
  sap_local<EO>(t, l0, l1, l2, l3);
  const int x0 = kSapB * c0 + l0, x1 = kSapB * c1 + l1, x2 = kSapB * c2 + l2, x3 = kSapB * c3 + l3;
  const int p = (x0 + x1 + x2 + x3) & 1;
  const size_t Ve = g.Ve, h = geo_half(g, x0, x1, x2, x3);
  const float2* Vp = V32 + (size_t)p * 36 * Ve;
  const float4* Hp = p ? Ho : He;
  float2* vb = sap_blk<36>(Vb, B);
  float4* cb = sap_blk<18>(Cb, B);
#pragma unroll 4
  for (int k = 0; k < 36; ++k) vb[k * kSapSites + t] = Vp[(size_t)(k / 9) * 9 * Ve + lk32_index(Ve, k % 9, h)];
#pragma unroll 6
  for (int k = 0; k < 18; ++k) {
    const float4 v = Hp[k * Ve + h];
    cb[k * kSapSites + t] = make_float4(-2.f * v.x, -2.f * v.y, -2.f * v.z, -2.f * v.w);
  }
  if (EO && p) {
    float4* ci = CIb + (size_t)B * 18 * (kSapSites / 2) + (t - kSapSites / 2);
#pragma unroll 6
    for (int k = 0; k < 18; ++k) {
      const float4 v = Hi[k * Ve + h];
      ci[k * (kSapSites / 2)] = make_float4(0.5f * v.x, 0.5f * v.y, 0.5f * v.z, 0.5f * v.w);
    }
  }
}

// The hops that cross the block's faces, a wave a direction MU: lane (a, b, c)
// takes the face sites whose other coordinates (in rising order of direction)
// are a, b, c.  face[MU][0]: forward from the sites l = 3, their own link times
// the neighbour's spinor; face[MU][1]: backward from l = 0, the neighbour's link.
// Both as the multiplied two-spinors, which the sites collect afterwards.  (In
// the site's own work-item each of the eight hops would run on a quarter of the
// lanes.)
constexpr int kFaceZero = 64, kFaceSlots = 66;
typedef float2 SapFace[2][6][kFaceSlots];

template <int MU, bool EO>
__device__ __forceinline__ void sap_face_hops(const Geo& g, const SapGeo& sb, const int c[4], int B, int lane,
                                              const float4* __restrict__ Xb, const float2* __restrict__ Vb,
                                              SapFace* face) {
  int l[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) l[m] = (lane >> (m < MU ? 4 - 2 * m : 6 - 2 * m)) & 3;
#pragma unroll
  for (int dir = 0; dir < 2; ++dir) {
    l[MU] = dir == 0 ? kSapB - 1 : 0;
    int x0 = kSapB * c[0] + l[0], x1 = kSapB * c[1] + l[1], x2 = kSapB * c[2] + l[2], x3 = kSapB * c[3] + l[3];
    bool neg;
    if (dir == 0)
      geo_step<MU, +1>(g, x0, x1, x2, x3, neg);
    else
      geo_step<MU, -1>(g, x0, x1, x2, x3, neg);
    const int bs = sap_bsite<EO>(sb, x0, x1, x2, x3);
    cx<float> s[12], u[9], h0[3], h1[3], w0[3], w1[3];
    sp_load(sap_blk<6>(Xb, bs >> 8), kSapSites, bs & 255, s);
    const float2* vb = dir == 0 ? sap_blk<36>(Vb, B) + sap_slot<EO>((l[0] << 6) | (l[1] << 4) | (l[2] << 2) | l[3])
                                : sap_blk<36>(Vb, bs >> 8) + (bs & 255);
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const float2 v = vb[(MU * 9 + k) * kSapSites];
      u[k] = mk(v.x, v.y);
    }
    if (dir == 0) {
      spin_project<MU, true>(s, h0, h1);
      sap_colour_mul<true>(u, h0, h1, w0, w1);
    } else {
      spin_project<MU, false>(s, h0, h1);
      sap_colour_mul<false>(u, h0, h1, w0, w1);
    }
    const float sg = MU == 0 && neg ? -1.f : 1.f;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      face[MU][dir][k][lane] = make_float2(sg * w0[k].re, sg * w0[k].im);
      face[MU][dir][3 + k][lane] = make_float2(sg * w1[k].re, sg * w1[k].im);
    }
  }
}

// acc += the hops along MU that leave the block at the site w
template <int MU>
__device__ __forceinline__ void sap_face_add(const SapFace* face, const SapSite& w, cx<float> acc[12]) {
  const int l[4] = {w.l0, w.l1, w.l2, w.l3};
  const int i = MU == 0   ? (w.l1 << 4) | (w.l2 << 2) | w.l3
                : MU == 1 ? (w.l0 << 4) | (w.l2 << 2) | w.l3
                : MU == 2 ? (w.l0 << 4) | (w.l1 << 2) | w.l3
                          : (w.l0 << 4) | (w.l1 << 2) | w.l2;
#pragma unroll
  for (int dir = 0; dir < 2; ++dir) {
    const int at = l[MU] == (dir == 0 ? kSapB - 1 : 0) ? i : kFaceZero;
    cx<float> w0[3], w1[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float2 a = face[MU][dir][k][at], b = face[MU][dir][3 + k][at];
      w0[k] = mk(a.x, a.y);
      w1[k] = mk(b.x, b.y);
    }
    if (dir == 0)
      spin_rebuild_add<MU, true>(acc, w0, w1);
    else
      spin_rebuild_add<MU, false>(acc, w0, w1);
  }
}

// (v, rho) / (v, v) over the first NW waves of the workgroup (one barrier).
template <int NW>
__device__ __forceinline__ cx<float> sap_alpha(SapLds& L, int t, const cx<float> v[12], const cx<float> rho[12]) {
  float are = 0.f, aim = 0.f, nn = 0.f;
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    are = fmaf(v[c].re, rho[c].re, are);  // conj(v) rho
    are = fmaf(v[c].im, rho[c].im, are);
    aim = fmaf(v[c].re, rho[c].im, aim);
    aim = fmaf(-v[c].im, rho[c].re, aim);
    nn = fmaf(v[c].re, v[c].re, nn);
    nn = fmaf(v[c].im, v[c].im, nn);
  }
  are = sap_wave_sum(are);
  aim = sap_wave_sum(aim);
  nn = sap_wave_sum(nn);
  const int wave = t >> 6;
  if ((t & 63) == 0) {
    L.red[0][wave] = are;
    L.red[1][wave] = aim;
    L.red[2][wave] = nn;
  }
  __syncthreads();
  are = aim = nn = 0.f;
#pragma unroll
  for (int k = 0; k < NW; ++k) {
    are += L.red[0][k];
    aim += L.red[1][k];
    nn += L.red[2][k];
  }
  // a block whose residual vanished stays put
  return nn > 0.f ? mk(are / nn, aim / nn) : mk(0.f, 0.f);
}

// The minimal-residual step along rho from v = -2 D rho: with a = (v, rho) /
// (v, v) = -alpha / 2, e += alpha rho and rho -= alpha D rho = a v.
__device__ __forceinline__ void sap_step(cx<float> a, const cx<float> v[12], cx<float> rho[12], cx<float> e[12]) {
  const cx<float> alpha = -2.f * a, na = -a;
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    sap_cmac(e[c], alpha, rho[c]);
    sap_cmac(rho[c], na, v[c]);
  }
}

// nmr minimal-residual steps on D_B from e = 0; rho: the residual
__device__ __forceinline__ void sap_solve(SapLds& L, int t, int nmr, const float4* __restrict__ cb,
                                          const cx<float> (*U)[9], cx<float> rho[12], cx<float> e[12]) {
  sap_zero(e);
  for (int step = 0; step < nmr; ++step) {
    // v = -2 D_B rho = hops(rho) - 2 H rho; every read of the previous step's
    // exchange buffers came before its reduction barrier
    cx<float> v[12];
    sap_publish<false>(L, t, rho, U);
    __syncthreads();
    sap_zero(v);
    sap_gather<false>(L, t, U, v);
    sap_clover_add<kSapSites>(cb, rho, v);
    sap_step(sap_alpha<4>(L, t, v, rho), v, rho, e);
  }
}

// The even-odd preconditioned solve: nmr steps on the block's Schur complement,
// then the odd sites by back substitution.  The two functions run side by side
// on the even and the odd waves and meet at the same barriers: the even sites
// hold rho = r_e, then the Schur residual, and return e_e; the odd sites hold
// rho = r_o and return e_o.  Sends and receives of one exchange touch the slots
// of opposite parities, so a wave may publish right after it gathered.  While
// the even waves work the odd ones request the clover inverse.
__device__ __forceinline__ void sap_solve_even(SapLds& L, int t, int nmr, bool odd_source,
                                               const float4* __restrict__ cb, const cx<float> (*U)[9],
                                               cx<float> rho[12], cx<float> e[12]) {
  __syncthreads();  // H_oo^-1 r_o / 2
  // r_e - D_eo H_oo^-1 r_o = r_e + hops(H_oo^-1 r_o / 2)
  if (odd_source) {
    sap_zero(e);  // free until the steps
    sap_gather<true>(L, t, U, e);
#pragma unroll
    for (int c = 0; c < 12; ++c) rho[c] = rho[c] + e[c];
  }
  sap_zero(e);
  for (int step = 0; step < nmr; ++step) {
    // v = -2 D_hat_B rho = hops(t_o) - 2 H_ee rho, t_o = (1/2) H_oo^-1 hops(rho)
    sap_publish<true>(L, t, rho, U);
    __syncthreads();
    __syncthreads();
    cx<float> v[12];
    sap_zero(v);
    sap_gather<true>(L, t, U, v);
    sap_clover_add<kSapSites>(cb, rho, v);
    sap_step(sap_alpha<2>(L, t, v, rho), v, rho, e);
  }
  sap_publish<true>(L, t, e, U);
  __syncthreads();
}

__device__ __forceinline__ void sap_solve_odd(SapLds& L, int t, int nmr, bool odd_source, const float4* __restrict__ ci,
                                              const cx<float> (*U)[9], const cx<float> rho[12], cx<float> e[12]) {
  constexpr int S = kSapSites / 2;
  cx<float> acc[12], to[12];
  if (odd_source) {
    sap_clover<S>(ci, rho, to);
    sap_publish<true>(L, t, to, U);
  }
  __syncthreads();
  for (int step = 0; step < nmr; ++step) {
    float r[36], r1[36];
    sap_clover_load<S, 0>(ci, r);
    sap_clover_load<S, 1>(ci, r1);
    __syncthreads();
    sap_zero(acc);
    sap_gather<true>(L, t, U, acc);
    sap_herm6(r, acc, to);
    sap_herm6(r1, acc + 6, to + 6);
    sap_publish<true>(L, t, to, U);
    __syncthreads();
    __syncthreads();  // the even sites' reduction
  }
  // e_o = H_oo^-1 (r_o - D_oe e_e) = (H_oo^-1 / 2) (2 r_o + hops(e_e))
  __syncthreads();
  sap_zero(acc);
  sap_gather<true>(L, t, U, acc);
#pragma unroll
  for (int c = 0; c < 12; ++c) acc[c] = 2.f * rho[c] + acc[c];
  sap_clover<S>(ci, acc, e);
}

// One half cycle on the blocks of `colour` (j = blockIdx.x; its partner is block
// j of the other colour, the other block of the pair {2 k3, 2 k3 + 1} along x3).
//   FIRST: the first of an application: x = 0, so the residual is the source,
//          read from the even half field eta_e (and the odd half eta_o when
//          given, else it is zero there) and copied to Eb for the block and its
//          partner;
//   else:  r = eta - D x from Eb and Xb; a block not yet visited has x = 0, and
//          only the hops across its faces count.
// last: the block's last visit: its x goes to out_e and, when given, out_o.  Xb
// gets it unless nobody reads it (keep_x).  EO: even-odd preconditioned block
// solves (waves 0, 1 hold the even sites).
template <bool FIRST, bool EO>
__global__ __launch_bounds__(kSapSites, 2) void k_sap_half(Geo g, SapGeo sb, int colour, int nmr,
                                                           bool visited, bool last, bool keep_x,
                                                           const float4* __restrict__ eta_e,
                                                           float4* __restrict__ Eb, float4* __restrict__ Xb,
                                                           const float2* __restrict__ Vb,
                                                           const float4* __restrict__ Cb,
                                                           const float4* __restrict__ CIb,
                                                           float4* __restrict__ out_e,
                                                           const float4* __restrict__ eta_o,
                                                           float4* __restrict__ out_o) {
  __shared__ SapLds L;
  const int j = blockIdx.x;
  int c[4];
  sap_block_coords(sb, colour, j, c[0], c[1], c[2], c[3]);
  const int B = colour * sb.nhalf + j;
  // EO: half the workgroups have their odd sites on waves 0, 1, so that the SIMDs
  // of a CU hold waves of both parities (with the even waves of both blocks on the
  // same two SIMDs the others idle while they work: 3 us more a half cycle)
  const int swap = EO && (((blockIdx.x >> 3) ^ (blockIdx.x >> 8)) & 1) ? kSapSites / 2 : 0;
  const SapSite w = sap_site<EO>(threadIdx.x ^ swap);
  // q: the site's parity (block origins are even), with EO the same in a wave
  const int t = w.t, q = EO ? __builtin_amdgcn_readfirstlane(w.t >> 7) : w.q;
  const int x0 = kSapB * c[0] + w.l0, x1 = kSapB * c[1] + w.l1, x2 = kSapB * c[2] + w.l2, x3 = kSapB * c[3] + w.l3;
  const size_t Ve = g.Ve;
  const float4* cb = sap_blk<18>(Cb, B) + t;
  const float4* ci = CIb + (size_t)B * 18 * (kSapSites / 2) + (t - kSapSites / 2);  // odd slots only
  float4* xb = sap_blk<6>(Xb, B);
  float4* eb = sap_blk<6>(Eb, B);

  // the site's four forward links stay in registers for the whole solve
  cx<float> U[4][9];
  {
    const float2* vb = sap_blk<36>(Vb, B) + t;
#pragma unroll
    for (int mu = 0; mu < 4; ++mu)
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        float2 v = vb[(mu * 9 + k) * kSapSites];
        U[mu][k] = mk(v.x, v.y);
      }
  }
  cx<float> rho[12];
  sap_zero(rho);
  if (FIRST) {
    if (q == 0 || eta_o) {
      // the partner's site in the same slot (same parity: x3 moves by 4)
      const int x3p = x3 + ((c[3] & 1) ? -kSapB : kSapB);
      const float4* src = q ? eta_o : eta_e;
      sp_load(src, Ve, geo_half(g, x0, x1, x2, x3), rho);
      if (!last) sp_store(eb, kSapSites, t, rho);
      cx<float> ep[12];
      sp_load(src, Ve, geo_half(g, x0, x1, x2, x3p), ep);
      sp_store(sap_blk<6>(Eb, (1 - colour) * sb.nhalf + j), kSapSites, t, ep);
    }
    sap_lds_init(L);
  } else {
    cx<float> acc[12];
    sap_zero(acc);
    if (visited) {
      cx<float> xs[12];
      sp_load(xb, kSapSites, t, xs);
      sap_lds_init(L);
      sap_publish<EO>(L, t, xs, U);
      __syncthreads();
      sap_gather<EO>(L, t, U, acc);
      __syncthreads();  // the faces take the place of the exchange buffers
    }
    SapFace* face = reinterpret_cast<SapFace*>(L.bw);
    static_assert(4 * sizeof(SapFace) <= sizeof(L.bw), "face hops");
    if (t < 48) face[t / 12][t / 6 & 1][t % 6][kFaceZero] = make_float2(0.f, 0.f);
    const int lane = t & 63;
    switch (__builtin_amdgcn_readfirstlane(t >> 6)) {
      case 0: sap_face_hops<0, EO>(g, sb, c, B, lane, Xb, Vb, face); break;
      case 1: sap_face_hops<1, EO>(g, sb, c, B, lane, Xb, Vb, face); break;
      case 2: sap_face_hops<2, EO>(g, sb, c, B, lane, Xb, Vb, face); break;
      default: sap_face_hops<3, EO>(g, sb, c, B, lane, Xb, Vb, face); break;
    }
    if (q == 0 || eta_o) sp_load(eb, kSapSites, t, rho);
    __syncthreads();
    sap_face_add<0>(face, w, acc);
    sap_face_add<1>(face, w, acc);
    sap_face_add<2>(face, w, acc);
    sap_face_add<3>(face, w, acc);
    if (visited) {
      cx<float> xs[12];
      sp_load(xb, kSapSites, t, xs);
      sap_clover_add<kSapSites>(cb, xs, acc);
    }
#pragma unroll
    for (int k = 0; k < 12; ++k) rho[k] = rho[k] + 0.5f * acc[k];
    __syncthreads();  // the exchange buffers take the place of the faces
    sap_lds_init(L);
  }

  cx<float> e[12];  // the block solution
  if (!EO) {
    sap_solve(L, t, nmr, cb, U, rho, e);
  } else if (q == 0) {
    sap_solve_even(L, t, nmr, !FIRST || eta_o, cb, U, rho, e);
  } else {
    sap_solve_odd(L, t, nmr, !FIRST || eta_o, ci, U, rho, e);
  }
  if (visited) {
    cx<float> xs[12];
    sp_load(xb, kSapSites, t, xs);
#pragma unroll
    for (int k = 0; k < 12; ++k) e[k] = e[k] + xs[k];
  }
  if (last && (q == 0 || out_o)) sp_store(q ? out_o : out_e, Ve, geo_half(g, x0, x1, x2, x3), e);
  if (keep_x) sp_store(xb, kSapSites, t, e);
}

// workspace roles (free in the solvers' table): block-order links, clover
// blocks, iterate, source and odd-site clover inverses
enum { W_SAP_VB = 8, W_SAP_CB = 9, W_SAP_XB = 13, W_SAP_EB = 14, W_SAP_CIB = 15 };

struct SapArgs {
  Geo g;
  SapGeo sb;
  int nmr;
  const float4* eta_e;
  float4 *Eb, *Xb;
  const float2* Vb;
  const float4 *Cb, *CIb;
  float4* out_e;
  const float4* eta_o;
  float4* out_o;
};

// half cycle `colour` of cycle cy of ncy
template <bool FIRST, bool EO>
void sap_launch(const SapArgs& a, int cy, int ncy, int colour, hipStream_t s) {
  const bool last = cy == ncy - 1;
  hipLaunchKernelGGL((k_sap_half<FIRST, EO>), dim3(a.sb.nhalf), dim3(kSapSites), 0, s, a.g, a.sb, colour, a.nmr,
                     cy > 0, last, !(last && colour == 1), a.eta_e, a.Eb, a.Xb, a.Vb, a.Cb, a.CIb, a.out_e, a.eta_o,
                     a.out_o);
}

}  // namespace

// Geometry the block colouring supports: an even number (at least two) of 4^4
// blocks along every direction and, with C* in k >= 2, an x1 shift of L1 that
// moves an even number of blocks (so neighbours across a shifted boundary still
// differ in colour).
bool sap_supported(const qxd_handle* h) {
  const Geo& g = h->geo;
  if (g.Le0 % (2 * kSapB) || g.Le1 % (2 * kSapB) || g.Le2 % (2 * kSapB) || g.Le3 % (2 * kSapB)) return false;
  return g.cstar < 2 || (g.L1 / kSapB) % 2 == 0;
}

namespace {

// The block-order copies of links and clover blocks for slot order eo (made
// when the links, the clover blocks or the slot order changed since the last).
// The inverse blocks on odd sites are copied for the even-odd block solver
// only: the plain one never reads CIb, which then aliases Cb.  The FP32 odd
// clover blocks are cast for the copy and released after it if no other call
// had them, since the block copy holds them from then on (at 128 x 64^3 they
// are 9.7 GB).
qxd_status sap_pack(qxd_handle* h, int eo, float2** Vb, float4** Cb, float4** CIb, SapGeo* sb, hipStream_t s) {
  const size_t V = (size_t)h->V;
  *Vb = (float2*)ws_get(h, W_SAP_VB, V * 36 * sizeof(float2));
  *Cb = (float4*)ws_get(h, W_SAP_CB, V * 18 * sizeof(float4));
  *CIb = eo ? (float4*)ws_get(h, W_SAP_CIB, V / 2 * 18 * sizeof(float4)) : *Cb;
  if (!*Vb || !*Cb || !*CIb) return QXD_ENOMEM;
  const Geo& g = h->geo;
  const int nblk = (g.Le0 / kSapB) * (g.Le1 / kSapB) * (g.Le2 / kSapB) * (g.Le3 / kSapB);
  *sb = SapGeo{g.Le1 / kSapB, g.Le2 / kSapB, g.Le3 / kSapB, nblk / 2};
  // the copies are tagged 2 setup_gen + eo
  const uint64_t tag = 2 * h->setup_gen + (uint64_t)eo;
  if (h->sap_gen != tag) {
    const bool had_ho = (h->copies & CP_HO32) != 0;
    QXD_TRY(ensure_copies(h, CP_V32 | CP_HE32 | CP_HO32 | (eo ? CP_HI32 : 0u), s));
    auto pack = eo ? k_sap_pack<true> : k_sap_pack<false>;
    hipLaunchKernelGGL(pack, dim3(nblk), dim3(kSapSites), 0, s, g, *sb, reinterpret_cast<const float2*>(h->V32),
                       reinterpret_cast<const float4*>(h->He32), reinterpret_cast<const float4*>(h->Ho32),
                       reinterpret_cast<const float4*>(eo ? h->Hi32 : h->Ho32), *Vb, *Cb, *CIb);
    QXD_HIP(hipGetLastError());
    if (!had_ho) {
      QXD_HIP(hipStreamSynchronize(s));
      release_copies(h, CP_HO32);
    }
    h->sap_gen = tag;
  }
  return QXD_OK;
}

}  // namespace

qxd_status sap_blocks(qxd_handle* h, int eo, const float2** Vb, const float4** Cb, SapGeo* sb, hipStream_t s) {
  if (!h->has_inverse) return QXD_ESTATE;
  if (!sap_supported(h)) return QXD_EGEOM;
  float2* vb;
  float4 *cb, *cib;
  QXD_TRY(sap_pack(h, eo, &vb, &cb, &cib, sb, s));
  *Vb = vb;
  *Cb = cb;
  return QXD_OK;
}

qxd_status sap_apply_internal(qxd_handle* h, int ncy, int nmr, int eo, float4* out_e, const float4* in_e,
                              hipStream_t s, const float4* in_o, float4* out_o) {
  if (ncy < 1 || nmr < 1 || ncy > 64 || nmr > 64 || (eo != 0 && eo != 1)) return QXD_EINVAL;
  if (!h->has_inverse) return QXD_ESTATE;
  if (!sap_supported(h)) return QXD_EGEOM;
  const size_t V = (size_t)h->V;
  float2* Vb;
  float4 *Cb, *CIb;
  SapGeo sb;
  QXD_TRY(sap_pack(h, eo, &Vb, &Cb, &CIb, &sb, s));
  float4* Xb = (float4*)ws_get(h, W_SAP_XB, V * 6 * sizeof(float4));
  float4* Eb = (float4*)ws_get(h, W_SAP_EB, V * 6 * sizeof(float4));
  if (!Xb || !Eb) return QXD_ENOMEM;
  const Geo& g = h->geo;
  const SapArgs a{g, sb, nmr, in_e, Eb, Xb, Vb, Cb, CIb, out_e, in_o, out_o};
  for (int cy = 0; cy < ncy; ++cy)
    for (int colour = 0; colour < 2; ++colour) {
      if (cy == 0 && colour == 0)
        eo ? sap_launch<true, true>(a, cy, ncy, colour, s) : sap_launch<true, false>(a, cy, ncy, colour, s);
      else
        eo ? sap_launch<false, true>(a, cy, ncy, colour, s) : sap_launch<false, false>(a, cy, ncy, colour, s);
    }
  QXD_HIP(hipGetLastError());
  return QXD_OK;
}

extern "C" qxd_status qxd_sap_apply(qxd_handle* h, int ncy, int nmr, int eo, void* out_e, const void* in_e,
                                    void* stream) {
  if (!h || !out_e || !in_e || out_e == in_e) return QXD_EINVAL;
  return sap_apply_internal(h, ncy, nmr, eo, (float4*)out_e, (const float4*)in_e, as_stream(stream));
}

extern "C" qxd_status qxd_sap_apply_full(qxd_handle* h, int ncy, int nmr, int eo, void* out, const void* in,
                                         void* stream) {
  if (!h || !out || !in || out == in) return QXD_EINVAL;
  const size_t half = (size_t)6 * h->Ve;
  return sap_apply_internal(h, ncy, nmr, eo, (float4*)out, (const float4*)in, as_stream(stream),
                            (const float4*)in + half, (float4*)out + half);
}
