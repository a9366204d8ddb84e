// Gauge part of the molecular dynamics (Sec. 2 and Sec. 4.3): the tree-level
// Symanzik action (1x1 plaquettes and 1x2 rectangles of the links), its
// force, the momentum and link steps of the integrator and the kinetic
// energy.  FP64 throughout (the accept/reject test compares energies in
// double precision, Sec. 5.4).
//
// Links and momenta use the packed 18-real FP64 link layout
// [parity][mu][9][Vh] (complex), the layout of LQCD_LINKS18 links, so the
// fermion force can be added into the same array.  Gauge links carry no
// boundary sign or staggered phase (those belong to the fermion operator).
//
// Force convention (shared with the fermion force): with dS = sum Re Tr[dU M],
// F = TA(U M), TA(W) = (W - W^dag)/2 - Tr(W - W^dag)/6, so that dS/deps =
// sum Tr[T F] for U -> exp(eps T) U.  For S_g = beta sum_loops w (1 - Re Tr
// W / 3), M_mu(x) = -(beta / 3) A_mu(x) with A the weighted sum of the staples
// of the link (the product of the other links of each loop through it).  The
// MD equations U' = i H U, H' = -i F conserve H^2/2 + S.
#include <hip/hip_runtime.h>

#include <cmath>

#include "gauge.h"
#include "m3.h"
#include "staple.h"
#include "tile.h"

namespace lqcd {

namespace {

constexpr int kGaugeBlock = 128;
constexpr int kMdBlock = 256;
constexpr int kMdLinksBlock = 64;
constexpr int kReduceBlock = 1024;

// Weighted staple sum of the link U_mu(x): Tr[U_mu(x) A] runs over every
// plaquette (weight c0) and every 1x2 rectangle (weight c1) through the link,
// each as the loop that starts along the link.
// SEL picks the staple shapes (bits): 1 plaquettes, 2 / 4 2x1 with the link
// first / second (upper), 8 / 16 the same lower, 32 / 64 1x2 upper / lower.
// The force splits the shapes over three launches to bound the live matrices.
constexpr int kStaplePass1 = 1 | 2 | 4, kStaplePass2 = 8 | 16, kStaplePass3 = 32 | 64;

template <int SEL>
__device__ M3 staples(const KGeom& g, const double2* __restrict__ U, const C4& x, int mu,
                      double c0, double c1) {
  M3 A = m_zero();
#pragma unroll 1
  for (int nu = 0; nu < 4; ++nu) {
    if (nu == mu) continue;
    const C4 xp = shift(g, x, mu, 1), xn = shift(g, x, nu, 1), xm = shift(g, x, nu, -1);
    const C4 xpm = shift(g, xp, nu, -1);
    // plaquettes: up U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag,
    //             down U_nu(x+mu-nu)^dag U_mu(x-nu)^dag U_nu(x-nu)
    if (SEL & 1) {
      M3 t = m_mul_dag(link(g, U, xp, nu), link(g, U, xn, mu));
      t = m_mul_dag(t, link(g, U, x, nu));
      m_axpy(c0, t, A);
      t = m_dag_mul(link(g, U, xpm, nu), m_dag_mul(link(g, U, xm, mu), link(g, U, xm, nu)));
      m_axpy(c0, t, A);
    }
    const C4 xmu = shift(g, x, mu, -1);
    const C4 x2p = shift(g, xp, mu, 1);
    // 2 x 1, link first, up:
    //   U_mu(x+mu) U_nu(x+2mu) U_mu(x+mu+nu)^dag U_mu(x+nu)^dag U_nu(x)^dag
    if (SEL & 2) {
      M3 t = m_mul(link(g, U, xp, mu), link(g, U, x2p, nu));
      t = m_mul_dag(t, link(g, U, shift(g, xp, nu, 1), mu));
      t = m_mul_dag(t, link(g, U, xn, mu));
      t = m_mul_dag(t, link(g, U, x, nu));
      m_axpy(c1, t, A);
    }
    // 2 x 1, link second, up:
    //   U_nu(x+mu) U_mu(x+nu)^dag U_mu(x-mu+nu)^dag U_nu(x-mu)^dag U_mu(x-mu)
    if (SEL & 4) {
      M3 t = m_mul_dag(link(g, U, xp, nu), link(g, U, xn, mu));
      t = m_mul_dag(t, link(g, U, shift(g, xmu, nu, 1), mu));
      t = m_mul_dag(t, link(g, U, xmu, nu));
      t = m_mul(t, link(g, U, xmu, mu));
      m_axpy(c1, t, A);
    }
    // 2 x 1, link first, down:
    //   U_mu(x+mu) U_nu(x+2mu-nu)^dag U_mu(x+mu-nu)^dag U_mu(x-nu)^dag U_nu(x-nu)
    if (SEL & 8) {
      M3 t = m_mul_dag(link(g, U, xp, mu), link(g, U, shift(g, x2p, nu, -1), nu));
      t = m_mul_dag(t, link(g, U, xpm, mu));
      t = m_mul_dag(t, link(g, U, xm, mu));
      t = m_mul(t, link(g, U, xm, nu));
      m_axpy(c1, t, A);
    }
    // 2 x 1, link second, down:
    //   U_nu(x+mu-nu)^dag U_mu(x-nu)^dag U_mu(x-mu-nu)^dag U_nu(x-mu-nu) U_mu(x-mu)
    if (SEL & 16) {
      const C4 xmm = shift(g, xmu, nu, -1);
      M3 t = m_dag_mul(link(g, U, xpm, nu), m_dag_mul(link(g, U, xm, mu), m_unit()));
      t = m_mul_dag(t, link(g, U, xmm, mu));
      t = m_mul(t, link(g, U, xmm, nu));
      t = m_mul(t, link(g, U, xmu, mu));
      m_axpy(c1, t, A);
    }
    // 1 x 2, up: U_nu(x+mu) U_nu(x+mu+nu) U_mu(x+2nu)^dag U_nu(x+nu)^dag U_nu(x)^dag
    if (SEL & 32) {
      M3 t = m_mul(link(g, U, xp, nu), link(g, U, shift(g, xp, nu, 1), nu));
      t = m_mul_dag(t, link(g, U, shift(g, xn, nu, 1), mu));
      t = m_mul_dag(t, link(g, U, xn, nu));
      t = m_mul_dag(t, link(g, U, x, nu));
      m_axpy(c1, t, A);
    }
    // 1 x 2, down:
    //   U_nu(x+mu-nu)^dag U_nu(x+mu-2nu)^dag U_mu(x-2nu)^dag U_nu(x-2nu) U_nu(x-nu)
    if (SEL & 64) {
      const C4 xm2 = shift(g, xm, nu, -1);
      M3 t = m_dag_mul(link(g, U, xpm, nu), m_dag_mul(link(g, U, shift(g, xpm, nu, -1), nu),
                                                      m_unit()));
      t = m_mul_dag(t, link(g, U, xm2, mu));
      t = m_mul(t, link(g, U, xm2, nu));
      t = m_mul(t, link(g, U, xm, nu));
      m_axpy(c1, t, A);
    }
  }
  return A;
}

// One thread per link in the link_thread order (segment = mu; both parities
// of 64 half indices per workgroup, so each (parity, mu, element) plane is
// written coalesced); the blocks of one XCD take consecutive chunks, and the
// half index runs through z slabs of tz slices with t inside the slab
// (tz = 0: lexicographic), so the neighbour links one thread loads are the
// ones its neighbours load, while still in that XCD's L2.
template <int SEL>
__global__ void __launch_bounds__(kGaugeBlock) k_gauge_force(KGeom g, const double2* __restrict__ U,
                                                             double beta, double c0, double c1,
                                                             int accumulate, int tz, double2* F) {
  LinkThread lt;
  if (!link_thread(g, int64_t(xcd_block(blockIdx.x, gridDim.x, 1)) * blockDim.x + threadIdx.x,
                   lt))
    return;
  const int h = tiled_half_index(g, lt.i, g.Ly, tz);
  const int par = lt.par, mu = lt.seg;
  const int pm = par * 4 + mu;
  const C4 x = site_c4(g, h, par);
  const M3 A = staples<SEL>(g, U, x, mu, c0, c1);
  M3 W = m_mul(link(g, U, x, mu), A);
  const double s = -beta / 3.0;
#pragma unroll
  for (int e = 0; e < 9; ++e) W.e[e] = make_double2(s * W.e[e].x, s * W.e[e].y);
  const M3 f = traceless_antiherm(W);
  double2* out = F + int64_t(pm) * 9 * g.Vh + h;
#pragma unroll
  for (int e = 0; e < 9; ++e) {
    double2 v = f.e[e];
    if (accumulate) {
      const double2 o = out[int64_t(e) * g.Vh];
      v.x += o.x;
      v.y += o.y;
    }
    out[int64_t(e) * g.Vh] = v;
  }
}

// F (+)= -beta/3 TA(U A), A the plaquette staples: the whole force without
// rectangles.  48^4: 3.1 ms, 24^3 x 48: 0.38 ms (6.0 and 0.63 with one thread per
// link in k_gauge_force's order, 19 matrices per link against 14 here).  Bound as
// the smearing.
__global__ void __launch_bounds__(256, 2) k_plaquette_force(KGeom g, const double2* __restrict__ U,
                                                            double beta, int accumulate, int ty,
                                                            int tz, double2* __restrict__ F) {
  __shared__ Near sh;
  const ChunkSite cs = chunk_site(g, ty, tz);
  const C4 x = site_c4(g, cs.h, cs.par);
  stage_links(g, U, cs, x, sh);
  const M3 A = staple_sum(g, U, cs, x, sh);
  const M3 f = a_full(ta(m_mul(lds_m3(sh[0][cs.task], cs.lane), A), -beta / 3.0));
  if (!cs.in) return;
  if (accumulate) {
    const M3 o = ld_m3(link_res(g, F, cs.par, cs.task), cs.h, g.Vh);
    st_m3(F + (int64_t(cs.par) * 4 + cs.task) * 9 * g.Vh + cs.h, g.Vh, m_add(o, f));
  } else {
    st_m3(F + (int64_t(cs.par) * 4 + cs.task) * 9 * g.Vh + cs.h, g.Vh, f);
  }
}

__global__ void __launch_bounds__(kReduceBlock) k_reduce_one(const double* __restrict__ part, int n,
                                                          double scale, double* __restrict__ out) {
  __shared__ double lds[kReduceBlock / 64];
  double s = strided_sum(part, n);
  s = block_sum(s, lds);
  if (threadIdx.x == 0) *out = scale * s;
}

// H <- H - i eps F, element-wise over the packed arrays
__global__ void __launch_bounds__(kMdBlock) k_md_momenta(int64_t n, const double2* __restrict__ F,
                                                         double eps, double2* __restrict__ H) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double2 f = F[i];
  double2 h = H[i];
  h.x = fma(eps, f.y, h.x);
  h.y = fma(-eps, f.x, h.y);
  H[i] = h;
}

// exp(X) by the characteristic equation X^3 = t X^2 - s X + q, t = tr X,
// s = (t^2 - tr X^2) / 2, q = det X: the Taylor series is a polynomial
// f0 + f1 X + f2 X^2 whose coefficients follow from a recursion of three complex
// numbers, so the matrices take one product (X^2) in place of the twelve of a
// Horner scheme.  X is scaled by a power of two to a Frobenius norm of at most 1
// (18 terms leave a remainder below 1e-17) and the result squared back.
__device__ M3 expm_su3(M3 X) {
  double nrm2 = 0.0;
#pragma unroll
  for (int e = 0; e < 9; ++e) nrm2 += X.e[e].x * X.e[e].x + X.e[e].y * X.e[e].y;
  double nrm = sqrt(nrm2);
  int sq = 0;
  while (nrm > 1.0 && sq < 40) {
    nrm *= 0.5;
    ++sq;
  }
  const double sc = ldexp(1.0, -sq);
#pragma unroll
  for (int e = 0; e < 9; ++e) X.e[e] = cscale<double>(sc, X.e[e]);
  const M3 X2 = m_mul(X, X);
  const double2 t = cadd<double>(cadd<double>(X.e[0], X.e[4]), X.e[8]);
  double2 ms = cadd<double>(cadd<double>(X2.e[0], X2.e[4]), X2.e[8]);  // -s
  cfma<double>(ms, neg(t), t);
  ms = cscale<double>(0.5, ms);
  // det X along the first row
  auto minor = [&](int i, int j) {
    double2 m = cmul<double>(X.e[3 + i], X.e[6 + j]);
    cfma<double>(m, neg(X.e[3 + j]), X.e[6 + i]);
    return m;
  };
  double2 q = cmul<double>(X.e[0], minor(1, 2));
  cfma<double>(q, X.e[1], minor(2, 0));
  cfma<double>(q, X.e[2], minor(0, 1));
  const double2 z = make_double2(0.0, 0.0);
  double2 f0 = make_double2(1.0, 0.0), f1 = z, f2 = z;
#pragma unroll
  for (int k = 18; k >= 1; --k) {  // f <- 1 + (X / k) f
    const double v = 1.0 / k;
    double2 n0 = cmul<double>(q, f2), n1 = f0, n2 = f1;
    cfma<double>(n1, ms, f2);
    cfma<double>(n2, t, f2);
    f0 = cscale<double>(v, n0);
    f0.x += 1.0;
    f1 = cscale<double>(v, n1);
    f2 = cscale<double>(v, n2);
  }
  M3 E;
#pragma unroll
  for (int e = 0; e < 9; ++e) {
    E.e[e] = e % 4 ? z : f0;
    cfma<double>(E.e[e], f1, X.e[e]);
    cfma<double>(E.e[e], f2, X2.e[e]);
  }
#pragma unroll 1
  for (int k = 0; k < sq; ++k) E = m_mul(E, E);
  return E;
}

// Gram-Schmidt on rows 0 and 1, row 2 = conj(row0 x row1): the nearest
// special-unitary matrix up to rounding, applied after each link update so
// that the links stay in SU(3) over many steps.
__device__ M3 reunitarize(M3 u) {
  double n0 = 0.0;
#pragma unroll
  for (int j = 0; j < 3; ++j) n0 += u.e[j].x * u.e[j].x + u.e[j].y * u.e[j].y;
  n0 = 1.0 / sqrt(n0);
#pragma unroll
  for (int j = 0; j < 3; ++j) u.e[j] = make_double2(n0 * u.e[j].x, n0 * u.e[j].y);
  double2 d = make_double2(0.0, 0.0);  // <row0, row1> = sum_j conj(row0_j) row1_j
#pragma unroll
  for (int j = 0; j < 3; ++j) cfmac<double>(d, u.e[j], u.e[3 + j]);
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const double2 p = cmul<double>(d, u.e[j]);
    u.e[3 + j].x -= p.x;
    u.e[3 + j].y -= p.y;
  }
  double n1 = 0.0;
#pragma unroll
  for (int j = 0; j < 3; ++j) n1 += u.e[3 + j].x * u.e[3 + j].x + u.e[3 + j].y * u.e[3 + j].y;
  n1 = 1.0 / sqrt(n1);
#pragma unroll
  for (int j = 0; j < 3; ++j) u.e[3 + j] = make_double2(n1 * u.e[3 + j].x, n1 * u.e[3 + j].y);
  // row2 = conj(row0 x row1)
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const int a = (j + 1) % 3, b = (j + 2) % 3;
    const double2 p = cmul<double>(u.e[a], u.e[3 + b]);
    const double2 q = cmul<double>(u.e[b], u.e[3 + a]);
    u.e[6 + j] = make_double2(p.x - q.x, -(p.y - q.y));
  }
  return u;
}

// U <- exp(i eps H) U, one thread per link.  Bound by HBM: 504 us at 32^3 x 48
// (2.7 GB, 5.4 TB/s); with 128 threads a workgroup and a Horner exponential 555 us,
// with one of the two 528 to 552, at four waves a SIMD 576.
__global__ void __launch_bounds__(kMdLinksBlock) k_md_links(KGeom g, const double2* __restrict__ H,
                                                          double eps, double2* __restrict__ U) {
  const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= int64_t(8) * g.Vh) return;
  const int h = int(idx % g.Vh);
  const int64_t base = (idx / g.Vh) * 9 * int64_t(g.Vh) + h;
  M3 X, u;
#pragma unroll
  for (int e = 0; e < 9; ++e) {
    const double2 v = H[base + int64_t(e) * g.Vh];
    X.e[e] = make_double2(-eps * v.y, eps * v.x);  // i eps H
    u.e[e] = U[base + int64_t(e) * g.Vh];
  }
  const M3 r = reunitarize(m_mul(expm_su3(X), u));
#pragma unroll
  for (int e = 0; e < 9; ++e) U[base + int64_t(e) * g.Vh] = r.e[e];
}

// per link Tr H^2 = sum_ab Re(H_ab H_ba)
__global__ void __launch_bounds__(kGaugeBlock) k_kinetic(KGeom g, const double2* __restrict__ H,
                                                         double* __restrict__ part) {
  __shared__ double lds[kGaugeBlock / 64];
  const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  double s = 0.0;
  if (idx < int64_t(8) * g.Vh) {
    const int h = int(idx % g.Vh);
    const int64_t base = (idx / g.Vh) * 9 * int64_t(g.Vh) + h;
    M3 m;
#pragma unroll
    for (int e = 0; e < 9; ++e) m.e[e] = H[base + int64_t(e) * g.Vh];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const double2 p = cmul<double>(m.e[3 * a + b], m.e[3 * b + a]);
        s += p.x;
      }
  }
  s = block_sum(s, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// U_out = exp(i theta) U_in per link, theta natural [4][V] (lex = 2 h + bit)
__global__ void __launch_bounds__(kMdBlock) k_u1_phases(KGeom g, const double2* __restrict__ U,
                                                        const double* __restrict__ theta,
                                                        double2* __restrict__ out) {
  const int64_t idx = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (idx >= int64_t(8) * g.Vh) return;
  const int h = int(idx % g.Vh);
  const int pm = int(idx / g.Vh);
  const int par = pm >> 2, mu = pm & 3;
  const Site s = decode_site(g, h, par);
  const int64_t lex = int64_t(s.x) + int64_t(g.Lx) * (s.y + int64_t(g.Ly) * (s.z + int64_t(g.Lz) * s.t));
  const int64_t V = int64_t(2) * g.Vh;
  double sn, cs;
  sincos(theta[mu * V + lex], &sn, &cs);
  const double2 u = make_double2(cs, sn);
  const int64_t base = int64_t(pm) * 9 * g.Vh + h;
#pragma unroll
  for (int e = 0; e < 9; ++e) out[base + int64_t(e) * g.Vh] = cmul<double>(u, U[base + int64_t(e) * g.Vh]);
}

int check_c1(double beta, double c1) {
  if (!std::isfinite(beta) || !std::isfinite(c1)) {
    set_error("beta and c1 must be finite");
    return LQCD_ERR_INVALID_ARG;
  }
  return LQCD_OK;
}

int reduce_to_host(const double* part, int nb, double scale, double* out_dev, double* host,
                   hipStream_t s) {
  hipLaunchKernelGGL(k_reduce_one, dim3(1), dim3(kReduceBlock), 0, s, part, nb, scale, out_dev);
  LQCD_LAUNCH_CHECK();
  LQCD_HIP_TRY(hipMemcpyAsync(host, out_dev, sizeof(double), hipMemcpyDeviceToHost, s));
  LQCD_HIP_TRY(hipStreamSynchronize(s));
  return LQCD_OK;
}

}  // namespace

int gauge_force_direct(const KGeom& k, const double2* U, double beta, double c1, int accumulate,
                       double2* F, hipStream_t s) {
  if (c1 == 0.0) {
    hipLaunchKernelGGL(k_plaquette_force, dim3(chunk_blocks(k.Vh)), dim3(256), 0, s, k, U, beta,
                       accumulate, chunk_tile(k.Ly, 16), chunk_tile(k.Lz, 7), F);
    LQCD_LAUNCH_CHECK();
    return LQCD_OK;
  }
  // F is linear in the staple sum, so the shapes split over three launches:
  // the later ones add TA(U (-beta/3) A_k) onto the first's result.
  const dim3 grid(unsigned(4 * link_threads_per_segment(k.Vh) / kGaugeBlock));
  const int tz = slab_tile(k.Lz);
  hipLaunchKernelGGL(k_gauge_force<kStaplePass1>, grid, dim3(kGaugeBlock), 0, s, k, U, beta,
                     1.0 - 8.0 * c1, c1, accumulate, tz, F);
  LQCD_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_gauge_force<kStaplePass2>, grid, dim3(kGaugeBlock), 0, s, k, U, beta,
                     1.0 - 8.0 * c1, c1, 1, tz, F);
  LQCD_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_gauge_force<kStaplePass3>, grid, dim3(kGaugeBlock), 0, s, k, U, beta,
                     1.0 - 8.0 * c1, c1, 1, tz, F);
  LQCD_LAUNCH_CHECK();
  return LQCD_OK;
}

}  // namespace lqcd

using namespace lqcd;

extern "C" {

int lqcd_apply_u1_phases(const lqcd_geom* g, const void* U64, const double* theta, void* out,
                         void* stream) {
  clear_error();
  int rc;
  if ((rc = check_geom(g)) || (rc = check_ptr(U64, "U64")) || (rc = check_ptr(out, "out")))
    return rc;
  if (!theta || (reinterpret_cast<uintptr_t>(theta) & 7)) {
    set_error("theta must be an 8-byte aligned device array of 4 V doubles");
    return LQCD_ERR_INVALID_ARG;
  }
  const KGeom k = make_kgeom(g);
  const int64_t n = int64_t(8) * k.Vh;
  hipLaunchKernelGGL(k_u1_phases, dim3(unsigned((n + kMdBlock - 1) / kMdBlock)), dim3(kMdBlock),
                     0, (hipStream_t)stream, k, (const double2*)U64, theta, (double2*)out);
  LQCD_LAUNCH_CHECK();
  return LQCD_OK;
}

size_t lqcd_gauge_workspace_bytes(const lqcd_geom* g) {
  if (check_geom(g)) return 0;
  const KGeom k = make_kgeom(g);
  return (size_t((int64_t(8) * k.Vh + kGaugeBlock - 1) / kGaugeBlock) + 32) * sizeof(double);
}

int lqcd_gauge_action(const lqcd_geom* g, const void* U64, double beta, double c1, double* S,
                      void* ws, size_t ws_bytes, void* stream) {
  clear_error();
  int rc;
  if ((rc = check_geom(g)) || (rc = check_ptr(U64, "U64")) || (rc = check_ptr(ws, "ws")) ||
      (rc = check_c1(beta, c1)))
    return rc;
  if (!S) {
    set_error("S must be a host pointer");
    return LQCD_ERR_INVALID_ARG;
  }
  if (ws_bytes < lqcd_gauge_workspace_bytes(g)) {
    set_error("gauge workspace of %zu bytes is too small: %zu needed", ws_bytes,
              lqcd_gauge_workspace_bytes(g));
    return LQCD_ERR_WORKSPACE;
  }
  const KGeom k = make_kgeom(g);
  const int nb = int(gauge_action_blocks(k));
  double* part = static_cast<double*>(ws);
  const hipStream_t s = (hipStream_t)stream;
  if ((rc = gauge_action_partials(k, (const double2*)U64, c1, part, s))) return rc;
  return reduce_to_host(part, nb, beta, part + nb + 16, S, s);
}

int lqcd_gauge_force(const lqcd_geom* g, const void* U64, double beta, double c1,
                     int32_t accumulate, void* F, void* stream) {
  clear_error();
  int rc;
  if ((rc = check_geom(g)) || (rc = check_ptr(U64, "U64")) || (rc = check_ptr(F, "F")) ||
      (rc = check_c1(beta, c1)))
    return rc;
  if (accumulate != 0 && accumulate != 1) {
    set_error("accumulate must be 0 or 1");
    return LQCD_ERR_INVALID_ARG;
  }
  if (F == U64) {
    set_error("F must not alias U64");
    return LQCD_ERR_INVALID_ARG;
  }
  return gauge_force_direct(make_kgeom(g), (const double2*)U64, beta, c1, accumulate,
                            (double2*)F, (hipStream_t)stream);
}

int lqcd_md_update_momenta(const lqcd_geom* g, const void* F, double eps, void* H,
                           void* stream) {
  clear_error();
  int rc;
  if ((rc = check_geom(g)) || (rc = check_ptr(F, "F")) || (rc = check_ptr(H, "H"))) return rc;
  if (!std::isfinite(eps)) {
    set_error("eps must be finite");
    return LQCD_ERR_INVALID_ARG;
  }
  if (F == H) {
    set_error("F must not alias H");
    return LQCD_ERR_INVALID_ARG;
  }
  const KGeom k = make_kgeom(g);
  const int64_t n = int64_t(8) * 9 * k.Vh;
  hipLaunchKernelGGL(k_md_momenta, dim3(unsigned((n + kMdBlock - 1) / kMdBlock)), dim3(kMdBlock),
                     0, (hipStream_t)stream, n, (const double2*)F, eps, (double2*)H);
  LQCD_LAUNCH_CHECK();
  return LQCD_OK;
}

int lqcd_md_update_links(const lqcd_geom* g, const void* H, double eps, void* U64,
                         void* stream) {
  clear_error();
  int rc;
  if ((rc = check_geom(g)) || (rc = check_ptr(H, "H")) || (rc = check_ptr(U64, "U64"))) return rc;
  if (!std::isfinite(eps)) {
    set_error("eps must be finite");
    return LQCD_ERR_INVALID_ARG;
  }
  if (H == U64) {
    set_error("H must not alias U64");
    return LQCD_ERR_INVALID_ARG;
  }
  const KGeom k = make_kgeom(g);
  const int64_t n = int64_t(8) * k.Vh;
  hipLaunchKernelGGL(k_md_links, dim3(unsigned((n + kMdLinksBlock - 1) / kMdLinksBlock)),
                     dim3(kMdLinksBlock), 0, (hipStream_t)stream, k, (const double2*)H, eps,
                     (double2*)U64);
  LQCD_LAUNCH_CHECK();
  return LQCD_OK;
}

int lqcd_kinetic_energy(const lqcd_geom* g, const void* H, double* K, void* ws, size_t ws_bytes,
                        void* stream) {
  clear_error();
  int rc;
  if ((rc = check_geom(g)) || (rc = check_ptr(H, "H")) || (rc = check_ptr(ws, "ws"))) return rc;
  if (!K) {
    set_error("K must be a host pointer");
    return LQCD_ERR_INVALID_ARG;
  }
  if (ws_bytes < lqcd_gauge_workspace_bytes(g)) {
    set_error("gauge workspace of %zu bytes is too small: %zu needed", ws_bytes,
              lqcd_gauge_workspace_bytes(g));
    return LQCD_ERR_WORKSPACE;
  }
  const KGeom k = make_kgeom(g);
  const int nb = int((int64_t(8) * k.Vh + kGaugeBlock - 1) / kGaugeBlock);
  double* part = static_cast<double*>(ws);
  const hipStream_t s = (hipStream_t)stream;
  hipLaunchKernelGGL(k_kinetic, dim3(nb), dim3(kGaugeBlock), 0, s, k, (const double2*)H, part);
  LQCD_LAUNCH_CHECK();
  return reduce_to_host(part, nb, 0.5, part + nb + 16, K, s);
}

}  // extern "C"
