// Stout smearing (Sec. 2: the Dirac operator uses k-times stout-smeared links)
// and the chain rule of the force through one smearing level.
//   U' = exp(X) U, X = TA(Omega), Omega = rho A^dag U^dag = rho (U A)^dag, A the
// plaquette staple sum of the link, so X = -rho TA(U A).
//
// One workgroup per 64 half indices of one parity, wave = direction of the link
// (chunk_site): the four directions of a site share most of the links around
// it, and the links that several waves use go through LDS.
#include <hip/hip_runtime.h>

#include <cmath>

#include "m3.h"
#include "staple.h"
#include "tile.h"

namespace lqcd {

namespace {

__device__ __forceinline__ M3 m_dag(const M3& a) {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) r.e[3 * i + j] = make_double2(a.e[3 * j + i].x, -a.e[3 * j + i].y);
  return r;
}

// ---- exp of a traceless anti-Hermitian X by its characteristic equation
//   X^3 = p X + q,  p = tr(X^2) / 2 (real),  q = det X = i d (imaginary),
// so that every polynomial in X is f0 + f1 X + f2 X^2 and the series is summed
// in those three complex numbers: one matrix product (X^2) in place of the 12
// of a Taylor polynomial.  X is scaled by a power of two to a Frobenius norm of
// at most 1 (18 terms leave a remainder below 1e-17), which smearing with the
// usual rho hardly ever needs, and the result squared back as a matrix: on the
// coefficients the squarings would lose accuracy as |X|^2.
struct Poly {
  double2 f0, f1, f2;
};

// Hermitian 3x3 matrix X^2.
struct Herm {
  double d0, d1, d2;
  double2 o01, o02, o12;
};

__device__ __forceinline__ Herm a_square(const Alg& a) {
  const double x2 = -(a.d.x + a.d.y);
  const double n01 = cnorm2<double>(a.o01), n02 = cnorm2<double>(a.o02),
               n12 = cnorm2<double>(a.o12);
  Herm r;
  r.d0 = -(a.d.x * a.d.x + n01 + n02);
  r.d1 = -(a.d.y * a.d.y + n01 + n12);
  r.d2 = -(x2 * x2 + n02 + n12);
  // (X^2)_01 = i (x0 + x1) X_01 - X_02 conj(X_12), and so on
  r.o01 = make_double2(x2 * a.o01.y, -x2 * a.o01.x);
  cfmac<double>(r.o01, neg(a.o12), a.o02);
  r.o02 = make_double2(a.d.y * a.o02.y, -a.d.y * a.o02.x);
  cfma<double>(r.o02, a.o01, a.o12);
  r.o12 = make_double2(a.d.x * a.o12.y, -a.d.x * a.o12.x);
  cfmac<double>(r.o12, neg(a.o01), a.o02);
  return r;
}

// Im det X of X = i Q (x_i the diagonal): -det Q
__device__ __forceinline__ double a_det(const Alg& a) {
  const double x0 = a.d.x, x1 = a.d.y, x2 = -(x0 + x1);
  const double2 ac = cmul<double>(a.o01, a.o12);
  const double im = fma(ac.y, a.o02.x, -(ac.x * a.o02.y));
  return -(x0 * x1 * x2 + 2.0 * im - x0 * cnorm2<double>(a.o12) - x1 * cnorm2<double>(a.o02) -
           x2 * cnorm2<double>(a.o01));
}

// the power of two that brings X to norm <= 1
__device__ __forceinline__ int scaling(const Alg& a) {
  const double x2 = a.d.x + a.d.y;
  double n = sqrt(a.d.x * a.d.x + a.d.y * a.d.y + x2 * x2 +
                  2.0 * (cnorm2<double>(a.o01) + cnorm2<double>(a.o02) + cnorm2<double>(a.o12)));
  int k = 0;
  while (n > 1.0 && k < 40) {
    n *= 0.5;
    ++k;
  }
  return k;
}

__device__ __forceinline__ Alg a_scale(double s, const Alg& a) {
  return Alg{cscale<double>(s, a.o01), cscale<double>(s, a.o02), cscale<double>(s, a.o12),
             cscale<double>(s, a.d)};
}

constexpr int kExpTerms = 18;

// z * i d
__device__ __forceinline__ double2 mul_id(double2 z, double d) {
  return make_double2(-d * z.y, d * z.x);
}

// Horner: f <- 1 + (X / k) f
__device__ __forceinline__ Poly exp_poly(double p, double d) {
  Poly f{make_double2(1.0, 0.0), make_double2(0.0, 0.0), make_double2(0.0, 0.0)};
#pragma unroll
  for (int k = kExpTerms; k >= 1; --k) {
    const double v = 1.0 / k;
    const double2 n0 = mul_id(f.f2, d * v);
    const double2 n1 = make_double2(v * fma(p, f.f2.x, f.f0.x), v * fma(p, f.f2.y, f.f0.y));
    f.f2 = cscale<double>(v, f.f1);
    f.f1 = n1;
    f.f0 = make_double2(1.0 + n0.x, n0.y);
  }
  return f;
}

// f0 + f1 X + f2 X^2 with H = X^2
__device__ __forceinline__ M3 evaluate(const Poly& f, const Alg& x, const Herm& h) {
  const double d2 = -(x.d.x + x.d.y);
  M3 r;
  auto diag = [&](double xi, double hi) {
    return make_double2(f.f0.x + fma(-f.f1.y, xi, f.f2.x * hi),
                        f.f0.y + fma(f.f1.x, xi, f.f2.y * hi));
  };
  auto off = [&](double2 xo, double2 ho, double2& u, double2& l) {
    const double2 a = cmul<double>(f.f1, xo), b = cmul<double>(f.f2, ho);
    u = cadd<double>(a, b);
    // below the diagonal X holds -conj, X^2 holds conj
    l = csub<double>(cmulc<double>(ho, f.f2), cmulc<double>(xo, f.f1));
  };
  r.e[0] = diag(x.d.x, h.d0);
  r.e[4] = diag(x.d.y, h.d1);
  r.e[8] = diag(d2, h.d2);
  off(x.o01, h.o01, r.e[1], r.e[3]);
  off(x.o02, h.o02, r.e[2], r.e[6]);
  off(x.o12, h.o12, r.e[5], r.e[7]);
  return r;
}

// One level: U' = exp(X) U.  24^3 x 32: 0.27 ms (0.43 with the directions as
// separate segments of the grid and a Taylor exponential).  Bound by waiting for
// 14 link matrices per link at the 8 waves a CU that registers and LDS allow:
// 3.6 GB from L2 (13 TB/s; a kernel that only reads L2 reaches 30), a quarter of
// the requests missing it, FP64 units 45 % busy.  Its HBM bytes would take 0.11 ms,
// its products 0.12 ms.  Only the sites' own links in LDS, for 12 waves a CU, made
// the plaquette force, which loads the same, 8 % slower.
__global__ void __launch_bounds__(256, 2) k_stout_smear(KGeom g, const double2* __restrict__ U,
                                                        double rho, int ty, int tz,
                                                        double2* __restrict__ out) {
  __shared__ Near sh;
  const ChunkSite cs = chunk_site(g, ty, tz);
  const C4 x = site_c4(g, cs.h, cs.par);
  stage_links(g, U, cs, x, sh);
  const M3 A = staple_sum(g, U, cs, x, sh);
  Alg X = ta(m_mul(lds_m3(sh[0][cs.task], cs.lane), A), -rho);
  const int sq = scaling(X);
  X = a_scale(ldexp(1.0, -sq), X);
  const Herm H = a_square(X);
  const double p = 0.5 * (H.d0 + H.d1 + H.d2), d = a_det(X);
  M3 E = evaluate(exp_poly(p, d), X, H);
#pragma unroll 1
  for (int k = 0; k < sq; ++k) E = m_mul(E, E);
  const M3 r = m_mul(E, lds_m3(sh[0][cs.task], cs.lane));
  if (cs.in) st_m3(out + (int64_t(cs.par) * 4 + cs.task) * 9 * g.Vh + cs.h, g.Vh, r);
}

// tr(X B) and tr(X^2 B)
__device__ __forceinline__ double2 tr_mul(const Alg& x, const M3& b) {
  const double d2 = -(x.d.x + x.d.y);
  double2 s = mul_id(b.e[0], x.d.x);
  s = cadd<double>(s, mul_id(b.e[4], x.d.y));
  s = cadd<double>(s, mul_id(b.e[8], d2));
  cfma<double>(s, x.o01, b.e[3]);
  cfma<double>(s, x.o02, b.e[6]);
  cfma<double>(s, x.o12, b.e[7]);
  cfmac<double>(s, neg(x.o01), b.e[1]);
  cfmac<double>(s, neg(x.o02), b.e[2]);
  cfmac<double>(s, neg(x.o12), b.e[5]);
  return s;
}

__device__ __forceinline__ double2 tr_mul(const Herm& h, const M3& b) {
  double2 s = cscale<double>(h.d0, b.e[0]);
  s = cadd<double>(s, cscale<double>(h.d1, b.e[4]));
  s = cadd<double>(s, cscale<double>(h.d2, b.e[8]));
  cfma<double>(s, h.o01, b.e[3]);
  cfma<double>(s, h.o02, b.e[6]);
  cfma<double>(s, h.o12, b.e[7]);
  cfmac<double>(s, h.o01, b.e[1]);
  cfmac<double>(s, h.o02, b.e[2]);
  cfmac<double>(s, h.o12, b.e[5]);
  return s;
}

// The coefficients' derivatives along a direction with p' = dp, q' = dq,
// carried through the same Horner steps.
__device__ __forceinline__ void exp_poly_tangent(double p, double d, double2 dp, double2 dq,
                                                 Poly& f, Poly& t) {
  const double2 z = make_double2(0.0, 0.0);
  f = Poly{make_double2(1.0, 0.0), z, z};
  t = Poly{z, z, z};
#pragma unroll
  for (int k = kExpTerms; k >= 1; --k) {
    const double v = 1.0 / k;
    double2 t0 = mul_id(t.f2, d);
    cfma<double>(t0, f.f2, dq);
    double2 t1 = make_double2(fma(p, t.f2.x, t.f0.x), fma(p, t.f2.y, t.f0.y));
    cfma<double>(t1, f.f2, dp);
    t.f2 = cscale<double>(v, t.f1);
    t.f1 = cscale<double>(v, t1);
    t.f0 = cscale<double>(v, t0);
    const double2 n0 = mul_id(f.f2, d * v);
    const double2 n1 = make_double2(v * fma(p, f.f2.x, f.f0.x), v * fma(p, f.f2.y, f.f0.y));
    f.f2 = cscale<double>(v, f.f1);
    f.f1 = n1;
    f.f0 = make_double2(1.0 + n0.x, n0.y);
  }
}

// acc += z m
__device__ __forceinline__ void add_scaled(double2 z, const M3& m, M3& acc) {
#pragma unroll
  for (int e = 0; e < 9; ++e) cfma<double>(acc.e[e], z, m.e[e]);
}

// E = exp(X) and TA(L), L = sum_k 1/k! sum_j X^j B X^(k-1-j) the Frechet
// derivative of exp at X along B.  With B = B0 + s, tr B0 = 0: the shift gives
// s E, and B0 changes p by tr(X B0) and q by tr(X^2 B0), so
//   L = s E + f1 B0 + f2 (X B0 + B0 X) + f0' + f1' X + f2' X^2.
// Of the scaled matrices, (E, L) -> (E E, E L + L E) for each halving.
__device__ __forceinline__ void exp_frechet(const Alg& X0, const M3& B, M3& E, Alg& L) {
  const int sq = scaling(X0);
  const double sc = ldexp(1.0, -sq);
  const Alg X = a_scale(sc, X0);
  const Herm H = a_square(X);
  const double p = 0.5 * (H.d0 + H.d1 + H.d2), d = a_det(X);
  const double2 s = make_double2((B.e[0].x + B.e[4].x + B.e[8].x) / 3.0,
                                 (B.e[0].y + B.e[4].y + B.e[8].y) / 3.0);
  M3 B0 = B;
  B0.e[0] = csub<double>(B0.e[0], s);
  B0.e[4] = csub<double>(B0.e[4], s);
  B0.e[8] = csub<double>(B0.e[8], s);
#pragma unroll
  for (int e = 0; e < 9; ++e) B0.e[e] = cscale<double>(sc, B0.e[e]);
  const double2 dp = tr_mul(X, B0), dq = tr_mul(H, B0);
  Poly f, t;
  exp_poly_tangent(p, d, dp, dq, f, t);
  M3 r = evaluate(t, X, H);
  add_scaled(f.f1, B0, r);
  add_scaled(f.f2, a_mul(X, B0), r);
  add_scaled(f.f2, m_mul_a(B0, X), r);
  __builtin_amdgcn_sched_barrier(0);  // B0 is done before E takes registers
  E = evaluate(f, X, H);
  add_scaled(cscale<double>(sc, s), E, r);
#pragma unroll 1
  for (int k = 0; k < sq; ++k) {
    r = m_add(m_mul(E, r), m_mul(r, E));
    E = m_mul(E, E);
  }
  L = ta(r, 1.0);
}

// Per link, from the raw gradient G' = M'^dag with respect to the smeared
// link: Lam = TA(L(X, U M')) (8 reals) and the local part
// Mloc = M' E + rho A Lam^dag of M.  24^3 x 32: 0.36 ms (0.78 when the derivative
// was a Taylor series of 2 x 2 block matrices, 40 products); bound as the
// smearing, with 0.4 GB more to and from HBM.
__global__ void __launch_bounds__(256, 2) k_stout_lambda(KGeom g, const double2* __restrict__ U,
                                                         double rho, int ty, int tz,
                                                         const double2* __restrict__ Gp,
                                                         double2* __restrict__ lam,
                                                         double2* __restrict__ Mloc) {
  __shared__ Near sh;
  const ChunkSite cs = chunk_site(g, ty, tz);
  const C4 x = site_c4(g, cs.h, cs.par);
  stage_links(g, U, cs, x, sh);
  Alg X;
  {
    const M3 A = staple_sum(g, U, cs, x, sh);
    X = ta(m_mul(lds_m3(sh[0][cs.task], cs.lane), A), -rho);
    __syncthreads();  // every wave is done with U_mu(x - mu): A waits there
#pragma unroll
    for (int e = 0; e < 9; ++e) sh[1][cs.task][e][cs.lane] = A.e[e];
  }
  const auto gr = link_res(g, Gp, cs.par, cs.task);
  M3 E;
  Alg l;
  exp_frechet(X, m_mul_dag(lds_m3(sh[0][cs.task], cs.lane), ld_m3(gr, cs.h, g.Vh)), E, l);
  if (!cs.in) return;
  const int64_t pm = int64_t(cs.par) * 4 + cs.task;
  double2* o = lam + pm * 4 * g.Vh + cs.h;
  o[0] = l.o01;
  o[int64_t(g.Vh)] = l.o02;
  o[int64_t(2) * g.Vh] = l.o12;
  o[int64_t(3) * g.Vh] = l.d;
  const M3 ml = m_add(m_dag_mul(ld_m3(gr, cs.h, g.Vh), E),
                      m_mul_a(lds_m3(sh[1][cs.task], cs.lane), a_scale(-rho, l)));  // Lam^dag = -Lam
  st_m3(Mloc + pm * 9 * g.Vh + cs.h, g.Vh, ml);
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t lam_res(const KGeom& g, const double2* lam,
                                                          int par, int mu) {
  return make_res(lam + (int64_t(par) * 4 + mu) * 4 * int64_t(g.Vh), 64u * uint32_t(g.Vh));
}

__device__ __forceinline__ Alg ld_lam(__amdgpu_buffer_rsrc_t r, int h, int Vh) {
  const uint32_t o = uint32_t(h) * 16u, s = uint32_t(Vh) * 16u;
  return Alg{ld_buf<double>(r, o, 0), ld_buf<double>(r, o, s), ld_buf<double>(r, o, 2 * s),
             ld_buf<double>(r, o, 3 * s)};
}

__device__ __forceinline__ Alg a_sub(const Alg& a, const Alg& b) {
  return Alg{csub<double>(a.o01, b.o01), csub<double>(a.o02, b.o02), csub<double>(a.o12, b.o12),
             csub<double>(a.d, b.d)};
}

// M of link (y, a) = Mloc + the terms of Re Tr[dA_mu(x) K_mu(x)], K = rho Lam^dag
// U = -rho Lam U, in which the link appears.  For every other direction m, with
// y- = y - m, y+ = y + m, ya = y + a:
//   lower plaquette  -rho Um(ya-)^dag { Ua(y-)^dag [Lam_m(y-) - Lam_a(y-)]
//                                      - Lam_m(ya-) Ua(y-)^dag } Um(y-)
//   upper plaquette  -rho { [Lam_m(ya) S - S Lam_m(y)] - W Lam_a(y+) Um(y)^dag },
//                     W = Um(ya) Ua(y+)^dag,  S = W Um(y)^dag
// (six terms of the staples' middle and outer links, with the matrices next to
// each other multiplied once).  Output: mode 0 F = TA(U M), mode 1 the raw
// gradient M^dag.  24^3 x 32: 0.43 ms (0.78 with K stored as full matrices and the
// six terms multiplied out); bound by 3 KB per link from L2 (5.4 GB).
__global__ void __launch_bounds__(256, 2) k_stout_gather(KGeom g, const double2* __restrict__ U,
                                                         const double2* __restrict__ lam,
                                                         const double2* __restrict__ Mloc,
                                                         double rho, int mode, int ty, int tz,
                                                         double2* __restrict__ out) {
  __shared__ Near sh;
  const ChunkSite cs = chunk_site(g, ty, tz);
  const C4 y = site_c4(g, cs.h, cs.par);
  stage_links(g, U, cs, y, sh);
  const int a = cs.task, h = cs.h, par = cs.par, opp = 1 - par, lane = cs.lane;
  const int ha = h + axis(g, y, a).off(1);
  const auto ua_o = link_res(g, U, opp, a);
  const auto la_o = lam_res(g, lam, opp, a);
  M3 S = m_zero();  // the terms over -rho
#pragma unroll 1
  for (int m = 0; m < 4; ++m) {
    if (m == a) continue;
    const Axis ym = axis(g, y, m);
    const int hp = h + ym.off(1), hm = h + ym.off(-1), ham = ha + ym.off(-1);
    const auto um_s = link_res(g, U, par, m), um_o = link_res(g, U, opp, m);
    const auto lm_s = lam_res(g, lam, par, m), lm_o = lam_res(g, lam, opp, m);
    {
      const M3 ud = m_dag(ld_m3(ua_o, hm, g.Vh));
      const Alg dl = a_sub(ld_lam(lm_o, hm, g.Vh), ld_lam(la_o, hm, g.Vh));
      M3 w = m_mul_a(ud, dl);
      const M3 v = a_mul(ld_lam(lm_s, ham, g.Vh), ud);
#pragma unroll
      for (int e = 0; e < 9; ++e) w.e[e] = csub<double>(w.e[e], v.e[e]);
      w = m_mul(w, lds_m3(sh[1][m], lane));
      S = m_add(S, m_dag_mul(ld_m3(um_s, ham, g.Vh), w));
    }
    {
      const M3 W = m_mul_dag(ld_m3(um_o, ha, g.Vh), ld_m3(ua_o, hp, g.Vh));
      const M3 um = lds_m3(sh[0][m], lane);
      const M3 st = m_mul_dag(W, um);
      S = m_add(S, a_mul(ld_lam(lm_o, ha, g.Vh), st));
      M3 w = m_mul_dag(m_mul_a(W, ld_lam(la_o, hp, g.Vh)), um);
      w = m_add(w, m_mul_a(st, ld_lam(lm_s, h, g.Vh)));
#pragma unroll
      for (int e = 0; e < 9; ++e) S.e[e] = csub<double>(S.e[e], w.e[e]);
    }
  }
  if (!cs.in) return;
  M3 M = ld_m3(link_res(g, Mloc, par, a), h, g.Vh);
  m_axpy(-rho, S, M);
  M3 r;
  if (mode == 0)
    r = a_full(ta(m_mul(lds_m3(sh[0][a], lane), M), 1.0));
  else
    r = m_dag(M);
  st_m3(out + (int64_t(par) * 4 + a) * 9 * g.Vh + h, g.Vh, r);
}

}  // namespace

}  // namespace lqcd

using namespace lqcd;

extern "C" {

int lqcd_stout_smear(const lqcd_geom* g, const void* U64, double rho, void* out, void* stream) {
  clear_error();
  int rc;
  if ((rc = check_geom(g)) || (rc = check_ptr(U64, "U64")) || (rc = check_ptr(out, "out")))
    return rc;
  if (!std::isfinite(rho)) {
    set_error("rho must be finite");
    return LQCD_ERR_INVALID_ARG;
  }
  if (out == U64) {
    set_error("out must not alias U64 (every link reads its neighbours)");
    return LQCD_ERR_INVALID_ARG;
  }
  const KGeom k = make_kgeom(g);
  hipLaunchKernelGGL(k_stout_smear, dim3(chunk_blocks(k.Vh)), dim3(256), 0, (hipStream_t)stream,
                     k, (const double2*)U64, rho, chunk_tile(k.Ly, 16), chunk_tile(k.Lz, 7),
                     (double2*)out);
  LQCD_LAUNCH_CHECK();
  return LQCD_OK;
}

size_t lqcd_stout_workspace_bytes(const lqcd_geom* g) {
  if (check_geom(g)) return 0;
  const KGeom k = make_kgeom(g);
  return size_t(2) * 8 * 9 * size_t(k.Vh) * sizeof(double2);
}

int lqcd_stout_force(const lqcd_geom* g, const void* U64, double rho, const void* G_smeared,
                     int32_t mode, void* out, void* ws, size_t ws_bytes, void* stream) {
  clear_error();
  int rc;
  if ((rc = check_geom(g)) || (rc = check_ptr(U64, "U64")) ||
      (rc = check_ptr(G_smeared, "G_smeared")) || (rc = check_ptr(out, "out")) ||
      (rc = check_ptr(ws, "ws")))
    return rc;
  if (!std::isfinite(rho)) {
    set_error("rho must be finite");
    return LQCD_ERR_INVALID_ARG;
  }
  if (mode != 0 && mode != 1) {
    set_error("mode must be 0 (projected) or 1 (raw), got %d", mode);
    return LQCD_ERR_INVALID_ARG;
  }
  if (ws_bytes < lqcd_stout_workspace_bytes(g)) {
    set_error("stout workspace of %zu bytes is too small: %zu needed", ws_bytes,
              lqcd_stout_workspace_bytes(g));
    return LQCD_ERR_WORKSPACE;
  }
  if (out == U64 || out == G_smeared) {
    set_error("out must not alias U64 or G_smeared");
    return LQCD_ERR_INVALID_ARG;
  }
  const KGeom k = make_kgeom(g);
  double2* Mloc = static_cast<double2*>(ws);
  double2* lam = Mloc + int64_t(8) * 9 * k.Vh;
  const hipStream_t s = (hipStream_t)stream;
  const dim3 grid(chunk_blocks(k.Vh));
  const int ty = chunk_tile(k.Ly, 16), tz = chunk_tile(k.Lz, 7);
  hipLaunchKernelGGL(k_stout_lambda, grid, dim3(256), 0, s, k, (const double2*)U64, rho, ty, tz,
                     (const double2*)G_smeared, lam, Mloc);
  LQCD_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_stout_gather, grid, dim3(256), 0, s, k, (const double2*)U64,
                     (const double2*)lam, (const double2*)Mloc, rho, mode, ty, tz, (double2*)out);
  LQCD_LAUNCH_CHECK();
  return LQCD_OK;
}

}  // extern "C"
