// 3x3 complex FP64 matrices held in registers, for the gauge-side kernels
// (products, the traceless anti-Hermitian projection, links by coordinates).
#pragma once

#include "common.h"
#include "su3.h"

namespace lqcd {

namespace {

struct M3 {
  double2 e[9];
};

__device__ __forceinline__ M3 m_zero() {
  M3 r;
#pragma unroll
  for (int i = 0; i < 9; ++i) r.e[i] = make_double2(0.0, 0.0);
  return r;
}

__device__ __forceinline__ M3 m_unit() {
  M3 r = m_zero();
  r.e[0].x = r.e[4].x = r.e[8].x = 1.0;
  return r;
}

// a b, a b^dag, a^dag b
__device__ __forceinline__ M3 m_mul(const M3& a, const M3& b) {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      double2 s = cmul<double>(a.e[3 * i], b.e[j]);
      cfma<double>(s, a.e[3 * i + 1], b.e[3 + j]);
      cfma<double>(s, a.e[3 * i + 2], b.e[6 + j]);
      r.e[3 * i + j] = s;
    }
  return r;
}

__device__ __forceinline__ M3 m_mul_dag(const M3& a, const M3& b) {
  M3 r;  // r_ij = sum_k a_ik conj(b_jk)
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      double2 s = cmulc<double>(b.e[3 * j], a.e[3 * i]);
      cfmac<double>(s, b.e[3 * j + 1], a.e[3 * i + 1]);
      cfmac<double>(s, b.e[3 * j + 2], a.e[3 * i + 2]);
      r.e[3 * i + j] = s;
    }
  return r;
}

__device__ __forceinline__ M3 m_dag_mul(const M3& a, const M3& b) {
  M3 r;  // r_ij = sum_k conj(a_ki) b_kj
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      double2 s = cmulc<double>(a.e[i], b.e[j]);
      cfmac<double>(s, a.e[3 + i], b.e[3 + j]);
      cfmac<double>(s, a.e[6 + i], b.e[6 + j]);
      r.e[3 * i + j] = s;
    }
  return r;
}

__device__ __forceinline__ void m_axpy(double w, const M3& a, M3& acc) {
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    acc.e[i].x = fma(w, a.e[i].x, acc.e[i].x);
    acc.e[i].y = fma(w, a.e[i].y, acc.e[i].y);
  }
}

// Coordinates with periodic wrap (named fields: a direction index chosen at
// run time selects among them, so nothing is indexed dynamically), and the
// link U_mu at a site.
struct C4 {
  int x, y, z, t;
};

__device__ __forceinline__ int wrap(int v, int L) { return v < 0 ? v + L : (v >= L ? v - L : v); }

__device__ __forceinline__ C4 shift(const KGeom& g, C4 s, int mu, int d) {
  if (mu == 0)
    s.x = wrap(s.x + d, g.Lx);
  else if (mu == 1)
    s.y = wrap(s.y + d, g.Ly);
  else if (mu == 2)
    s.z = wrap(s.z + d, g.Lz);
  else
    s.t = wrap(s.t + d, g.Lt);
  return s;
}

__device__ __forceinline__ int half_index(const KGeom& g, const C4& s) {
  return (s.x >> 1) + g.Lxh * (s.y + g.Ly * (s.z + g.Lz * s.t));
}

__device__ __forceinline__ M3 link(const KGeom& g, const double2* __restrict__ U, const C4& s,
                                   int mu) {
  const int par = (s.x + s.y + s.z + s.t) & 1;
  const int h = half_index(g, s);
  const double2* p = U + (int64_t(par) * 4 + mu) * 9 * int64_t(g.Vh) + h;
  M3 r;
#pragma unroll
  for (int e = 0; e < 9; ++e) r.e[e] = p[int64_t(e) * g.Vh];
  return r;
}

__device__ __forceinline__ C4 site_c4(const KGeom& g, int h, int par) {
  const Site s = decode_site(g, h, par);
  return C4{s.x, s.y, s.z, s.t};
}

// TA(W) = (W - W^dag)/2 - Tr(W - W^dag)/6
__device__ __forceinline__ M3 traceless_antiherm(const M3& w) {
  M3 r;
  const double tr_im = (w.e[0].y + w.e[4].y + w.e[8].y) / 3.0;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const double2 a = w.e[3 * i + j], b = w.e[3 * j + i];
      r.e[3 * i + j] = make_double2(0.5 * (a.x - b.x), 0.5 * (a.y + b.y) - (i == j ? tr_im : 0.0));
    }
  return r;
}

// Half-index displacements along one direction: off(d) is the half index of
// the site d steps away minus the site's own (periodic wrap, |d| <= 2).
// Displacements along two directions add, because stepping along one leaves
// the other coordinates alone; the parity changes with the sum of the steps.
struct Axis {
  int c, L, st;  // coordinate, extent, half-index stride (0 marks x)
  __device__ __forceinline__ int off(int d) const {
    const int v = wrap(c + d, L);
    return st == 0 ? (v >> 1) - (c >> 1) : (v - c) * st;
  }
};

__device__ __forceinline__ Axis axis(const KGeom& g, const C4& s, int mu) {
  return mu == 0   ? Axis{s.x, g.Lx, 0}
         : mu == 1 ? Axis{s.y, g.Ly, g.sy}
         : mu == 2 ? Axis{s.z, g.Lz, g.sz}
                   : Axis{s.t, g.Lt, g.st};
}

// The [parity][mu] block of a link field as a buffer resource (parity and mu
// uniform over the wave), and the matrix of half index h in it.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t link_res(const KGeom& g,
                                                           const double2* __restrict__ U, int par,
                                                           int mu) {
  return make_res(U + (int64_t(par) * 4 + mu) * 9 * int64_t(g.Vh), 144u * uint32_t(g.Vh));
}

__device__ __forceinline__ M3 ld_m3(__amdgpu_buffer_rsrc_t r, int h, int Vh) {
  M3 m;
#pragma unroll
  for (int e = 0; e < 9; ++e)
    m.e[e] = ld_buf<double>(r, uint32_t(h) * 16u, uint32_t(e) * uint32_t(Vh) * 16u);
  return m;
}

// Traceless anti-Hermitian 3x3 matrix: entries 01, 02, 12 and the imaginary
// parts of 00 and 11.  Stored as four complex planes.
struct Alg {
  double2 o01, o02, o12, d;
};

__device__ __forceinline__ Alg a_zero() {
  const double2 z = make_double2(0.0, 0.0);
  return Alg{z, z, z, z};
}

__device__ __forceinline__ void a_axpy(double w, const Alg& a, Alg& s) {
  s.o01 = make_double2(fma(w, a.o01.x, s.o01.x), fma(w, a.o01.y, s.o01.y));
  s.o02 = make_double2(fma(w, a.o02.x, s.o02.x), fma(w, a.o02.y, s.o02.y));
  s.o12 = make_double2(fma(w, a.o12.x, s.o12.x), fma(w, a.o12.y, s.o12.y));
  s.d = make_double2(fma(w, a.d.x, s.d.x), fma(w, a.d.y, s.d.y));
}

__device__ __forceinline__ double2 neg(double2 a) { return make_double2(-a.x, -a.y); }

// A u (the entries below the diagonal are minus the conjugates)
__device__ __forceinline__ M3 a_mul(const Alg& a, const M3& u) {
  const double d2 = -(a.d.x + a.d.y);
  M3 t;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    double2 s = make_double2(-a.d.x * u.e[j].y, a.d.x * u.e[j].x);
    cfma<double>(s, a.o01, u.e[3 + j]);
    cfma<double>(s, a.o02, u.e[6 + j]);
    t.e[j] = s;
    s = make_double2(-a.d.y * u.e[3 + j].y, a.d.y * u.e[3 + j].x);
    cfmac<double>(s, neg(a.o01), u.e[j]);
    cfma<double>(s, a.o12, u.e[6 + j]);
    t.e[3 + j] = s;
    s = make_double2(-d2 * u.e[6 + j].y, d2 * u.e[6 + j].x);
    cfmac<double>(s, neg(a.o02), u.e[j]);
    cfmac<double>(s, neg(a.o12), u.e[3 + j]);
    t.e[6 + j] = s;
  }
  return t;
}

// u A
__device__ __forceinline__ M3 m_mul_a(const M3& u, const Alg& a) {
  const double d2 = -(a.d.x + a.d.y);
  M3 t;
#pragma unroll
  for (int i = 0; i < 9; i += 3) {
    double2 s = make_double2(-a.d.x * u.e[i].y, a.d.x * u.e[i].x);
    cfmac<double>(s, neg(a.o01), u.e[i + 1]);
    cfmac<double>(s, neg(a.o02), u.e[i + 2]);
    t.e[i] = s;
    s = make_double2(-a.d.y * u.e[i + 1].y, a.d.y * u.e[i + 1].x);
    cfma<double>(s, a.o01, u.e[i]);
    cfmac<double>(s, neg(a.o12), u.e[i + 2]);
    t.e[i + 1] = s;
    s = make_double2(-d2 * u.e[i + 2].y, d2 * u.e[i + 2].x);
    cfma<double>(s, a.o02, u.e[i]);
    cfma<double>(s, a.o12, u.e[i + 1]);
    t.e[i + 2] = s;
  }
  return t;
}

// s TA(w)
__device__ __forceinline__ Alg ta(const M3& w, double s) {
  const double tr = (w.e[0].y + w.e[4].y + w.e[8].y) / 3.0, h = 0.5 * s;
  return Alg{make_double2(h * (w.e[1].x - w.e[3].x), h * (w.e[1].y + w.e[3].y)),
             make_double2(h * (w.e[2].x - w.e[6].x), h * (w.e[2].y + w.e[6].y)),
             make_double2(h * (w.e[5].x - w.e[7].x), h * (w.e[5].y + w.e[7].y)),
             make_double2(s * (w.e[0].y - tr), s * (w.e[4].y - tr))};
}

// the full matrix
__device__ __forceinline__ M3 a_full(const Alg& a) {
  M3 r;
  r.e[0] = make_double2(0.0, a.d.x);
  r.e[4] = make_double2(0.0, a.d.y);
  r.e[8] = make_double2(0.0, -(a.d.x + a.d.y));
  r.e[1] = a.o01;
  r.e[2] = a.o02;
  r.e[5] = a.o12;
  r.e[3] = make_double2(-a.o01.x, a.o01.y);
  r.e[6] = make_double2(-a.o02.x, a.o02.y);
  r.e[7] = make_double2(-a.o12.x, a.o12.y);
  return r;
}

// A matrix of the wave's 64 lanes in LDS, one element after the other.
__device__ __forceinline__ M3 lds_m3(const double2 (&s)[9][64], int lane) {
  M3 m;
#pragma unroll
  for (int e = 0; e < 9; ++e) m.e[e] = s[e][lane];
  return m;
}

// a b, with a read from LDS as it is used (no registers held for it)
__device__ __forceinline__ M3 lds_mul(const double2 (&a)[9][64], int lane, const M3& b) {
  M3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      double2 s = cmul<double>(a[3 * i][lane], b.e[j]);
      cfma<double>(s, a[3 * i + 1][lane], b.e[3 + j]);
      cfma<double>(s, a[3 * i + 2][lane], b.e[6 + j]);
      r.e[3 * i + j] = s;
    }
  return r;
}

}  // namespace

}  // namespace lqcd
