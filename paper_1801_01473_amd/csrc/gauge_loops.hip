// The Symanzik gauge force through loop fields (Sec. 4.3: the 1x1 and 1x2
// rectangles are the building blocks of the gauge force).
//
// For a plane of directions a < b and a site x, with the links of that plane,
//   l(x)  the plaquette        a, b, -a, -b
//   ra(x) the 2x1 rectangle    a, a, b, -a, -a, -b
//   rb(x) the 1x2 rectangle    a, b, b, -a, -b, -b
// closed loops at x, of which only the traceless anti-Hermitian part TA is
// needed: F_a(x) = -(beta/3) sum of w TA(loop at x that starts along a) over
// the loops through the link (x, a), and TA commutes with moving a loop's
// base point, TA(V^dag W V) = V^dag TA(W) V for unitary V (a site near a link that
// is not unitary to rounding has its staples multiplied out instead).  Every loop through
// (x, a) is one of l, ra, rb based at x, x-a, x-b, x-2b or x-a-b, moved to x
// along its own links, reversed (sign -) where (x, a) is its upper side:
//   F_a/(-beta/3) = c0 l(x) + c1 (ra(x) + rb(x))
//     - Ub(x-b)^dag [ c0 l(x-b) + c1 ra(x-b) + c1 Ub(x-2b)^dag rb(x-2b) Ub(x-2b) ] Ub(x-b)
//     + c1 Ua(x-a)^dag [ ra(x-a) - Ub(x-a-b)^dag ra(x-a-b) Ub(x-a-b) ] Ua(x-a)
// summed over b (the last transport once for the sum).  For b < a the stored
// loops of the plane (b, a) run the other way round: l -> -l, ra -> -rb,
// rb -> -ra.
//
// Pass 1 (k_loops, one thread per site and plane): 11 SU(3) products; TA of the
// loops, stored as 8 reals each.  Pass 2 (k_loop_force, one thread per link):
// 10 transports V^dag A V, about 0.64 of two products each.  That is 66 + 51
// products per site, against 204 when the plaquette staples of each plane
// were stored as full matrices and 340 with every staple multiplied out, and
// 2 launches instead of 12.  Both passes are bound by their memory path, not
// by arithmetic (with the products taken out of a copy they took the same
// time): pass 1 by HBM (12.3 GB read past L2 for 3.1 GB of links, 6.1 GB written,
// 3.6 ms at 48^4), pass 2 by what misses L2 (60 % of its requests, 24.3 GB at 6.4
// TB/s, 3.8 ms: the sites in flight on an XCD have 9 MB of fields, links and
// forces), so the links that the waves of a workgroup share go through LDS
// (4.5 -> 3.7 ms).
// 48^4: 25.7 ms with stored staples, 7.1 ms now (7.0 without the look at the links).
#include <hip/hip_runtime.h>

#include <cmath>

#include "gauge.h"
#include "m3.h"
#include "tile.h"

namespace lqcd {

namespace {

// TA(a b^dag)
__device__ __forceinline__ Alg ta_mul_dag(const M3& a, const M3& b) {
  return ta(m_mul_dag(a, b), 1.0);
}

// U^dag A U
__device__ __forceinline__ Alg transport(const M3& u, const Alg& a) {
  const M3 t = a_mul(a, u);
  auto entry = [&](int i, int j) {
    double2 s = cmulc<double>(u.e[i], t.e[j]);
    cfmac<double>(s, u.e[3 + i], t.e[3 + j]);
    cfmac<double>(s, u.e[6 + i], t.e[6 + j]);
    return s;
  };
  auto diag = [&](int i) {  // imaginary part only
    double s = fma(u.e[i].x, t.e[i].y, -(u.e[i].y * t.e[i].x));
    s = fma(u.e[3 + i].x, t.e[3 + i].y, fma(-u.e[3 + i].y, t.e[3 + i].x, s));
    return fma(u.e[6 + i].x, t.e[6 + i].y, fma(-u.e[6 + i].y, t.e[6 + i].x, s));
  };
  return Alg{entry(0, 1), entry(0, 2), entry(1, 2), make_double2(diag(0), diag(1))};
}

// The planes whose loop fields one pass pair holds: slot s has the fields
//   0: c0 l + c1 (ra + rb), the sum that both directions take at x itself
//      (c0 l + c1 ra is that minus c1 rb), -beta/3 included,  1: ra,  2: rb.
struct Planes {
  int n;
  int a[6], b[6];
  int slot[4][4];  // plane of two directions, -1: not in this pass
  int dirs;        // bit mu: the pass writes F_mu
  int add;         // bit mu: add to F_mu instead of writing it
  int sh;          // log2 of the chunk of half indices
};

constexpr size_t kPlaneBytes = 3 * 128;  // loop fields of a plane per half index, both parities

// Loop fields are stored by chunks of 2^sh half indices, [chunk][parity][slot]
// [field][4][2^sh], so that what a wave reads around a site lies in a few
// contiguous regions instead of one page per plane of the lattice (3 % of the
// force at 48^4).  The chunk divides Vh (a multiple of 8): the largest of 64,
// 32, 16, 8, so the fields fill Vh entries exactly.
inline int chunk_shift(int Vh) {
  int s = 6;
  while (Vh & ((1 << s) - 1)) --s;
  return s;
}

__device__ __forceinline__ double2* field_at(double2* P, const Planes& pl, int slot, int f,
                                             int par, int h) {
  const int64_t c = int64_t(h >> pl.sh) * 2 + par;
  return P + ((c * (pl.n * 12) + (slot * 3 + f) * 4) << pl.sh) + (h & ((1 << pl.sh) - 1));
}

__device__ __forceinline__ Alg ld_alg(const double2* __restrict__ P, const Planes& pl, int slot,
                                      int f, int par, int h) {
  const double2* p = field_at(const_cast<double2*>(P), pl, slot, f, par, h);
  const int n = 1 << pl.sh;
  return Alg{p[0], p[n], p[2 * n], p[3 * n]};
}

// Stores past the caches (NT) where the fields of a pass exceed the 256 MB
// last-level cache, so that they leave the links there: 48^4 3.59 -> 3.44 ms in
// k_loops, 3.73 -> 3.66 in k_loop_force; smaller lattices read both back from it.
constexpr int64_t kStreamFieldBytes = int64_t(256) << 20;

template <bool NT>
__device__ __forceinline__ void st(double2* p, double2 v) {
  if constexpr (NT) {
    typedef double V2 __attribute__((ext_vector_type(2)));
    __builtin_nontemporal_store(V2{v.x, v.y}, reinterpret_cast<V2*>(p));
  } else {
    *p = v;
  }
}

template <bool NT>
__device__ __forceinline__ void st_alg(double2* __restrict__ P, const Planes& pl, int slot, int f,
                                       int par, int h, const Alg& a) {
  double2* p = field_at(P, pl, slot, f, par, h);
  const int n = 1 << pl.sh;
  st<NT>(p, a.o01);
  st<NT>(p + n, a.o02);
  st<NT>(p + 2 * n, a.o12);
  st<NT>(p + 3 * n, a.d);
}

// What a wave of the plane kernels works with: one plane of 64 sites of one
// parity, its links by displacement, and the links U_mu(x) and U_mu(x + mu) of
// the workgroup's sites in LDS (three planes use each of them, twice each).
using Ahead = double2[2][4][9][64];

struct PlaneSite {
  __amdgpu_buffer_rsrc_t a_s, b_s, a_o, b_o;  // links leaving sites of the same / other parity
  int h, a1, b1, ab, a2, b2;                  // x, x + a, x + b, x + a + b, x + 2a, x + 2b
};

__device__ __forceinline__ PlaneSite plane_site(const KGeom& g, const double2* __restrict__ U,
                                                const ChunkSite& cs, int n, int a, int b,
                                                Ahead& sh) {
  const int h = cs.h, par = cs.par, opp = 1 - par;
  const C4 x = site_c4(g, h, par);
  for (int m = cs.task; m < 8; m += n) {
    const int mu = m & 3, far = m >> 2;
    const M3 u = ld_m3(link_res(g, U, far ? opp : par, mu),
                       h + (far ? axis(g, x, mu).off(1) : 0), g.Vh);
#pragma unroll
    for (int e = 0; e < 9; ++e) sh[far][mu][e][cs.lane] = u.e[e];
  }
  const Axis xa = axis(g, x, a), xb = axis(g, x, b);
  PlaneSite p;
  p.h = h;
  p.a1 = h + xa.off(1);
  p.b1 = h + xb.off(1);
  p.ab = p.a1 + (p.b1 - h);
  p.a2 = h + xa.off(2);
  p.b2 = h + xb.off(2);
  p.a_s = link_res(g, U, par, a);
  p.b_s = link_res(g, U, par, b);
  p.a_o = link_res(g, U, opp, a);
  p.b_o = link_res(g, U, opp, b);
  __syncthreads();
  return p;
}

// One workgroup per 64 half indices of both parities, wave = plane.
template <bool NT>
__global__ void __launch_bounds__(768, 3) k_loops(KGeom g, const double2* __restrict__ U,
                                                  const Planes pl, double w0, double w1, int ty,
                                                  int tz, double2* __restrict__ P) {
  __shared__ Ahead ahead[2];
  const ChunkSite cs = chunk_pair_site(g, pl.n, ty, tz);
  Ahead& sh = ahead[cs.par];
  const int lane = cs.lane, task = cs.task, a = pl.a[task], b = pl.b[task];
  const PlaneSite p = plane_site(g, U, cs, pl.n, a, b, sh);
  if (!cs.in) return;
  // (the barriers keep the compiler from loading every section's links at
  // once: 168 registers without spilling, three waves a SIMD)
  const M3 c1 = lds_mul(sh[0][a], lane, ld_m3(p.b_o, p.a1, g.Vh));  // a, b
  __builtin_amdgcn_sched_barrier(0);
  const M3 c2 = lds_mul(sh[0][b], lane, ld_m3(p.a_o, p.b1, g.Vh));  // b, a
  Alg sum = a_zero();
  a_axpy(w0, ta_mul_dag(c1, c2), sum);
  __builtin_amdgcn_sched_barrier(0);
  {
    const M3 r = m_mul(c2, ld_m3(p.a_s, p.ab, g.Vh));  // b, a, a
    const M3 e = lds_mul(sh[1][a], lane, ld_m3(p.b_s, p.a2, g.Vh));
    const M3 l = lds_mul(sh[0][a], lane, e);  // a, a, b
    const Alg ra = ta_mul_dag(l, r);
    st_alg<NT>(P, pl, task, 1, cs.par, p.h, ra);
    a_axpy(w1, ra, sum);
  }
  __builtin_amdgcn_sched_barrier(0);
  {
    const M3 l = m_mul(c1, ld_m3(p.b_s, p.ab, g.Vh));  // a, b, b
    const M3 e = lds_mul(sh[1][b], lane, ld_m3(p.a_s, p.b2, g.Vh));
    const M3 r = lds_mul(sh[0][b], lane, e);  // b, b, a
    const Alg rb = ta_mul_dag(l, r);
    st_alg<NT>(P, pl, task, 2, cs.par, p.h, rb);
    a_axpy(w1, rb, sum);
  }
  st_alg<NT>(P, pl, task, 0, cs.par, p.h, sum);
}

// Re Tr[a b^dag]
__device__ __forceinline__ double re_tr_dag(const M3& a, const M3& b) {
  double s = 0.0;
#pragma unroll
  for (int e = 0; e < 9; ++e) s = fma(a.e[e].x, b.e[e].x, fma(a.e[e].y, b.e[e].y, s));
  return s;
}

// The action of the loops whose first corner is x, one plane per wave as in
// k_loops: w (1 - Re Tr / 3) of the plaquette and of both rectangles, 8 products
// per plane (the last one of each loop is only a trace).  24^3 x 48: 0.30 ms, bound
// by the latency of 44 link matrices per site, 4.2 GB, of which L2 holds 86 %
// (14 TB/s at 12 waves a CU; one parity a workgroup, 6 waves a CU, 0.38 ms); one
// thread per site over all loops, 13 products per plane, took 1.03 ms.
__global__ void __launch_bounds__(768, 3) k_loop_action(KGeom g, const double2* __restrict__ U,
                                                        const Planes pl, double c0, double c1,
                                                        int ty, int tz,
                                                        double* __restrict__ part) {
  __shared__ Ahead ahead[2];
  __shared__ double lds[12];
  const ChunkSite cs = chunk_pair_site(g, pl.n, ty, tz);
  Ahead& sh = ahead[cs.par];
  const int lane = cs.lane, a = pl.a[cs.task], b = pl.b[cs.task];
  const PlaneSite p = plane_site(g, U, cs, pl.n, a, b, sh);
  const M3 ca = lds_mul(sh[0][a], lane, ld_m3(p.b_o, p.a1, g.Vh));  // a, b
  __builtin_amdgcn_sched_barrier(0);
  const M3 cb = lds_mul(sh[0][b], lane, ld_m3(p.a_o, p.b1, g.Vh));  // b, a
  double s = c0 * (1.0 - re_tr_dag(ca, cb) / 3.0);
  if (c1 != 0.0) {
    __builtin_amdgcn_sched_barrier(0);
    {
      const M3 r = m_mul(cb, ld_m3(p.a_s, p.ab, g.Vh));  // b, a, a
      const M3 e = lds_mul(sh[1][a], lane, ld_m3(p.b_s, p.a2, g.Vh));
      s += c1 * (1.0 - re_tr_dag(lds_mul(sh[0][a], lane, e), r) / 3.0);
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      const M3 l = m_mul(ca, ld_m3(p.b_s, p.ab, g.Vh));  // a, b, b
      const M3 e = lds_mul(sh[1][b], lane, ld_m3(p.a_s, p.b2, g.Vh));
      s += c1 * (1.0 - re_tr_dag(l, lds_mul(sh[0][b], lane, e)) / 3.0);
    }
  }
  s = block_sum(cs.in ? s : 0.0, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// Whether a link's rows are orthonormal to rounding (2^-46: links of one update or
// exponential are within some 2^-50, and drift as the root of the products taken).
// A transport V^dag TA(W) V stands for TA(V^-1 W V), so it may only pass along such
// links; an error of d in V^dag V would enter the force about six times.
__device__ __forceinline__ bool unitary(const M3& u) {
  constexpr double kTol = 0x1p-46;
  double worst = 0.0;
#pragma unroll
  for (int i = 0; i < 9; i += 3) {
    double n = -1.0;
#pragma unroll
    for (int e = i; e < i + 3; ++e) n = fma(u.e[e].x, u.e[e].x, fma(u.e[e].y, u.e[e].y, n));
    double2 d = make_double2(0.0, 0.0);
    const int j = (i + 3) % 9;
#pragma unroll
    for (int e = 0; e < 3; ++e) cfmac<double>(d, u.e[i + e], u.e[j + e]);
    worst += fabs(n) + fabs(d.x) + fabs(d.y);  // (a sum: NaN stays)
  }
  return worst <= kTol;
}

// TA of U_a(x) times the weighted staples of the link (x, a) in its plane with b,
// each multiplied out along its path from x + a to x: for the sites whose loops
// cannot be moved along their links (all of them, single-precision links: 48^4
// 24.1 ms, 8^4 94 us; one link of 8^4 135 us, a chain of 108 steps).  The steps of a path, two bits each from the lowest:
// 0 +a, 1 +b, 2 -a, 3 -b; the paths below the link have b reversed.
__device__ __forceinline__ Alg direct_loops(const KGeom& g, const double2* __restrict__ U,
                                            const C4& x, int par, int a, int b, double w0,
                                            double w1) {
  constexpr int kSteps[4] = {
      1 | 2 << 2 | 3 << 4,                        // +b -a -b
      0 | 1 << 2 | 2 << 4 | 2 << 6 | 3 << 8,      // +a +b -a -a -b
      1 | 2 << 2 | 2 << 4 | 3 << 6 | 0 << 8,      // +b -a -a -b +a
      1 | 1 << 2 | 2 << 4 | 3 << 6 | 3 << 8,      // +b +b -a -b -b
  };
  M3 sum = m_zero();
#pragma unroll 1
  for (int k = 0; k < 8; ++k) {
    const int q = k >> 1;
    int code = q == 0 ? kSteps[0] : q == 1 ? kSteps[1] : q == 2 ? kSteps[2] : kSteps[3];
    M3 t = m_unit();
    C4 s = shift(g, x, a, 1);
    int p = 1 - par;
#pragma unroll 1
    for (int n = q == 0 ? 3 : 5; n > 0; --n, code >>= 2) {
      const int mu = code & 1 ? b : a;
      const bool back = ((code >> 1) ^ (code & k & 1)) & 1;
      if (back) s = shift(g, s, mu, -1);
      const M3 u = ld_m3(link_res(g, U, back ? 1 - p : p, mu), half_index(g, s), g.Vh);
#pragma unroll
      for (int i = 0; i < 9; i += 3) {  // row by row, in place
        double2 r[3];
        if (back) {
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            r[j] = cmulc<double>(u.e[3 * j], t.e[i]);
            cfmac<double>(r[j], u.e[3 * j + 1], t.e[i + 1]);
            cfmac<double>(r[j], u.e[3 * j + 2], t.e[i + 2]);
          }
        } else {
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            r[j] = cmul<double>(t.e[i], u.e[j]);
            cfma<double>(r[j], t.e[i + 1], u.e[3 + j]);
            cfma<double>(r[j], t.e[i + 2], u.e[6 + j]);
          }
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) t.e[i + j] = r[j];
      }
      if (!back) s = shift(g, s, mu, 1);
      p = 1 - p;
    }
    m_axpy(q == 0 ? w0 : w1, t, sum);
  }
  return ta(m_mul(ld_m3(link_res(g, U, par, a), half_index(g, x), g.Vh), sum), 1.0);
}

// One workgroup per 64 half indices of one parity, wave = direction a.  The
// links U_mu(x - mu), U_mu(x - 2 mu) of the transports, which three or four
// waves use, go through LDS: 20 link matrices per site from L2 instead of 40.
template <bool NT>
__global__ void __launch_bounds__(256, 2) k_loop_force(KGeom g, const double2* __restrict__ U,
                                                       const double2* __restrict__ P,
                                                       const Planes pl, double w0, double w1,
                                                       int ty, int tz, double2* __restrict__ F) {
  __shared__ double2 sh[4][2][9][64];  // U_mu(x - mu), U_mu(x - 2 mu)
  __shared__ bool movable[4][64];      // loops can be moved along both
  const ChunkSite cs = chunk_site(g, ty, tz);
  const int h = cs.h, par = cs.par, opp = 1 - par, lane = cs.lane, a = cs.task;
  const C4 x = site_c4(g, h, par);
  {
    const Axis xa = axis(g, x, a);
    const M3 u1 = ld_m3(link_res(g, U, opp, a), h + xa.off(-1), g.Vh);
    const M3 u2 = ld_m3(link_res(g, U, par, a), h + xa.off(-2), g.Vh);
#pragma unroll
    for (int e = 0; e < 9; ++e) {
      sh[a][0][e][lane] = u1.e[e];
      sh[a][1][e][lane] = u2.e[e];
    }
    movable[a][lane] = unitary(u1) & unitary(u2);
  }
  __syncthreads();
  bool ok = movable[0][lane] & movable[1][lane] & movable[2][lane] & movable[3][lane];
  const int am = axis(g, x, a).off(-1);
  Alg f = a_zero(), q = a_zero();
#pragma unroll 1
  for (int b = 0; b < 4; ++b) {
    if (b == a) continue;
    const int s = pl.slot[a][b];
    if (s < 0) continue;
    const double sg = a < b ? 1.0 : -1.0;
    const int fa = a < b ? 1 : 2, fb = 3 - fa;  // fields of ra, rb
    const Axis xb = axis(g, x, b);
    const int hb = h + xb.off(-1), h2 = h + xb.off(-2);
    Alg z = ld_alg(P, pl, s, 0, opp, hb);
    Alg y = transport(lds_m3(sh[b][1], lane), ld_alg(P, pl, s, fb, par, h2));
    a_axpy(-1.0, ld_alg(P, pl, s, fb, opp, hb), y);
    a_axpy(w1, y, z);
    z = transport(lds_m3(sh[b][0], lane), z);
    a_axpy(-sg, z, f);
    a_axpy(sg, ld_alg(P, pl, s, 0, par, h), f);
    a_axpy(sg, ld_alg(P, pl, s, fa, opp, h + am), q);
    const M3 v = ld_m3(link_res(g, U, par, b), hb + am, g.Vh);
    y = transport(v, ld_alg(P, pl, s, fa, par, hb + am));
    ok = ok & unitary(v);
    a_axpy(-sg, y, q);
  }
  if (!cs.in || !((pl.dirs >> a) & 1)) return;
  a_axpy(w1, transport(lds_m3(sh[a][0], lane), q), f);
  if (!ok) {
    f = a_zero();
#pragma unroll 1
    for (int b = 0; b < 4; ++b)
      if (b != a && pl.slot[a][b] >= 0) a_axpy(1.0, direct_loops(g, U, x, par, a, b, w0, w1), f);
  }
  double2* out = F + (int64_t(par) * 4 + a) * 9 * g.Vh + h;
  const M3 v = a_full(f);
  const bool add = (pl.add >> a) & 1;
#pragma unroll
  for (int e = 0; e < 9; ++e) {
    double2 z = v.e[e];
    if (add) {
      const double2 o = out[int64_t(e) * g.Vh];
      z.x += o.x;
      z.y += o.y;
    }
    st<NT>(out + int64_t(e) * g.Vh, z);
  }
}

// The passes over planes [lo, hi) of the list 01, 02, 03, 12, 13, 23.
Planes plane_pass(int lo, int hi, int accumulate, int* seen) {
  Planes p{};
  for (auto& r : p.slot)
    for (int& v : r) v = -1;
  int used = 0, i = 0;
  for (int a = 0; a < 4; ++a)
    for (int b = a + 1; b < 4; ++b, ++i) {
      if (i < lo || i >= hi) continue;
      p.slot[a][b] = p.slot[b][a] = p.n;
      p.a[p.n] = a;
      p.b[p.n] = b;
      ++p.n;
      used |= (1 << a) | (1 << b);
    }
  p.dirs = used;
  p.add = accumulate ? 15 : *seen;
  *seen |= used;
  return p;
}

}  // namespace

unsigned gauge_action_blocks(const KGeom& k) { return chunk_pair_blocks(k.Vh); }

int gauge_action_partials(const KGeom& k, const double2* U, double c1, double* part,
                          hipStream_t s) {
  int seen = 0;
  const Planes p = plane_pass(0, 6, 0, &seen);
  hipLaunchKernelGGL(k_loop_action, dim3(gauge_action_blocks(k)), dim3(128 * p.n), 0, s, k, U, p,
                     1.0 - 8.0 * c1, c1, chunk_tile(k.Ly, 16), chunk_tile(k.Lz, 7), part);
  LQCD_LAUNCH_CHECK();
  return LQCD_OK;
}

}  // namespace lqcd

using namespace lqcd;

extern "C" {

size_t lqcd_gauge_force_staples_workspace_bytes(const lqcd_geom* g) {
  if (check_geom(g)) return 0;
  const KGeom k = make_kgeom(g);
  return size_t(4) * 2 * 9 * size_t(k.Vh) * sizeof(double2);
}

int lqcd_gauge_force_staples(const lqcd_geom* g, const void* U64, double beta, double c1,
                             int32_t accumulate, void* F, void* ws, size_t ws_bytes,
                             void* stream) {
  clear_error();
  int rc;
  if ((rc = check_geom(g)) || (rc = check_ptr(U64, "U64")) || (rc = check_ptr(F, "F")) ||
      (rc = check_ptr(ws, "ws")))
    return rc;
  if (!std::isfinite(beta) || !std::isfinite(c1)) {
    set_error("beta and c1 must be finite");
    return LQCD_ERR_INVALID_ARG;
  }
  if (accumulate != 0 && accumulate != 1) {
    set_error("accumulate must be 0 or 1");
    return LQCD_ERR_INVALID_ARG;
  }
  if (F == U64 || ws == U64 || ws == F) {
    set_error("F, U64 and ws must be distinct buffers");
    return LQCD_ERR_INVALID_ARG;
  }
  const size_t need = lqcd_gauge_force_staples_workspace_bytes(g);
  if (ws_bytes < need) {
    set_error("gauge force workspace of %zu bytes is too small: %zu needed", ws_bytes, need);
    return LQCD_ERR_WORKSPACE;
  }
  const KGeom k = make_kgeom(g);
  const hipStream_t s = (hipStream_t)stream;
  const double2* U = static_cast<const double2*>(U64);
  double2* P = static_cast<double2*>(ws);
  double2* out = static_cast<double2*>(F);
  if (c1 == 0.0) return gauge_force_direct(k, U, beta, 0.0, accumulate, out, s);
  // The required workspace holds the loop fields of three planes (two pass
  // pairs, the second adding to F); given room for all six, one pair writes F.
  const int step = ws_bytes >= 6 * kPlaneBytes * size_t(k.Vh) ? 6 : 3;
  const int ty = chunk_tile(k.Ly, 16), tz = chunk_tile(k.Lz, 7);
  const double w0 = -beta / 3.0 * (1.0 - 8.0 * c1), w1 = -beta / 3.0 * c1;
  int seen = 0;
  for (int lo = 0; lo < 6; lo += step) {
    Planes p = plane_pass(lo, lo + step, accumulate, &seen);
    p.sh = chunk_shift(k.Vh);
    const bool nt = int64_t(p.n) * int64_t(kPlaneBytes) * k.Vh > kStreamFieldBytes;
    hipLaunchKernelGGL(nt ? k_loops<true> : k_loops<false>, dim3(chunk_pair_blocks(k.Vh)),
                       dim3(128 * p.n), 0, s, k, U, p, w0, w1, ty, tz, P);
    LQCD_LAUNCH_CHECK();
    hipLaunchKernelGGL(nt ? k_loop_force<true> : k_loop_force<false>, dim3(chunk_blocks(k.Vh)),
                       dim3(256), 0, s, k, U, P, p, w0, w1, ty, tz, out);
    LQCD_LAUNCH_CHECK();
  }
  return LQCD_OK;
}

}  // extern "C"
