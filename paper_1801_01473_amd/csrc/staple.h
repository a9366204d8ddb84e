// The plaquette staples of a link, by workgroups of 64 half indices of one parity
// whose waves are the link's directions (chunk_site).  The four directions of a
// site share most of the links around it: those that several waves use go
// through LDS.
#pragma once

#include "m3.h"
#include "tile.h"

namespace lqcd {

__device__ __forceinline__ M3 m_add(M3 a, const M3& b) {
#pragma unroll
  for (int e = 0; e < 9; ++e) a.e[e] = make_double2(a.e[e].x + b.e[e].x, a.e[e].y + b.e[e].y);
  return a;
}

__device__ __forceinline__ void st_m3(double2* p, int Vh, const M3& m) {
#pragma unroll
  for (int e = 0; e < 9; ++e) p[int64_t(e) * Vh] = m.e[e];
}

// The links U_mu(x) and U_mu(x - mu), mu = 0..3, of the workgroup's sites.
using Near = double2[2][4][9][64];

__device__ __forceinline__ void stage_links(const KGeom& g, const double2* __restrict__ U,
                                            const ChunkSite& cs, const C4& x, Near& sh) {
  const int mu = cs.task;
  const M3 u = ld_m3(link_res(g, U, cs.par, mu), cs.h, g.Vh);
  const M3 v = ld_m3(link_res(g, U, 1 - cs.par, mu), cs.h + axis(g, x, mu).off(-1), g.Vh);
#pragma unroll
  for (int e = 0; e < 9; ++e) {
    sh[0][mu][e][cs.lane] = u.e[e];
    sh[1][mu][e][cs.lane] = v.e[e];
  }
  __syncthreads();
}

// Sum of the six plaquette staples of the link (x, a), a = cs.task:
//   U_b(x+a) U_a(x+b)^dag U_b(x)^dag + U_b(x+a-b)^dag U_a(x-b)^dag U_b(x-b)
__device__ __forceinline__ M3 staple_sum(const KGeom& g, const double2* __restrict__ U,
                                         const ChunkSite& cs, const C4& x, const Near& sh) {
  const int a = cs.task, h = cs.h, opp = 1 - cs.par;
  const int ha = h + axis(g, x, a).off(1);
  const auto a_o = link_res(g, U, opp, a);
  M3 A = m_zero();
#pragma unroll 1
  for (int b = 0; b < 4; ++b) {
    if (b == a) continue;
    const Axis xb = axis(g, x, b);
    const int up = xb.off(1), dn = xb.off(-1);
    const M3 t = m_mul_dag(ld_m3(link_res(g, U, opp, b), ha, g.Vh), ld_m3(a_o, h + up, g.Vh));
    A = m_add(A, m_mul_dag(t, lds_m3(sh[0][b], cs.lane)));
    const M3 d = m_dag_mul(ld_m3(a_o, h + dn, g.Vh), lds_m3(sh[1][b], cs.lane));
    A = m_add(A, m_dag_mul(ld_m3(link_res(g, U, cs.par, b), ha + dn, g.Vh), d));
  }
  return A;
}

}  // namespace lqcd
