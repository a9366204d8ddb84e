// Fermion force and rational pseudofermion action.
//
// The action of Eq. (1) with M^(-1/4) in rational form is
//   S = sum_j [ alpha_0 |phi_j|^2 + sum_i alpha_i Re <phi_j, X_ji> ],
//   X_ji = (A + sigma_i)^-1 phi_j,  A = m^2 + D_oe^dag D_oe  (D_eo = -D_oe^dag).
// Its variation is dS = -sum alpha_i <X, dA X> = -2 sum alpha_i Re <chi, dD_oe X>
// with chi = D_oe X, which, link by link, is dS = sum Re Tr[dU_mu(x) M_mu(x)] with
//   x odd : M_mu(x) = -sum alpha eta_mu(x) s_mu(x) X(x+mu) chi(x)^dag
//   x even: M_mu(x) = +sum alpha eta_mu(x) s_mu(x) chi(x+mu) X(x)^dag.
// Every link touches exactly one odd site as either its forward link (x odd)
// or the backward link of x+mu (x even), so one odd site y owns the eight
// links of its star and writes each of them once: no atomics.
//
// Work split: a workgroup takes 64 odd sites and wave mu owns their links (y, mu)
// and (y - mu, mu).  For each (pseudofermion, shift) pair a lane computes the
// direction-mu part of chi(y) = (D_oe X)(y) with its two links, the four parts
// are added through LDS (same order in every wave), and the lane adds the two
// outer products into its two 3x3 accumulators.  chi is never written to memory.
// At the end the lane projects U M to the traceless anti-Hermitian part (mode 0)
// or writes M^dag (mode 1, torch's gradient).
//
// At 32^3 x 48 with 48 pairs the kernel takes 1.63 ms (1.74 ms with four lanes
// of one wave per site and two shuffles per pair): 464 M vector instructions
// keep the FP64 units busy 55 % of the time at the 1.9-2.0 GHz that the card
// holds under them, 15 GB of loads go through L1 (11 GB from L2, 5.2 GB from
// memory against 2.7 GB that must be read).  With every X read from L2 it would
// take 1.42 ms.  Two lanes per link at twice the waves (1.67 ms), loads one pair
// ahead (1.63 ms, but 3 % slower where few waves are in flight), the next pair's
// hop over this pair's LDS reads (1.65 ms) and two sites' waves in a workgroup
// (1.71 ms) gain nothing.
#include <hip/hip_runtime.h>

#include <cmath>
#include <mutex>

#include "common.h"
#include "solver.h"
#include "su3.h"
#include "tile.h"

namespace lqcd {

namespace {

constexpr int kForceBlock = 256;  // 4 directions x 64 odd sites

// Up to 256 workgroups, one a CU, a workgroup has two groups of four waves that
// take every other pair: a wave is then bound by the latency of one pair after
// the other, 0.7 us.  4 x 12 pairs: 8^4 30 us (40 with one group), 12^4 34 us (42);
// past one workgroup a CU it loses, 16^4 78 us (74), with 4 pairs 26 us (18).
constexpr int kForceGroupsVh = 64 * 256;
constexpr int kActionBlock = 256;
constexpr int kCombineBlock = 256;

struct Alphas {
  double a[kMaxShift];
};

// Block partials and the final sum of lqcd_action_noalloc live here instead of
// in a caller workspace: 1 MiB, i.e. ceil(Vh/256) + 32 doubles for any Vh up to
// 33.5 million, more than the largest lattice the library accepts.  Each device
// holds its own copy until the process ends.  Host code never passes this name
// to a kernel (on the host it is only a stand-in for the symbol): it uses the
// device address that hipGetSymbolAddress returns for the current device.
constexpr size_t kActionScratchDoubles = size_t(1) << 17;
static __device__ __align__(256) double scratch[kActionScratchDoubles];

constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_dev[kMaxScratchDevices] = {};

template <int G>
__global__ void __launch_bounds__(G * kForceBlock, 2) k_force(const KGeom g,
                                                          const double2* __restrict__ U,
                                                          const double2* __restrict__ X, int npf,
                                                          int nshift, const Alphas al, int mode,
                                                          int accumulate, int ty, int tz,
                                                          double2* __restrict__ F) {
  // Every even X is read by its eight odd neighbours, for every pair, so the
  // sites sharing neighbours run close together and on one XCD (one L2):
  // consecutive blocks of an XCD take consecutive sites of a (y, z)-tiled
  // order with t inside the tile, and the waves of a workgroup, in step
  // over the pairs, find most of a site's neighbours in L1.
  __shared__ double2 parts[G][2][4][3][64];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int mu = w & 3, grp = w >> 2;
  double2 (&part)[2][4][3][64] = parts[grp];
  const int i0 = xcd_block(blockIdx.x, gridDim.x, 1) * 64 + lane;
  const bool in = i0 < g.Vh;  // lanes past Vh work on the first site and store nothing
  const int h = tiled_half_index(g, in ? i0 : 0, ty, tz);  // odd site
  const Site s = decode_site(g, h, 1);
  int fwd[4], bwd[4];
  neighbours(g, s, h, fwd, bwd);
  const int hf = mu == 0 ? fwd[0] : mu == 1 ? fwd[1] : mu == 2 ? fwd[2] : fwd[3];
  const int hb = mu == 0 ? bwd[0] : mu == 1 ? bwd[1] : mu == 2 ? bwd[2] : bwd[3];
  const int ep = ((mu >= 1 ? s.x : 0) + (mu >= 2 ? s.y : 0) + (mu >= 3 ? s.z : 0)) & 1;
  double sf = ep ? -1.0 : 1.0, sb = -sf;  // eta_mu(y) s_mu(y), -eta_mu(y-mu) s_mu(y-mu)
  if (mu == 3 && g.anti) {
    if (s.t == g.Lt - 1) sf = -sf;
    if (s.t == 0) sb = -sb;
  }
  const int64_t pstride = int64_t(4) * 9 * g.Vh;
  Su3<double> Uf, Ub;
  load_link<double, 9>(U + pstride + int64_t(mu) * 9 * g.Vh, h, g.Vh, Uf);  // (y, mu), y odd
  load_link<double, 9>(U + int64_t(mu) * 9 * g.Vh, hb, g.Vh, Ub);           // (y-mu, mu), even

  Su3<double> Mf, Mb;
#pragma unroll
  for (int e = 0; e < 9; ++e) Mf.e[e] = Mb.e[e] = mk<double>(0, 0);
  // The hop coefficients sf/2, sb/2 (a sign and a power of two, so exactly)
  // go into the links, which then give the direction-mu part of chi directly.
#pragma unroll
  for (int e = 0; e < 9; ++e) {
    Uf.e[e] = cscale<double>(0.5 * sf, Uf.e[e]);
    Ub.e[e] = cscale<double>(0.5 * sb, Ub.e[e]);
  }

  const int npair = npf * nshift;
  const uint32_t of = uint32_t(hf) * uint32_t(sizeof(double2));
  const uint32_t ob = uint32_t(hb) * uint32_t(sizeof(double2));
  const int64_t cs = int64_t(g.Vh) * sizeof(double2);
  const char* p = reinterpret_cast<const char*>(X) + 3 * cs * grp;
  auto load_x = [&](cplx<double>* vf, cplx<double>* vb) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      vf[c] = *reinterpret_cast<const double2*>(p + c * cs + of);
      vb[c] = *reinterpret_cast<const double2*>(p + c * cs + ob);
    }
  };
  // step of the loop, this group's pair and its shift
  int j = 0, k = grp, i = G > 1 && grp >= nshift ? 0 : grp;
  const int steps = (npair + G - 1) / G;
  auto pair = [&](const cplx<double>* xf, const cplx<double>* xb, cplx<double>* nf,
                  cplx<double>* nb, double2 (&pk)[4][3][64]) {
    // direction-mu part of chi(y) = 1/2 [sf U_mu(y) X(y+mu) + sb U_mu(y-mu)^dag X(y-mu)]
    cplx<double> y1[3], y2[3];
    mat_vec<double>(Uf, xf, y1);
    adj_mat_vec<double>(Ub, xb, y2);
#pragma unroll
    for (int c = 0; c < 3; ++c) pk[mu][c][lane] = cadd<double>(y1[c], y2[c]);
    // the loads of the pair after the next, in flight over the barrier and the outer products
    if (k + 2 * G < npair) p += G * 3 * cs;
    load_x(nf, nb);
    // One barrier per step: a wave writes a buffer again two steps later, after a
    // barrier that every wave reaches only when it has read this one.
    __syncthreads();
    // chi already carries the 1/2 of D_oe; the 1/2 of dD_oe and the factor 2 of
    // the variation cancel, so M takes alpha * eta * s with no further factor:
    //   M_mu(y)   = -sf sum alpha X(y+mu) chi(y)^dag
    //   M_mu(y-mu) = -sb sum alpha chi(y) X(y-mu)^dag
    // and the sums without -sf, -sb are kept.
    if (G == 1 || k < npair) {
      cplx<double> chi[3];
#pragma unroll
      for (int c = 0; c < 3; ++c)
        chi[c] = cscale<double>(al.a[i],
                                cadd<double>(cadd<double>(pk[0][c][lane], pk[1][c][lane]),
                                             cadd<double>(pk[2][c][lane], pk[3][c][lane])));
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          cfmac<double>(Mf.e[3 * a + b], chi[b], xf[a]);
          cfmac<double>(Mb.e[3 * a + b], xb[b], chi[a]);
        }
    }
    ++j;
    k += G;
    i += G;
    if (i >= nshift) i -= nshift;
    if (G > 1 && i >= nshift) i -= nshift;
  };
  // three register sets and two LDS buffers in turn, without copies
  cplx<double> xf[3][3], xb[3][3];
  load_x(xf[0], xb[0]);
  if (k + G < npair) p += G * 3 * cs;
  load_x(xf[1], xb[1]);
  while (true) {
    pair(xf[0], xb[0], xf[2], xb[2], part[j & 1]);
    if (j == steps) break;
    pair(xf[1], xb[1], xf[0], xb[0], part[j & 1]);
    if (j == steps) break;
    pair(xf[2], xb[2], xf[1], xb[1], part[j & 1]);
    if (j == steps) break;
  }
  if constexpr (G == 2) {  // group 0 ends with the sum of the forward side, group 1 of the backward
    double2 (&x)[4][9][64] = *reinterpret_cast<double2 (*)[4][9][64]>(&parts[0][0][0][0][0]);
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      Su3<double>& M = side == 0 ? Mf : Mb;
      __syncthreads();
      if (grp != side)
#pragma unroll
        for (int e = 0; e < 9; ++e) x[mu][e][lane] = M.e[e];
      __syncthreads();
      if (grp == side)
#pragma unroll
        for (int e = 0; e < 9; ++e) M.e[e] = cadd<double>(M.e[e], x[mu][e][lane]);
    }
  }
  if (!in) return;
  // U M = (2 s U') (-s M') = -2 U' M'; for the raw M the factor is -s
#pragma unroll
  for (int e = 0; e < 9; ++e) {
    Mf.e[e] = cscale<double>(mode == 1 ? -sf : -2.0, Mf.e[e]);
    Mb.e[e] = cscale<double>(mode == 1 ? -sb : -2.0, Mb.e[e]);
  }

  // outputs: forward link at (parity 1, mu, h), backward link at (parity 0, mu, hb)
  for (int side = 0; side < 2; ++side) {
    if (G == 2 && side != grp) continue;
    const Su3<double>& M = side == 0 ? Mf : Mb;
    const Su3<double>& Ul = side == 0 ? Uf : Ub;
    double2* out = F + (side == 0 ? pstride : 0) + int64_t(mu) * 9 * g.Vh + (side == 0 ? h : hb);
    cplx<double> res[9];
    if (mode == 1) {
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) res[3 * a + b] = conj_of<double>(M.e[3 * b + a]);
    } else {
      cplx<double> W[9];
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          cplx<double> w = cmul<double>(Ul.e[3 * a], M.e[b]);
          cfma<double>(w, Ul.e[3 * a + 1], M.e[3 + b]);
          cfma<double>(w, Ul.e[3 * a + 2], M.e[6 + b]);
          W[3 * a + b] = w;
        }
      // TA(W) = (W - W^dag)/2 - Tr(W - W^dag)/6; Tr(W - W^dag) = 2 i Im Tr W
      const double im_tr = (W[0].y + W[4].y + W[8].y) / 3.0;
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          const cplx<double> w = W[3 * a + b], wt = W[3 * b + a];
          res[3 * a + b] = mk<double>(0.5 * (w.x - wt.x), 0.5 * (w.y + wt.y) - (a == b ? im_tr : 0.0));
        }
    }
#pragma unroll
    for (int e = 0; e < 9; ++e) {
      cplx<double> v = res[e];
      if (accumulate) {
        const double2 o = out[int64_t(e) * g.Vh];
        v.x += o.x;
        v.y += o.y;
      }
      out[int64_t(e) * g.Vh] = v;
    }
  }
}

// partials[blk] = sum over the block's even sites of
//   sum_j [alpha0 |phi_j|^2 + sum_i alpha_i Re <phi_j, X_ji>]
__global__ void __launch_bounds__(kActionBlock) k_action(int Vh, const double2* __restrict__ phi,
                                                         const double2* __restrict__ X, int npf,
                                                         int nshift, double alpha0,
                                                         const Alphas al,
                                                         double* __restrict__ part) {
  __shared__ double lds[kActionBlock / 64];
  const int h = blockIdx.x * blockDim.x + threadIdx.x;
  double s = 0.0;
  if (h < Vh) {
    const int64_t vs = int64_t(3) * Vh;
    for (int j = 0; j < npf; ++j) {
      double2 f[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        f[c] = phi[j * vs + int64_t(c) * Vh + h];
        s += alpha0 * (f[c].x * f[c].x + f[c].y * f[c].y);
      }
      for (int i = 0; i < nshift; ++i) {
        const double2* Xk = X + (int64_t(j) * nshift + i) * vs;
        double d = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const double2 x = Xk[int64_t(c) * Vh + h];
          d += f[c].x * x.x + f[c].y * x.y;  // Re(conj(phi) X)
        }
        s += al.a[i] * d;
      }
    }
  }
  s = block_sum(s, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

__global__ void __launch_bounds__(kActionBlock) k_sum(const double* __restrict__ part, int n,
                                                      double* __restrict__ out) {
  __shared__ double lds[kActionBlock / 64];
  double s = strided_sum(part, n);
  s = block_sum(s, lds);
  if (threadIdx.x == 0) *out = s;
}

// y_j = alpha0 b_j + sum_i alpha_i X_ji for every complex element e of the
// [3][Vh] even-site vectors (blockIdx.y = j).  The terms are added in a fixed
// order (alpha0 b first, then i = 0, 1, ...), so the result is reproducible.
// y may be b (each element is read before it is written), never X.
__global__ void __launch_bounds__(kCombineBlock) k_rational_combine(
    int64_t n, const double2* __restrict__ b, const double2* X, int nshift, double alpha0,
    Alphas al, double2* y) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const int64_t j = blockIdx.y;
  const double2 bv = b[j * n + e];
  double re = alpha0 * bv.x, im = alpha0 * bv.y;
  const double2* xj = X + j * nshift * n + e;
  constexpr int kChunk = 8;  // loads issued together before their products
  for (int i0 = 0; i0 < nshift; i0 += kChunk) {
    double2 v[kChunk];
#pragma unroll
    for (int u = 0; u < kChunk; ++u)
      if (i0 + u < nshift) v[u] = xj[int64_t(i0 + u) * n];
#pragma unroll
    for (int u = 0; u < kChunk; ++u)
      if (i0 + u < nshift) {
        re = fma(al.a[i0 + u], v[u].x, re);
        im = fma(al.a[i0 + u], v[u].y, im);
      }
  }
  y[j * n + e] = make_double2(re, im);
}

// Device address of the current device's copy of `scratch`, looked up once per
// device.  Returns NULL (error text set) if the device or the lookup fails.
double* action_scratch_ptr() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxScratchDevices) {
    set_error("no usable current HIP device (device %d) for the action scratch array", dev);
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      set_error("hipGetSymbolAddress(scratch) failed on device %d: %s", dev,
                hipGetErrorString(e));
      return nullptr;
    }
    g_scratch_dev[dev] = static_cast<double*>(p);
  }
  return g_scratch_dev[dev];
}

int check_alpha(int32_t nshift, const double* alpha) {
  if (nshift < 1 || nshift > kMaxShift) {
    set_error("nshift = %d must be in [1, %d]", nshift, kMaxShift);
    return LQCD_ERR_INVALID_ARG;
  }
  if (!alpha) {
    set_error("alpha must be a host array of nshift doubles");
    return LQCD_ERR_INVALID_ARG;
  }
  for (int i = 0; i < nshift; ++i)
    if (!std::isfinite(alpha[i])) {
      set_error("alpha[%d] is not finite", i);
      return LQCD_ERR_INVALID_ARG;
    }
  return LQCD_OK;
}

}  // namespace

}  // namespace lqcd

using namespace lqcd;

extern "C" {

int lqcd_fermion_force(const lqcd_geom* g, const void* U64, int32_t npf, int32_t nshift,
                       const double* alpha, const void* X, int32_t mode, int32_t accumulate,
                       void* F, void* stream) {
  clear_error();
  int rc;
  if ((rc = check_geom(g)) || (rc = check_ptr(U64, "U64")) || (rc = check_ptr(X, "X")) ||
      (rc = check_ptr(F, "F")) || (rc = check_alpha(nshift, alpha)))
    return rc;
  if (npf < 1 || npf > 64) {
    set_error("npf = %d must be in [1, 64]", npf);
    return LQCD_ERR_INVALID_ARG;
  }
  if (mode != 0 && mode != 1) {
    set_error("mode must be 0 (projected) or 1 (raw), got %d", mode);
    return LQCD_ERR_INVALID_ARG;
  }
  if (accumulate != 0 && accumulate != 1) {
    set_error("accumulate must be 0 or 1");
    return LQCD_ERR_INVALID_ARG;
  }
  if (F == U64 || F == X) {
    set_error("F must not alias U64 or X");
    return LQCD_ERR_INVALID_ARG;
  }
  const KGeom k = make_kgeom(g);
  Alphas al{};
  for (int i = 0; i < nshift; ++i) al.a[i] = alpha[i];
  const unsigned grid = unsigned((k.Vh + 63) / 64);
  // (y, z) tiles keep a site's +-z and +-t neighbours near in launch order: 48^4, 96
  // pairs, 12.1 ms without, 11.0 with 16 x 6 tiles (59 GB read), 10.4 with 8 x 6 (45).
  // On large lattices tiles of eight rows, where they divide Ly, ms of 16 (else the
  // next divisor) and 8:   12 pairs      48 pairs       96 pairs
  //   32^3 x 48           0.601 0.592   1.612 1.592   2.992 2.968
  //   32^3 x 64           0.866 0.841   2.169 2.164   4.028 4.001
  //   40^4                0.992 0.980   2.672 2.662   5.012 4.989
  //   48^4                2.030 2.018   5.591 5.535  11.006 10.423
  // but 36^4 0.666 with 12 and 0.692 with 6 rows, 44^4 within 1 %, 32^3 x 40 0.510
  // 0.513, and 24^4, 48 pairs, 0.367 with 12 and 0.372 with 8.
  const bool large = k.Vh >= 3 << 18 && k.Ly % 8 == 0;
  const int rows = chunk_tile(k.Ly, large ? 8 : 16), tz = chunk_tile(k.Lz, 7);
  // An odd number of rows, which Ly = 18, 22, 26, 30 have, loses 1 to 5 % against whole
  // ones: 18^4 46.0 45.0 us with 12 pairs, 117.3 115.9 with 48; 22^4 101.1 99.7, 272.2
  // 268.5; 30^4 348.8 336.1, 896.9 891.2 (even ones lose up to 4 %: 24^4 356 366).
  const int ty = rows % 2 && k.Ly <= 30 ? k.Ly : rows;
  if (k.Vh <= kForceGroupsVh && npf * nshift >= 2)
    hipLaunchKernelGGL(k_force<2>, dim3(grid), dim3(2 * kForceBlock), 0, (hipStream_t)stream, k,
                       (const double2*)U64, (const double2*)X, npf, nshift, al, mode, accumulate,
                       ty, tz, (double2*)F);
  else
    hipLaunchKernelGGL(k_force<1>, dim3(grid), dim3(kForceBlock), 0, (hipStream_t)stream, k,
                       (const double2*)U64, (const double2*)X, npf, nshift, al, mode, accumulate,
                       ty, tz, (double2*)F);
  LQCD_LAUNCH_CHECK();
  return LQCD_OK;
}

size_t lqcd_action_workspace_bytes(const lqcd_geom* g) {
  if (check_geom(g)) return 0;
  const KGeom k = make_kgeom(g);
  return (size_t((k.Vh + kActionBlock - 1) / kActionBlock) + 32) * sizeof(double);
}

}  // extern "C"

namespace lqcd {
namespace {

int check_action_args(const lqcd_geom* g, int32_t npf, int32_t nshift, double alpha0,
                      const double* alpha, const void* phi, const void* X, const double* S) {
  int rc;
  if ((rc = check_geom(g)) || (rc = check_ptr(phi, "phi")) || (rc = check_ptr(X, "X")) ||
      (rc = check_alpha(nshift, alpha)))
    return rc;
  if (!S) {
    set_error("S must be a host pointer");
    return LQCD_ERR_INVALID_ARG;
  }
  if (npf < 1 || npf > 64) {
    set_error("npf = %d must be in [1, 64]", npf);
    return LQCD_ERR_INVALID_ARG;
  }
  if (!std::isfinite(alpha0)) {
    set_error("alpha0 is not finite");
    return LQCD_ERR_INVALID_ARG;
  }
  return LQCD_OK;
}

// The two reduction launches of the action into `part` (ceil(Vh/256) + 32
// doubles of device memory), then the result to the host.
int run_action(const lqcd_geom* g, int32_t npf, int32_t nshift, double alpha0,
               const double* alpha, const void* phi, const void* X, double* S, double* part,
               hipStream_t s) {
  const KGeom k = make_kgeom(g);
  Alphas al{};
  for (int i = 0; i < nshift; ++i) al.a[i] = alpha[i];
  const int nb = (k.Vh + kActionBlock - 1) / kActionBlock;
  double* out = part + nb + 16;
  hipLaunchKernelGGL(k_action, dim3(nb), dim3(kActionBlock), 0, s, k.Vh, (const double2*)phi,
                     (const double2*)X, npf, nshift, alpha0, al, part);
  LQCD_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_sum, dim3(1), dim3(kActionBlock), 0, s, part, nb, out);
  LQCD_LAUNCH_CHECK();
  LQCD_HIP_TRY(hipMemcpyAsync(S, out, sizeof(double), hipMemcpyDeviceToHost, s));
  LQCD_HIP_TRY(hipStreamSynchronize(s));
  return LQCD_OK;
}

}  // namespace
}  // namespace lqcd

extern "C" {

int lqcd_action(const lqcd_geom* g, int32_t npf, int32_t nshift, double alpha0,
                const double* alpha, const void* phi, const void* X, double* S, void* ws,
                size_t ws_bytes, void* stream) {
  clear_error();
  int rc;
  if ((rc = check_action_args(g, npf, nshift, alpha0, alpha, phi, X, S)) ||
      (rc = check_ptr(ws, "ws")))
    return rc;
  const size_t need = lqcd_action_workspace_bytes(g);
  if (ws_bytes < need) {
    set_error("action workspace of %zu bytes is too small: %zu needed", ws_bytes, need);
    return LQCD_ERR_WORKSPACE;
  }
  return run_action(g, npf, nshift, alpha0, alpha, phi, X, S, static_cast<double*>(ws),
                    (hipStream_t)stream);
}

int lqcd_action_noalloc(const lqcd_geom* g, int32_t npf, int32_t nshift, double alpha0,
                        const double* alpha, const void* phi, const void* X, double* S,
                        void* stream) {
  clear_error();
  int rc;
  if ((rc = check_action_args(g, npf, nshift, alpha0, alpha, phi, X, S))) return rc;
  const size_t need = lqcd_action_workspace_bytes(g);
  if (need > kActionScratchDoubles * sizeof(double)) {
    set_error("lattice needs %zu bytes of action scratch, above the fixed %zu-byte array", need,
              kActionScratchDoubles * sizeof(double));
    return LQCD_ERR_WORKSPACE;
  }
  double* part = action_scratch_ptr();
  if (!part) return LQCD_ERR_HIP;
  return run_action(g, npf, nshift, alpha0, alpha, phi, X, S, part, (hipStream_t)stream);
}

int lqcd_rational_combine(const lqcd_geom* g, int32_t nrhs, int32_t nshift, double alpha0,
                          const double* alpha, const void* b, const void* X, void* y,
                          void* stream) {
  clear_error();
  int rc;
  if ((rc = check_geom(g)) || (rc = check_ptr(b, "b")) || (rc = check_ptr(X, "X")) ||
      (rc = check_ptr(y, "y")) || (rc = check_alpha(nshift, alpha)))
    return rc;
  if (nrhs < 1 || nrhs > 64) {
    set_error("nrhs = %d must be in [1, 64]", nrhs);
    return LQCD_ERR_INVALID_ARG;
  }
  if (!std::isfinite(alpha0)) {
    set_error("alpha0 is not finite");
    return LQCD_ERR_INVALID_ARG;
  }
  const KGeom k = make_kgeom(g);
  const int64_t n = int64_t(3) * k.Vh;
  const char* xb = static_cast<const char*>(X);
  const char* yb = static_cast<const char*>(y);
  const int64_t xbytes = int64_t(nrhs) * nshift * n * int64_t(sizeof(double2));
  const int64_t ybytes = int64_t(nrhs) * n * int64_t(sizeof(double2));
  if (yb < xb + xbytes && xb < yb + ybytes) {
    set_error("y must not overlap X");
    return LQCD_ERR_INVALID_ARG;
  }
  Alphas al{};
  for (int i = 0; i < nshift; ++i) al.a[i] = alpha[i];
  const dim3 grid(unsigned((n + kCombineBlock - 1) / kCombineBlock), unsigned(nrhs));
  hipLaunchKernelGGL(k_rational_combine, grid, dim3(kCombineBlock), 0, (hipStream_t)stream, n,
                     (const double2*)b, (const double2*)X, nshift, alpha0, al, (double2*)y);
  LQCD_LAUNCH_CHECK();
  return LQCD_OK;
}

}  // extern "C"
