// Reductions of block partials inside kernels of any workgroup size, and the
// step length of CG computed from them.
#pragma once

#include "common.h"
#include "solver.h"

namespace lqcd {

// Partial counts up to this can go through the reduction below in every
// workgroup of a kernel, instead of a kernel of one workgroup.
constexpr int kFusedPartials = 2 * kScalarThreads;

// Whether that pays: nb workgroups a right-hand side then read nb partials each
// from L2, nb^2 nrhs doubles in all and twice that for the step length.  A whole
// iteration with the scalars inside and in kernels of their own, us, 8 shifts:
//   FP64, 1 system   8^4 18.0 22.8   16^4 29.3 37.2   22^3 x 24 (nb 1997) 69.7 76.5
//   FP64, 2          16^4 36.1 41.8  20^4 (1250) 63.0 65.5; 22^3 x 24 loses
//   FP64, 4          16^4 (512) 50.6 56.9; with 8: 12^3 x 24 (324) 58.0 60.8
//   FP32, 1          16^4 22.7 27.7  22^3 x 24 42.8 46.2;   3: 16^4 36.2 38.8
// In pairs a workgroup sums two systems' partials, four arrays, and the stencil
// they hide behind is the shortest:
//   2 systems  8^3 x 16 (64) 27.0 28.9  12^3 x 16 (216) 28.6 31.1  12^3 x 24 33.2 32.9
//   4          8^4 (32) 28.5 29.8       12^2 x 8 x 16 (144) 33.4 33.1  16^4 47.0 43.0
//   8          8^3 x 16 31.6 32.7       144 39.4 37.6  12^3 x 24 53.2 45.1
inline bool fused_partials_pay(int64_t nb, int nrhs, bool pairs) {
  const int64_t most = int64_t(1) << (pairs ? 17 : nrhs <= 2 ? 22 : 20);
  return nb <= kFusedPartials && nb * nb * nrhs <= most;
}

// The sums of K arrays of n[k] <= kFusedPartials doubles by a workgroup of 256
// threads, in the order in which a workgroup of kScalarThreads threads (wg_sum)
// adds them -- 16 groups of 64, a butterfly in each, the groups in order -- so
// with the same bits.  All loads are issued before the first butterfly.  Every
// thread gets the results.
constexpr int kSmallBlock = 256;

template <int K>
struct SmallSums {
  static constexpr int W = kScalarThreads / 64, NW = kSmallBlock / 64, M = W / NW;
  double v[K][M];
  // issues the loads
  __device__ __forceinline__ void load(const double* const (&p)[K], const int (&n)[K]) {
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const int i = (int(threadIdx.x >> 6) + NW * m) * 64 + int(threadIdx.x & 63);
        v[k][m] = i < n[k] ? p[k][i] : 0.0;
      }
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (n[k] > kScalarThreads)
#pragma unroll
        for (int m = 0; m < M; ++m) {
          const int i = kScalarThreads + (int(threadIdx.x >> 6) + NW * m) * 64 +
                        int(threadIdx.x & 63);
          v[k][m] += i < n[k] ? p[k][i] : 0.0;
        }
  }
  // sums groups of 64 into LDS; a barrier goes between this and sum()
  __device__ __forceinline__ void reduce(double (&lds)[K][W]) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int m = 0; m < M; ++m) v[k][m] += __shfl_xor(v[k][m], off, 64);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int m = 0; m < M; ++m) lds[k][(threadIdx.x >> 6) + NW * m] = v[k][m];
  }
  __device__ __forceinline__ static double sum(const double (&lds)[W]) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) s += lds[w];
    return s;
  }
};

// What the step length depends on; read with the other flags of a kernel.
struct StepState {
  double rho, m2s;
  int done;
};

__device__ __forceinline__ StepState step_state(const SysState& S) {
  return StepState{S.rho, S.m2s, S.done};
}

// Step length of the base system from |p|^2 and |D_oe p|^2; false: the system
// is finished, or the curvature <p, A p> is not a positive number (err).
__device__ __forceinline__ bool cg_step(const StepState& S, double tt, double pp, double* a,
                                        bool* err) {
  *err = false;
  *a = 0.0;
  if (S.done) return false;
  const double pAp = S.m2s * pp + tt;
  if (!(pAp > 0.0) || !(pAp == pAp && fabs(pAp) <= 1.7e308)) {
    *err = true;
    return false;
  }
  *a = S.rho / pAp;
  return true;
}

// The state after the step length is known, by kMaxShift threads of one
// wavefront: s in [0, kMaxShift) is the thread's number (others do nothing) and
// the shift it advances.  Other workgroups of the launch may read rho, m2s, done
// and live: none is stored here, an error ends the system in store_beta.
__device__ __forceinline__ void store_step(SysState& S, GlobalFlags* gf, int nshift, bool ok,
                                           bool err, double a, double pp, int s) {
  if (s < 0 || s >= kMaxShift) return;
  // values another thread stores below are read before (one wavefront)
  const double rho = S.rho, a_old = S.a_old, b_old = S.b_old;
  const int iters = S.iters;
  if (s < nshift) {
    const bool up = ok && S.active[s];
    S.upd[s] = up ? 1 : 0;
    if (up) {
      const double z = S.zeta[s], zo = S.zeta_old[s];
      const double zn =
          z * zo * a_old / (a * b_old * (zo - z) + zo * a_old * (1.0 + S.delta[s] * a));
      S.zeta_new[s] = zn;
      S.a_s[s] = a * zn / z;
    }
  }
  if (s != 0) return;
  S.restart = 0;
  S.upd_any = ok ? 1 : 0;
  S.rho_k = rho;
  S.iter_k = iters;
  if (ok || err) S.pp = pp;
  if (ok) S.a = a;
  if (err) {
    S.err = 1;
    gf->error = 1;
  }
}

// What an update of the base direction takes from the state.  Fused: what the
// step length left there; a system that was finished before its first iteration
// (a zero right-hand side beside others) never had one, and the loads from the
// residual ring are issued before `go` is looked at, so its slot is 0.
struct BaseStep {
  bool go;
  double zs, bs;  // p = zs r + bs p  (fused: bs = |r|^2 / bs, once |r|^2 is known)
  int slot;       // ring slot of the new residual (before % R), never negative
};

__host__ __device__ __forceinline__ BaseStep base_step(const SysState& S, int base, bool fused) {
  const bool go = S.upd_any != 0;
  if (fused) return BaseStep{go, S.zeta_new[base], S.rho_k, go ? S.iter_k + 1 : 0};
  return BaseStep{go, S.zeta[base], S.b_s[base], S.iters};
}

__device__ __forceinline__ void finish_step(BaseStep& u, double rr) {
  u.go = u.go && rr == rr && fabs(rr) <= 1.7e308;
  u.bs = rr / u.bs;
}

// The state after the residual norm rr is known, by a whole workgroup: thread s
// advances shift s, then every thread its share of the window coefficients
// (wc, deferred shift updates):
//   x_s += a_s p_s   ->  cx_s += a_s cp_s
//   p_s  = zeta_s r + b_s p_s  ->  cp_s = b_s cp_s, cp_s[n+1] = zeta_s
// where index n+1 is the residual after this iteration (ring slot n).  S.rho_k,
// S.iter_k, S.zeta_new and (fused) S.upd_any stay as the step length left them, so
// other workgroups of the same launch may read those.
struct BetaArgs {
  int max_iter = 0;
  double rel_delta2 = 0.0;  // reliable-update trigger
  double sw2 = 0.0;         // FP64 -> FP32 switch level
  int fp64 = 0;             // arithmetic of this phase
  int fused = 0;            // the launch's other workgroups update the base direction
  WinCoef* wc = nullptr;    // window coefficients of every system, or none
  int win = 1;
};

struct BetaShared {
  double a[kMaxShift], b[kMaxShift], z[kMaxShift];
  int u[kMaxShift];
  int n;
};

__device__ __forceinline__ void store_beta(SysState& S, GlobalFlags* gf, int nshift, double rr,
                                           const BetaArgs& ba, WinCoef* wc, BetaShared& sh) {
  const int s = threadIdx.x;
  if (s < 64) {  // one wavefront: its reads of the state come before its stores
    bool go = S.upd_any != 0;
    const int wpos = S.wpos, err = S.err;
    const bool bad = go && (!(rr == rr && fabs(rr) <= 1.7e308) || (wc && wpos >= ba.win));
    if (bad) go = false;
    const double rho = S.rho_k, a_step = S.a;
    const double beta = go ? rr / rho : 0.0;
    bool up = false;
    if (go && s < nshift) {
      up = S.upd[s] != 0;
      sh.u[s] = up ? 1 : 0;
      if (up) {
        const double zn = S.zeta_new[s], z = S.zeta[s];
        const double ratio = zn / z;
        const double bs = beta * ratio * ratio;
        S.b_s[s] = bs;
        S.zeta_old[s] = z;
        S.zeta[s] = zn;
        S.dirty[s] = 1;
        if (wc) S.wdirty[s] = 1;
        sh.a[s] = S.a_s[s];
        sh.b[s] = bs;
        sh.z[s] = zn;
        if (zn * zn * rr <= S.target2) S.active[s] = 0;
      }
    }
    const int nupd = __popcll(__ballot(up));
    if (s == 0) {
      sh.n = -1;
      if (bad) {
        S.err = 1;
        if (!ba.fused) S.upd_any = 0;
        gf->error = 1;
      }
      if (bad || err) {  // found here or by the step length
        S.done = 1;
        S.live = 0;
      }
      if (go) {
        S.a_old = a_step;
        S.b_old = beta;
        S.rho = rr;
        S.iters += 1;
        if (ba.fp64) {
          S.iters64 += 1;
          S.upd64 += nupd;
        } else {
          S.upd32 += nupd;
        }
        if (rr < ba.rel_delta2 * S.r2ref) gf->rel_req = 1;
        if (rr <= ba.sw2 * S.bnorm2) S.lowres = 1;
        if (rr <= S.target2 || S.iters >= ba.max_iter) {
          S.done = 1;
          S.live = 0;
          S.conv = rr <= S.target2 ? 1 : 0;
        }
        if (wc) {
          sh.n = wpos;
          S.wpos = wpos + 1;
        }
      }
    }
  }
  __syncthreads();
  const int n = sh.n;
  if (n < 0) return;
  for (int i = threadIdx.x; i < nshift * kWinRow; i += blockDim.x) {
    const int k = i / kWinRow, q = i % kWinRow;
    if (!sh.u[k]) continue;
    if (q <= n) {
      const double cp = wc->cp[k][q];
      wc->cx[k][q] = fma(sh.a[k], cp, wc->cx[k][q]);
      wc->cp[k][q] = sh.b[k] * cp;
    } else if (q == n + 1) {
      wc->cp[k][q] = sh.z[k];
    }
  }
}

}  // namespace lqcd
