// D_oe / D_eo with the four directions of a site on four waves (k_dslash_split),
// for lattices too small to fill the chip with one thread per site.
//
// One workgroup takes 64 output sites and up to B right-hand sides; wave mu
// loads the two links and the two neighbours of direction mu and multiplies
// them, the eight products per site meet in LDS, and the waves finish one
// (right-hand side, colour) each: the chain of memory round trips per site is
// one deep instead of four, and four times as many waves are in flight.  The
// products are added in k_dslash's order, so the result has the same bits (the
// factor +-1/2 is exact).
//
// 16^4, one right-hand side, kernel times: D_oe FP32 12-real 6.7 -> 4.9 us, FP64
// 12-real 9.8 -> 8.3 us; FP64 18-real 10.7 -> 8.9 us (41 MB past the L2s: the
// last-level cache's rate).  From 26^4 on one thread per site fills the chip.
//
// With DslashCall::sys the fused CG update also computes its step length from
// the partials of D_oe and of the direction, in every workgroup, while the
// stencil's loads are in flight: one launch less per iteration (16^4: 9.0 us and
// 6.0 us for the one-workgroup kernel -> 6.9 us in FP32).
#include <hip/hip_runtime.h>

#include "dslash.h"
#include "su3.h"
#include "sysred.h"

namespace lqcd {

namespace {

constexpr int kSplitBlock = kSmallBlock;  // 64 sites x 4 directions

// Slot of right-hand side j's residual of its iteration it.
__device__ __forceinline__ int64_t ring_slot(const DslashCall& a, int j, int it) {
  return a.r_iter ? int64_t(j) * a.r_slots + it % a.r_slots : int64_t(j);
}

// PR: right-hand sides in interleaved pairs (DslashCall::pairs; B = 2).
template <typename R, int NE, int B, int MODE, typename RO, bool PR>
__global__ void __launch_bounds__(kSplitBlock) k_dslash_split(const DslashCall a, const int xcd,
                                                              const int ngroups) {
  __shared__ cplx<R> sh[B][4][2][3][64];  // +-1/2 U v of each hop
  __shared__ double red[2 * B][kScalarThreads / 64];
  __shared__ double lds[B][4];
  const int halt = a.halt ? *a.halt : 0;
  const KGeom& g = a.g;
  const int nblk = gridDim.x / ngroups;
  const int lb0 = xcd_block(blockIdx.x, gridDim.x, xcd);
  const int lb = a.rev ? int(gridDim.x) - 1 - lb0 : lb0;
  const int blk = lb / ngroups;
  const int rhs0 = (lb % ngroups) * B;
  // every flag and scalar of the systems in one round trip
  bool lv[B];
  bool any = false;
  int it[B];
  StepState ss[B];
  double m2s[B], al[B];
#pragma unroll
  for (int b = 0; b < B; ++b) {
    const int j = rhs0 + b, jl = j < a.nrhs ? j : a.nrhs - 1;
    lv[b] = j < a.nrhs && (a.live == nullptr || a.live[j * a.live_stride] != 0);
    any |= lv[b];
    it[b] = (MODE == DM_CG || MODE == DM_RES) && a.r_iter ? a.r_iter[jl * a.r_iter_stride] : 0;
    m2s[b] = MODE != DM_PLAIN && a.m2s ? a.m2s[jl * a.m2s_stride] : a.m2s_c;
    al[b] = 0.0;
    if constexpr (MODE == DM_CG) {
      if (a.sys)
        ss[b] = step_state(a.sys[jl]);
      else
        al[b] = a.alpha[jl * a.alpha_stride];
    }
  }
  if (halt || !any) {  // uniform over the block; one round trip for all flags
    if (MODE == DM_CG && a.sys && blk == 0 && threadIdx.x < B && rhs0 + int(threadIdx.x) < a.nrhs) {
      SysState& S = a.sys[rhs0 + threadIdx.x];  // finished systems: no update follows
      S.upd_any = 0;
      S.restart = 0;
    }
    return;
  }

  const int lane = threadIdx.x & 63;
  const int mu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int idx = blk * 64 + lane;
  const bool in = idx < g.Vh;
  const int h = in ? idx : 0;  // lanes past Vh work on site 0 and store nothing
  const Site s = decode_site(g, h, a.out_par);
  constexpr uint32_t cb = sizeof(cplx<R>);
  const uint32_t csoff = uint32_t(g.Vh) * cb;

  int fwd, bwd;
  if (mu == 0) {
    const int xp = s.x + 1 == g.Lx ? 0 : s.x + 1, xm = s.x == 0 ? g.Lx - 1 : s.x - 1;
    fwd = h - (s.x >> 1) + (xp >> 1);
    bwd = h - (s.x >> 1) + (xm >> 1);
  } else {
    const int L = mu == 1 ? g.Ly : (mu == 2 ? g.Lz : g.Lt);
    const int st = mu == 1 ? g.sy : (mu == 2 ? g.sz : g.st);
    const int c = mu == 1 ? s.y : (mu == 2 ? s.z : s.t);
    fwd = h + (c + 1 == L ? -(L - 1) * st : st);
    bwd = h + (c == 0 ? (L - 1) * st : -st);
  }
  const int ep = ((mu >= 1 ? s.x : 0) + (mu >= 2 ? s.y : 0) + (mu >= 3 ? s.z : 0)) & 1;
  R cf = ep ? R(-0.5) : R(0.5), cw = cf;
  if (mu == 3 && g.anti) {
    if (s.t == g.Lt - 1) cf = -cf;
    if (s.t == 0) cw = -cw;
  }
  const int64_t lb_ = link_block<NE>(g.Vh);
  const uint32_t link_bytes = uint32_t(lb_) * cb;
  const cplx<R>* U = static_cast<const cplx<R>*>(a.U);
  const auto rf = make_res(U + (int64_t(a.out_par) * 4 + mu) * lb_, link_bytes);
  const auto rb = make_res(U + (int64_t(1 - a.out_par) * 4 + mu) * lb_, link_bytes);
  Su3<R> uf, ub;
  cplx<R> vf[B][3], vb[B][3];
  R thf = R(0), thb = R(0);
#pragma unroll
  for (int e = 0; e < stored_planes<NE>(); ++e) {
    uf.e[e] = ld_buf<R>(rf, uint32_t(h) * cb, uint32_t(e) * csoff);
    ub.e[e] = ld_buf<R>(rb, uint32_t(bwd) * cb, uint32_t(e) * csoff);
  }
  if constexpr (NE == 8) {
    thf = ld_buf_real<R>(rf, uint32_t(h) * uint32_t(sizeof(R)), 6u * csoff);
    thb = ld_buf_real<R>(rb, uint32_t(bwd) * uint32_t(sizeof(R)), 6u * csoff);
  }
  if constexpr (PR) {
    const int jr = rhs0 < a.nrhs ? rhs0 : a.nrhs - 2;
    const auto rin = make_res(static_cast<const cplx<R>*>(a.in) + int64_t(jr) * a.in_stride,
                              6u * csoff);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      ld_buf_pair(rin, 2u * uint32_t(fwd) * cb, uint32_t(c) * 2u * csoff, vf[0][c], vf[1][c]);
      ld_buf_pair(rin, 2u * uint32_t(bwd) * cb, uint32_t(c) * 2u * csoff, vb[0][c], vb[1][c]);
    }
  } else {
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int jr = rhs0 + b < a.nrhs ? rhs0 + b : a.nrhs - 1;
      const auto rin = make_res(static_cast<const cplx<R>*>(a.in) + int64_t(jr) * a.in_stride,
                                3u * csoff);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        vf[b][c] = ld_buf<R>(rin, uint32_t(fwd) * cb, uint32_t(c) * csoff);
        vb[b][c] = ld_buf<R>(rin, uint32_t(bwd) * cb, uint32_t(c) * csoff);
      }
    }
  }

  // The wave's share of the epilogue: colours of one right-hand side (or of the
  // pair); own-site operands are loaded before the workgroup meets.
  constexpr int Q = PR ? 2 : 1;             // right-hand sides per item
  constexpr int NI = (B / Q) * 3;           // items of the workgroup
  constexpr int NW = (NI + 3) / 4;          // items of a wave
  cplx<R> dv[NW][Q], rv[NW][Q];
  double2 bv[NW];
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const int k = mu + 4 * i, q = k / 3, c = k - 3 * q;
    if (k >= NI) continue;
    if constexpr (MODE != DM_PLAIN) {
      if constexpr (PR) {
        const int jp = rhs0 < a.nrhs ? rhs0 : a.nrhs - 2;
        ld_once_pair<false>(static_cast<const cplx<R>*>(a.diag) + int64_t(jp) * a.diag_stride +
                                2 * (int64_t(c) * g.Vh + h),
                            dv[i][0], dv[i][1]);
      } else {
        const int jl = rhs0 + q < a.nrhs ? rhs0 + q : a.nrhs - 1;
        dv[i][0] = (static_cast<const cplx<R>*>(a.diag) + int64_t(jl) * a.diag_stride +
                    int64_t(c) * g.Vh)[h];
        if constexpr (MODE == DM_RES)
          bv[i] = (static_cast<const double2*>(a.b) + int64_t(jl) * a.b_stride +
                   int64_t(c) * g.Vh)[h];
      }
      if constexpr (MODE == DM_CG) {
#pragma unroll
        for (int e = 0; e < Q; ++e) {
          const int j = rhs0 + q * Q + e, jl = j < a.nrhs ? j : a.nrhs - 1;
          int itn = 0;
#pragma unroll
          for (int bb = 0; bb < B; ++bb)
            if (bb == q * Q + e) itn = it[bb];
          rv[i][e] = (static_cast<const cplx<R>*>(a.r) + ring_slot(a, jl, itn) * a.r_stride +
                      int64_t(c) * g.Vh)[h];
        }
      }
    }
  }
  SmallSums<2 * B> parts;
  if constexpr (MODE == DM_CG) {
    if (a.sys) {
      const double* p[2 * B];
      int n[2 * B];
#pragma unroll
      for (int b = 0; b < B; ++b) {
        const int j = rhs0 + b < a.nrhs ? rhs0 + b : a.nrhs - 1;
        p[2 * b] = a.step_t + int64_t(j) * a.step_nt;
        n[2 * b] = a.step_nt;
        p[2 * b + 1] = a.step_p + int64_t(j) * a.step_np;
        n[2 * b + 1] = a.step_np;
      }
      parts.load(p, n);
    }
  }

  complete_link<R, NE>(uf);
  complete_link<R, NE>(ub);
  if constexpr (NE == 8) {
    apply_u1<R>(uf, thf);
    apply_u1<R>(ub, thb);
  }
#pragma unroll
  for (int b = 0; b < B; ++b) {
    cplx<R> y[3];
    mat_vec<R>(uf, vf[b], y);
#pragma unroll
    for (int c = 0; c < 3; ++c) sh[b][mu][0][c][lane] = cscale<R>(cf, y[c]);
    adj_mat_vec<R>(ub, vb[b], y);
#pragma unroll
    for (int c = 0; c < 3; ++c) sh[b][mu][1][c][lane] = cscale<R>(-cw, y[c]);
  }
  if constexpr (MODE == DM_CG) {
    if (a.sys) parts.reduce(red);
  }
  __syncthreads();
  if constexpr (MODE == DM_CG) {
    if (a.sys) {
#pragma unroll
      for (int b = 0; b < B; ++b) {
        if (rhs0 + b >= a.nrhs) continue;
        const double tt = parts.sum(red[2 * b]), pp = parts.sum(red[2 * b + 1]);
        bool err;
        lv[b] = cg_step(ss[b], tt, pp, &al[b], &err);
        // (the last wave has the least of the epilogue)
        if (blk == 0)
          store_step(a.sys[rhs0 + b], a.flags, a.nshift, lv[b], err, al[b], pp,
                     int(threadIdx.x) - (kSplitBlock - 64));
      }
    }
  }

  double nrm[B];
#pragma unroll
  for (int b = 0; b < B; ++b) nrm[b] = 0.0;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const int k = mu + 4 * i, q = k / 3, c = k - 3 * q;
    if (k >= NI || !in) continue;
    cplx<R> acc[Q];
#pragma unroll
    for (int e = 0; e < Q; ++e) {
      cplx<R> z = mk<R>(0, 0);
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int d = 0; d < 2; ++d) z = cadd<R>(z, sh[q * Q + e][m][d][c][lane]);
      acc[e] = z;
    }
    if constexpr (PR && MODE == DM_PLAIN) {
      if (lv[0] || lv[1])
        st_once_pair<false>(static_cast<cplx<R>*>(a.out) + int64_t(rhs0) * a.out_stride +
                                2 * (int64_t(c) * g.Vh + h),
                            acc[0], acc[1]);
    }
#pragma unroll
    for (int e = 0; e < Q; ++e) {
      const int b = q * Q + e, j = rhs0 + b;
      double v = 0.0;
      bool live = false;
      double alpha = 0.0, md = 0.0;
      int itn = 0;
#pragma unroll
      for (int bb = 0; bb < B; ++bb)
        if (bb == b) {
          live = lv[bb];
          alpha = al[bb];
          md = m2s[bb];
          itn = it[bb];
        }
      if (!live) continue;
      if constexpr (MODE == DM_PLAIN) {
        if constexpr (!PR)
          (static_cast<cplx<R>*>(a.out) + int64_t(j) * a.out_stride + int64_t(c) * g.Vh)[h] = acc[e];
        v = cnorm2<R>(acc[e]);
      } else if constexpr (MODE == DM_AXPY) {
        (static_cast<cplx<R>*>(a.out) + int64_t(j) * a.out_stride + int64_t(c) * g.Vh)[h] =
            mk<R>(fma(R(md), dv[i][e].x, -acc[e].x), fma(R(md), dv[i][e].y, -acc[e].y));
      } else if constexpr (MODE == DM_CG) {
        const R av = R(alpha);
        const R wx = fma(R(md), dv[i][e].x, -acc[e].x);
        const R wy = fma(R(md), dv[i][e].y, -acc[e].y);
        cplx<R> rn = rv[i][e];
        rn.x = fma(-av, wx, rn.x);
        rn.y = fma(-av, wy, rn.y);
        (static_cast<cplx<R>*>(a.r) + ring_slot(a, j, itn + 1) * a.r_stride + int64_t(c) * g.Vh)[h] = rn;
        v = cnorm2<R>(rn);
      } else {  // DM_RES, R = double
        const double rx = bv[i].x - fma(md, (double)dv[i][e].x, -(double)acc[e].x);
        const double ry = bv[i].y - fma(md, (double)dv[i][e].y, -(double)acc[e].y);
        if (a.r)
          (static_cast<cplx<RO>*>(a.r) + ring_slot(a, j, itn) * a.r_stride + int64_t(c) * g.Vh)[h] =
              mk<RO>(RO(rx), RO(ry));
        v = fma(rx, rx, ry * ry);
      }
#pragma unroll
      for (int bb = 0; bb < B; ++bb)
        if (bb == b) nrm[bb] += v;
    }
  }
  if (a.partials) {
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const double sum = block_sum(nrm[b], lds[b]);
      if (threadIdx.x == 0 && lv[b]) a.partials[int64_t(rhs0 + b) * nblk + blk] = sum;
    }
  }
}

template <typename R, int NE, int B, int MODE, typename RO, bool PR>
int launch_split(const DslashCall& c, const DslashCfg& cfg, hipStream_t st) {
  const int ngroups = (c.nrhs + B - 1) / B;
  hipLaunchKernelGGL((k_dslash_split<R, NE, B, MODE, RO, PR>),
                     dim3(dslash_nblocks(c.g, cfg) * ngroups), dim3(kSplitBlock), 0, st, c,
                     cfg.xcd, ngroups);
  LQCD_LAUNCH_CHECK();
  return LQCD_OK;
}

template <typename R, int NE, int MODE, typename RO>
int split_b(const DslashCall& c, const DslashCfg& cfg, hipStream_t st) {
  if constexpr (sizeof(R) == 4 && (NE == 6 || NE == 9) && (MODE == DM_PLAIN || MODE == DM_CG)) {
    if (c.pairs) return launch_split<R, NE, 2, MODE, RO, true>(c, cfg, st);
  }
  return cfg.rhs_block == 2 ? launch_split<R, NE, 2, MODE, RO, false>(c, cfg, st)
                            : launch_split<R, NE, 1, MODE, RO, false>(c, cfg, st);
}

template <typename R, int NE>
int split_mode(const DslashCall& c, const DslashCfg& cfg, hipStream_t st) {
  switch (c.mode) {
    case DM_PLAIN: return split_b<R, NE, DM_PLAIN, R>(c, cfg, st);
    case DM_AXPY: return split_b<R, NE, DM_AXPY, R>(c, cfg, st);
    default: return split_b<R, NE, DM_CG, R>(c, cfg, st);
  }
}

template <typename R>
int split_fmt(const DslashCall& c, const DslashCfg& cfg, hipStream_t st) {
  switch (c.fmt) {
    case LQCD_LINKS12: return split_mode<R, 6>(c, cfg, st);
    case LQCD_LINKS12D: return split_mode<R, 7>(c, cfg, st);
    case LQCD_LINKS12T: return split_mode<R, 8>(c, cfg, st);
    default: return split_mode<R, 9>(c, cfg, st);
  }
}

}  // namespace

bool dslash_split_supported(const DslashCall& c, const DslashCfg& f) {
  return f.sp == 1 && f.block == kSplitBlock && (f.rhs_block == 1 || f.rhs_block == 2) &&
         (!c.pairs || f.rhs_block == 2) && f.tz == 0 && f.ty == 0 && f.tm == 0 && f.mf == 0;
}

int dslash_split_launch(const DslashCall& c, const DslashCfg& cfg, hipStream_t st) {
  if (!dslash_split_supported(c, cfg)) {
    set_error("the direction-split stencil needs 256 threads, an RHS block of 1 or 2 (2 for "
              "right-hand-side pairs) and no tiles");
    return LQCD_ERR_UNSUPPORTED;
  }
  if (c.mode == DM_RES) {
    if (c.prec != LQCD_F64 || c.fmt != LQCD_LINKS18) {
      set_error("residual mode needs FP64 18-real links");
      return LQCD_ERR_UNSUPPORTED;
    }
    return c.r_prec == LQCD_F32 ? split_b<double, 9, DM_RES, float>(c, cfg, st)
                                : split_b<double, 9, DM_RES, double>(c, cfg, st);
  }
  return c.prec == LQCD_F64 ? split_fmt<double>(c, cfg, st) : split_fmt<float>(c, cfg, st);
}

}  // namespace lqcd
