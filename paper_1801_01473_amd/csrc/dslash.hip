// The hopping term D_oe / D_eo (Sec. 2): launch dispatch over precision and
// link format, the launch-configuration tuner and the C ABI entry points.  The
// kernels are in dslash_kernel.h (k_dslash) and dslash_tm.hip (t-march); each
// (precision, format) instantiation compiles in its own dslash_inst_*.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <tuple>
#include <vector>

#include "dslash.h"
#include "sysred.h"

namespace lqcd {

int dslash_launch(const DslashCall& c, const DslashCfg& cfg, hipStream_t st) {
  if (cfg.block != 64 && cfg.block != 128 && cfg.block != 256) {
    set_error("unsupported dslash block size %d", cfg.block);
    return LQCD_ERR_UNSUPPORTED;
  }
  if (c.pairs) {
    const int64_t vs = int64_t(3) * c.g.Vh;
    if (c.prec != LQCD_F32 || (c.fmt != LQCD_LINKS12 && c.fmt != LQCD_LINKS18) ||
        (c.mode != DM_PLAIN && c.mode != DM_CG) || c.nrhs % 2 != 0 || cfg.rhs_block % 2 != 0 ||
        cfg.tm > 0 || cfg.mf == 1 || c.in_stride < vs ||
        (c.mode == DM_PLAIN && c.out_stride < vs) || (c.mode == DM_CG && c.diag_stride < vs)) {
      set_error("right-hand-side pairs need FP32 12- or 18-real links, the plain or fused CG "
                "mode, an even number of right-hand sides and RHS block, k_dslash, and rows "
                "of at least 3 Vh values");
      return LQCD_ERR_UNSUPPORTED;
    }
  }
  if (c.sys && (cfg.sp != 1 || c.mode != DM_CG)) {
    set_error("the step length inside the stencil needs the direction-split CG update");
    return LQCD_ERR_UNSUPPORTED;
  }
  if (cfg.tm > 0) return dslash_tm_launch(c, cfg, st);
  if (cfg.sp == 1) return dslash_split_launch(c, cfg, st);
  if (cfg.mf == 1) return dslash_mfma_launch(c, cfg, st);
  if (cfg.tz < 0 || (cfg.tz > 0 && c.g.Lz % cfg.tz != 0) || cfg.ty < 0 ||
      (cfg.ty > 0 && c.g.Ly % cfg.ty != 0)) {
    set_error("tile %d x %d (y, z) must divide Ly = %d, Lz = %d", cfg.ty, cfg.tz, c.g.Ly, c.g.Lz);
    return LQCD_ERR_UNSUPPORTED;
  }
  if (c.mode == DM_RES) {
    if (c.prec != LQCD_F64 || c.fmt != LQCD_LINKS18) {
      set_error("residual mode needs FP64 18-real links");
      return LQCD_ERR_UNSUPPORTED;
    }
    return dslash_launch_res(c, cfg, st);
  }
  if (c.prec == LQCD_F64)
    return c.fmt == LQCD_LINKS12    ? dslash_launch_fmt<double, 6>(c, cfg, st)
           : c.fmt == LQCD_LINKS12D ? dslash_launch_fmt<double, 7>(c, cfg, st)
           : c.fmt == LQCD_LINKS12T ? dslash_launch_fmt<double, 8>(c, cfg, st)
                                    : dslash_launch_fmt<double, 9>(c, cfg, st);
  return c.fmt == LQCD_LINKS12    ? dslash_launch_fmt<float, 6>(c, cfg, st)
         : c.fmt == LQCD_LINKS12D ? dslash_launch_fmt<float, 7>(c, cfg, st)
         : c.fmt == LQCD_LINKS12T ? dslash_launch_fmt<float, 8>(c, cfg, st)
                                  : dslash_launch_fmt<float, 9>(c, cfg, st);
}

// ----------------------------------------------------------------- tuner

namespace {

using TuneKey = std::tuple<int, int, int, int, int, int, int, int, int, int, std::string>;
std::mutex g_tune_mu;
std::map<TuneKey, DslashCfg> g_tune;

DslashCfg default_cfg(int nrhs, int forced, int prec, int pairs) {
  DslashCfg c;
  c.block = 256;
  c.xcd = 1;
  c.lf = prec == LQCD_F32 ? 1 : 0;
  int b = 1;
  while (b * 2 <= std::min(nrhs, 8)) b *= 2;
  c.rhs_block = forced > 0 ? forced : b;
  if (pairs && c.rhs_block < 2) c.rhs_block = 2;
  return c;
}

bool tuning_enabled() {
  const char* e = std::getenv("LQCD_TUNE");
  return !(e && e[0] == '0');
}

bool tuning_verbose() {
  const char* e = std::getenv("LQCD_TUNE_VERBOSE");
  return e && e[0] == '1';
}

// ---- optional on-disk tuning cache (LQCD_TUNE_CACHE=file) ----------------
// One line per tuned shape:
// "<key>;<block>,<B>,<xcd>,<tz>,<nt>,<occ>,<ilv>,<lf>,<hh>,<ty>[,<ns>[,<tm>,<tp>[,<sp>]]]"
// where the key names the cache format, the GPU architecture and CU count,
// the geometry, precision, link format, RHS count, forced RHS block, mode,
// pairs and, where it matters, the kind of caller (caller_kind).  Lines that do not parse, or whose configuration is not valid for
// the shape, are ignored (that shape is tuned again).
constexpr int kTuneCacheFormat = 1;

// Half volumes up to which the direction-split stencil is a candidate.
constexpr int kSplitMaxVh = 1 << 18;

// Half volumes up to which the plain modes also try it with one right-hand side a
// pass over the links when there are several: more workgroups, an eighth off a
// launch on the smallest lattices (8^4, 2 systems 7.2 and 8.2 us), but the links are
// read again for each.  On one link field that pays further up (FP64 D_oe, 16^4, 2
// systems 12.4 13.5 us, 16^3 x 32 18.4 19.8, 18^4, 3 systems 19.0 20.9), and solves,
// which run on one, try it everywhere (DslashCall::solve).  A program with fields past
// the last-level cache in turn loses by it from there on, which the timings below on
// one field would not tell: A x, FP64, 12^4, 3 systems 12.7 14.2 us; 16^4, 2 systems
// 21.7 20.3, 4 systems 30.7 26.1; 20^4, 3 systems 55.7 51.7; FP32 16^4, 4 systems
// 19.0 16.2.
constexpr int kSplitOncePerRhsVh = 1 << 14;

// What the split kernel saves elsewhere when the solve takes its scalars into the
// CG kernels (DslashCall::fusable, fused_partials_pay): their one-workgroup kernels,
// 5 and 4 us a launch at 16^4, against about 1 us more in the CG kernels each.  Its
// times in CG mode are ranked with this credit; the solves that use it gain 4 to 8 us
// an iteration from 4^4 to 22^3 x 24 (the table at fused_partials_pay).
constexpr float kFusedCreditMs = 0.006f;

bool credit_applies(const DslashCall& c) {
  return c.mode == DM_CG && fused_partials_pay((c.g.Vh + 63) / 64, c.nrhs, c.pairs != 0);
}

constexpr char kSeparate[] = "/sep", kSolve[] = "/solve";

// Callers that get a choice of their own, tuned and kept apart: CG updates that the
// credit would apply to but whose solve cannot use it, and D_oe of a solve where a
// plain call does not try all that it does.
std::string caller_kind(const DslashCall& c, int forced) {
  if (credit_applies(c) && !c.fusable) return kSeparate;
  if (c.solve && c.mode == DM_PLAIN && c.nrhs > 1 && !c.pairs && !forced &&
      c.g.Vh > kSplitOncePerRhsVh && c.g.Vh <= kSplitMaxVh)
    return kSolve;
  return "";
}

const char* tune_cache_path() {
  const char* e = std::getenv("LQCD_TUNE_CACHE");
  return (e && e[0]) ? e : nullptr;
}

std::string tune_cache_key(const DslashCall& c, int forced) {
  int dev = 0;
  hipDeviceProp_t prop;
  std::string arch = "unknown";
  int cus = 0;
  if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess) {
    arch = prop.gcnArchName;
    cus = prop.multiProcessorCount;
  }
  for (char& ch : arch)
    if (ch == ';' || ch == ' ') ch = '_';
  char buf[256];
  std::snprintf(buf, sizeof(buf), "v%d/%s/%dcu/%dx%dx%dx%d/p%d/f%d/n%d/b%d/m%d%s%s",
                kTuneCacheFormat, arch.c_str(), cus, c.g.Lx, c.g.Ly, c.g.Lz, c.g.Lt, c.prec, c.fmt,
                c.nrhs, forced, c.mode, c.pairs ? "/pairs" : "",
                caller_kind(c, forced).c_str());
  return buf;
}

bool cfg_valid(const DslashCall& c, const DslashCfg& f, int forced) {
  const bool b_ok = f.rhs_block == 1 || f.rhs_block == 2 || f.rhs_block == 4 || f.rhs_block == 8;
  return (f.block == 64 || f.block == 128 || f.block == 256) && b_ok &&
         (!forced || f.rhs_block == forced) && (f.xcd == 0 || f.xcd == 1) && f.tz >= 0 &&
         (f.tz == 0 || c.g.Lz % f.tz == 0) && f.ty >= 0 && (f.ty == 0 || c.g.Ly % f.ty == 0) &&
         (f.nt == 0 || f.nt == 1) && (f.lf == 0 || f.lf == 1) && (f.hh == 0 || f.hh == 1) &&
         (f.ns == 0 || (f.ns == 1 && f.nt == 1)) &&
         (f.ilv == 0 || f.ilv == 1) && f.occ >= 0 && dslash_lds_bytes(f) >= 0 &&
         dslash_lds_bytes(f) <= 64 * 1024 && f.tm >= 0 &&
         (f.tm == 0 || dslash_tm_supported(c, f)) &&
         (f.sp == 0 || (f.sp == 1 && dslash_split_supported(c, f))) &&
         (!c.pairs || (f.rhs_block % 2 == 0 && f.tm == 0 && f.mf == 0));
}

// The last valid entry for the key, if any.  A line of the solves with the credit in
// which another kernel won all the same holds for those without it.
bool tune_cache_lookup(const char* path, const std::string& key, const DslashCall& c, int forced,
                       DslashCfg* out) {
  FILE* f = std::fopen(path, "r");
  if (!f) return false;
  const std::string with_credit = caller_kind(c, forced) == kSeparate
                                      ? key.substr(0, key.size() - std::strlen(kSeparate))
                                      : key;
  char line[512];
  bool found = false;
  while (std::fgets(line, sizeof(line), f)) {
    char* semi = std::strchr(line, ';');
    if (!semi) continue;
    *semi = '\0';
    if (key != line && with_credit != line) continue;
    DslashCfg v;
    const int n = std::sscanf(semi + 1, "%d,%d,%d,%d,%d,%d,%d,%d,%d,%d,%d,%d,%d,%d", &v.block,
                              &v.rhs_block, &v.xcd, &v.tz, &v.nt, &v.occ, &v.ilv, &v.lf, &v.hh,
                              &v.ty, &v.ns, &v.tm, &v.tp, &v.sp);
    if (n != 10 && n != 11 && n != 13 && n != 14) continue;
    if (!cfg_valid(c, v, forced) || (key != line && v.sp == 1)) continue;
    *out = v;
    found = true;
  }
  std::fclose(f);
  return found;
}

void tune_cache_store(const char* path, const std::string& key, const DslashCfg& v) {
  FILE* f = std::fopen(path, "a");
  if (!f) return;  // the cache is an optimisation; an unwritable file only costs tuning
  std::fprintf(f, "%s;%d,%d,%d,%d,%d,%d,%d,%d,%d,%d,%d,%d,%d,%d\n", key.c_str(), v.block,
               v.rhs_block, v.xcd, v.tz, v.nt, v.occ, v.ilv, v.lf, v.hh, v.ty, v.ns, v.tm, v.tp,
               v.sp);
  std::fclose(f);
}

}  // namespace

void dslash_clear_tuning() {
  std::lock_guard<std::mutex> lk(g_tune_mu);
  g_tune.clear();
}

int dslash_tuned(const DslashCall& c, int forced, hipStream_t st, DslashCfg* out) {
  if (forced != 0 && forced != 1 && forced != 2 && forced != 4 && forced != 8) {
    set_error("rhs_block must be 0 (tuned), 1, 2, 4 or 8, got %d", forced);
    return LQCD_ERR_INVALID_ARG;
  }
  if (c.pairs && forced == 1) {
    set_error("right-hand-side pairs need an RHS block of 2, 4 or 8");
    return LQCD_ERR_INVALID_ARG;
  }
  // LQCD_DSLASH_CFG="block,rhs_block,xcd,tz[,nt,occ,ilv,lf,hh,ty,ns,tm,tp,mf,sp]" pins the
  // configuration (testing, profiling).  A t-march or matrix-core configuration
  // applies only where that kernel exists (t-march: 8 right-hand sides or more,
  // 12-real links, the plain and fused modes; matrix cores: FP32, 12-real, plain
  // mode without norms); other calls fall back to its k_dslash settings.
  if (const char* e = std::getenv("LQCD_DSLASH_CFG")) {
    DslashCfg f;
    if (std::sscanf(e, "%d,%d,%d,%d,%d,%d,%d,%d,%d,%d,%d,%d,%d,%d,%d", &f.block, &f.rhs_block,
                    &f.xcd, &f.tz, &f.nt, &f.occ, &f.ilv, &f.lf, &f.hh, &f.ty, &f.ns, &f.tm,
                    &f.tp, &f.mf, &f.sp) >= 4) {
      if (forced) f.rhs_block = forced;
      if (c.pairs && f.rhs_block == 1) f.rhs_block = 2;  // pairs load two rows at once
      if (f.tm > 0 && (c.nrhs < 8 || !dslash_tm_supported(c, f))) {
        f.tm = 0;
        if (f.rhs_block > c.nrhs) f.rhs_block = 1;
      }
      if (f.mf == 1 && !dslash_mfma_supported(c, f)) f.mf = 0;
      if (f.sp == 1 && !dslash_split_supported(c, f)) f.sp = 0;
      *out = f;
      return LQCD_OK;
    }
  }
  const TuneKey key{c.g.Lx, c.g.Ly, c.g.Lz,  c.g.Lt, c.prec, c.fmt,
                    c.nrhs, forced, c.mode, c.pairs, caller_kind(c, forced)};
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    auto it = g_tune.find(key);
    if (it != g_tune.end()) {
      *out = it->second;
      return LQCD_OK;
    }
  }
  DslashCfg best = default_cfg(c.nrhs, forced, c.mode == DM_RES ? LQCD_F64 : c.prec, c.pairs);
  if (!tuning_enabled()) {
    *out = best;
    return LQCD_OK;
  }
  const char* cache_path = tune_cache_path();
  const std::string cache_key = cache_path ? tune_cache_key(c, forced) : std::string();
  if (cache_path && tune_cache_lookup(cache_path, cache_key, c, forced, &best)) {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tune[key] = best;
    *out = best;
    return LQCD_OK;
  }

  // Candidates are timed in the caller's mode (the fused CG update with its
  // own-site loads, or plain) with FP64 norm partials, on private scratch
  // fields and the caller's links, so no caller data is touched.
  // Stage 1: workgroup size, RHS block, XCD remap, z-slab traversal, RHS
  // interleave.  Stage 2: (y, z) tiles for the three fastest, each with and
  // without one hop per iteration, non-temporal link loads and own-site
  // streams.  Stage 3: the three fastest so far with the other schedules
  // (loads first, one hop per iteration, non-temporal links and streams) and
  // occupancy caps.  Stage 4: the five fastest re-timed, best median.
  std::vector<DslashCfg> cand;
  for (int blk : {64, 128, 256})
    for (int b : {1, 2, 4, 8}) {
      if (forced ? b != forced : b > c.nrhs) continue;
      if (c.pairs && b == 1) continue;  // pairs load two rows at once
      for (int x : {0, 1})
        for (int tz : {0, 2, 4, 8}) {
          if (tz && (c.g.Lz % tz || tz >= c.g.Lz)) continue;
          for (int ilv : {0, 1}) {
            if (ilv && b >= c.nrhs) continue;  // a single RHS group has nothing to interleave
            DslashCfg v = best;
            v.block = blk;
            v.rhs_block = b;
            v.xcd = x;
            v.tz = tz;
            v.ty = 0;
            v.ilv = ilv;
            cand.push_back(v);
          }
        }
    }

  // the direction-split kernel, where one thread per site leaves the chip idle
  if (c.g.Vh <= kSplitMaxVh)
    for (int b : {1, 2}) {
      if (forced ? b != forced : b > c.nrhs) continue;
      if (c.pairs && b == 1) continue;
      if (b == 1 && c.nrhs > 1 && !forced && c.mode != DM_CG && !c.solve &&
          c.g.Vh > kSplitOncePerRhsVh)
        continue;
      for (int x : {0, 1}) {
        DslashCfg v;
        v.block = 256;
        v.rhs_block = b;
        v.xcd = x;
        v.sp = 1;
        cand.push_back(v);
      }
    }

  const size_t vec = size_t(3) * c.g.Vh * 2 * (c.prec == LQCD_F32 ? 4 : 8);
  const bool cg = c.mode == DM_CG;
  // [in][out or r][diag][partials][alpha]
  const size_t fields = (cg ? 3 : 2) * vec * c.nrhs;
  const size_t npart = dslash_partials_max(c.g, c.nrhs);
  const size_t sbytes = fields + npart * 8 + size_t(c.nrhs) * 8;
  void* scratch = nullptr;
  LQCD_HIP_TRY(hipStreamSynchronize(st));
  LQCD_HIP_TRY(hipMalloc(&scratch, sbytes));
  // non-zero data (0x3f bytes: ~0.75 in FP32, ~3e-4 in FP64, also the CG step
  // length) so timings match real fields and the CG update stays finite
  LQCD_HIP_TRY(hipMemsetAsync(scratch, 0x3f, sbytes, st));
  constexpr int kMaxReps = 8;
  hipEvent_t ev[2 * kMaxReps];
  for (auto& e : ev) LQCD_HIP_TRY(hipEventCreate(&e));

  // Built from scratch: only the shape, parity, precision and links are the
  // caller's; every field pointer (residual ring, right-hand side, flags) is
  // either a scratch field below or left null.
  DslashCall t;
  t.g = c.g;
  t.out_par = c.out_par;
  t.nrhs = c.nrhs;
  t.U = c.U;
  t.mode = cg ? DM_CG : DM_PLAIN;
  t.in = scratch;
  t.in_stride = int64_t(3) * c.g.Vh;
  t.out = static_cast<char*>(scratch) + vec * c.nrhs;
  t.out_stride = int64_t(3) * c.g.Vh;
  if (cg) {
    t.r = t.out;
    t.r_stride = t.out_stride;
    t.diag = static_cast<char*>(scratch) + 2 * vec * c.nrhs;
    t.diag_stride = int64_t(3) * c.g.Vh;
    t.m2s = nullptr;
    t.m2s_c = 0.01;
    t.alpha = reinterpret_cast<const double*>(static_cast<char*>(scratch) + fields + npart * 8);
    t.alpha_stride = 1;
  }
  t.partials = reinterpret_cast<double*>(static_cast<char*>(scratch) + fields);
  t.prec = c.prec;
  t.fmt = c.fmt;
  t.pairs = c.pairs;  // same bytes per field, read and written as pairs
  if (c.mode == DM_RES) {  // the residual kernels run on FP64 18-real links
    t.prec = LQCD_F64;
    t.fmt = LQCD_LINKS18;
  }

  // Median time of one launch.  As in the solver, the input field has just
  // been written when the stencil runs (part of it is still cached), so it is
  // rewritten before each timed launch.
  auto time_cfg = [&](const DslashCfg& cfg, int reps, float* med) -> int {
    for (int i = 0; i < reps; ++i) {
      if (hipMemsetAsync(scratch, 0x3f, vec * c.nrhs, st) != hipSuccess) return LQCD_ERR_HIP;
      (void)hipEventRecord(ev[2 * i], st);
      dslash_launch(t, cfg, st);
      (void)hipEventRecord(ev[2 * i + 1], st);
    }
    if (hipEventSynchronize(ev[2 * reps - 1]) != hipSuccess) return LQCD_ERR_HIP;
    float ts[kMaxReps];
    for (int i = 0; i < reps; ++i) (void)hipEventElapsedTime(&ts[i], ev[2 * i], ev[2 * i + 1]);
    std::sort(ts, ts + reps);
    *med = ts[reps / 2];
    return LQCD_OK;
  };

  const float credit = credit_applies(c) && c.fusable ? kFusedCreditMs : 0.f;
  auto ranked = [&](float ms, const DslashCfg& cfg) { return cfg.sp == 1 ? ms - credit : ms; };
  float best_ms = 1e30f;
  int rc = LQCD_OK;
  std::vector<std::pair<float, DslashCfg>> timed;
  const size_t stage1 = cand.size();
  size_t stage2 = size_t(-1);
  auto top3 = [&]() {
    std::vector<std::pair<float, DslashCfg>> s1;
    for (const auto& tk : timed)
      if (tk.second.sp == 0) s1.push_back(tk);  // the split kernel has no schedules
    std::sort(s1.begin(), s1.end(),
              [](const std::pair<float, DslashCfg>& a, const std::pair<float, DslashCfg>& b) {
                return a.first < b.first;
              });
    if (s1.size() > 3) s1.resize(3);
    return s1;
  };
  for (size_t ci = 0; ci < cand.size() && rc == LQCD_OK; ++ci) {
    const DslashCfg cfg = cand[ci];
    float ms = 0;
    const bool runs = dslash_launch(t, cfg, st) == LQCD_OK;  // warm-up
    if (!runs) clear_error();  // skip what cannot launch
    if (runs && time_cfg(cfg, 3, &ms) != LQCD_OK) {
      set_error("dslash tuning run failed");
      rc = LQCD_ERR_HIP;
      break;
    }
    if (runs && tuning_verbose())
      fprintf(stderr,
              "[lqcd tune] L=%dx%dx%dx%d prec=%d fmt=%d nrhs=%d mode=%d block=%d B=%d xcd=%d "
              "ty=%d tz=%d nt=%d occ=%d ilv=%d lf=%d hh=%d ns=%d tm=%d tp=%d sp=%d: %.2f us\n",
              c.g.Lx, c.g.Ly, c.g.Lz, c.g.Lt, t.prec, t.fmt, c.nrhs, t.mode, cfg.block,
              cfg.rhs_block, cfg.xcd, cfg.ty, cfg.tz, cfg.nt, cfg.occ, cfg.ilv, cfg.lf, cfg.hh,
              cfg.ns, cfg.tm, cfg.tp, cfg.sp, 1000.0 * ms);
    ms = ranked(ms, cfg);
    if (runs) timed.push_back({ms, cfg});
    if (runs && ms < best_ms) {
      best_ms = ms;
      best = cfg;
    }
    if (ci + 1 == stage1) {  // stage 2: (y, z) tiles of the best three
      // The tile and the one-hop schedule interact (a tile pays off most with
      // one hop per iteration), so both are crossed here.  The seeds cover
      // both block-to-XCD maps: the remap that wins untiled can lose tiled.
      auto seeds = top3();
      if (seeds.size() == 3 && seeds[0].second.xcd == seeds[1].second.xcd &&
          seeds[1].second.xcd == seeds[2].second.xcd) {
        const std::pair<float, DslashCfg>* other = nullptr;
        for (const auto& tk : timed)
          if (tk.second.sp == 0 && tk.second.xcd != seeds[0].second.xcd &&
              (!other || tk.first < other->first))
            other = &tk;
        if (other) seeds[2] = *other;
      }
      for (const auto& tk : seeds)
        for (int ty : {0, 4, 8, 12, 16, 24})
          for (int tz : {2, 4, 6, 8, 12})
            for (int hh : {0, 1}) {
              if ((ty && (c.g.Ly % ty || ty >= c.g.Ly)) || c.g.Lz % tz || tz >= c.g.Lz) continue;
              DslashCfg v = tk.second;
              v.ty = ty;
              v.tz = tz;
              v.nt = 1;
              v.ns = 1;
              v.hh = hh;
              cand.push_back(v);
            }
      stage2 = cand.size();
    } else if (ci + 1 == stage2) {  // stage 3: schedules and occupancy caps
      for (const auto& tk : top3())
        for (int ntns : {0, 1, 3})  // bit 0: non-temporal links, bit 1: own-site streams too
          for (int lf : {0, 1})
            for (int hh : {0, 1})
              for (int occ : {0, 2, 3, 4}) {
                DslashCfg v = tk.second;
                const int nt = ntns & 1, ns = ntns >> 1;
                if (nt == v.nt && ns == v.ns && lf == v.lf && hh == v.hh && occ == v.occ)
                  continue;
                v.nt = nt;
                v.ns = ns;
                v.lf = lf;
                v.hh = hh;
                v.occ = occ;
                const int lds = dslash_lds_bytes(v);
                if (lds < 0 || lds > 64 * 1024) continue;
                cand.push_back(v);
              }
      // the t-march kernel, where it exists: eight right-hand sides per
      // column, a few chunk lengths along t, lanes per column, XCD maps
      if (c.nrhs >= 8 && (!forced || forced == 8))
        for (int blk : {64, 128, 256})
          for (int tp : {2, 4})
            for (int tm : {4, 6, 8, 12, 16, 24})
              for (int x : {0, 1})
                for (int occ : {0, 2}) {
                  DslashCfg v;
                  v.block = blk;
                  v.rhs_block = 8;
                  v.xcd = x;
                  v.nt = 1;
                  v.ns = 1;
                  v.tm = tm;
                  v.tp = tp;
                  v.occ = occ;
                  const int lds = dslash_lds_bytes(v);
                  if (lds < 0 || lds > 64 * 1024 || !dslash_tm_supported(t, v)) continue;
                  cand.push_back(v);
                }
    }
  }
  // Stage 4: single short timings are noisy and the minimum over ~200 of them
  // favours lucky ones; re-time the five fastest in interleaved rounds and
  // keep the best median.
  if (rc == LQCD_OK && timed.size() > 1) {
    std::sort(timed.begin(), timed.end(),
              [](const std::pair<float, DslashCfg>& a, const std::pair<float, DslashCfg>& b) {
                return a.first < b.first;
              });
    const size_t nf = std::min<size_t>(5, timed.size());
    constexpr int kRounds = 3;
    std::vector<std::vector<float>> rt(nf);
    for (int round = 0; round < kRounds && rc == LQCD_OK; ++round)
      for (size_t k = 0; k < nf; ++k) {
        float ms = 0;
        if (time_cfg(timed[k].second, 5, &ms) != LQCD_OK) {
          set_error("dslash tuning run failed");
          rc = LQCD_ERR_HIP;
          break;
        }
        rt[k].push_back(ranked(ms, timed[k].second));
      }
    if (rc == LQCD_OK) {
      float best_med = 1e30f;
      for (size_t k = 0; k < nf; ++k) {
        std::sort(rt[k].begin(), rt[k].end());
        const float med = rt[k][rt[k].size() / 2];
        if (med < best_med) {
          best_med = med;
          best = timed[k].second;
        }
      }
      best_ms = best_med;
    }
  }
  for (auto& e : ev) (void)hipEventDestroy(e);
  (void)hipFree(scratch);
  if (rc != LQCD_OK) return rc;
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tune[key] = best;
  }
  if (cache_path) tune_cache_store(cache_path, cache_key, best);
  if (tuning_verbose())
    fprintf(stderr,
            "[lqcd tune] chosen L=%dx%dx%dx%d prec=%d fmt=%d nrhs=%d mode=%d: block=%d B=%d "
            "xcd=%d ty=%d tz=%d nt=%d occ=%d ilv=%d lf=%d hh=%d ns=%d tm=%d tp=%d sp=%d (%.2f us)\n",
            c.g.Lx, c.g.Ly, c.g.Lz, c.g.Lt, t.prec, t.fmt, c.nrhs, t.mode, best.block,
            best.rhs_block, best.xcd, best.ty, best.tz, best.nt, best.occ, best.ilv, best.lf,
            best.hh, best.ns, best.tm, best.tp, best.sp,
            1000.0 * (best_ms + (best.sp == 1 ? credit : 0.f)));
  *out = best;
  return LQCD_OK;
}

}  // namespace lqcd

// ----------------------------------------------------------------- C ABI

using namespace lqcd;

namespace {

int hop_entry(const lqcd_geom* g, int prec, int fmt, const void* U, const void* in, void* out,
              int32_t nrhs, void* stream, int out_par, const char* name) {
  clear_error();
  int st;
  if ((st = check_geom(g)) || (st = check_prec_fmt(prec, fmt)) || (st = check_ptr(U, "U")) ||
      (st = check_ptr(in, "in")) || (st = check_ptr(out, "out")) || (st = check_nrhs(nrhs)))
    return st;
  if (in == out) {
    set_error("%s: in and out must not alias", name);
    return LQCD_ERR_INVALID_ARG;
  }
  DslashCall c;
  c.g = make_kgeom(g);
  c.out_par = out_par;
  c.prec = prec;
  c.fmt = fmt;
  c.nrhs = nrhs;
  c.mode = DM_PLAIN;
  c.U = U;
  c.in = in;
  c.in_stride = int64_t(3) * c.g.Vh;
  c.out = out;
  c.out_stride = c.in_stride;
  hipStream_t s = (hipStream_t)stream;
  DslashCfg cfg;
  if ((st = dslash_tuned(c, 0, s, &cfg))) return st;
  return dslash_launch(c, cfg, s);
}

}  // namespace

extern "C" {

int lqcd_doe(const lqcd_geom* g, int prec, int fmt, const void* U, const void* in_even,
             void* out_odd, int32_t nrhs, void* stream) {
  return hop_entry(g, prec, fmt, U, in_even, out_odd, nrhs, stream, 1, "lqcd_doe");
}

int lqcd_deo(const lqcd_geom* g, int prec, int fmt, const void* U, const void* in_odd,
             void* out_even, int32_t nrhs, void* stream) {
  return hop_entry(g, prec, fmt, U, in_odd, out_even, nrhs, stream, 0, "lqcd_deo");
}

int lqcd_apply_A(const lqcd_geom* g, int prec, int fmt, const void* U, double mass, double sigma,
                 const void* in_even, void* out_even, void* tmp_odd, int32_t nrhs,
                 void* stream) {
  clear_error();
  int st;
  if ((st = check_ptr(tmp_odd, "tmp_odd")) || (st = check_ptr(out_even, "out_even"))) return st;
  if (tmp_odd == in_even || tmp_odd == out_even || in_even == out_even) {
    set_error("lqcd_apply_A: in, out and tmp must be distinct buffers");
    return LQCD_ERR_INVALID_ARG;
  }
  if (!(mass == mass) || !(sigma == sigma)) {
    set_error("lqcd_apply_A: mass and sigma must be finite");
    return LQCD_ERR_INVALID_ARG;
  }
  if ((st = hop_entry(g, prec, fmt, U, in_even, tmp_odd, nrhs, stream, 1, "lqcd_apply_A")))
    return st;
  DslashCall c;
  c.g = make_kgeom(g);
  c.out_par = 0;
  c.prec = prec;
  c.fmt = fmt;
  c.nrhs = nrhs;
  c.mode = DM_AXPY;
  c.U = U;
  c.in = tmp_odd;
  c.in_stride = int64_t(3) * c.g.Vh;
  c.out = out_even;
  c.out_stride = c.in_stride;
  c.diag = in_even;
  c.diag_stride = c.in_stride;
  c.m2s_c = mass * mass + sigma;
  hipStream_t s = (hipStream_t)stream;
  DslashCfg cfg;
  if ((st = dslash_tuned(c, 0, s, &cfg))) return st;
  return dslash_launch(c, cfg, s);
}

}  // extern "C"
