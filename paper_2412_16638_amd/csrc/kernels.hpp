// kernels.hpp -- the gfx950 kernels of one time step.
//
// Per implicit stage i (sigma = tau a_ii), following the paper's split of explicit FP64
// work and implicit low-precision (LP) solves (Section "Implementation of the
// Mixed-precision Runge--Kutta methods"):
//   k_stage_rhs  (FP64)  rhs = u + tau sum_{j<i}(a^h_ij k_j + a^eps_ij k^eps_j); y = rhs
//   k_residual   (FP64)  k = K y (+ g) ; res = rhs - y + sigma k ; ||res||, ||rhs|| ; outer decision
//   k_cg_begin / k_gm_begin   res -> LP, scaled to unit RMS (FP16 range; Section "Method
//                        stability in the context of mixed precision" on rescaling)
//   k_cg_dir, k_cg_upd   fused preconditioned CG iteration (heat, SPD)
//   k_gm_matvec, k_gm_orth   one right-preconditioned GMRES Arnoldi step (the block-Jacobi
//                        apply of the next direction is fused into k_gm_orth / k_gm_begin)
//   k_promote / k_gm_finish   y += scale * delta (LP -> FP64)
//   ... k_residual again; the stage ends when ||res|| <= outer_tol ||rhs||.
//   k_keps       (FP64)  k^eps_i = (y - rhs) / sigma (only for tableaus with eps off-diagonals)
// and per step k_combine (FP64) u += tau sum_i b_i k_i.
// All kernels of a solve read the device control record first and return at once when the
// phase they belong to has finished, so the host may enqueue ahead of the convergence test.
#pragma once

#include "device.hpp"
#include "zmarch.hpp"

namespace mprk {

// Basis vectors handled per chunk in the GMRES kernels (their loads are issued back to back):
// 64 bytes per lane per chunk.
template <typename S, int VEC>
__host__ __device__ constexpr int basis_chunk() {
  return 64 / (int)(sizeof(S) * VEC) < 1 ? 1 : 64 / (int)(sizeof(S) * VEC) > 8 ? 8 : 64 / (int)(sizeof(S) * VEC);
}

// Whether a kernel loads this lane's block-Jacobi rows up front, together with its other
// independent loads (when they fit in 128 bytes per lane), or after its vector work.
template <typename S, int VEC, int BS>
__host__ __device__ constexpr bool bj_early() {
  return BS > 0 && sizeof(S) * VEC * BS <= 128;
}

struct CombArgs {
  const double* v[2 * MAXS];
  double c[2 * MAXS];
  int nv;
  const double* pv;  // k_stage_rhs: start value y = rhs + pc pv (+ pc2 pv2) when set
  double pc;
  const double* pv2;
  double pc2;
  unsigned long long* empty;  // slots of the one-launch stage that follows, emptied here
  int nempty;
  long long* rec;  // that stage's record, cleared here: a halted stage leaves it so
};

// ------------------------------------------------------------------------------------------
// FP64 explicit parts
// ------------------------------------------------------------------------------------------

// rhs = u + sum_j c_j v_j ; y = rhs, or rhs + pc pv with a start value pv.  reset: RESET_STAGE
// clears the stage record, RESET_STEP also the step's gating flags, RESET_CALL the strict halt of
// an earlier call.  A halted call, and one with a one-launch stage that timed out, opens every later
// stage finished, so its solve kernels return at once.
template <int VEC, int FL>
__global__ __launch_bounds__(TPB) void k_stage_rhs(Launch ln, const double* __restrict__ u,
                                                   CombArgs a, double* __restrict__ rhs,
                                                   double* __restrict__ y, Ctl* ctl, int reset) {
  count_work(ctl, KC_STAGE_RHS);
  if (a.empty && blockIdx.x == 0)
    for (int i = threadIdx.x; i < a.nempty; i += TPB) a.empty[i] = GRP_EMPTY;
  if (a.rec && blockIdx.x == 0 && threadIdx.x < 8) a.rec[threadIdx.x] = 0;
  if (reset && blockIdx.x == 0 && threadIdx.x == 0) {
    if (reset & RESET_CALL) ctl->halt = 0;
    ctl->outer_done = ctl->halt | ctl->bar.error;
    ctl->inner_done = 0;
    ctl->passes = 0;
    ctl->iters = 0;
    ctl->total_iters = 0;
    ctl->nonfinite = 0;
    ctl->converged = 0;
    ctl->J = 0;
    ctl->outer_rel = 0.0;
    ctl->res_norm = 0.0;
    ctl->rhs_norm = 0.0;
    if (reset & RESET_STEP) {
      ctl->step_nonfinite = 0;
      ctl->step_held = ctl->halt;
    }
  }
  const int L = xcd_block(ln.G);
  for (int it = 0; it < ln.nit; ++it) {
    const int g = (L * ln.nit + it) * TPB + threadIdx.x;
    if (g >= ln.ng) break;
    const int e = g * VEC;
    double acc[VEC];
    loadg<double, double, VEC, FL>(u, e, ln.n, acc);
    for (int j = 0; j < a.nv; ++j) {
      double t[VEC];
      loadg<double, double, VEC, FL>(a.v[j], e, ln.n, t);
      const double c = a.c[j];
#pragma unroll
      for (int v = 0; v < VEC; ++v) acc[v] += c * t[v];
    }
    storeg<double, double, VEC, FL>(rhs, e, ln.n, acc);
    if (a.pv) {
      double t[VEC];
      loadg<double, double, VEC, FL>(a.pv, e, ln.n, t);
#pragma unroll
      for (int v = 0; v < VEC; ++v) acc[v] += a.pc * t[v];
      if (a.pv2) {
        loadg<double, double, VEC, FL>(a.pv2, e, ln.n, t);
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] += a.pc2 * t[v];
      }
    }
    storeg<double, double, VEC, FL>(y, e, ln.n, acc);
  }
}

// CSR row products of one wavefront's 64 consecutive rows gw .. gw + 63 (rows from ng on are
// empty): lane l returns sum_k val[k] x[col[k]] over row gw + l, x given by functor F.  The rows'
// entries [rowptr[gw], rowptr[gw + 64]) are one contiguous run: consecutive lanes read
// consecutive entries (coalesced column and value loads, CSR_U of them in flight per lane), each
// product goes to the wave's own LDS slice and each lane then adds its row's products in entry
// order.  Only the wave takes part (no workgroup barrier).  Runs longer than 64 CSR_U entries
// (rows averaging more than CSR_U entries) are summed row by row instead.  Every lane of the
// wave calls it with the same gw.
constexpr int CSR_U = 8;

// orders the wave's LDS writes before its lanes read each other's values
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// first row of the calling lane's wavefront among the workgroup's rows g0 .. g0 + TPB - 1
__device__ __forceinline__ int wave_row0(int g0) {
  return g0 + 64 * __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

template <typename C, typename SV, typename F>
__device__ __forceinline__ C csr_wave_row(const Csr& m, const SV* __restrict__ val, int gw, int ng,
                                          const F& f) {
  __shared__ C prod[TPB / 64][CSR_U * 64];
  const int lane = threadIdx.x & 63;
  C* buf = prod[threadIdx.x >> 6];
  const int g = gw + lane;
  const int b0 = m.rowptr[gw], b1 = m.rowptr[min(gw + 64, ng)];
  const int rb = g < ng ? m.rowptr[g] : 0;
  const int re = g < ng ? m.rowptr[g + 1] : 0;
  C acc = C(0);
  if (b1 - b0 > CSR_U * 64) {  // uniform over the wave
    for (int k = rb; k < re; ++k) acc += (C)val[k] * f.one(m.col[k]);
    return acc;
  }
  if (b1 == b0) return acc;  // every row of the wave is empty
  // entry loads are unconditional (indices clamped into the run) so that all of them are in
  // flight together; the products of clamped slots land past the run's end in the slice
  int cl[CSR_U];
  SV vl[CSR_U];
  C xv[CSR_U];
#pragma unroll
  for (int u = 0; u < CSR_U; ++u) {
    const int k = min(b0 + u * 64 + lane, b1 - 1);
    cl[u] = m.col[k];
    vl[u] = val[k];
  }
#pragma unroll
  for (int u = 0; u < CSR_U; ++u) xv[u] = f.one(cl[u]);
#pragma unroll
  for (int u = 0; u < CSR_U; ++u) buf[u * 64 + lane] = (C)vl[u] * xv[u];
  wave_sync();
  // the row's products are read CSR_U at a time (clamped reads, added in entry order)
  for (int k0 = rb; k0 < re; k0 += CSR_U) {
    C pv[CSR_U];
#pragma unroll
    for (int u = 0; u < CSR_U; ++u) pv[u] = buf[min(k0 + u, b1 - 1) - b0];
#pragma unroll
    for (int u = 0; u < CSR_U; ++u)
      if (k0 + u < re) acc += pv[u];
  }
  wave_sync();  // the next call writes the slice again
  return acc;
}

// FMT 0: matrix-free stencil (VEC values per thread); FMT 1: CSR (one row per group, VEC = 1)
// with the row product csum from csr_wave_row.
template <int VEC, int FMT, int FL, typename P = NoPre>
__device__ __forceinline__ void k64_group(const Geo& geo, const Coef<double>& K,
                                          const double* __restrict__ y, int g, double csum,
                                          double (&yc)[VEC], double (&ky)[VEC], const P& pre = P()) {
  if constexpr (FMT == 0) {
    In1<double, double, VEC> f{y};
    stencil_group<double, VEC, FL>(geo, K, g * VEC, f, yc, ky, pre);
  } else {
    static_assert(VEC == 1, "CSR kernels use one row per group");
    pre();
    yc[0] = y[g];
    ky[0] = csum;
  }
}

// The stage's outer decision from the residual kernel's totals (||res||^2, ||rhs||^2,
// non-finite count): norms, the unit-RMS scale of the next LP right-hand side, convergence,
// pass limit or the one-solve mode's single pass, the strict halt.  One thread.
__device__ __forceinline__ void residual_decision(const double* tot, const SolveCfg& cfg, Ctl* ctl) {
  const double rn = sqrt(tot[0]), bn = sqrt(tot[1]);
  const double rel = bn > 0.0 ? rn / bn : rn;
  ctl->res_norm = rn;
  ctl->rhs_norm = bn;
  ctl->outer_rel = rel;
  int done = 0;
  if (tot[2] != 0.0 || !__builtin_isfinite(rn) || !__builtin_isfinite(bn)) {
    ctl->nonfinite = 1;
    ctl->step_nonfinite = 1;
    done = 1;
  } else {
    ctl->converged = rel <= cfg.outer_tol;
    if (cfg.paper_mode) {
      // one LP solve and no residual test: the stage counts as converged when that solve
      // stopped on its own tolerance (not on its iteration cap or a breakdown)
      done = ctl->passes >= 1;
      ctl->converged = done && ctl->inner_conv;
    } else {
      done = ctl->converged || ctl->passes >= cfg.max_passes || rn == 0.0;
    }
    if (done && !ctl->converged) {
      ctl->missed += 1;
      if (cfg.strict) {
        ctl->step_held = 1;
        ctl->halt = 1;
      }
    }
  }
  ctl->scale = rn > 0.0 ? rn / cfg.sqrtN : 1.0;
  ctl->outer_done = done;
}

// FP64 explicit evaluation and stage residual: k = K y ; res = rhs - y + sigma k ; ||res||^2,
// ||rhs||^2, non-finite count.
// The last block decides whether the stage is finished (outer residual loop).
template <int VEC, int FMT, int FL>
__global__ __launch_bounds__(TPB) void k_residual(Launch ln, Geo geo, Coef<double> K, Csr csr,
                                                  const double* __restrict__ kval,
                                                  const double* __restrict__ y,
                                                  const double* __restrict__ rhs,
                                                  double* __restrict__ kout,
                                                  double* __restrict__ res, FTerms fx,
                                                  SolveCfg cfg, Ctl* ctl, Red red) {
  if (ctl->outer_done) return;
  count_work(ctl, KC_RESIDUAL);
  const double* __restrict__ force = fx.g;
  const int L = xcd_block(ln.G);
  double acc[3] = {0.0, 0.0, 0.0};
  for (int it = 0; it < ln.nit; ++it) {
    const int g0 = (L * ln.nit + it) * TPB;
    const int g = g0 + threadIdx.x;
    const int gw = FMT == 1 ? wave_row0(g0) : g;  // CSR: the wave leaves together
    if (gw >= ln.ng) break;
    // for CSR, rhs and the forcing are loaded ahead of the staged row products (rows past the
    // end load row ng - 1 unused)
    const int e = FMT == 1 ? min(g, ln.ng - 1) : g * VEC;
    double yc[VEC], ky[VEC], b[VEC], rr[VEC], fv[VEC];
    loadg<double, double, VEC, FL>(rhs, e, ln.n, b);
    if (force) loadg<double, double, VEC, FL>(force, e, ln.n, fv);
    double csum = 0.0;
    if constexpr (FMT == 1) {
      csum = csr_wave_row<double, double>(csr, kval, gw, ln.ng, In1<double, double, 1>{y});
      if (g >= ln.ng) break;
    }
    // the stencil's seven loads are kept in flight together (an empty loader selects the
    // scheduling barrier; moving rhs into the group measured slower)
    k64_group<VEC, FMT, FL>(geo, K, y, g, csum, yc, ky, [] {});
    if (force) {  // constant forcing: f(y) = K y + g, so the stage solves y - sigma f(y) = rhs
#pragma unroll
      for (int v = 0; v < VEC; ++v) ky[v] += fv[v];
    }
    if (fx.react) {  // reaction: f(y) = K y + g + R(y); the outer loop is then a simplified Newton
#pragma unroll
      for (int v = 0; v < VEC; ++v) ky[v] += fx.R(yc[v]);
    }
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      rr[v] = b[v] - yc[v] + cfg.sigma * ky[v];
      acc[0] += rr[v] * rr[v];
      acc[1] += b[v] * b[v];
      acc[2] += (__builtin_isfinite(rr[v]) && __builtin_isfinite(ky[v])) ? 0.0 : 1.0;
    }
    storeg<double, double, VEC, FL>(kout, e, ln.n, ky);
    storeg<double, double, VEC, FL>(res, e, ln.n, rr);
  }
  __shared__ double tot[3];
  if (!reduce_to_last<3>(acc, 3, red, L, ln.G, tot)) return;
  if (threadIdx.x == 0) residual_decision(tot, cfg, ctl);
}

// Per-group work of the z-marching residual: rhs (and the forcing) of the next plane loaded
// ahead; res = rhs - y + sigma (K y + g), the k and res stores and the norm partials.
template <int VEC>
struct ResidualBody {
  const double* __restrict__ rhs;
  const double* __restrict__ force;
  FTerms fx;
  double* __restrict__ kout;
  double* __restrict__ res;
  double sigma;
  double bn[VEC], bc[VEC], fn[VEC], fc[VEC];
  double acc[3];
  __device__ __forceinline__ void pre(int e) {
    loadv<double, double, VEC>(rhs + e, bn);
    if (force) loadv<double, double, VEC>(force + e, fn);
  }
  __device__ __forceinline__ void next() {
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      bc[v] = bn[v];
      fc[v] = fn[v];
    }
  }
  __device__ __forceinline__ void fin(int e, const double (&yc)[VEC], const double (&kin)[VEC]) {
    double ky[VEC], rr[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      ky[v] = force ? kin[v] + fc[v] : kin[v];
      if (fx.react) ky[v] += fx.R(yc[v]);
      rr[v] = bc[v] - yc[v] + sigma * ky[v];
      acc[0] += rr[v] * rr[v];
      acc[1] += bc[v] * bc[v];
      acc[2] += (__builtin_isfinite(rr[v]) && __builtin_isfinite(ky[v])) ? 0.0 : 1.0;
    }
    storev<double, double, VEC>(kout + e, ky);
    storev<double, double, VEC>(res + e, rr);
  }
};

// k_residual with z-marching tiles (stencil format; same arithmetic per value).
template <int VEC>
__global__ __launch_bounds__(TPB) void k_residual_zm(ZLaunch zl, Geo geo, Coef<double> K,
                                                     const double* __restrict__ y,
                                                     const double* __restrict__ rhs,
                                                     double* __restrict__ kout,
                                                     double* __restrict__ res, FTerms fx,
                                                     SolveCfg cfg, Ctl* ctl, Red red) {
  if (ctl->outer_done) return;
  count_work(ctl, KC_RESIDUAL);
  extern __shared__ double zm_lds[];
  const int L = xcd_block(zl.G);
  ResidualBody<VEC> body{rhs, fx.g, fx, kout, res, cfg.sigma, {}, {}, {}, {}, {0.0, 0.0, 0.0}};
  auto src = [&](int e, double (&o)[VEC], bool) { loadv<double, double, VEC>(y + e, o); };
  zmarch<double, VEC>(geo, K, zl, L, src, body, zm_lds);
  __shared__ double tot[3];
  if (!reduce_to_last<3>(body.acc, 3, red, L, zl.G, tot)) return;
  if (threadIdx.x == 0) residual_decision(tot, cfg, ctl);
}

// y = K x (mode 0) or y = x - sigma K x (mode 1), FP64, no reduction (verification access);
// mode 0 adds the terms fx (an explicit stage's slope f(x) = K x + g + R(x)).
template <int VEC, int FMT, int FL>
__global__ __launch_bounds__(TPB) void k_apply64(Launch ln, Geo geo, Coef<double> K, Csr csr,
                                                 const double* __restrict__ kval,
                                                 const double* __restrict__ x,
                                                 double* __restrict__ y, double sigma, int mode,
                                                 FTerms fx) {
  const double* __restrict__ force = fx.g;
  const int L = xcd_block(ln.G);
  for (int it = 0; it < ln.nit; ++it) {
    const int g0 = (L * ln.nit + it) * TPB;
    const int g = g0 + threadIdx.x;
    double csum = 0.0;
    if constexpr (FMT == 1) {
      const int gw = wave_row0(g0);
      if (gw >= ln.ng) break;
      csum = csr_wave_row<double, double>(csr, kval, gw, ln.ng, In1<double, double, 1>{x});
    }
    if (g >= ln.ng) break;
    double xc[VEC], kx[VEC];
    k64_group<VEC, FMT, FL>(geo, K, x, g, csum, xc, kx);
    if (force) {  // mode 0 with forcing: y = K x + g (an explicit stage's slope)
      double fv[VEC];
      loadg<double, double, VEC, FL>(force, g * VEC, ln.n, fv);
#pragma unroll
      for (int v = 0; v < VEC; ++v) kx[v] += fv[v];
    }
    if (fx.react) {
#pragma unroll
      for (int v = 0; v < VEC; ++v) kx[v] += fx.R(xc[v]);
    }
    if (mode == 1) {
#pragma unroll
      for (int v = 0; v < VEC; ++v) kx[v] = xc[v] - sigma * kx[v];
    }
    storeg<double, double, VEC, FL>(y, g * VEC, ln.n, kx);
  }
}

// Steps replayed from a graph keep each stage's final head record (the 64-byte prefix of Ctl)
// on the device; the steered path copies it to the host after each stage instead.
static __global__ void k_stage_snapshot(Ctl* ctl, int slot) {
  const long long* head = reinterpret_cast<const long long*>(ctl);
  if (threadIdx.x < 8) ctl->srec[slot][threadIdx.x] = head[threadIdx.x];
}

// The replays of a call start with the strict halt of an earlier call released (the steered
// path does this in its first stage-rhs launch).
static __global__ void k_release_halt(Ctl* ctl) {
  if (threadIdx.x == 0) ctl->halt = 0;
}

// k^eps = (y - rhs) / sigma : the low-precision slope of an implicit stage.
template <int VEC, int FL>
__global__ __launch_bounds__(TPB) void k_keps(Launch ln, const double* __restrict__ y,
                                              const double* __restrict__ rhs, double inv_sigma,
                                              double* __restrict__ keps) {
  const int L = xcd_block(ln.G);
  for (int it = 0; it < ln.nit; ++it) {
    const int g = (L * ln.nit + it) * TPB + threadIdx.x;
    if (g >= ln.ng) break;
    double a[VEC], b[VEC];
    loadg<double, double, VEC, FL>(y, g * VEC, ln.n, a);
    loadg<double, double, VEC, FL>(rhs, g * VEC, ln.n, b);
#pragma unroll
    for (int v = 0; v < VEC; ++v) a[v] = (a[v] - b[v]) * inv_sigma;
    storeg<double, double, VEC, FL>(keps, g * VEC, ln.n, a);
  }
}

// u += sum_j c_j v_j (step combination), skipped when the step hit a non-finite residual, was held or
// timed out.
template <int VEC, int FL>
__global__ __launch_bounds__(TPB) void k_combine(Launch ln, double* __restrict__ u, CombArgs a,
                                                 Ctl* ctl) {
  const int nonfin = ctl->step_nonfinite, held = ctl->step_held;
  const int late = ctl->bar.error;  // a one-launch stage timed out: the host runs the step again
  const int bad = nonfin | held | late;
  count_work(ctl, KC_COMBINE);
  if (blockIdx.x == 0 && threadIdx.x == 0 && !late) {
    if (nonfin) ctl->bad_steps += 1;
    else if (held) ctl->held_steps += 1;
    else ctl->good_steps += 1;
  }
  if (bad) return;
  const int L = xcd_block(ln.G);
  for (int it = 0; it < ln.nit; ++it) {
    const int g = (L * ln.nit + it) * TPB + threadIdx.x;
    if (g >= ln.ng) break;
    const int e = g * VEC;
    double acc[VEC];
    loadg<double, double, VEC, FL>(u, e, ln.n, acc);
    for (int j = 0; j < a.nv; ++j) {
      double t[VEC];
      loadg<double, double, VEC, FL>(a.v[j], e, ln.n, t);
      const double c = a.c[j];
#pragma unroll
      for (int v = 0; v < VEC; ++v) acc[v] += c * t[v];
    }
    storeg<double, double, VEC, FL>(u, e, ln.n, acc);
  }
}

// ------------------------------------------------------------------------------------------
// LP operators
// ------------------------------------------------------------------------------------------

// w = M v for one group; for CSR M v = v - msig * (Kt v) with Kt the scaled LP values, the row
// product csum = (Kt v)_g coming from csr_wave_row.
template <typename S, typename C, int VEC, int FMT, int FL, typename F, typename P = NoPre>
__device__ __forceinline__ void mlp_group(const Geo& geo, const Coef<C>& M, C msig, int g, C csum,
                                          const F& f, C (&ctr)[VEC], C (&w)[VEC],
                                          const P& pre = P()) {
  if constexpr (FMT == 0) {
    stencil_group<C, VEC, FL, S>(geo, M, g * VEC, f, ctr, w, pre);
  } else {
    static_assert(VEC == 1, "CSR kernels use one row per group");
    ctr[0] = f.one(g);
    w[0] = ctr[0] - msig * csum;
  }
}

template <typename S, typename C, int VEC, int FMT, int FL>
__global__ __launch_bounds__(TPB) void k_apply_lp(Launch ln, Geo geo, Coef<C> M, Csr csr,
                                                  const S* __restrict__ mval, C msig,
                                                  const S* __restrict__ x, S* __restrict__ y) {
  const int L = xcd_block(ln.G);
  const In1<C, S, VEC> f{x};
  for (int it = 0; it < ln.nit; ++it) {
    const int g0 = (L * ln.nit + it) * TPB;
    const int g = g0 + threadIdx.x;
    C csum = C(0);
    if constexpr (FMT == 1) {
      const int gw = wave_row0(g0);
      if (gw >= ln.ng) break;
      csum = csr_wave_row<C, S>(csr, mval, gw, ln.ng, f);
    }
    if (g >= ln.ng) break;
    C ctr[VEC], w[VEC];
    mlp_group<S, C, VEC, FMT, FL>(geo, M, msig, g, csum, f, ctr, w);
    storeg<S, C, VEC, FL>(y, g * VEC, ln.n, w);
  }
}

template <typename S, typename C, int VEC, int BS, int AD, int FL>
__global__ __launch_bounds__(TPB) void k_bj_apply(Launch ln, const S* __restrict__ r,
                                                  S* __restrict__ z, BJ<S> dinv) {
  const int L = xcd_block(ln.G);
  for (int it = 0; it < ln.nit; ++it) {
    const int g = (L * ln.nit + it) * TPB + threadIdx.x;
    const bool valid = g < ln.ng;
    C rv[VEC], zv[VEC];
    if (valid) loadg<C, S, VEC, FL>(r, g * VEC, ln.n, rv);
    else {
#pragma unroll
      for (int v = 0; v < VEC; ++v) rv[v] = C(0);
    }
    bj_apply_lane<C, S, VEC, BS, AD>(dinv, g * VEC, valid, rv, zv);
    if (valid) storeg<S, C, VEC, FL>(z, g * VEC, ln.n, zv);
  }
}

// ------------------------------------------------------------------------------------------
// Preconditioned CG in LP (heat).  BS = 0: no preconditioner (z is r).
// ------------------------------------------------------------------------------------------

// Start of a CG pass: r = LP(res / scale), z = BJ(r), rz = (r, z), rr = (r, r)
template <typename S, typename C, int VEC, int BS, int AD, int FL>
__global__ __launch_bounds__(TPB) void k_cg_begin(Launch ln, const double* __restrict__ res,
                                                  S* __restrict__ r, S* __restrict__ z,
                                                  BJ<S> dinv, SolveCfg cfg,
                                                  Ctl* ctl, Red red) {
  if (ctl->outer_done) return;
  count_work(ctl, KC_CG_BEGIN);
  const double inv = 1.0 / ctl->scale;
  const int L = xcd_block(ln.G);
  double acc[2] = {0.0, 0.0};
  for (int it = 0; it < ln.nit; ++it) {
    const int g = (L * ln.nit + it) * TPB + threadIdx.x;
    const bool valid = g < ln.ng;
    const int e = valid ? g * VEC : 0;  // an invalid lane reads group 0 and discards it
    double t[VEC];
    loadg<double, double, VEC, FL>(res, e, ln.n, t);
    BJRows<S, VEC, bj_early<S, VEC, BS>() ? BS : 1> R;
    if constexpr (bj_early<S, VEC, BS>()) bj_load<S, VEC, BS, AD>(dinv, e, valid, R);
    C rv[VEC], zv[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) rv[v] = valid ? rnd<S, C>((C)(t[v] * inv)) : C(0);
    constexpr int ZR = FL ? 1 : AD == 2 ? (BS >= 4 ? 2 : 1) : 0;
    C prz = C(0), prr = C(0);
    if constexpr (BS > 0) {
      if constexpr (bj_early<S, VEC, BS>()) bj_mul<C, S, VEC, BS, AD, ZR>(dinv, e, R, valid, rv, zv);
      else bj_apply_lane<C, S, VEC, BS, AD, ZR>(dinv, e, valid, rv, zv);
#pragma unroll
      for (int v = 0; v < VEC; ++v) zv[v] = rnd<S, C>(zv[v]);
    }
    if (valid) {
      storev<S, C, VEC>(r + e, rv);
      if constexpr (BS > 0) storev<S, C, VEC>(z + e, zv);
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        if constexpr (FL) {
          acc[1] += (double)(rv[v] * rv[v]);
          if constexpr (BS > 0) acc[0] += (double)(rv[v] * zv[v]);
        } else {
          prr += rv[v] * rv[v];
          if constexpr (BS > 0) prz += rv[v] * zv[v];
        }
      }
    }
    if constexpr (!FL) {
      acc[0] += (double)prz;
      acc[1] += (double)prr;
    }
  }
  __shared__ double tot[2];
  if (!reduce_to_last<2>(acc, 2, red, L, ln.G, tot)) return;
  if (threadIdx.x == 0) {
    const double rr = tot[1];
    const double rz = BS > 0 ? tot[0] : rr;
    const double bn = sqrt(rr);
    ctl->rz = rz;
    ctl->rr = rr;
    ctl->beta = 0.0;
    ctl->iters = 0;
    ctl->tol = fmax(fmax(cfg.rtol * bn, cfg.atol / ctl->scale),
                    outer_target(cfg, ctl, ctl->scale));
    ctl->inner_conv = bn <= ctl->tol;
    ctl->inner_done = ctl->inner_conv || cfg.maxit <= 0;
  }
}

// p_new = z + beta p_old (p_new = z in the first iteration), q = M p_new, pq = (p_new, q).
// p is double-buffered because neighbours read p_old at the halo while p_new is written.
template <typename S, typename C, int VEC, int FMT, int FL>
__global__ __launch_bounds__(TPB) void k_cg_dir(Launch ln, Geo geo, Coef<C> M, Csr csr,
                                                const S* __restrict__ mval, C msig,
                                                const S* __restrict__ z,
                                                const S* __restrict__ pold, S* __restrict__ pnew,
                                                S* __restrict__ q, Ctl* ctl, Red red) {
  if (ctl->outer_done | ctl->inner_done) return;
  count_work(ctl, KC_CG_DIR);
  const int first = ctl->iters == 0;
  const InAxpy<C, S, VEC> f{z, first ? z : pold, first ? C(0) : (C)ctl->beta};
  const int L = xcd_block(ln.G);
  double acc[1] = {0.0};
  for (int it = 0; it < ln.nit; ++it) {
    const int g0 = (L * ln.nit + it) * TPB;
    const int g = g0 + threadIdx.x;
    C csum = C(0);
    if constexpr (FMT == 1) {
      const int gw = wave_row0(g0);
      if (gw >= ln.ng) break;
      csum = csr_wave_row<C, S>(csr, mval, gw, ln.ng, f);
    }
    if (g >= ln.ng) break;
    C p[VEC], w[VEC];
    mlp_group<S, C, VEC, FMT, FL>(geo, M, msig, g, csum, f, p, w);
    if constexpr (FL) {  // (stencil: zero past the end, the vectors are padded; CSR has rows alone)
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        w[v] = rnd<S, C>(w[v]);
        acc[0] += (double)(p[v] * w[v]);
      }
    } else {
      C s = C(0);
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        w[v] = rnd<S, C>(w[v]);
        s += as_fp32<S, C>(p[v]) * w[v];
      }
      acc[0] += (double)s;
    }
    storev<S, C, VEC>(pnew + g * VEC, p);
    storev<S, C, VEC>(q + g * VEC, w);
  }
  __shared__ double tot[1];
  if (!reduce_to_last<1>(acc, 1, red, L, ln.G, tot)) return;
  if (threadIdx.x == 0) {
    const double pq = tot[0];
    ctl->pq = pq;
    if (!(pq > 0.0) || !__builtin_isfinite(pq)) {
      ctl->inner_done = 1;  // breakdown: keep the current iterate
      ctl->inner_conv = 0;
      ctl->alpha = 0.0;
    } else {
      ctl->alpha = ctl->rz / pq;
    }
  }
}

// x += alpha p (x = alpha p first), r -= alpha q, z = BJ(r), rz, rr; convergence test.
template <typename S, typename C, int VEC, int BS, int AD, int FL>
__global__ __launch_bounds__(TPB) void k_cg_upd(Launch ln, S* __restrict__ x,
                                                const S* __restrict__ p, S* __restrict__ r,
                                                const S* __restrict__ q, S* __restrict__ z,
                                                BJ<S> dinv, SolveCfg cfg,
                                                Ctl* ctl, Red red) {
  if (ctl->outer_done | ctl->inner_done) return;
  count_work(ctl, KC_CG_UPD);
  const int first = ctl->iters == 0;
  const C alpha = (C)ctl->alpha;
  const int L = xcd_block(ln.G);
  double acc[2] = {0.0, 0.0};
  for (int it = 0; it < ln.nit; ++it) {
    const int g = (L * ln.nit + it) * TPB + threadIdx.x;
    const bool valid = g < ln.ng;
    const int e = valid ? g * VEC : 0;  // an invalid lane reads group 0 and discards it
    // all loads first (x is read but unused in the first iteration)
    C rv[VEC], zv[VEC], pv[VEC], qv[VEC], xv[VEC];
    loadv<C, S, VEC>(p + e, pv);
    loadv<C, S, VEC>(q + e, qv);
    loadv<C, S, VEC>(r + e, rv);
    loadv<C, S, VEC>(x + e, xv);
    BJRows<S, VEC, bj_early<S, VEC, BS>() ? BS : 1> R;
    if constexpr (bj_early<S, VEC, BS>()) bj_load<S, VEC, BS, AD>(dinv, e, valid, R);
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      xv[v] = first ? alpha * pv[v] : xv[v] + alpha * pv[v];
      if constexpr (FL || AD == 2) {
        xv[v] = rnd2<S, C>(xv[v]);
        rv[v] = rnd_fma<S, C>(-alpha, qv[v], rv[v]);
        if (!valid || (FL && e + v >= ln.n)) rv[v] = C(0);
      } else {
        rv[v] = valid ? rnd<S, C>(rv[v] - alpha * qv[v]) : C(0);
      }
    }
    if (valid) {
      storev<S, C, VEC>(x + e, xv);
      storev<S, C, VEC>(r + e, rv);
    }
    constexpr int ZR = FL || AD == 2 ? 1 : 0;
    C prz = C(0), prr = C(0);
    if constexpr (BS > 0) {
      if constexpr (bj_early<S, VEC, BS>()) bj_mul<C, S, VEC, BS, AD, ZR>(dinv, e, R, valid, rv, zv);
      else bj_apply_lane<C, S, VEC, BS, AD, ZR>(dinv, e, valid, rv, zv);
#pragma unroll
      for (int v = 0; v < VEC; ++v) zv[v] = rnd<S, C>(zv[v]);
      if (valid) storev<S, C, VEC>(z + e, zv);
    }
    if (valid) {
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        if constexpr (FL) {
          acc[1] += (double)(rv[v] * rv[v]);
          if constexpr (BS > 0) acc[0] += (double)(rv[v] * zv[v]);
        } else {
          prr += rv[v] * rv[v];
          if constexpr (BS > 0) prz += rv[v] * zv[v];
        }
      }
    }
    if constexpr (!FL) {
      acc[0] += (double)prz;
      acc[1] += (double)prr;
    }
  }
  __shared__ double tot[2];
  if (!reduce_to_last<2>(acc, 2, red, L, ln.G, tot)) return;
  if (threadIdx.x == 0) {
    const double rr = tot[1];
    const double rz = BS > 0 ? tot[0] : rr;
    const int its = ctl->iters + 1;
    ctl->iters = its;
    ctl->total_iters += 1;
    ctl->life_iters += 1;
    ctl->beta = rz / ctl->rz;
    ctl->rz = rz;
    ctl->rr = rr;
    const bool fin = __builtin_isfinite(rr) && __builtin_isfinite(rz);
    ctl->inner_conv = fin && sqrt(rr) <= ctl->tol;
    ctl->inner_done = !fin || ctl->inner_conv || its >= cfg.maxit;
  }
}

// End of a CG pass: y += scale * x ; one LP pass done.
template <typename S, typename C, int VEC, int FL>
__global__ __launch_bounds__(TPB) void k_promote(Launch ln, double* __restrict__ y,
                                                 const S* __restrict__ x, Ctl* ctl) {
  if (ctl->outer_done) return;
  count_work(ctl, KC_PROMOTE);
  const double s = ctl->scale;
  const int have = ctl->iters > 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (ctl->passes < MAXPASS) ctl->pass_iters[ctl->passes] = ctl->iters;
    ctl->passes += 1;
    ctl->life_passes += 1;
  }
  if (!have) return;
  const int L = xcd_block(ln.G);
  for (int it = 0; it < ln.nit; ++it) {
    const int g = (L * ln.nit + it) * TPB + threadIdx.x;
    if (g >= ln.ng) break;
    double yv[VEC];
    C xv[VEC];
    loadg<double, double, VEC, FL>(y, g * VEC, ln.n, yv);
    loadv<C, S, VEC>(x + g * VEC, xv);
#pragma unroll
    for (int v = 0; v < VEC; ++v) yv[v] += s * (double)xv[v];
    storeg<double, double, VEC, FL>(y, g * VEC, ln.n, yv);
  }
}

// ------------------------------------------------------------------------------------------
// Right-preconditioned GMRES(m) in LP (advection-diffusion).  Inner products are taken in
// the RMS sense ((x, y) / N) so stored basis vectors have O(1) entries (FP16 range); basis
// vector i is vscale[i] times the stored vector i.  One cycle per outer pass: the restart
// residual is the FP64 residual of the outer loop.
// ------------------------------------------------------------------------------------------

// Start of a GMRES cycle: V_0 = LP(res / scale) ; zt = BJ(V_0) (the preconditioned direction of the first
// Arnoldi step, before normalisation; BJ is linear) ; beta = ||V_0||_rms.
template <typename S, typename C, int VEC, int BS, int AD, int FL>
__global__ __launch_bounds__(TPB) void k_gm_begin(Launch ln, const double* __restrict__ res,
                                                  S* __restrict__ v0, S* __restrict__ zt,
                                                  BJ<S> dinv, SolveCfg cfg,
                                                  Ctl* ctl, Red red) {
  if (ctl->outer_done) return;
  count_work(ctl, KC_GM_BEGIN);
  const double inv = 1.0 / ctl->scale;
  const int L = xcd_block(ln.G);
  double acc[1] = {0.0};
  for (int it = 0; it < ln.nit; ++it) {
    const int g = (L * ln.nit + it) * TPB + threadIdx.x;
    const bool valid = g < ln.ng;
    const int e = valid ? g * VEC : 0;  // an invalid lane reads group 0 and discards it
    double t[VEC];
    loadg<double, double, VEC, FL>(res, e, ln.n, t);
    BJRows<S, VEC, bj_early<S, VEC, BS>() ? BS : 1> R;
    if constexpr (bj_early<S, VEC, BS>()) bj_load<S, VEC, BS, AD>(dinv, e, valid, R);
    __builtin_amdgcn_sched_barrier(0);  // res and the rows in flight together
    C rv[VEC];
    C s = C(0);
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      rv[v] = valid ? rnd<S, C>((C)(t[v] * inv)) : C(0);
      if constexpr (FL) acc[0] += (double)(rv[v] * rv[v]);
      else s += rv[v] * rv[v];
    }
    if (valid) storev<S, C, VEC>(v0 + e, rv);
    if constexpr (BS > 0) {
      C zv[VEC];
      if constexpr (bj_early<S, VEC, BS>()) bj_mul<C, S, VEC, BS, AD, (FL || AD == 2 ? 1 : 0)>(dinv, e, R, valid, rv, zv);
      else bj_apply_lane<C, S, VEC, BS, AD, (FL || AD == 2 ? 1 : 0)>(dinv, e, valid, rv, zv);
      if (valid) storev<S, C, VEC>(zt + e, zv);
    }
    if constexpr (!FL) acc[0] += (double)s;
  }
  __shared__ double tot[1];
  if (!reduce_to_last<1>(acc, 1, red, L, ln.G, tot)) return;
  if (threadIdx.x == 0) {
    const double beta = sqrt(tot[0] * cfg.invN);
    ctl->vscale[0] = beta > 0.0 ? 1.0 / beta : 0.0;
    ctl->g[0] = beta;
    for (int i = 1; i <= MAXM; ++i) ctl->g[i] = 0.0;
    ctl->J = 0;
    ctl->iters = 0;
    ctl->tol = fmax(fmax(cfg.rtol * beta, cfg.atol / (ctl->scale * cfg.sqrtN)),
                    outer_target(cfg, ctl, ctl->scale * cfg.sqrtN));
    ctl->inner_conv = (beta <= ctl->tol) || beta == 0.0;
    ctl->inner_done = ctl->inner_conv || cfg.maxit <= 0;
  }
}

// Completes Hessenberg column j, whose entries 0..j are already in H, with the subdiagonal
// entry hn = h_{j+1,j}: the earlier Givens rotations and a new one, the rotated right-hand side
// g, the iteration counters, J = j + 1 and the inner stopping test on the residual estimate
// |g_{j+1}| (hn = 0 is an exact breakdown: the solve is exact).  One thread.
__device__ __forceinline__ void gm_complete_column(Ctl* ctl, const SolveCfg& cfg, int j, double hn) {
  double* col = ctl->H + j * (MAXM + 1);
  col[j + 1] = hn;
  for (int i = 0; i < j; ++i) {  // previous rotations
    const double a = col[i], b = col[i + 1];
    col[i] = ctl->cs[i] * a + ctl->sn[i] * b;
    col[i + 1] = -ctl->sn[i] * a + ctl->cs[i] * b;
  }
  const double a = col[j], b = col[j + 1];
  const double den = sqrt(a * a + b * b);
  const double c = den > 0.0 ? a / den : 1.0;
  const double sn = den > 0.0 ? b / den : 0.0;
  ctl->cs[j] = c;
  ctl->sn[j] = sn;
  col[j] = den;
  col[j + 1] = 0.0;
  ctl->g[j + 1] = -sn * ctl->g[j];
  ctl->g[j] = c * ctl->g[j];
  const int its = ctl->iters + 1;
  ctl->iters = its;
  ctl->total_iters += 1;
  ctl->life_iters += 1;
  const int J = j + 1;
  ctl->J = J;
  const double resid = fabs(ctl->g[J]);
  const bool fin = __builtin_isfinite(resid) && __builtin_isfinite(den);
  const bool conv = fin && (resid <= ctl->tol || hn == 0.0);
  const bool stop = !fin || conv || J >= cfg.m || its >= cfg.maxit;
  ctl->inner_conv = conv;
  if (stop) ctl->inner_done = 1;
  if (!fin) {  // drop this cycle: the promoted correction is zero
    for (int i = 0; i <= J; ++i) ctl->g[i] = 0.0;
  }
}

// The launch of Arnoldi step j is compiled for a bound NDM >= j + 1 on the number of basis
// vectors it touches (the host knows j: every step of a cycle is enqueued in order), so that
// its per-lane dot accumulators and coefficients take NDM registers, not MAXD.  A launch whose
// step exceeds its bound flags the solve as failed instead of computing.
__device__ __forceinline__ bool gm_bound_exceeded(Ctl* ctl, int nd, int ndm) {
  if (nd <= ndm) return false;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctl->nonfinite = 1;
    ctl->step_nonfinite = 1;
    ctl->inner_done = 1;
    ctl->inner_conv = 0;
  }
  return true;
}

// w = M BJ(v_j) (PREC: z + j zstride holds BJ of the stored vector j, scaled here by vscale[j];
// zstride = 0 for a single preconditioned-direction buffer) or w = M v_j ; V_{j+1} := LP(w) ;
// d_i = (V_i, LP(w)) for i <= j.
template <typename S, typename C, int VEC, int FMT, int PREC, int NDM, int FL>
__global__ __launch_bounds__(TPB) void k_gm_matvec(Launch ln, Geo geo, Coef<C> M, Csr csr,
                                                   const S* __restrict__ mval, C msig,
                                                   const S* __restrict__ z, size_t zstride,
                                                   S* __restrict__ V, size_t vstride, SolveCfg cfg,
                                                   Ctl* ctl, Red red) {
  if (ctl->outer_done | ctl->inner_done) return;
  const int j = ctl->J;
  const int nd = j + 1;
  if (gm_bound_exceeded(ctl, nd, NDM)) return;
  count_work(ctl, KC_GM_MATVEC, nd);
  S* wout = V + (size_t)(j + 1) * vstride;
  const int L = xcd_block(ln.G);
  // flat groups add every product in FP64 (a group of one did), else a group's are added in C
  using D = std::conditional_t<FL == 1, double, C>;
  D dacc[NDM];
#pragma unroll
  for (int i = 0; i < NDM; ++i) dacc[i] = D(0);
  constexpr int CH = basis_chunk<S, VEC>() < NDM ? basis_chunk<S, VEC>() : NDM;
  const InScaled<C, S, VEC> f{PREC ? z + (size_t)j * zstride : V + (size_t)j * vstride,
                              (C)ctl->vscale[j]};
  for (int it = 0; it < ln.nit; ++it) {
    const int g0 = (L * ln.nit + it) * TPB;
    const int g = g0 + threadIdx.x;
    const int gw = FMT == 1 ? wave_row0(g0) : g;  // CSR: the wave leaves together
    if (gw >= ln.ng) break;
    const int e = g * VEC;
    // the first chunk of basis vectors (nd >= 1) is loaded together with the stencil inputs
    // (for CSR ahead of the staged row products; rows past the end load row ng - 1 unused)
    const int el = FMT == 1 ? min(g, ln.ng - 1) : e;
    Vec<S, VEC> v0[CH];
#pragma unroll
    for (int k = 0; k < CH; ++k)
      v0[k] = *reinterpret_cast<const Vec<S, VEC>*>(V + (size_t)min(k, nd - 1) * vstride + el);
    C csum = C(0);
    if constexpr (FMT == 1) {
      csum = csr_wave_row<C, S>(csr, mval, gw, ln.ng, f);
      if (g >= ln.ng) break;
    }
    C ctr[VEC], w[VEC];
    mlp_group<S, C, VEC, FMT, FL>(geo, M, msig, g, csum, f, ctr, w);
#pragma unroll
    for (int v = 0; v < VEC; ++v) w[v] = rnd<S, C>(w[v]);
    storev<S, C, VEC>(wout + e, w);
#pragma unroll
    for (int k = 0; k < CH; ++k) {
      D s = D(0);
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        if constexpr (FL) s += (double)((C)v0[k].v[v] * w[v]);
        else s += (C)v0[k].v[v] * w[v];
      }
      dacc[k] += (k < nd) ? s : D(0);
    }
    // remaining basis vectors in chunks of CH whose loads are issued together (indices past
    // nd are clamped to a valid vector and their contribution discarded)
#pragma unroll
    for (int c = CH; c < NDM; c += CH) {
      if (c < nd) {
        C vv[CH][VEC];
#pragma unroll
        for (int k = 0; k < CH; ++k)
          loadv<C, S, VEC>(V + (size_t)min(c + k, nd - 1) * vstride + e, vv[k]);
#pragma unroll
        for (int k = 0; k < CH; ++k) {
          if (c + k < NDM) {
            D s = D(0);
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
              if constexpr (FL) s += (double)(vv[k][v] * w[v]);
              else s += vv[k][v] * w[v];
            }
            dacc[c + k] += (c + k < nd) ? s : D(0);
          }
        }
      }
    }
  }
  double acc[NDM];
#pragma unroll
  for (int i = 0; i < NDM; ++i) acc[i] = (double)dacc[i];
  __shared__ double tot[NDM];
  if (!reduce_to_last<NDM>(acc, nd, red, L, ln.G, tot)) return;
  if (threadIdx.x < nd) {
    ctl->hcol[threadIdx.x] = ctl->vscale[threadIdx.x] * tot[threadIdx.x] * cfg.invN;
    ctl->hacc[threadIdx.x] = 0.0;
  }
}

// Re-orthogonalisation pass of classical Gram-Schmidt (CGS2), between k_gm_matvec and
// k_gm_orth: w' = w - sum_{i<=j} h_ij v_i is formed and stored (in the storage type), then its
// products d_i = (V_i, w') are taken in the same launch (the basis chunks are read again,
// normally from cache).  The first pass's h moves to hacc and d becomes the coefficient set
// that k_gm_orth subtracts; the Hessenberg column is h + d.
template <typename S, typename C, int VEC, int NDM, int FL>
__global__ __launch_bounds__(TPB) void k_gm_reorth(Launch ln, S* __restrict__ V, size_t vstride,
                                                   SolveCfg cfg, Ctl* ctl, Red red) {
  if (ctl->outer_done | ctl->inner_done) return;
  const int j = ctl->J;
  const int nd = j + 1;
  if (gm_bound_exceeded(ctl, nd, NDM)) return;
  count_work(ctl, KC_GM_REORTH, nd);
  C cf[NDM];
#pragma unroll
  for (int i = 0; i < NDM; ++i) cf[i] = i < nd ? (C)(ctl->hcol[i] * ctl->vscale[i]) : C(0);
  S* w = V + (size_t)(j + 1) * vstride;
  const int L = xcd_block(ln.G);
  constexpr int CH = basis_chunk<S, VEC>() < NDM ? basis_chunk<S, VEC>() : NDM;
  using D = std::conditional_t<FL == 1, double, C>;  // (as k_gm_matvec)
  D dacc[NDM];
#pragma unroll
  for (int i = 0; i < NDM; ++i) dacc[i] = D(0);
  for (int it = 0; it < ln.nit; ++it) {
    const int g = (L * ln.nit + it) * TPB + threadIdx.x;
    if (g >= ln.ng) break;
    const int e = g * VEC;
    C wv[VEC];
    loadv<C, S, VEC>(w + e, wv);
    // w' = w - V h over chunks of CH basis vectors (indices past nd are clamped to a valid
    // vector; their coefficient is zero)
#pragma unroll
    for (int c = 0; c < NDM; c += CH) {
      if (c < nd) {
        C vv[CH][VEC];
#pragma unroll
        for (int k = 0; k < CH; ++k)
          loadv<C, S, VEC>(V + (size_t)min(c + k, nd - 1) * vstride + e, vv[k]);
#pragma unroll
        for (int k = 0; k < CH; ++k) {
          if (c + k < NDM) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) wv[v] -= cf[c + k] * vv[k][v];
          }
        }
      }
    }
#pragma unroll
    for (int v = 0; v < VEC; ++v) wv[v] = FL && e + v >= ln.n ? C(0) : rnd<S, C>(wv[v]);
    storev<S, C, VEC>(w + e, wv);
    // d = V^T w' (the stored, rounded w')
#pragma unroll
    for (int c = 0; c < NDM; c += CH) {
      if (c < nd) {
        C vv[CH][VEC];
#pragma unroll
        for (int k = 0; k < CH; ++k)
          loadv<C, S, VEC>(V + (size_t)min(c + k, nd - 1) * vstride + e, vv[k]);
#pragma unroll
        for (int k = 0; k < CH; ++k) {
          if (c + k < NDM) {
            D s = D(0);
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
              if constexpr (FL) s += (double)(vv[k][v] * wv[v]);
              else s += vv[k][v] * wv[v];
            }
            dacc[c + k] += (c + k < nd) ? s : D(0);
          }
        }
      }
    }
  }
  double acc[NDM];
#pragma unroll
  for (int i = 0; i < NDM; ++i) acc[i] = (double)dacc[i];
  __shared__ double tot[NDM];
  if (!reduce_to_last<NDM>(acc, nd, red, L, ln.G, tot)) return;
  if (threadIdx.x < nd) {
    ctl->hacc[threadIdx.x] = ctl->hcol[threadIdx.x];
    ctl->hcol[threadIdx.x] = ctl->vscale[threadIdx.x] * tot[threadIdx.x] * cfg.invN;
  }
}

// w -= sum_{i<=j} h_ij v_i (classical Gram-Schmidt, coefficients from k_gm_matvec, or from
// k_gm_reorth in the second pass of CGS2); h_{j+1,j} = ||w||; Givens update of the Hessenberg column; residual estimate |g_{j+1}|.
// With a preconditioner (BS > 0) also BJ(w), the next step's preconditioned direction before
// normalisation, stored at zt + (j + 1) zstride (zstride = 0: the single buffer zt).
template <typename S, typename C, int VEC, int BS, int NDM, int AD, int FL>
__global__ __launch_bounds__(TPB) void k_gm_orth(Launch ln, S* __restrict__ V, size_t vstride,
                                                 S* __restrict__ zt, size_t zstride, BJ<S> dinv,
                                                 SolveCfg cfg, Ctl* ctl, Red red) {
  if (ctl->outer_done | ctl->inner_done) return;
  const int j = ctl->J;
  const int nd = j + 1;
  if (gm_bound_exceeded(ctl, nd, NDM)) return;
  count_work(ctl, KC_GM_ORTH, nd);
  C cf[NDM];
#pragma unroll
  for (int i = 0; i < NDM; ++i) cf[i] = i < nd ? (C)(ctl->hcol[i] * ctl->vscale[i]) : C(0);
  S* w = V + (size_t)(j + 1) * vstride;
  S* zw = zt + (size_t)(j + 1) * zstride;
  const int L = xcd_block(ln.G);
  constexpr int CH = basis_chunk<S, VEC>() < NDM ? basis_chunk<S, VEC>() : NDM;
  constexpr bool EARLY = bj_early<S, VEC, BS>();
  double acc[1] = {0.0};
  for (int it = 0; it < ln.nit; ++it) {
    const int g = (L * ln.nit + it) * TPB + threadIdx.x;
    const bool valid = g < ln.ng;
    const int e = valid ? g * VEC : 0;  // an invalid lane reads group 0 and discards it
    // every load that does not depend on a value is issued first: w, the first chunk of basis
    // vectors (nd >= 1) and the block-Jacobi rows
    Vec<S, VEC> wr = *reinterpret_cast<const Vec<S, VEC>*>(w + e);
    Vec<S, VEC> v0[CH];
#pragma unroll
    for (int k = 0; k < CH; ++k)
      v0[k] = *reinterpret_cast<const Vec<S, VEC>*>(V + (size_t)min(k, nd - 1) * vstride + e);
    BJRows<S, VEC, EARLY ? BS : 1> R;
    if constexpr (EARLY) bj_load<S, VEC, BS, AD>(dinv, e, valid, R);
    // keep them in flight together (the scheduler would otherwise wait for w and the basis
    // chunk before issuing the block-Jacobi rows: a second memory round trip)
    __builtin_amdgcn_sched_barrier(0);
    C wv[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) wv[v] = (C)wr.v[v];
    // flat groups with a small basis round w - V h with its last product (the groups of one that
    // they replace did); every other form rounds the finished sum
    constexpr bool LAST = FL == 1 && NDM <= 8;
#pragma unroll
    for (int k = 0; k < CH; ++k) {  // cf is zero past nd
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        if constexpr (LAST && CH == NDM) {
          if (k == NDM - 1) {
            wv[v] = rnd_fma<S, C>(-cf[k], (C)v0[k].v[v], wv[v]);
            continue;
          }
        }
        wv[v] -= cf[k] * (C)v0[k].v[v];
      }
    }
#pragma unroll
    for (int c = CH; c < NDM; c += CH) {
      if (c < nd) {
        C vv[CH][VEC];
#pragma unroll
        for (int k = 0; k < CH; ++k)
          loadv<C, S, VEC>(V + (size_t)min(c + k, nd - 1) * vstride + e, vv[k]);
#pragma unroll
        for (int k = 0; k < CH; ++k) {
          if (c + k < NDM) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
              if constexpr (LAST) {
                if (c + k == NDM - 1) {
                  wv[v] = rnd_fma<S, C>(-cf[c + k], vv[k][v], wv[v]);
                  continue;
                }
              }
              wv[v] -= cf[c + k] * vv[k][v];
            }
          }
        }
      }
    }
    C s = C(0);
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      if constexpr (FL || AD == 2) {
        wv[v] = valid && !(FL && e + v >= ln.n) ? rnd2<S, C>(wv[v]) : C(0);
      } else {
        wv[v] = valid ? rnd<S, C>(wv[v]) : C(0);
      }
      if constexpr (FL) acc[0] += (double)(wv[v] * wv[v]);
      else s += wv[v] * wv[v];
    }
    if (valid) storev<S, C, VEC>(w + e, wv);
    if constexpr (BS > 0) {
      C zv[VEC];
      if constexpr (EARLY) bj_mul<C, S, VEC, BS, AD, (FL || AD == 2 ? 1 : 0)>(dinv, e, R, valid, wv, zv);
      else bj_apply_lane<C, S, VEC, BS, AD, (FL || AD == 2 ? 1 : 0)>(dinv, e, valid, wv, zv);
      if (valid) storev<S, C, VEC>(zw + e, zv);
    }
    if constexpr (!FL) acc[0] += (double)s;
  }
  __shared__ double tot[1];
  if (!reduce_to_last<1>(acc, 1, red, L, ln.G, tot)) return;
  if (threadIdx.x == 0) {
    const double hn = sqrt(tot[0] * cfg.invN);
    double* col = ctl->H + j * (MAXM + 1);
    for (int i = 0; i <= j; ++i) col[i] = ctl->hacc[i] + ctl->hcol[i];
    gm_complete_column(ctl, cfg, j, hn);
    ctl->vscale[j + 1] = hn > 0.0 ? 1.0 / hn : 0.0;
  }
}

// Per-group work of k_gm_zmatvec: the first chunk of basis vectors of the next plane loaded
// ahead; w = LP(out) stored as V_{j+1}; its products with V_0 .. V_j.
template <typename S, typename C, int VEC, int NDM>
struct GmMatvecBody {
  static constexpr int CH = basis_chunk<S, VEC>() < NDM ? basis_chunk<S, VEC>() : NDM;
  const S* __restrict__ V;
  size_t vstride;
  int nd;
  S* __restrict__ wout;
  Vec<S, VEC> vn[CH], vc[CH];
  C dacc[NDM];
  __device__ __forceinline__ void pre(int e) {
#pragma unroll
    for (int k = 0; k < CH; ++k)
      vn[k] = *reinterpret_cast<const Vec<S, VEC>*>(V + (size_t)min(k, nd - 1) * vstride + e);
  }
  __device__ __forceinline__ void next() {
#pragma unroll
    for (int k = 0; k < CH; ++k) vc[k] = vn[k];
  }
  __device__ __forceinline__ void fin(int e, const C (&)[VEC], const C (&out)[VEC]) {
    C w[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) w[v] = rnd<S, C>(out[v]);
    storev<S, C, VEC>(wout + e, w);
#pragma unroll
    for (int k = 0; k < CH; ++k) {
      C s = C(0);
#pragma unroll
      for (int v = 0; v < VEC; ++v) s += (C)vc[k].v[v] * w[v];
      dacc[k] += (k < nd) ? s : C(0);
    }
#pragma unroll
    for (int c = CH; c < NDM; c += CH) {
      if (c < nd) {
        C vv[CH][VEC];
#pragma unroll
        for (int k = 0; k < CH; ++k)
          loadv<C, S, VEC>(V + (size_t)min(c + k, nd - 1) * vstride + e, vv[k]);
#pragma unroll
        for (int k = 0; k < CH; ++k) {
          if (c + k < NDM) {
            C s = C(0);
#pragma unroll
            for (int v = 0; v < VEC; ++v) s += vv[k][v] * w[v];
            dacc[c + k] += (c + k < nd) ? s : C(0);
          }
        }
      }
    }
  }
};

// k_gm_matvec on z-marching tiles (stencil format): w = M (vscale_j z_j) with z_j = BJ(V_j)
// (PREC) or V_j, stored as V_{j+1}; d_i = (V_i, w) for i <= j.
template <typename S, typename C, int VEC, int PREC, int NDM>
__global__ __launch_bounds__(TPB) void k_gm_zmatvec(ZLaunch zl, Geo geo, Coef<C> M,
                                                    const S* __restrict__ z, S* __restrict__ V,
                                                    size_t vstride, SolveCfg cfg, Ctl* ctl,
                                                    Red red) {
  if (ctl->outer_done | ctl->inner_done) return;
  const int j = ctl->J;
  const int nd = j + 1;
  if (gm_bound_exceeded(ctl, nd, NDM)) return;
  count_work(ctl, KC_GM_MATVEC, nd);
  extern __shared__ double zm_lds_d[];
  C* lds = reinterpret_cast<C*>(zm_lds_d);
  const int L = xcd_block(zl.G);
  const S* zin = PREC ? z : V + (size_t)j * vstride;
  const C sj = (C)ctl->vscale[j];
  auto src = [&](int e, C (&o)[VEC], bool) {
    loadv<C, S, VEC>(zin + e, o);
#pragma unroll
    for (int v = 0; v < VEC; ++v) o[v] *= sj;
  };
  GmMatvecBody<S, C, VEC, NDM> body{V, vstride, nd, V + (size_t)(j + 1) * vstride, {}, {}, {}};
#pragma unroll
  for (int i = 0; i < NDM; ++i) body.dacc[i] = C(0);
  zmarch<C, VEC>(geo, M, zl, L, src, body, lds);
  double acc[NDM];
#pragma unroll
  for (int i = 0; i < NDM; ++i) acc[i] = (double)body.dacc[i];
  __shared__ double tot[NDM];
  if (!reduce_to_last<NDM>(acc, nd, red, L, zl.G, tot)) return;
  if (threadIdx.x < nd) {
    ctl->hcol[threadIdx.x] = ctl->vscale[threadIdx.x] * tot[threadIdx.x] * cfg.invN;
    ctl->hacc[threadIdx.x] = 0.0;
  }
}

// ------------------------------------------------------------------------------------------
// GMRES Arnoldi steps on z-marching tiles (stencil format), the update of step j folded into
// the product of step j + 1.  The separate form reads the basis twice per step (the products
// in k_gm_matvec, the update in k_gm_orth) and writes and re-reads the product w; here one
// launch per step forms v_j = w_{j-1} - sum_i h_{i,j-1} v_i from the stored product and the
// basis (halo groups recompute it from the same values), stores v_j, applies block-Jacobi and
// the stencil to it through the tile, stores the new product w_j and takes its products with
// the basis.  The norm of v_j, the subdiagonal entry of column j - 1, is only known at the end
// of that launch, so column j - 1's Givens rotation and stopping test run there, and the
// stencil input is scaled by an estimate of 1 / ||v_j|| (from ||w_{j-1}||^2 - sum h^2) only to
// keep stored values O(1): the exact factor (zc) is carried into the next column.  After the
// cycle's last step a streaming launch (k_gm_zclose) forms the last norm and column.
// Products are alternately stored in W0 and W1 (halo groups of step j read w_{j-1} while
// owners write w_j).
// ------------------------------------------------------------------------------------------

// Per-group work of the first product: w_0 = LP(M (vscale_0 zt)) stored; (V_0, w_0), ||w_0||^2.
template <typename S, typename C, int VEC>
struct GmFirstBody {
  const S* __restrict__ v0;
  S* __restrict__ wout;
  Vec<S, VEC> vn, vc;
  C d0, ww;
  __device__ __forceinline__ void pre(int e) { vn = *reinterpret_cast<const Vec<S, VEC>*>(v0 + e); }
  __device__ __forceinline__ void next() { vc = vn; }
  __device__ __forceinline__ void fin(int e, const C (&)[VEC], const C (&out)[VEC]) {
    C w[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      w[v] = rnd<S, C>(out[v]);
      d0 += (C)vc.v[v] * w[v];
      ww += w[v] * w[v];
    }
    storev<S, C, VEC>(wout + e, w);
  }
};

// First product of a cycle: the stencil input is vscale_0 BJ(V_0) (stored by k_gm_begin in zin)
// or vscale_0 V_0 without a preconditioner (zin = V_0).
template <typename S, typename C, int VEC>
__global__ __launch_bounds__(TPB) void k_gm_zfirst(ZLaunch zl, Geo geo, Coef<C> M,
                                                   const S* __restrict__ zin,
                                                   const S* __restrict__ V, S* __restrict__ wout,
                                                   SolveCfg cfg, Ctl* ctl, Red red) {
  if (ctl->outer_done | ctl->inner_done) return;
  count_work(ctl, KC_GM_MATVEC, 1);
  extern __shared__ double zm_lds_d[];
  C* lds = reinterpret_cast<C*>(zm_lds_d);
  const int L = xcd_block(zl.G);
  const C s0 = (C)ctl->vscale[0];
  auto src = [&](int e, C (&o)[VEC], bool) {
    loadv<C, S, VEC>(zin + e, o);
#pragma unroll
    for (int v = 0; v < VEC; ++v) o[v] *= s0;
  };
  GmFirstBody<S, C, VEC> body{V, wout, {}, {}, C(0), C(0)};
  zmarch<C, VEC>(geo, M, zl, L, src, body, lds);
  double acc[2] = {(double)body.d0, (double)body.ww};
  __shared__ double tot[2];
  if (!reduce_to_last<2>(acc, 2, red, L, zl.G, tot)) return;
  if (threadIdx.x == 0) {
    // the stored product is c0 = s0 ||V_0|| times the product of the normalised vector
    const double c0 = ctl->vscale[0] > 0.0 ? (double)s0 / ctl->vscale[0] : 0.0;
    const double t = ctl->vscale[0] * tot[0] * cfg.invN;
    ctl->hcol[0] = c0 > 0.0 ? t / c0 : 0.0;
    ctl->hacc[0] = 0.0;
    ctl->zc = c0;
    const double ww = tot[1] * cfg.invN;
    const double est = fmax(ww - t * t, 1e-6 * ww);
    ctl->znext = est > 0.0 ? 1.0 / sqrt(est) : 1.0;
  }
}

// Per-group work of a folded step: w_j = LP(M z) stored; (V_i, w_j) for i <= j, ||w_j||^2.
template <typename S, typename C, int VEC, int NDM>
struct GmStepBody {
  const S* __restrict__ V;
  size_t vstride;
  int nd;
  S* __restrict__ wout;
  C dacc[NDM];
  C ww;
  __device__ __forceinline__ void pre(int) {}
  __device__ __forceinline__ void next() {}
  __device__ __forceinline__ void fin(int e, const C (&)[VEC], const C (&out)[VEC]) {
    constexpr int CH = basis_chunk<S, VEC>() < NDM ? basis_chunk<S, VEC>() : NDM;
    C w[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      w[v] = rnd<S, C>(out[v]);
      ww += w[v] * w[v];
    }
    storev<S, C, VEC>(wout + e, w);
#pragma unroll
    for (int c = 0; c < NDM; c += CH) {
      if (c < nd) {
        C vv[CH][VEC];
#pragma unroll
        for (int k = 0; k < CH; ++k)
          loadv<C, S, VEC>(V + (size_t)min(c + k, nd - 1) * vstride + e, vv[k]);
#pragma unroll
        for (int k = 0; k < CH; ++k) {
          if (c + k < NDM) {
            C s = C(0);
#pragma unroll
            for (int v = 0; v < VEC; ++v) s += vv[k][v] * w[v];
            dacc[c + k] += (c + k < nd) ? s : C(0);
          }
        }
      }
    }
  }
};

// Folded Arnoldi step j (j = J + 1 >= 1): v_j from w_{j-1} (win) and the basis, stored; the
// stencil of vscale-estimate * BJ(v_j) through the tile into w_j (wout); column j - 1 completed
// with ||v_j||; column j's entries for the next launch.
template <typename S, typename C, int VEC, int BS, int NDM, int AD = 0>
__global__ __launch_bounds__(TPB) void k_gm_zstep(ZLaunch zl, Geo geo, Coef<C> M,
                                                  S* __restrict__ V, size_t vstride,
                                                  const S* __restrict__ win,
                                                  S* __restrict__ wout, BJ<S> dinv,
                                                  SolveCfg cfg, Ctl* ctl, Red red) {
  if (ctl->outer_done | ctl->inner_done) return;
  const int j = ctl->J + 1;
  const int nd = j + 1;
  if (gm_bound_exceeded(ctl, nd, NDM)) return;
  count_work(ctl, KC_GM_STEP, nd);
  extern __shared__ double zm_lds_d[];
  C* lds = reinterpret_cast<C*>(zm_lds_d);
  const int L = xcd_block(zl.G);
  // update coefficients of the stored basis: v_j = w_{j-1} - sum_{i<j} a_i V_i
  C a[NDM];
#pragma unroll
  for (int i = 0; i < NDM; ++i) a[i] = i < j ? (C)(ctl->zc * ctl->hcol[i] * ctl->vscale[i]) : C(0);
  const C sc = (C)ctl->znext;
  S* vj = V + (size_t)j * vstride;
  constexpr int CH = basis_chunk<S, VEC>() < NDM ? basis_chunk<S, VEC>() : NDM;
  C nv = C(0);
  auto src = [&](int e, C (&o)[VEC], bool own) {
    C v[VEC];
    loadv<C, S, VEC>(win + e, v);
#pragma unroll
    for (int c = 0; c < NDM; c += CH) {
      if (c < j) {
        C vv[CH][VEC];
#pragma unroll
        for (int k = 0; k < CH; ++k)
          loadv<C, S, VEC>(V + (size_t)min(c + k, j - 1) * vstride + e, vv[k]);
#pragma unroll
        for (int k = 0; k < CH; ++k) {
          if (c + k < NDM) {
#pragma unroll
            for (int q = 0; q < VEC; ++q) v[q] -= a[c + k] * vv[k][q];
          }
        }
      }
    }
#pragma unroll
    for (int q = 0; q < VEC; ++q) v[q] = rnd<S, C>(v[q]);
    if (own) {
      storev<S, C, VEC>(vj + e, v);
#pragma unroll
      for (int q = 0; q < VEC; ++q) nv += v[q] * v[q];
    }
    if constexpr (BS > 0) {
      C zv[VEC];
      bj_apply_lane<C, S, VEC, BS, AD>(dinv, e, true, v, zv);
#pragma unroll
      for (int q = 0; q < VEC; ++q) o[q] = sc * zv[q];
    } else {
#pragma unroll
      for (int q = 0; q < VEC; ++q) o[q] = sc * v[q];
    }
  };
  GmStepBody<S, C, VEC, NDM> body{V, vstride, nd, wout, {}, C(0)};
#pragma unroll
  for (int i = 0; i < NDM; ++i) body.dacc[i] = C(0);
  // lanes of one block-Jacobi block exchange values when a block spans several groups
  zmarch<C, VEC, (BS > VEC ? BS / VEC : 1)>(geo, M, zl, L, src, body, lds);
  double acc[NDM + 2];
  acc[0] = (double)nv;
  acc[1] = (double)body.ww;
#pragma unroll
  for (int i = 0; i < NDM; ++i) acc[2 + i] = (double)body.dacc[i];
  __shared__ double tot[NDM + 2];
  if (!reduce_to_last<NDM + 2>(acc, nd + 2, red, L, zl.G, tot)) return;
  if (threadIdx.x == 0) {
    const double beta = sqrt(tot[0] * cfg.invN);  // ||v_j|| (stored, rms)
    const int jc = j - 1;                         // the column completed here
    double* col = ctl->H + jc * (MAXM + 1);
    for (int i = 0; i <= jc; ++i) col[i] = ctl->hcol[i];
    const double zc = ctl->zc;
    ctl->vscale[j] = beta > 0.0 ? 1.0 / beta : 0.0;
    gm_complete_column(ctl, cfg, jc, zc > 0.0 ? beta / zc : 0.0);
    // column j's entries (used by the next launch unless the solve stops here)
    const double cj = (double)sc * beta;
    const double ww = tot[1] * cfg.invN;
    double est = ww;
    for (int i = 0; i <= j; ++i) {
      const double t = ctl->vscale[i] * tot[2 + i] * cfg.invN;
      ctl->hcol[i] = cj > 0.0 ? t / cj : 0.0;
      ctl->hacc[i] = 0.0;
      est -= t * t;
    }
    ctl->zc = cj;
    est = fmax(est, 1e-6 * ww);
    ctl->znext = est > 0.0 ? 1.0 / sqrt(est) : 1.0;
  }
}

// Last column of a cycle of folded steps: ||w_J - sum_{i<=J} h_{iJ} v_i|| (no store), then
// column J's Givens rotation and stopping test.
template <typename S, typename C, int VEC, int NDM>
__global__ __launch_bounds__(TPB) void k_gm_zclose(Launch ln, const S* __restrict__ V,
                                                   size_t vstride, const S* __restrict__ win,
                                                   SolveCfg cfg, Ctl* ctl, Red red) {
  if (ctl->outer_done | ctl->inner_done) return;
  const int J = ctl->J;
  const int nd = J + 1;
  if (gm_bound_exceeded(ctl, nd, NDM)) return;
  count_work(ctl, KC_GM_CLOSE, nd);
  C a[NDM];
#pragma unroll
  for (int i = 0; i < NDM; ++i) a[i] = i < nd ? (C)(ctl->zc * ctl->hcol[i] * ctl->vscale[i]) : C(0);
  const int L = xcd_block(ln.G);
  constexpr int CH = basis_chunk<S, VEC>() < NDM ? basis_chunk<S, VEC>() : NDM;
  C nv = C(0);
  for (int it = 0; it < ln.nit; ++it) {
    const int g = (L * ln.nit + it) * TPB + threadIdx.x;
    if (g >= ln.ng) break;
    const int e = g * VEC;
    C v[VEC];
    loadv<C, S, VEC>(win + e, v);
#pragma unroll
    for (int c = 0; c < NDM; c += CH) {
      if (c < nd) {
        C vv[CH][VEC];
#pragma unroll
        for (int k = 0; k < CH; ++k)
          loadv<C, S, VEC>(V + (size_t)min(c + k, nd - 1) * vstride + e, vv[k]);
#pragma unroll
        for (int k = 0; k < CH; ++k) {
          if (c + k < NDM) {
#pragma unroll
            for (int q = 0; q < VEC; ++q) v[q] -= a[c + k] * vv[k][q];
          }
        }
      }
    }
#pragma unroll
    for (int q = 0; q < VEC; ++q) {
      v[q] = rnd<S, C>(v[q]);
      nv += v[q] * v[q];
    }
  }
  double acc[1] = {(double)nv};
  __shared__ double tot[1];
  if (!reduce_to_last<1>(acc, 1, red, L, ln.G, tot)) return;
  if (threadIdx.x == 0) {
    const double beta = sqrt(tot[0] * cfg.invN);
    double* col = ctl->H + J * (MAXM + 1);
    for (int i = 0; i <= J; ++i) col[i] = ctl->hcol[i];
    const double zc = ctl->zc;
    ctl->vscale[J + 1] = beta > 0.0 ? 1.0 / beta : 0.0;
    gm_complete_column(ctl, cfg, J, zc > 0.0 ? beta / zc : 0.0);
  }
}

// End of a GMRES cycle: y += scale * BJ(sum_{i<J} ysol_i v_i) ; one LP pass done.  The J x J
// triangular least-squares system is solved here by every block (J <= 32), so a cycle the
// host ends early (fewer iterations enqueued than the device would run) is still promoted.
// NDM bounds J: the host passes the number of Arnoldi steps it enqueued in this cycle.
template <typename S, typename C, int VEC, int BS, int NDM, int AD, int FL>
__global__ __launch_bounds__(TPB) void k_gm_finish(Launch ln, double* __restrict__ y,
                                                   const S* __restrict__ V, size_t vstride,
                                                   BJ<S> dinv, Ctl* ctl) {
  if (ctl->outer_done) return;
  const int J = ctl->J;
  count_work(ctl, KC_GM_FINISH, J);
  const double sc = ctl->scale;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (ctl->passes < MAXPASS) ctl->pass_iters[ctl->passes] = ctl->iters;
    ctl->passes += 1;
    ctl->life_passes += 1;
  }
  if (J == 0) return;
  if (J > NDM) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      ctl->nonfinite = 1;
      ctl->step_nonfinite = 1;
    }
    return;
  }
  __shared__ double ys[MAXM];
  if (threadIdx.x == 0) {
    for (int i = J - 1; i >= 0; --i) {
      double acc = ctl->g[i];
      for (int k = i + 1; k < J; ++k) acc -= ctl->H[k * (MAXM + 1) + i] * ys[k];
      const double d = ctl->H[i * (MAXM + 1) + i];
      ys[i] = (d != 0.0 && __builtin_isfinite(acc)) ? acc / d : 0.0;
    }
  }
  __syncthreads();
  C cf[NDM];
#pragma unroll
  for (int i = 0; i < NDM; ++i) cf[i] = i < J ? (C)(ys[i] * ctl->vscale[i]) : C(0);
  const int L = xcd_block(ln.G);
  constexpr int CH = basis_chunk<S, VEC>() < NDM ? basis_chunk<S, VEC>() : NDM;
  for (int it = 0; it < ln.nit; ++it) {
    const int g = (L * ln.nit + it) * TPB + threadIdx.x;
    const bool valid = g < ln.ng;
    const int e = valid ? g * VEC : 0;  // an invalid lane reads group 0 and discards it
    // independent loads first: the first chunk of basis vectors (J >= 1), the block-Jacobi
    // rows and y
    Vec<S, VEC> v0[CH];
#pragma unroll
    for (int k = 0; k < CH; ++k)
      v0[k] = *reinterpret_cast<const Vec<S, VEC>*>(V + (size_t)min(k, J - 1) * vstride + e);
    BJRows<S, VEC, bj_early<S, VEC, BS>() ? BS : 1> R;
    if constexpr (bj_early<S, VEC, BS>()) bj_load<S, VEC, BS, AD>(dinv, e, valid, R);
    double yv[VEC];
    loadg<double, double, VEC, FL>(y, e, ln.n, yv);
    C t[VEC], zv[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) t[v] = C(0);
#pragma unroll
    for (int k = 0; k < CH; ++k) {  // cf is zero past J
#pragma unroll
      for (int v = 0; v < VEC; ++v) t[v] += cf[k] * (C)v0[k].v[v];
    }
#pragma unroll
    for (int c = CH; c < NDM; c += CH) {
      if (c < J) {
        C vv[CH][VEC];
#pragma unroll
        for (int k = 0; k < CH; ++k)
          loadv<C, S, VEC>(V + (size_t)min(c + k, J - 1) * vstride + e, vv[k]);
#pragma unroll
        for (int k = 0; k < CH; ++k) {
          if (c + k < NDM) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) t[v] += cf[c + k] * vv[k][v];
          }
        }
      }
    }
#pragma unroll
    for (int v = 0; v < VEC; ++v) t[v] = valid ? t[v] : C(0);
    if constexpr (BS > 0) {
      if constexpr (bj_early<S, VEC, BS>()) bj_mul<C, S, VEC, BS, AD>(dinv, e, R, valid, t, zv);
      else bj_apply_lane<C, S, VEC, BS, AD>(dinv, e, valid, t, zv);
    } else {
#pragma unroll
      for (int v = 0; v < VEC; ++v) zv[v] = t[v];
    }
    if (valid) {
#pragma unroll
      for (int v = 0; v < VEC; ++v) yv[v] += sc * (double)zv[v];
      storeg<double, double, VEC, FL>(y, e, ln.n, yv);
    }
  }
}

// ------------------------------------------------------------------------------------------
// Setup (not on the timed path)
// ------------------------------------------------------------------------------------------

// Deterministic non-constant fill (autotuner test state): x[i] = sin(a i) + 0.5 cos(b i).
static __global__ void k_fill_pattern(long n, double a, double b, double* __restrict__ x) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] = sin(a * (double)i) + 0.5 * cos(b * (double)i);
}

// In-place Gauss-Jordan inverse of an n x n (n <= BJ_MAX) matrix with partial pivoting.
__host__ __device__ inline int gj_invert(double (&a)[BJ_MAX][BJ_MAX], double (&inv)[BJ_MAX][BJ_MAX], int n) {
  for (int i = 0; i < BJ_MAX; ++i)
    for (int k = 0; k < BJ_MAX; ++k) inv[i][k] = (i == k) ? 1.0 : 0.0;
  for (int col = 0; col < n; ++col) {
    int piv = col;
    double best = fabs(a[col][col]);
    for (int i = col + 1; i < n; ++i)
      if (fabs(a[i][col]) > best) {
        best = fabs(a[i][col]);
        piv = i;
      }
    if (!(best > 0.0)) return 1;
    if (piv != col)
      for (int k = 0; k < BJ_MAX; ++k) {
        double t = a[col][k];
        a[col][k] = a[piv][k];
        a[piv][k] = t;
        t = inv[col][k];
        inv[col][k] = inv[piv][k];
        inv[piv][k] = t;
      }
    const double d = 1.0 / a[col][col];
    for (int k = 0; k < BJ_MAX; ++k) {
      a[col][k] *= d;
      inv[col][k] *= d;
    }
    for (int i = 0; i < n; ++i) {
      if (i == col) continue;
      const double f = a[i][col];
      if (f == 0.0) continue;
      for (int k = 0; k < BJ_MAX; ++k) {
        a[i][k] -= f * a[col][k];
        inv[i][k] -= f * inv[col][k];
      }
    }
  }
  return 0;
}

// Row i of slot blk's inverse goes to chunk blk * BS + i (lay == 0) or to its place in the
// interleaved layout for lanes of `lay` rows (lay = 1, 4 or 8).
template <typename S>
__device__ inline void bj_store(S* dinv, int blk, int BS, int n, const double (&inv)[BJ_MAX][BJ_MAX],
                                int lay) {
  for (int i = 0; i < BS; ++i) {
    const int r = blk * BS + i;
    const size_t chunk = lay == 8 ? bj_chunk<8>(r) : lay == 4 ? bj_chunk<4>(r)
                       : lay == 1 ? bj_chunk<1>(r) : (size_t)r;
    for (int k = 0; k < BS; ++k) {
      double v = (i < n && k < n) ? inv[i][k] : (i == k ? 1.0 : 0.0);
      dinv[chunk * BS + k] = (S)v;
    }
  }
}

// Block blk's inverse in the adaptive-precision layout (mode 4) for lanes of `lay` rows: each
// row in its chunk's type (tag 0 FP8 E4M3, rounded to nearest even; 1 FP16, 2 FP32, 3 FP64) at
// the chunk's byte offset.
__device__ inline void bj_store_adaptive(void* base, const int* tag, const long long* aoff, int blk,
                                         int BS, int n, const double (&inv)[BJ_MAX][BJ_MAX], int lay) {
  for (int i = 0; i < BS; ++i) {
    const int r = blk * BS + i;
    const int g = r / lay, q = r % lay;
    const int ch = g >> 6;
    const size_t ent = ((size_t)q * 64 + (g & 63)) * BS;
    char* p = (char*)base + aoff[ch];
    for (int k = 0; k < BS; ++k) {
      const double v = (i < n && k < n) ? inv[i][k] : (i == k ? 1.0 : 0.0);
      if (tag[ch] == 0)
        ((unsigned char*)p)[ent + k] =
            (unsigned char)(__builtin_amdgcn_cvt_pk_fp8_f32((float)v, 0.0f, 0, false) & 0xff);
      else if (tag[ch] == 1) ((half_t*)p)[ent + k] = (half_t)v;
      else if (tag[ch] == 2) ((float*)p)[ent + k] = (float)v;
      else ((double*)p)[ent + k] = v;
    }
  }
}

// The rows past the last block that the last lane's group of `lay` rows still covers (blocks smaller
// than a group) are stored as zero: such a lane multiplies them by zero inputs, which whatever lay
// in the workspace could turn into NaN.  tag == nullptr: the layouts of bj_store.
template <typename S>
__device__ inline void bj_store_tail(S* dinv, const int* tag, const long long* aoff, int nblk, int BS,
                                     int lay) {
  const int per = tag && lay == 1 ? 64 : lay;  // (mode 4 with lay = 1 serves groups of any width)
  if (per < 1) return;
  for (int r = nblk * BS; r % per != 0; ++r) {
    if (tag) {
      const int g = r / lay, q = r % lay;
      const int ch = g >> 6;
      const int eb = 1 << tag[ch];  // bytes per entry
      char* p = (char*)dinv + aoff[ch] + ((size_t)q * 64 + (g & 63)) * BS * eb;
      for (int k = 0; k < BS * eb; ++k) p[k] = 0;
    } else {
      const size_t chunk = lay == 8 ? bj_chunk<8>(r) : lay == 4 ? bj_chunk<4>(r) : bj_chunk<1>(r);
      for (int k = 0; k < BS; ++k) dinv[chunk * BS + k] = (S)0;
    }
  }
}

// Diagonal blocks of M = I - sigma K for the stencil operator (Mc = stencil of M in FP64).
// Slot i receives the inverse of block reps[i] (reps == nullptr: block i, stored in the
// layout `lay`), so the per-block table and the table of distinct blocks come from the same
// arithmetic.
template <typename S>
__global__ void k_bj_setup_stencil(int nslot, int BS, Geo geo, Coef<double> Mc, S* dinv,
                                   int* fail, const int* reps, int lay, const int* atag,
                                   const long long* aoff) {
  const int slot = blockIdx.x * blockDim.x + threadIdx.x;
  if (slot >= nslot) return;
  const int blk = reps ? reps[slot] : slot;
  const int r0 = blk * BS;
  const int n = min(BS, geo.N - r0);
  double a[BJ_MAX][BJ_MAX], inv[BJ_MAX][BJ_MAX];
  for (int i = 0; i < BJ_MAX; ++i)
    for (int k = 0; k < BJ_MAX; ++k) a[i][k] = 0.0;
  for (int i = 0; i < n; ++i) {
    const int row = r0 + i;
    const Nbr nb = neighbours<1>(geo, row);
    a[i][i] += Mc.c;
    const int idx[6] = {nb.xm, nb.xp, nb.ym, nb.yp, nb.zm, nb.zp};
    const double cf[6] = {Mc.xm, Mc.xp, Mc.ym, Mc.yp, Mc.zm, Mc.zp};
    for (int d = 0; d < 6; ++d) {
      const int c = idx[d];
      if (c >= r0 && c < r0 + n) a[i][c - r0] += cf[d];
    }
  }
  if (gj_invert(a, inv, n)) atomicOr(fail, 1);
  if (atag) bj_store_adaptive(dinv, atag, aoff, slot, BS, n, inv, lay);
  else bj_store<S>(dinv, slot, BS, n, inv, reps ? 0 : lay);
  if (!reps && slot == nslot - 1) bj_store_tail<S>(dinv, atag, aoff, nslot, BS, lay);
}

// Diagonal blocks of M = I - sigma K from the FP64 CSR values of K (slots as above).
template <typename S>
__global__ void k_bj_setup_csr(int nslot, int BS, int N, Csr csr, const double* kval, double sigma,
                               S* dinv, int* fail, const int* reps, int lay, const int* atag,
                               const long long* aoff) {
  const int slot = blockIdx.x * blockDim.x + threadIdx.x;
  if (slot >= nslot) return;
  const int blk = reps ? reps[slot] : slot;
  const int r0 = blk * BS;
  const int n = min(BS, N - r0);
  double a[BJ_MAX][BJ_MAX], inv[BJ_MAX][BJ_MAX];
  for (int i = 0; i < BJ_MAX; ++i)
    for (int k = 0; k < BJ_MAX; ++k) a[i][k] = (i == k && i < n) ? 1.0 : 0.0;
  for (int i = 0; i < n; ++i) {
    const int row = r0 + i;
    for (int k = csr.rowptr[row]; k < csr.rowptr[row + 1]; ++k) {
      const int c = csr.col[k];
      if (c >= r0 && c < r0 + n) a[i][c - r0] -= sigma * kval[k];
    }
  }
  if (gj_invert(a, inv, n)) atomicOr(fail, 1);
  if (atag) bj_store_adaptive(dinv, atag, aoff, slot, BS, n, inv, lay);
  else bj_store<S>(dinv, slot, BS, n, inv, reps ? 0 : lay);
  if (!reps && slot == nslot - 1) bj_store_tail<S>(dinv, atag, aoff, nslot, BS, lay);
}

// LP copy of the CSR values of K, scaled by a power of two into [-1, 1].
template <typename S>
__global__ void k_csr_lp_values(long nnz, const double* __restrict__ kval, double inv_kscale,
                                S* __restrict__ out) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nnz) out[i] = (S)(kval[i] * inv_kscale);
}

}  // namespace mprk
