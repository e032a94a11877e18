// One implicit stage of a small CG problem in one launch: the FP64 residual loop around the
// preconditioned CG of kernels.hpp, with exchanges between workgroups in place of kernel
// boundaries.
//
// A small grid is bound by waits, not by bytes: a reducing kernel of the per-kernel path takes
// about 5 us (launch, one memory round trip, the reduction's ticket) plus a gap, an iteration
// needs two, and the host waits for the device's decision at every stage's end.  Here an
// iteration costs two exchanges and one read of z, and the host waits once per call.  Each
// workgroup keeps its part of x, r and q in registers, and the search direction on its part and
// the planes beside it in LDS, where p = z + beta p is formed again from z, so z is all that
// travels.  Three workgroups to a CU by registers (FP32 117 to 131, FP64 140 to 168) and LDS; gate.hpp
// keeps what waits for each other within what the device holds.
//
// A step of heat with SDIRK3 and block-Jacobi (8), per-kernel path -> here: FP32 8^3 440 -> 105 us,
// 16^3 505 -> 200, 37^3 840 -> 545, 50^3 1020 -> 740; FP64 8^3 465 -> 120, 27^3 875 -> 640,
// 50^3 1380 -> 1130.
// With a counter barrier, p and q in memory and caches invalidated at each barrier 37^3 took 902.
#pragma once

#include "group.hpp"
#include "kernels.hpp"

namespace mprk {

struct StagePlan {
  int nwg;    // workgroups (co-resident), 0: the per-kernel path
  int chunk;  // unknowns per workgroup, a multiple of 64 (block-Jacobi blocks never straddle)
  int slab;   // most unknowns of a workgroup's part and the planes beside it
};

constexpr int STAGE_WGS_PER_CU = 3;   // by registers and LDS
constexpr int STAGE_PART = 4 * TPB;   // a workgroup's part: one group of four unknowns per thread
constexpr int STAGE_SLAB_MAX = 6500;  // FP64 values, so that three workgroups' slabs fit a CU's LDS

// Stencil input from the slab in LDS: unknowns o .. of the grid, around its end where periodic.
template <typename C, int VEC>
struct InSlab {
  static constexpr int pin = 0;
  const C* lds;
  int o, N;
  __device__ __forceinline__ int at(int i) const {
    int l = i - o;
    l += l < 0 ? N : 0;
    return l >= N ? l - N : l;
  }
  __device__ __forceinline__ void uvec(int i, C (&v)[VEC]) const {
    const C* p = lds + at(i);
#pragma unroll
    for (int k = 0; k < VEC; ++k) v[k] = p[k];
  }
  __device__ __forceinline__ void vec(int i, C (&v)[VEC]) const { uvec(i, v); }
  __device__ __forceinline__ C one(int i) const { return lds[at(i)]; }
};

// Every value of the slab [o, o + L) of src, four at a time, to put(place, values); up to U groups'
// loads of a thread in flight together.
template <typename S, int T, bool DEV, typename F>
__device__ __forceinline__ void read_slab(const S* src, int N, int o, int L, const F& put) {
  constexpr int U = sizeof(S) == 8 ? 2 : 4;
  const DevVec<S> d(src, N);
  for (int i0 = (int)threadIdx.x * 4; i0 < L; i0 += U * 4 * T) {
    S v[U][4];
    int g[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * 4 * T;
      g[u] = o + (i < L ? i : i0);
      if (g[u] < 0) g[u] += N;
      if (g[u] >= N) g[u] -= N;
      if constexpr (DEV) d.template vec<4>(g[u], v[u]);
      else loadg<S, S, 4, 1>(src, g[u], N, v[u]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * 4 * T;
      if (i >= L) break;
      if (DEV && g[u] + 4 > N && i + N - g[u] < L) {  // around the end of the grid
#pragma unroll
        for (int k = 0; k < 4; ++k) v[u][k] = d.one(g[u] + k < N ? g[u] + k : g[u] + k - N);
      }
      put(i, v[u]);
    }
  }
}

// y: start value in, solution out (N values, element aligned); rhs, kout: FP64 vectors of the
// workspace; z: an LP vector of it, padded to whole groups.  slot: record of the stage's final head
// (srec), or >= MAXSTG for none.  part: nwg > 1: 3 GRP_ND nwg slots, EMPTY before the launch.
// Dynamic LDS: slab + 4 FP64 values.
template <typename S, typename C, int BS, bool many>
__global__ __launch_bounds__(TPB, STAGE_WGS_PER_CU) void k_cg_stage(
    StagePlan pl, Geo geo, Coef<double> K, double* y, const double* __restrict__ rhs, double* kout, S* z,
    BJ<S> dinv, FTerms fx, SolveCfg cfg, Ctl* ctl, double* part, int slot) {
  if (ctl->outer_done) return;  // (a halted call: uniform over the grid, written before the launch)
  constexpr int VEC = 4, T = TPB;
  extern __shared__ double stage_lds[];
  double* yl = stage_lds;
  C* pd = reinterpret_cast<C*>(stage_lds);
  const int N = geo.N;
  const int wl = blockIdx.x;
  const int r0 = wl * pl.chunk;
  const int r1 = min(N, r0 + pl.chunk);
  int o = 0, L = N;
  if (many && pl.slab < N) {
    o = r0 - geo.plane;
    L = r1 + geo.plane - o;
    if (geo.bc == 0) {
      o = max(o, 0);
      L = min(N, r1 + geo.plane) - o;
    }
  }
  const int e = r0 + (int)threadIdx.x * VEC;
  const bool valid = e < r1;
  const bool lead = wl == 0 && threadIdx.x == 0;
  int epoch = 0;
  auto reduce = [&](auto& a, auto& t) {
    constexpr int ND = sizeof(a) / sizeof(double);
    if constexpr (many) {
      group_exchange<ND, T>(a, (unsigned long long*)part, &ctl->bar, pl.nwg, wl, epoch, t);
    } else {
      int parity = 0;
      group_reduce<ND, T>(a, part, &ctl->bar, 1, 0, parity, t);
    }
  };
  auto store_z = [&](const C (&v)[VEC]) {
    if constexpr (many) store_shared_group<S, C, VEC>(z + r0, e - r0, pl.chunk, v);
    else storev<S, C, VEC>(z + e, v);
  };
  const Coef<C> M = coef_cast<C>(coef_stage(K, cfg.sigma));
  int passes = 0;
  bool inner_conv = false;
  const int maxp = cfg.paper_mode ? 1 : cfg.max_passes;
  for (;;) {
    // ---- FP64 residual: k = K y (+ g + R(y)) ; res = rhs - y + sigma k ----
    double acc[3] = {0.0, 0.0, 0.0};
    double rs[VEC], b[VEC], fv[VEC];
    const int el = valid ? e : r0;
    loadg<double, double, VEC, 1>(rhs, el, N, b);
    if (fx.g) loadg<double, double, VEC, 1>(fx.g, el, N, fv);
    read_slab<double, T, many>(y, N, o, L, [&](int i, const double (&v)[4]) {
#pragma unroll
      for (int k = 0; k < 4; ++k) yl[i + k] = v[k];
    });
    __syncthreads();
    if (valid) {
      double yc[VEC], ky[VEC];
      const InSlab<double, VEC> f{yl, o, N};
      int eh = e;
      asm volatile("" : "+v"(eh));
      stencil_group<double, VEC, 1>(geo, K, eh, f, yc, ky);
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        if (fx.g) ky[v] += fv[v];
        if (fx.react) ky[v] += fx.R(yc[v]);
        rs[v] = b[v] - yc[v] + cfg.sigma * ky[v];
        acc[0] += rs[v] * rs[v];
        acc[1] += b[v] * b[v];
        acc[2] += (__builtin_isfinite(rs[v]) && __builtin_isfinite(ky[v])) ? 0.0 : 1.0;
      }
      storeg<double, double, VEC, 1>(kout, e, N, ky);
    } else {
#pragma unroll
      for (int v = 0; v < VEC; ++v) rs[v] = 0.0;
    }
    double t[3];
    reduce(acc, t);
    const double rn = sqrt(t[0]), bn = sqrt(t[1]);
    const double rel = bn > 0.0 ? rn / bn : rn;
    if (lead) residual_decision(t, cfg, ctl);
    if (t[2] != 0.0 || !__builtin_isfinite(rn) || !__builtin_isfinite(bn)) break;
    if (cfg.paper_mode ? passes >= 1 : (rel <= cfg.outer_tol || passes >= maxp || rn == 0.0)) break;
    const double scale = rn > 0.0 ? rn / cfg.sqrtN : 1.0;
    const double inv = 1.0 / scale;
    // ---- r = LP(res / scale), z = BJ(r) ----
    C rr[VEC], xx[VEC], pp[VEC], qq[VEC];
    double a2[2] = {0.0, 0.0};
    // z = BJ(r) (r itself without one), its part of (r, z) and (r, r).  (A thread's rows of the
    // inverse and its neighbours' places are the same in every iteration, but kept over the loop
    // they spill: the opaque copies have each iteration form them again.  FP64 with blocks of 8 spills
    // 10 to 12 registers all the same.)
    auto precondition = [&]() {
      C zv[VEC];
      if constexpr (BS > 0) {
        BJRows<S, VEC, BS> rows;
        BJ<S> d = dinv;
        asm volatile("" : "+s"(d.inv));
        bj_load<S, VEC, BS, 2>(d, e, valid, rows);
        bj_mul<C, S, VEC, BS, 2>(dinv, e, rows, valid, rr, zv);
        if (valid) store_z(zv);
      } else {
        if (valid) store_z(rr);
      }
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        if constexpr (BS > 0) a2[0] += valid ? (double)(rr[v] * zv[v]) : 0.0;
        a2[1] += (double)(rr[v] * rr[v]);
      }
    };
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      rr[v] = rnd<S, C>((C)(rs[v] * inv));
      xx[v] = C(0);
    }
    precondition();
    double t2[2];
    reduce(a2, t2);
    double rz = BS > 0 ? t2[0] : t2[1];
    const double tol = fmax(fmax(cfg.rtol * sqrt(t2[1]), cfg.atol / scale),
                            cfg.outer_stop ? 0.5 * cfg.outer_tol * bn / scale : 0.0);
    inner_conv = sqrt(t2[1]) <= tol;
    bool inner_done = inner_conv || cfg.maxit <= 0;
    double beta = 0.0;
    int its = 0;
    while (!inner_done) {
      // ---- p = z + beta p ; q = M p ; (p, q) ----
      const C bt = (C)beta;
      read_slab<S, T, many>(z, N, o, L, [&](int i, const S (&v)[4]) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          pd[i + k] = its > 0 ? rnd_fma<S, C>(bt, pd[i + k], (C)v[k]) : (C)v[k];
      });
      __syncthreads();
      double a1[1] = {0.0};
      if (valid) {
        const InSlab<C, VEC> f{pd, o, N};
        int eh = e;
        asm volatile("" : "+v"(eh));
        stencil_group<C, VEC, 1, S>(geo, M, eh, f, pp, qq);
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
          qq[v] = rnd<S, C>(qq[v]);
          a1[0] += (double)(pp[v] * qq[v]);
        }
      } else {
#pragma unroll
        for (int v = 0; v < VEC; ++v) pp[v] = qq[v] = C(0);
      }
      double t1[1];
      reduce(a1, t1);
      const double pq = t1[0];
      if (!(pq > 0.0) || !__builtin_isfinite(pq)) {  // breakdown: keep the current iterate
        inner_conv = false;
        break;
      }
      const C alpha = (C)(rz / pq);
      // ---- x += alpha p ; r -= alpha q ; z = BJ(r) ; (r, z), (r, r) ----
      a2[0] = a2[1] = 0.0;
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        xx[v] = its == 0 ? alpha * pp[v] : xx[v] + alpha * pp[v];
        rr[v] = rnd_fma<S, C>(-alpha, qq[v], rr[v]);
      }
      precondition();
      reduce(a2, t2);
      ++its;
      const double rzn = BS > 0 ? t2[0] : t2[1];
      beta = rzn / rz;
      rz = rzn;
      const bool fin = __builtin_isfinite(t2[1]) && __builtin_isfinite(rz);
      inner_conv = fin && sqrt(t2[1]) <= tol;
      inner_done = !fin || inner_conv || its >= cfg.maxit;
    }
    // ---- y += scale x ----
    if (its > 0 && valid) {
      double yv[VEC];
      loadg<double, double, VEC, 1>(y, e, N, yv);  // (this thread's own last values)
#pragma unroll
      for (int v = 0; v < VEC; ++v) yv[v] += scale * (double)xx[v];
      if constexpr (!many) {
        storeg<double, double, VEC, 1>(y, e, N, yv);
      } else {
#pragma unroll
        for (int v = 0; v < VEC; ++v)
          if (e + v < N) store_shared(y + e + v, yv[v]);
      }
    }
    if (lead) {
      if (passes < MAXPASS) ctl->pass_iters[passes] = its;
      ctl->iters = its;
      ctl->total_iters += its;
      ctl->life_iters += its;
      ctl->life_passes += 1;
      ctl->inner_conv = inner_conv;
      ctl->passes = passes + 1;
    }
    ++passes;
    if constexpr (many) {  // y complete before the next residual
      const double none[1] = {0.0};
      double u[1];
      reduce(none, u);
    } else {
      __syncthreads();
    }
  }
  if (lead && slot < MAXSTG) {
    const long long* head = reinterpret_cast<const long long*>(ctl);
#pragma unroll
    for (int i = 0; i < 8; ++i) ctl->srec[slot][i] = head[i];
  }
}

}  // namespace mprk
