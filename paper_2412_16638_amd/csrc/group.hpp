// Several workgroups on one solve inside one launch: data exchange, barrier and reduction (the
// batched stage kernel and the single-problem one).  All workgroups of a group must be
// co-resident; every barrier wait is bounded (a timeout raises an error flag and the kernel still
// runs to its end).
#pragma once

#include "device.hpp"

namespace mprk {

constexpr int GRP_ND = 4;             // most values of one group reduction
constexpr int GRP_WGS = 128;          // most workgroups of a group exchange
constexpr long BAR_SPIN_LIMIT = 1L << 22;

// Data one workgroup writes and another reads inside a stage launch (the stencil inputs y, p
// and z, and the reduction partials) are written with device-scope stores, which are coherent
// across the XCDs once complete.  A barrier therefore needs no L2 writeback: every wave waits
// for its own stores to complete before its workgroup arrives, and after the barrier every wave
// invalidates its non-coherent cached lines (agent-scope acquire) before reading other
// workgroups' rows.  Data a thread writes and only the same thread reads back (its own rows of
// r, x, q, res, rhs, k) stay plain stores.
template <typename T>
__device__ __forceinline__ void store_shared(T* p, T v) {
  if constexpr (sizeof(T) == 2) {
    unsigned short b;
    __builtin_memcpy(&b, &v, 2);
    __hip_atomic_store(reinterpret_cast<unsigned short*>(p), b, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  } else {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// The group at element e of a workgroup's chunk, which starts at `base` (uniform over the wave) and
// holds `chunk` elements: device-scope stores of 16 bytes where a group has them (8-byte atomic
// stores would each write half of every 16 bytes through to memory).
template <typename S, typename C, int VEC>
__device__ __forceinline__ void store_shared_group(S* base, int e, int chunk, const C (&o)[VEC]) {
  constexpr int B = sizeof(S) * VEC;
  Vec<S, VEC> t;
#pragma unroll
  for (int v = 0; v < VEC; ++v) t.v[v] = (S)o[v];
  if constexpr (B % 16 == 0) {
    typedef unsigned quad __attribute__((ext_vector_type(4)));
    constexpr int SC1 = 16;  // cache policy: device scope
    quad w[B / 16];
    __builtin_memcpy(w, &t, B);
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(base, 0, chunk * (int)sizeof(S), 0x00020000);
#pragma unroll
    for (int i = 0; i < B / 16; ++i)
      __builtin_amdgcn_raw_buffer_store_b128(w[i], rs, e * (int)sizeof(S) + 16 * i, 0, SC1);
  } else if constexpr (B == 8) {
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(base + e),
                       __builtin_bit_cast(unsigned long long, t), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else {
#pragma unroll
    for (int v = 0; v < VEC; ++v) store_shared(base + e + v, (S)o[v]);
  }
}

__device__ __forceinline__ void wait_own_stores() {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(0);
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

__device__ __forceinline__ unsigned int load_u32_dev(const unsigned int* p) {
  return __hip_atomic_load(const_cast<unsigned int*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Barrier over a group's nwg workgroups (generation counter; bounded spin).
__device__ __forceinline__ void group_barrier(GroupBar* c, int nwg) {
  if (nwg > 1) wait_own_stores();
  __syncthreads();
  if (nwg > 1) {
    if (threadIdx.x == 0) {
      // the generation is read (and the read completed) before this arrival is counted
      const unsigned gen = load_u32_dev(&c->gen);
      wait_own_stores();
      const unsigned arrived = __hip_atomic_fetch_add(&c->count, 1u, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT);
      if (arrived == (unsigned)nwg - 1u) {
        __hip_atomic_store(&c->count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        wait_own_stores();  // the reset is visible before the next generation opens
        __hip_atomic_fetch_add(&c->gen, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else {
        // Polls go to the line that arrivals are counted on, so a large group must not poll hard:
        // with s_sleep(1) one 28^3 problem on 343 workgroups takes 5.14 ms for two FP32 steps, with
        // 2 4.73; FP64 36^3 on 365 8.4 and 7.2 ms.  Groups of 8 are as fast either way (0.44 ms).
        long spins = 0;
        while (load_u32_dev(&c->gen) == gen) {
          __builtin_amdgcn_s_sleep(2);
          if (++spins > BAR_SPIN_LIMIT) {
            __hip_atomic_store(&c->error, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            break;
          }
        }
      }
    }
    __syncthreads();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
}

// Group reduction of ND values over workgroups of T threads; every workgroup returns the same
// totals.  Each publishes its partials (device-scope stores), passes the group barrier, then
// sums all the group's partials itself in workgroup order (every thread a strided slice of all
// values at once, fixed shuffle tree and wave order), so all workgroups take identical decisions
// without a second round trip.  Partials (2 GRP_ND nwg values) are double-buffered by `parity`
// (a fast workgroup may publish the next reduction's partials while a slow one reads these).
template <int ND, int T>
__device__ __forceinline__ void group_reduce(const double (&v)[ND], double* part0, GroupBar* bar, int nwg,
                                             int wl, int& parity, double (&out)[ND]) {
  static_assert(ND <= GRP_ND, "the partials hold GRP_ND values");
  constexpr int NW = T / 64;
  __shared__ double wsum[NW][ND];
  __shared__ double wt[NW][ND];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int d = 0; d < ND; ++d) {
    const double s = wave_sum(v[d]);
    if (lane == 0) wsum[wave][d] = s;
  }
  __syncthreads();
  if (nwg == 1) {
#pragma unroll
    for (int d = 0; d < ND; ++d) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) s += wsum[w][d];
      out[d] = s;
    }
    __syncthreads();  // the next reduction writes the wave sums again
    return;
  }
  double* part = part0 + (size_t)parity * GRP_ND * nwg;
  if (threadIdx.x < ND) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) s += wsum[w][threadIdx.x];
    store_dev(part + (size_t)threadIdx.x * nwg + wl, s);
  }
  group_barrier(bar, nwg);
  double s[ND];
#pragma unroll
  for (int d = 0; d < ND; ++d) s[d] = 0.0;
#pragma unroll 1
  for (int w = threadIdx.x; w < nwg; w += T) {
#pragma unroll
    for (int d = 0; d < ND; ++d) s[d] += load_dev(part + (size_t)d * nwg + w);
  }
#pragma unroll
  for (int d = 0; d < ND; ++d) {
    const double t = wave_sum(s[d]);
    if (lane == 0) wt[wave][d] = t;
  }
  __syncthreads();
#pragma unroll
  for (int d = 0; d < ND; ++d) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += wt[w][d];
    out[d] = t;
  }
  parity ^= 1;  // (the next write of wt is behind the next barrier)
}

// A vector of n values that other workgroups write inside the launch, read at device scope (past
// this XCD's caches): no cache has to be invalidated between two phases, so what a workgroup
// reads back of its own stays in them.
template <typename S>
struct DevVec {
  __amdgpu_buffer_rsrc_t rs;
  __device__ __forceinline__ DevVec(const S* p, int n)
      : rs(__builtin_amdgcn_make_buffer_rsrc(const_cast<S*>(p), 0, n * (int)sizeof(S), 0x00020000)) {}
  static constexpr int SC1 = 16;  // cache policy: device scope
  template <int VEC>
  __device__ __forceinline__ void vec(int i, S (&o)[VEC]) const {
    typedef unsigned quad __attribute__((ext_vector_type(4)));
    constexpr int B = sizeof(S) * VEC;
    static_assert(B % 16 == 0, "whole 16-byte loads");
    quad w[B / 16];
#pragma unroll
    for (int k = 0; k < B / 16; ++k)
      w[k] = __builtin_amdgcn_raw_buffer_load_b128(rs, i * (int)sizeof(S) + 16 * k, 0, SC1);
    __builtin_memcpy(o, w, B);
  }
  __device__ __forceinline__ S one(int i) const {
    if constexpr (sizeof(S) == 8) {
      typedef unsigned pair __attribute__((ext_vector_type(2)));
      const pair w = __builtin_amdgcn_raw_buffer_load_b64(rs, i * 8, 0, SC1);
      return __builtin_bit_cast(S, w);
    } else {
      return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b32(rs, i * 4, 0, SC1));
    }
  }
};

// Exchange of ND values over up to GRP_WGS workgroups in one round trip, barrier and reduction at once.
// A workgroup publishes its partials once its data stores have completed; every workgroup's first
// wave polls the partials themselves (two workgroups per lane), which read as EMPTY until published,
// and adds them in a fixed order.  Three buffers of slots: exchange e uses buffer e % 3; when it
// is complete every workgroup is past reading buffer (e - 1) % 3, whose slots (all GRP_ND: that
// exchange may have had more values) their owners then empty for exchange e + 2; that is completed
// before they publish e + 1, which every reader of e + 2 has seen.  All slots are EMPTY before the
// launch.  A counter to arrive at, a generation to poll and partials to read afterwards would take
// four dependent trips to memory.

__device__ __forceinline__ unsigned long long load_u64_dev(const unsigned long long* p) {
  return __hip_atomic_load(const_cast<unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_u64_dev(unsigned long long* p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int ND, int T>
__device__ __forceinline__ void group_exchange(const double (&v)[ND], unsigned long long* slots, GroupBar* bar,
                                               int nwg, int wl, int& epoch, double (&out)[ND]) {
  static_assert(ND <= GRP_ND, "the slots hold GRP_ND values");
  constexpr int NW = T / 64;
  __shared__ double wsum[NW][ND];
  __shared__ double tot[ND];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int d = 0; d < ND; ++d) {
    const double s = wave_sum(v[d]);
    if (lane == 0) wsum[wave][d] = s;
  }
  wait_own_stores();
  __syncthreads();
  if (wave == 0) {
    unsigned long long* cur = slots + (size_t)(epoch % 3) * GRP_ND * nwg;
    unsigned long long* old = slots + (size_t)((epoch + 2) % 3) * GRP_ND * nwg;
    if (lane < ND) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) s += wsum[w][lane];
      unsigned long long b = __builtin_bit_cast(unsigned long long, s);
      if (b == GRP_EMPTY) b = 0x7ff8000000000000ULL;
      store_u64_dev(cur + lane * nwg + wl, b);
    }
    constexpr int PL = GRP_WGS / 64;
    unsigned long long b[ND][PL];
    bool wait = lane < nwg;
#pragma unroll
    for (int d = 0; d < ND; ++d)
#pragma unroll
      for (int k = 0; k < PL; ++k) b[d][k] = 0;
    for (long spins = 0; __any(wait); ++spins) {
      if (spins > BAR_SPIN_LIMIT) {
        __hip_atomic_store(&bar->error, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
      if (wait) {
        bool all = true;
#pragma unroll
        for (int d = 0; d < ND; ++d)
#pragma unroll
          for (int k = 0; k < PL; ++k)
            if (lane + 64 * k < nwg) b[d][k] = load_u64_dev(cur + d * nwg + lane + 64 * k);
#pragma unroll
        for (int d = 0; d < ND; ++d)
#pragma unroll
          for (int k = 0; k < PL; ++k) all = all && b[d][k] != GRP_EMPTY;
        wait = !all;
      }
    }
#pragma unroll
    for (int d = 0; d < ND; ++d) {
      double s = 0.0;
#pragma unroll
      for (int k = 0; k < PL; ++k) s += __builtin_bit_cast(double, b[d][k]);
      s = wave_sum(s);
      if (lane == 0) tot[d] = s;
    }
    if (lane < GRP_ND) store_u64_dev(old + lane * nwg + wl, GRP_EMPTY);
  }
  __syncthreads();
#pragma unroll
  for (int d = 0; d < ND; ++d) out[d] = tot[d];
  ++epoch;
  __syncthreads();  // the next exchange writes tot and wsum again
}

}  // namespace mprk
