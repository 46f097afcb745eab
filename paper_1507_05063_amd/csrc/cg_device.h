// Device helpers shared by the CG sweep kernels and of the one-launch solves.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "excmg_internal.h"

namespace excmg {

namespace {

constexpr int kXcds = 8;

// Bijection from the hardware workgroup id to a logical tile id such that logical ids [x*per, (x+1)*per) run on XCD x.
__device__ __forceinline__ int xcd_remap(int b, int nb) {
  const int per = nb / kXcds, rem = nb % kXcds;
  const int x = b % kXcds, l = b / kXcds;
  const int start = (x < rem) ? x * (per + 1) : rem * (per + 1) + (x - rem) * per;
  return start + l;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Tile shape of the stencil sweeps (x is the fast axis: one wavefront covers one 64-node row segment).
constexpr int TX = 64;
__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// Loads and stores of data a sweep touches once: non-temporal (streaming) when NTP, so that they do not displace the
// operand's halo lines, which neighbouring tiles read again, from the caches.
template <bool NTP, typename T>
__device__ __forceinline__ T ld1(const T *p) {
  if constexpr (NTP) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool NTP, typename T>
__device__ __forceinline__ void st1(T v, T *p) {
  if constexpr (NTP) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// f(integral_constant<int, 0>), ..., f(integral_constant<int, N - 1>), in that order
template <typename F, int... Q>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, Q...>) {
  (f(std::integral_constant<int, Q>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// a node of a plane by its byte offset there (32 bits: the launchers refuse larger planes), so that a load is one
// uniform base and one 32-bit offset
template <typename T>
__device__ __forceinline__ T *at_byte(T *plane, unsigned off) {
  return reinterpret_cast<T *>(reinterpret_cast<std::conditional_t<std::is_const_v<T>, const char, char> *>(plane) +
                               off);
}

// p, known to point to global memory (the compiler cannot tell for a pointer that is itself read from memory, and takes
// the slower flat instructions)
template <typename T>
__device__ __forceinline__ T *as_global(T *p) {
  return (T *)(__attribute__((address_space(1))) T *)p;
}

template <typename T>
__device__ __forceinline__ T *at_plane(T *a, unsigned bytes, unsigned k) {
  using C = std::conditional_t<std::is_const_v<T>, const char, char>;
  return reinterpret_cast<T *>(reinterpret_cast<C *>(a) + (unsigned long long)bytes * k);
}

// Sums of K values over the whole grid of a launch (or one problem's nb workgroups), in the workgroup that finishes
// last: every workgroup writes its partials past the XCD's own L2 (agent-scope stores), waits for them and counts
// itself in; the last one to do so reads all partials the same way and adds them in workgroup order.  Only the
// values themselves are coherent; nothing else is fenced (an agent-scope fence writes back the XCD's L2).  This saves
// the separate reduction launch.  True in every thread of the last workgroup, tot valid in thread 0; the count is
// back at 0 then.
template <int K, int NTB>
__device__ __forceinline__ bool last_sums(double (&v)[K], double *parts, unsigned *count, int bid, int nb,
                                          double (&tot)[K]) {
  constexpr int NW = NTB / 64;
  __shared__ double sh[K][NW];
  __shared__ int last;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const double x = wave_sum(v[k]);
    if (lane == 0) sh[k][w] = x;
  }
  __syncthreads();
  // lane k < K of the first wave adds the waves' sums of value k
  auto waves = [&]() {
    double x = 0.0;
    if (lane < K) {
#pragma unroll 1
      for (int q = 0; q < NW; ++q) x += sh[lane][q];
    }
    return x;
  };
  if (threadIdx.x < 64) {
    const double x = waves();
    if (lane < K)
      __hip_atomic_store(&parts[(long long)lane * nb + bid], x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (lane == 0)
      last = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)nb - 1;
  }
  __syncthreads();
  if (!last) return false;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    double x = 0.0;
    for (int q = threadIdx.x; q < nb; q += NTB)
      x += __hip_atomic_load(&parts[(long long)k * nb + q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    x = wave_sum(x);
    if (lane == 0) sh[k][w] = x;
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    const double x = waves();
#pragma unroll
    for (int k = 0; k < K; ++k) tot[k] = __shfl(x, k, 64);
    if (lane == 0) __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  return true;
}

// entry e of a batched launch; nothing writes the tables while a kernel runs, so its fields are read as constants
// (scalar loads)
__device__ __forceinline__ const BatchEntry &entry_at(const BatchList &L, int e) {
  typedef const BatchEntry *P;
  const P p = *(const P *)(__attribute__((address_space(4))) const P *)(L.ent + e);
  return *(const BatchEntry *)(__attribute__((address_space(4))) const BatchEntry *)p;
}

// entry of flattened workgroup b: the largest e with pre[e] <= b (entries with no workgroups have pre[e] = pre[e+1])
__device__ __forceinline__ int find_entry(const int *pre, int n, int b) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (pre[mid] <= b) lo = mid;
    else hi = mid;
  }
  return lo;
}

// copy of a CG state's scalars for the host; the finest grid's completion time is stamped once
__device__ __forceinline__ void mirror(const BatchEntry &E, const CgState *cs, BatchStatus *stat, int slot, bool final_state) {
  BatchMirror &m = stat[E.problem].m[slot];
  m.done = cs->done;
  m.iter = cs->iter;
  m.status = cs->status;
  m.abort = cs->abort;
  m.rho = cs->rho;
  m.bnorm2 = cs->bnorm2;
  m.rho0 = cs->rho0;
  m.stop2 = cs->stop2;
  if (final_state && E.finest && cs->done && !cs->abort && stat[E.problem].t_done == 0)
    stat[E.problem].t_done = (long long)wall_clock64();
}

}  // namespace

}  // namespace excmg
