// Terms of the dual bound, Eq. (3), recomputed from the input costs and the
// messages in FP64, one wave each:
//   node term  min_s [theta_u(s) + sum_{e incident to u} phi_{e->u}(s)]
//   edge term  min_{s,t} [theta_e(s,t) - phi_e[0](s) - phi_e[1](t)]
// A node's sum runs over its incidences in slot order; minima are exact and
// order-free.  Both are bound by memory: the edge terms read every table
// once (16 bytes a load where rows allow), a node's messages are read 16
// incidences at a time.  On 200 nodes and 64 labels (326 MB of tables) the two
// took 123 and 63 us in launches of their own, one entry and one incidence at
// a time; mplpxx_dual_bound took 246 us there and takes 114 us, some 45 of
// them the call's copies and waits.
#pragma once
#include "device_common.h"

namespace mplpxx {

__device__ __forceinline__ double dmin(double a, double b) { return __builtin_fmin(a, b); }

// exact minimum over the 64 lanes
__device__ __forceinline__ double wave_min64(double x) {
  x = row16_min(x);
  {
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    x = dmin(dbl_of(lo[0], hi[0]), dbl_of(lo[1], hi[1]));
  }
  const unsigned long long b = (unsigned long long)__double_as_longlong(x);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
  return dmin(dbl_of(lo[0], hi[0]), dbl_of(lo[1], hi[1]));
}

template <typename T>
__device__ __forceinline__ double node_term(const T* __restrict__ unary, const T* __restrict__ phi,
                                            const int* __restrict__ inc, int k0, int k1, int L) {
  constexpr int B = 16;
  const int lane = threadIdx.x & 63;
  double mn = __builtin_inf();
  for (int x0 = 0; x0 < L; x0 += 64) {
    const int x = min(x0 + lane, L - 1);
    double acc = (double)unary[x];
    for (int kb = k0; kb < k1; kb += 64) {
      const int code_v = inc[min(kb + lane, k1 - 1)];
      const int cnt = min(64, k1 - kb);
      for (int j = 0; j < cnt; j += B) {
        T v[B];
#pragma unroll
        for (int i = 0; i < B; ++i) {
          const int code = __builtin_amdgcn_readlane(code_v, min(j + i, 63));
          v[i] = phi[(size_t)code * L + x];  // (code = 2 slot + side)
        }
#pragma unroll
        for (int i = 0; i < B; ++i) acc = j + i < cnt ? acc + (double)v[i] : acc;
      }
    }
    mn = dmin(mn, acc);
  }
  return wave_min64(mn);
}

// tab: the slot's table, or its parameters (potts: the cost kind); ph its
// messages; sh: 2 L values of LDS of this wave.  V entries a load (V divides
// L; V = 1 for structured costs).
template <typename T, int V>
__device__ __forceinline__ double edge_term(const T* __restrict__ tab, const T* __restrict__ ph, int L, int potts, T* sh) {
  const int lane = threadIdx.x & 63;
  for (int i = lane; i < 2 * L; i += 64) sh[i] = ph[i];
  wave_sync();
  // entries V lane, V (lane + 64), ...: position (s, t) advanced without
  // divisions
  const int ds = 64 * V / L, dt = 64 * V - ds * L;
  int s = V * lane / L, t = V * lane - s * L;
  double mn = __builtin_inf();
  const int total = L * L;
#pragma unroll 4
  for (int i = V * lane; i < total; i += 64 * V) {
    T x[V];
    if (V == 1 && sizeof(T) == 4 && potts) {
      x[0] = (T)structured_cost(potts, reinterpret_cast<const float*>(tab), s, t);
    } else {
#pragma unroll
      for (int k = 0; k < V; ++k) x[k] = tab[i + k];
    }
#pragma unroll
    for (int k = 0; k < V; ++k) mn = dmin(mn, (double)x[k] - (double)sh[s] - (double)sh[L + t + k]);
    s += ds;
    t += dt;
    if (t >= L) {
      t -= L;
      ++s;
    }
  }
  return wave_min64(mn);
}

}  // namespace mplpxx
