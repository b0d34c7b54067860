// Dual bound (Eq. (3)), per-iteration dual traces, primal rounding (Eq. (5))
// and energy (Eq. (1)) of MPLP++ on gfx950, plus small utility kernels.
//
// The certified dual bound is recomputed from the input costs and the
// messages, never from the incrementally updated unaries:
//   node term  min_s [theta_u(s) + sum_{e incident to u} phi_{e->u}(s)]
//   edge term  min_{s,t} [theta_e(s,t) - phi_e[0](s) - phi_e[1](t)]
// with every sum in FP64 (Eq. (2) and Eq. (3)).  All reductions use a fixed
// order, so the result is deterministic.
#include <algorithm>

#include "device_common.h"
#include "dual_terms.h"

namespace mplpxx {

// fixed-order block reduction of one double per thread (blockDim power of 2)
template <int NT, bool kMin>
__device__ __forceinline__ double block_reduce(double v, double* sh) {
  const int tid = threadIdx.x;
  sh[tid] = v;
  __syncthreads();
#pragma unroll
  for (int s = NT / 2; s >= 1; s >>= 1) {
    if (tid < s) sh[tid] = kMin ? dmin(sh[tid], sh[tid + s]) : sh[tid] + sh[tid + s];
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

// th(s, t) of the edge in `slot`: its table, or, for structured costs (their
// parameters per slot), the expanded table entry
template <typename T>
__device__ __forceinline__ T table_at(const T* tables, int slot, int L, int s, int t, int potts) {
  if constexpr (sizeof(T) == 4) {
    if (potts) return structured_cost(potts, tables + (size_t)slot * cost_params(potts), s, t);
  }
  return tables[(size_t)slot * L * L + (size_t)s * L + t];
}

// out = sum(a[0..na)) + sum(b[0..nb)), fixed order, one workgroup for each of
// the grid's states (their terms one after another)
__global__ void __launch_bounds__(1024) k_sum2(const double* __restrict__ a, int na, const double* __restrict__ b,
                                               int nb, double* __restrict__ out) {
  __shared__ double sh[1024];
  a += (size_t)blockIdx.x * na;
  b += (size_t)blockIdx.x * nb;
  double acc = 0.0;
  for (int i = threadIdx.x; i < na; i += 1024) acc += a[i];
  for (int i = threadIdx.x; i < nb; i += 1024) acc += b[i];
  acc = block_reduce<1024, false>(acc, sh);
  if (threadIdx.x == 0) out[blockIdx.x] = acc;
}

// Node and edge terms of Eq. (3) in one launch (dual_terms.h): waves [0, n)
// take a node each, the others a slot; grid y: the state, of `states` message
// arrays one after another.
template <typename T, int V>
__global__ void __launch_bounds__(256) k_dual_terms(const T* __restrict__ unaries, const T* __restrict__ tables,
                                                    const T* __restrict__ phi, const int* __restrict__ node_ptr,
                                                    const int* __restrict__ inc, int n, int L, int m, int potts,
                                                    double* __restrict__ node_min, double* __restrict__ edge_min) {
  __shared__ T sh[4][2 * MPLPXX_MAX_LABELS];
  phi += (size_t)blockIdx.y * m * 2 * L;
  node_min += (size_t)blockIdx.y * n;
  edge_min += (size_t)blockIdx.y * m;
  const int w = uni((int)(blockIdx.x * 4 + (threadIdx.x >> 6))), lane = threadIdx.x & 63;
  if (w < n) {
    const double mn = node_term(unaries + (size_t)w * L, phi, inc, uni(node_ptr[w]), uni(node_ptr[w + 1]), L);
    if (lane == 0) node_min[w] = mn;
  } else if (w - n < m) {
    const int slot = w - n;
    const size_t step = potts ? (size_t)cost_params(potts) : (size_t)L * L;
    const double mn = edge_term<T, V>(tables + slot * step, phi + (size_t)slot * 2 * L, L, potts, sh[threadIdx.x >> 6]);
    if (lane == 0) edge_min[slot] = mn;
  }
}

template <typename T>
hipError_t launch_dual(const T* unaries, const T* tables, const T* phi, const int* node_ptr, const int* inc, int n,
                       int L, int m, double* node_min, double* edge_min, double* out, hipStream_t st, int potts,
                       int states) {
  const dim3 grid((unsigned)((n + (size_t)m + 3) / 4), (unsigned)states);
  // (a vector of 16 bytes stays inside a row, and is aligned, where its width divides L)
  constexpr int V = 16 / sizeof(T);
  if (!potts && L % V == 0)
    hipLaunchKernelGGL((k_dual_terms<T, V>), grid, dim3(256), 0, st, unaries, tables, phi, node_ptr, inc, n, L, m, potts,
                       node_min, edge_min);
  else
    hipLaunchKernelGGL((k_dual_terms<T, 1>), grid, dim3(256), 0, st, unaries, tables, phi, node_ptr, inc, n, L, m, potts,
                       node_min, edge_min);
  hipLaunchKernelGGL(k_sum2, dim3(states), dim3(1024), 0, st, node_min, n, edge_min, m, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Traces: sum_u min_s U_u(s) in FP64 per iteration.
// ---------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(64) k_trace_nodes(const T* __restrict__ U, const T* __restrict__ Ulo, int L,
                                                    double* __restrict__ row) {
  const int u = blockIdx.x;
  double mn = __builtin_inf();
  for (int s = threadIdx.x; s < L; s += 64) {
    const size_t i = (size_t)u * L + s;
    mn = dmin(mn, (double)U[i] + (Ulo ? (double)Ulo[i] : 0.0));
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) mn = dmin(mn, __shfl_xor(mn, o, 64));
  if (threadIdx.x == 0) row[u] = mn;
}

template <typename T>
hipError_t launch_trace_nodes(const T* U, const T* Ulo, int n, int L, double* row, hipStream_t st) {
  hipLaunchKernelGGL(k_trace_nodes<T>, dim3(n), dim3(64), 0, st, U, Ulo, L, row);
  return hipGetLastError();
}

// Edge terms of Eq. (3) for the trace of one iteration: out[slot] =
// min_{s,t} [theta(s,t) - phi[0](s) - phi[1](t)] in FP64, stored as FP32 (the
// FP32 engines' terms are rounding-level numbers, far inside FP32 range).
template <typename T>
__global__ void __launch_bounds__(256) k_trace_edges(const T* __restrict__ tables, const T* __restrict__ phi, int L,
                                                     float* __restrict__ out) {
  __shared__ double sh[256];
  const int slot = blockIdx.x;
  const T* tab = tables + (size_t)slot * L * L;
  const T* p0 = phi + (size_t)slot * 2 * L;
  const T* p1 = p0 + L;
  double mn = __builtin_inf();
  for (int i = threadIdx.x; i < L * L; i += 256) {
    const int s = i / L, t = i - s * L;
    mn = dmin(mn, ((double)tab[i] - (double)p0[s]) - (double)p1[t]);
  }
  mn = block_reduce<256, true>(mn, sh);
  if (threadIdx.x == 0) out[slot] = (float)mn;
}

template <typename T>
hipError_t launch_trace_edges(const T* tables, const T* phi, int m, int L, float* out, hipStream_t st) {
  if (m <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_trace_edges<T>, dim3(m), dim3(256), 0, st, tables, phi, L, out);
  return hipGetLastError();
}

// One workgroup per iteration: sum of the node minima (nodes without edges
// keep their input unary) plus, when trace_e is given, the edge terms (the
// minimum over the W partial minima of each slot), in a fixed order.
template <typename T>
__global__ void __launch_bounds__(256) k_trace_sum(const double* __restrict__ trace_nodes,
                                                   const float* __restrict__ trace_e, int m, int W,
                                                   const T* __restrict__ U, const int* __restrict__ deg, int n, int L,
                                                   double* __restrict__ out) {
  __shared__ double sh[256];
  const int it = blockIdx.x;
  double acc = 0.0;
  for (int u = threadIdx.x; u < n; u += 256) {
    double v;
    if (deg[u] > 0) {
      v = trace_nodes[(size_t)it * n + u];
    } else {
      v = __builtin_inf();
      for (int s = 0; s < L; ++s) v = dmin(v, (double)U[(size_t)u * L + s]);
    }
    acc += v;
  }
  if (trace_e) {
    for (int e = threadIdx.x; e < m; e += 256) {
      const float* w = trace_e + ((size_t)it * m + e) * W;
      float v = w[0];
      for (int k = 1; k < W; ++k) v = __builtin_fminf(v, w[k]);
      acc += (double)v;
    }
  }
  acc = block_reduce<256, false>(acc, sh);
  if (threadIdx.x == 0) out[it] = acc;
}

template <typename T>
hipError_t launch_trace_sum(double* trace_nodes, const float* trace_e, int m, int W, const T* U, const int* deg, int n,
                            int L, int iters, double* out, hipStream_t st) {
  if (iters <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_trace_sum<T>, dim3(iters), dim3(256), 0, st, trace_nodes, trace_e, m, W, U, deg, n, L, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Primal rounding, Eq. (5), and energy, Eq. (1).
//
// Eq. (5) labels the nodes in ascending order, each after its lower
// neighbours.  k_decode gives every node a workgroup of its own and lets the
// labels themselves order them: a workgroup reads everything that does not
// depend on a label at once, polls the labels of its lower neighbours, and
// reads the table row a label selects as soon as that label is there.  Nodes
// without an edge between them run side by side, and on a complete graph only
// the newest label's row is on the chain from one node to the next (it comes
// from a copy of that edge's table in LDS).  What bounds it is that chain: one
// label store, one poll, one sum and one minimum per dependent node, 1.7 us on
// a complete graph of 200 nodes and 64 labels (one workgroup walking the
// nodes took 14 us a node there, its reads one after another).  Whole calls,
// before and after: that graph 2966 -> 405 us, 1000 nodes of degree 50 at 16
// labels 4874 -> 233 us, 20 nodes at 8 labels 101 -> 98 us.  Sleeping between
// polls only made the chain longer (405 -> 418 us with s_sleep 1).
//
// Nodes are numbered by an arrival ticket, so a workgroup only waits for
// workgroups that have started: the launch needs no co-residency.
//
// Several states of one model (one message array after another) are labelled
// in one launch, the tickets taking node 0 of every state, then node 1 of
// every state: their chains run side by side.
//
// Sums are in FP64 and in one order whatever the graph: wave w sums the
// incidences w, w+16, ... of the node (lane = label), and the 16 partial sums
// are added in wave order after the reparametrized unary.
// ---------------------------------------------------------------------------
constexpr int kDecW = 16;               // waves per node = partial sums
// nodes of a launch (the threads of one are a 32-bit number: 2^22 - 1 nodes at most)
constexpr int kDecodeLaunch = 1 << 21;
constexpr size_t kDecStage = 44 * 1024;  // largest table copied to LDS (with the partial sums within 64 KB)

__global__ void k_decode_init(int* __restrict__ labels, int n, int* __restrict__ ticket) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) labels[i] = -1;
  if (i == 0) *ticket = 0;
}

// PER: labels per lane (1 up to 64 labels, 2 up to 128); B: incidences a wave
// holds in registers at once (all of its share up to degree 16 B)
template <typename T, int PER, int B>
__global__ void __launch_bounds__(kDecW * 64) k_decode(const T* __restrict__ unaries, const T* __restrict__ tables,
                                                       const T* __restrict__ phi, const SlotInfo* __restrict__ slots,
                                                       const int* __restrict__ node_ptr, const int* __restrict__ inc,
                                                       int n, int L, int m, int states, int potts, int stage,
                                                       int* __restrict__ labels, int* __restrict__ ticket, int* __restrict__ err,
                                                       long long spin_limit) {
  static_assert(B <= 64, "one lane polls each incidence of a block");
  __shared__ double part[kDecW][64 * PER];
  __shared__ int s_u, s_near, s_near_slot;
  extern __shared__ __align__(16) unsigned char dec_lds[];
  T* near_phi = reinterpret_cast<T*>(dec_lds);  // [L], then the table [L][L]
  T* near_tab = near_phi + L;
  const int tid = threadIdx.x;
  const int w = tid >> 6, lane = tid & 63;
  if (tid == 0) {
    s_u = atomicAdd(ticket, 1);
    s_near = -1;
    s_near_slot = -1;
  }
  __syncthreads();
  const int t = uni(s_u);
  const int u = uni(t / states), state = t - u * states;
  phi += (size_t)state * m * 2 * L;
  labels += (size_t)state * n;
  const int k0 = uni(node_ptr[u]), k1 = uni(node_ptr[u + 1]);
  const int deg = k1 - k0;
  {
    // the largest lower neighbour is (on dense graphs) the last to be
    // labelled: what its label selects from goes to LDS before it is known
    int nb = -1;
    for (int k = k0 + tid; k < k1; k += kDecW * 64) {
      const int code = inc[k];
      if (code & 1) nb = max(nb, slots[code >> 1].u);
    }
    if (nb >= 0) atomicMax(&s_near, nb);
    __syncthreads();
    for (int k = k0 + tid; k < k1; k += kDecW * 64) {
      const int code = inc[k];
      if ((code & 1) && slots[code >> 1].u == s_near) s_near_slot = code >> 1;
    }
    __syncthreads();
    if (s_near_slot >= 0) {
      for (int i = tid; i < L; i += kDecW * 64) near_phi[i] = phi[(size_t)s_near_slot * 2 * L + i];
      if (stage) {
        const T* src = tables + (size_t)s_near_slot * L * L;
        for (int i = tid; i < L * L; i += kDecW * 64) near_tab[i] = src[i];
      }
    }
    __syncthreads();
  }
  const int near_slot = uni(s_near_slot);
  double acc[PER], un[PER];
#pragma unroll
  for (int c = 0; c < PER; ++c) {
    acc[c] = 0.0;
    un[c] = (double)unaries[(size_t)u * L + min(lane + 64 * c, L - 1)];
  }
  // this wave's incidences w, w + 16, ... in blocks of B
  for (int k = k0 + w; k < k1; k += kDecW * B) {
    const int cnt = min(B, (k1 - k + kDecW - 1) / kDecW);
    // lane i holds incidence i of the block: its code, and the lower
    // neighbour whose label it needs (-1: none, u is the lower node)
    int code_v = 0, nbr_v = -1;
    if (lane < cnt) {
      code_v = inc[k + lane * kDecW];
      if (code_v & 1) nbr_v = slots[code_v >> 1].u;
    }
    T msg[B][PER], th[B][PER], py[B];
#pragma unroll
    for (int i = 0; i < B; ++i) {
      if (i < cnt) {
        const int code = __builtin_amdgcn_readlane(code_v, i);
        const T* p = phi + (size_t)(code >> 1) * 2 * L + (size_t)(code & 1) * L;
#pragma unroll
        for (int c = 0; c < PER; ++c) msg[i][c] = p[min(lane + 64 * c, L - 1)];
      }
    }
    unsigned long long want = __ballot(nbr_v >= 0);
    long long spins = 0;
    while (want) {
      int y_v = -1;
      if ((want >> lane) & 1) y_v = ld_dev(labels + nbr_v);
      unsigned long long got = __ballot(y_v >= 0);
      if (!got) {
        if (++spins > spin_limit || ((spins & 255) == 0 && ld_dev(err) != 0)) {
          // (the call fails; label 0 lets every other wait end)
          if (lane == 0 && spins > spin_limit) report_timeout(err, -1, u, 0, 0);
          y_v = 0;
          got = want;
        } else {
          continue;
        }
      }
#pragma unroll
      for (int i = 0; i < B; ++i) {
        if ((got >> i) & 1) {
          const int slot = __builtin_amdgcn_readlane(code_v, i) >> 1;
          const int y = __builtin_amdgcn_readlane(y_v, i);
          const bool near = slot == near_slot;
          py[i] = near ? near_phi[y] : phi[(size_t)slot * 2 * L + y];
#pragma unroll
          for (int c = 0; c < PER; ++c) {
            const int x = min(lane + 64 * c, L - 1);
            th[i][c] = near && stage ? near_tab[y * L + x] : table_at(tables, slot, L, y, x, potts);
          }
        }
      }
      want &= ~got;
    }
    // in incidence order: the message into u (part of its reparametrized
    // unary, Eq. 2), then theta^phi_{vu}(x*_v, x) of a lower neighbour v
#pragma unroll
    for (int i = 0; i < B; ++i) {
      if (i < cnt) {
        const bool lower = __builtin_amdgcn_readlane(code_v, i) & 1;
#pragma unroll
        for (int c = 0; c < PER; ++c) {
          acc[c] += (double)msg[i][c];
          if (lower) acc[c] += (double)th[i][c] - (double)py[i] - (double)msg[i][c];
        }
      }
    }
  }
#pragma unroll
  for (int c = 0; c < PER; ++c) part[w][lane + 64 * c] = acc[c];
  __syncthreads();
  if (w != 0) return;
  // cost and argmin over labels; ties go to the smallest label (the exact
  // minimum first, then the first lane that holds it)
  double v[PER], best = __builtin_inf();
#pragma unroll
  for (int c = 0; c < PER; ++c) {
    const int x = lane + 64 * c;
    v[c] = un[c];
#pragma unroll
    for (int ww = 0; ww < kDecW; ++ww) v[c] += part[ww][x];
    if (x < L) best = dmin(best, v[c]);
  }
  best = wave_min64(best);
  int arg = 0;
#pragma unroll
  for (int c = PER - 1; c >= 0; --c) {
    const unsigned long long at = __ballot(lane + 64 * c < L && v[c] == best);
    if (at) arg = 64 * c + __ffsll((unsigned long long)at) - 1;
  }
  if (lane == 0) st_dev(labels + u, arg);
}

// the terms of the energy of Eq. (1): node u's unary and slot's pairwise cost
// at the labelling
template <typename T>
__global__ void __launch_bounds__(256) k_energy_terms(const T* __restrict__ unaries, const T* __restrict__ tables,
                                                      const SlotInfo* __restrict__ slots,
                                                      const int* __restrict__ labels, int n, int L, int m, int potts,
                                                      double* __restrict__ node_e, double* __restrict__ edge_e) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  labels += (size_t)blockIdx.y * n;
  node_e += (size_t)blockIdx.y * n;
  edge_e += (size_t)blockIdx.y * m;
  if (i < (size_t)n) {
    node_e[i] = (double)unaries[i * L + labels[i]];
  } else if (i - n < (size_t)m) {
    const int slot = (int)(i - n);
    edge_e[slot] = (double)table_at(tables, slot, L, labels[slots[slot].u], labels[slots[slot].v], potts);
  }
}

template <typename T>
hipError_t launch_decode(const T* unaries, const T* tables, const T* phi, const SlotInfo* slots, const int* node_ptr,
                         const int* inc, int n, int L, int m, int* labels, int* ticket, double* node_e, double* edge_e,
                         double* energy, int* err, long long spin_limit, hipStream_t st, int potts, int states) {
  const int all = n * states;
  hipLaunchKernelGGL(k_decode_init, dim3((unsigned)(((size_t)all + 255) / 256)), dim3(256), 0, st, labels, all, ticket);
  const size_t tab = (size_t)L * L * sizeof(T);
  const int stage = !potts && m > 0 && tab <= kDecStage;
  const size_t dyn = L * sizeof(T) + (stage ? tab : 0);
  constexpr int B1 = sizeof(T) == 4 ? 16 : 8;
  // (the tickets run on from one launch to the next)
  for (int left = all; left > 0; left -= kDecodeLaunch) {
    const dim3 grid(std::min(left, kDecodeLaunch));
    if (L <= 64)
      hipLaunchKernelGGL((k_decode<T, 1, B1>), grid, dim3(kDecW * 64), dyn, st, unaries, tables, phi, slots,
                         node_ptr, inc, n, L, m, states, potts, stage, labels, ticket, err, spin_limit);
    else
      hipLaunchKernelGGL((k_decode<T, 2, B1 / 2>), grid, dim3(kDecW * 64), dyn, st, unaries, tables, phi, slots,
                         node_ptr, inc, n, L, m, states, potts, stage, labels, ticket, err, spin_limit);
  }
  hipLaunchKernelGGL(k_energy_terms<T>, dim3((unsigned)(((size_t)n + m + 255) / 256), states), dim3(256), 0, st, unaries,
                     tables, slots, labels, n, L, m, potts, node_e, edge_e);
  hipLaunchKernelGGL(k_sum2, dim3(states), dim3(1024), 0, st, node_e, n, edge_e, m, energy);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Utilities: finiteness check of device inputs, table packing from a device
// copy in the caller's layout, integer fill (used instead of memset so that
// the same code can sit inside captured graphs).
// ---------------------------------------------------------------------------
template <typename T>
__global__ void k_check_finite(const T* __restrict__ p, size_t count, int* __restrict__ flag) {
  bool bad = false;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < count; i += (size_t)gridDim.x * blockDim.x)
    bad |= sizeof(T) == 4 ? !(__builtin_fabs((double)p[i]) <= MPLPXX_F32_MAX_COST) : !__builtin_isfinite(p[i]);
  if (bad) atomicOr(flag, 1);
}

template <typename T>
hipError_t launch_check_finite(const T* p, size_t count, int* flag, hipStream_t st) {
  if (count == 0) return hipSuccess;
  size_t blocks = (count + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_check_finite<T>, dim3((unsigned)blocks), dim3(256), 0, st, p, count, flag);
  return hipGetLastError();
}

// dst slot i <- src edge slot_edge[i], transposed when slot_flip[i]
template <typename S, typename D>
__global__ void __launch_bounds__(256) k_pack_tables(const S* __restrict__ src, D* __restrict__ dst,
                                                     const int* __restrict__ slot_edge,
                                                     const int* __restrict__ slot_flip, int L) {
  const int slot = blockIdx.x;
  const S* s = src + (size_t)slot_edge[slot] * L * L;
  D* d = dst + (size_t)slot * L * L;
  const bool flip = slot_flip[slot] != 0;
  for (int i = threadIdx.x; i < L * L; i += 256) {
    const int r = i / L, c = i - r * L;
    d[i] = (D)(flip ? s[(size_t)c * L + r] : s[i]);
  }
}

template <typename S, typename D>
hipError_t launch_pack_tables(const S* src, D* dst, const int* slot_edge, const int* slot_flip, int m, int L,
                              hipStream_t st) {
  if (m == 0) return hipSuccess;
  hipLaunchKernelGGL((k_pack_tables<S, D>), dim3(m), dim3(256), 0, st, src, dst, slot_edge, slot_flip, L);
  return hipGetLastError();
}
template hipError_t launch_pack_tables<float, float>(const float*, float*, const int*, const int*, int, int, hipStream_t);
template hipError_t launch_pack_tables<double, double>(const double*, double*, const int*, const int*, int, int, hipStream_t);
template hipError_t launch_pack_tables<double, float>(const double*, float*, const int*, const int*, int, int, hipStream_t);

// messages in the caller's edge order from slot order
template <typename T>
__global__ void __launch_bounds__(128) k_phi_by_edge(const T* __restrict__ phi_slot, const int* __restrict__ slot_of_edge,
                                                     int m, int row, T* __restrict__ out) {
  for (size_t e = blockIdx.x; e < (size_t)m; e += gridDim.x) {
    const T* src = phi_slot + (size_t)slot_of_edge[e] * row;
    for (int i = threadIdx.x; i < row; i += 128) out[e * row + i] = src[i];
  }
}

template <typename T>
hipError_t launch_phi_by_edge(const T* phi_slot, const int* slot_of_edge, int m, int L, T* out, hipStream_t st) {
  if (m <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_phi_by_edge<T>, dim3(stride_blocks(m)), dim3(128), 0, st, phi_slot, slot_of_edge, m, 2 * L, out);
  return hipGetLastError();
}

__global__ void k_fill_int(int* __restrict__ p, int value, size_t count) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < count; i += (size_t)gridDim.x * blockDim.x)
    p[i] = value;
}

template <typename S, typename D>
__global__ void k_convert(const S* __restrict__ src, D* __restrict__ dst, size_t count) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < count; i += (size_t)gridDim.x * blockDim.x)
    dst[i] = (D)src[i];
}

hipError_t launch_convert(const float* src, double* dst, size_t count, hipStream_t st) {
  if (count == 0) return hipSuccess;
  const size_t blocks = std::min<size_t>((count + 255) / 256, 4096);
  hipLaunchKernelGGL((k_convert<float, double>), dim3((unsigned)blocks), dim3(256), 0, st, src, dst, count);
  return hipGetLastError();
}

hipError_t launch_convert(const double* src, float* dst, size_t count, hipStream_t st) {
  if (count == 0) return hipSuccess;
  const size_t blocks = std::min<size_t>((count + 255) / 256, 4096);
  hipLaunchKernelGGL((k_convert<double, float>), dim3((unsigned)blocks), dim3(256), 0, st, src, dst, count);
  return hipGetLastError();
}

hipError_t launch_fill_int(int* p, int value, size_t count, hipStream_t st) {
  if (count == 0) return hipSuccess;
  size_t blocks = (count + 255) / 256;
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(k_fill_int, dim3((unsigned)blocks), dim3(256), 0, st, p, value, count);
  return hipGetLastError();
}

#define MPLPXX_INST(T)                                                                                              \
  template hipError_t launch_dual<T>(const T*, const T*, const T*, const int*, const int*, int, int, int, double*,  \
                                     double*, double*, hipStream_t, int, int);                                    \
  template hipError_t launch_trace_nodes<T>(const T*, const T*, int, int, double*, hipStream_t);                             \
  template hipError_t launch_trace_edges<T>(const T*, const T*, int, int, float*, hipStream_t);               \
  template hipError_t launch_trace_sum<T>(double*, const float*, int, int, const T*, const int*, int, int, int,   \
                                          double*, hipStream_t);     \
  template hipError_t launch_decode<T>(const T*, const T*, const T*, const SlotInfo*, const int*, const int*, int, \
                                       int, int, int*, int*, double*, double*, double*, int*, long long,           \
                                       hipStream_t, int, int);                                                     \
  template hipError_t launch_phi_by_edge<T>(const T*, const int*, int, int, T*, hipStream_t);                      \
  template hipError_t launch_check_finite<T>(const T*, size_t, int*, hipStream_t);
MPLPXX_INST(float)
MPLPXX_INST(double)
#undef MPLPXX_INST

}  // namespace mplpxx
