// Adjoint (reverse mode) of K unrolled MPLP++ iterations.
//
// Loss: D_K = sum_u min_s U_u(s) after K iterations from phi = 0.  After an
// edge's (H) update its reparametrized pairwise term theta - r - q has row
// minima 0 (Sec. 4, after (H)), so it stays identically 0 under small input
// changes and the dual bound of Eq. (3) reduces to the node terms.
//
// Forward of one update (three-minimization form of (H)), with the argmin
// records the reverse needs (lowest index on ties); in FP32 the unaries are
// updated with the same compensated sum as in the other engines, which
// changes no derivative:
//   p(s) = min_t [th(s,t) + a_v(t)]   t1(s) = argmin
//   b(s) = (a_u(s) - p(s)) / 2
//   q(t) = min_s [th(s,t) + b(s)]     s2(t) = argmin
//   r(s) = min_t [th(s,t) - q(t)]     t3(s) = argmin
//   phi0' = r, phi1' = q, U_u' = a_u + r, U_v' = a_v + q,
//   a_u = U_u - phi0, a_v = U_v - phi1.
// Reverse, given the adjoints Ub_u', Ub_v' of the new unaries and pb0', pb1'
// of the new messages:
//   rb = pb0' + Ub_u',  qb = pb1' + Ub_v'
//   r:  thb(s, t3(s)) += rb(s);  qb(t3(s)) -= rb(s)
//   q:  thb(s2(t), t) += qb(t);  bb(s2(t)) += qb(t)
//   b:  ab_u = Ub_u' + bb / 2;   pb = -bb / 2
//   p:  thb(s, t1(s)) += pb(s);  ab_v = Ub_v' + sum over s with t1(s)=t of pb(s)
//   Ub_u = ab_u, pb0 = -ab_u, Ub_v = ab_v, pb1 = -ab_v.
// Every scatter is done by one thread per target in ascending index order, so
// the result is deterministic.  Per-matching kernels: one workgroup per
// edge, one launch per matching (the edges of a matching are independent in
// reverse as forward).  Persistent FP64 kernels (L <= 64, below): one launch
// per segment, with the same arithmetic in the same order.
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "host_util.h"
#include "mailbox64.h"

namespace mplpxx {

template <typename T> __device__ __forceinline__ T inf_of();
template <> __device__ __forceinline__ float inf_of<float>() { return __builtin_inff(); }
template <> __device__ __forceinline__ double inf_of<double>() { return __builtin_inf(); }

constexpr int kAdjNT = 256;

// Forward of one matching with argmin records: rec[slot][0..L) = t1,
// [L..2L) = s2, [2L..3L) = t3.  Same values, bit for bit, as the other engines
// (each entry one IEEE add, exact minimum).
template <typename T>
__global__ void __launch_bounds__(kAdjNT) k_step_record(const T* __restrict__ tables, T* __restrict__ phi,
                                                        T* __restrict__ U, T* __restrict__ Ulo,
                                                        const SlotInfo* __restrict__ slots, int L, int slot_begin,
                                                        unsigned char* __restrict__ rec) {
  constexpr bool kComp = std::is_same<T, float>::value;
  __shared__ T au[MPLPXX_MAX_LABELS], av[MPLPXX_MAX_LABELS], b[MPLPXX_MAX_LABELS], q[MPLPXX_MAX_LABELS];
  __shared__ T hu[MPLPXX_MAX_LABELS], lu[MPLPXX_MAX_LABELS], ou[MPLPXX_MAX_LABELS];
  __shared__ T hv[MPLPXX_MAX_LABELS], lv[MPLPXX_MAX_LABELS], ov[MPLPXX_MAX_LABELS];
  __shared__ T cuv[2];
  const int slot = slot_begin + blockIdx.x;
  const SlotInfo si = slots[slot];
  const T* th = tables + (size_t)slot * L * L;
  T* ph = phi + (size_t)slot * 2 * L;
  T* Uu = U + (size_t)si.u * L;
  T* Uv = U + (size_t)si.v * L;
  unsigned char* rc = rec + (size_t)slot * 3 * L;
  const int tid = threadIdx.x;
  T delta = T(0);
  if constexpr (!kComp) {
    for (int i = tid; i < L; i += kAdjNT) {
      au[i] = Uu[i] - ph[i];
      av[i] = Uv[i] - ph[L + i];
    }
  } else {
    // centred passes, as in the other FP32 engines (device_common.h)
    for (int i = tid; i < L; i += kAdjNT) {
      hu[i] = Uu[i];
      lu[i] = Ulo[(size_t)si.u * L + i];
      ou[i] = ph[i];
      hv[i] = Uv[i];
      lv[i] = Ulo[(size_t)si.v * L + i];
      ov[i] = ph[L + i];
    }
    __syncthreads();
    const int wave = tid >> 6, lane = tid & 63;
    if (wave < 2) {
      const T* h = wave == 0 ? hu : hv;
      T c = inf_of<T>();
      for (int i = lane; i < L; i += 64) c = vmin(c, h[i]);
      c = col4_min(row16_min(c));
      if (lane == 0) cuv[wave] = c;
    }
    __syncthreads();
    for (int i = tid; i < L; i += kAdjNT) {
      au[i] = ((hu[i] - cuv[0]) + lu[i]) - ou[i];
      av[i] = ((hv[i] - cuv[1]) + lv[i]) - ov[i];
    }
    delta = T(0.5) * (cuv[0] - cuv[1]);
  }
  __syncthreads();
  for (int s = tid; s < L; s += kAdjNT) {  // pass 1
    T mn = inf_of<T>();
    int arg = 0;
    for (int t = 0; t < L; ++t) {
      const T x = th[(size_t)s * L + t] + av[t];
      if (x < mn) { mn = x; arg = t; }
    }
    b[s] = T(0.5) * (au[s] - mn);
    rc[s] = (unsigned char)arg;
  }
  __syncthreads();
  for (int t = tid; t < L; t += kAdjNT) {  // pass 2
    T mn = inf_of<T>();
    int arg = 0;
    for (int s = 0; s < L; ++s) {
      const T x = th[(size_t)s * L + t] + b[s];
      if (x < mn) { mn = x; arg = s; }
    }
    q[t] = mn;
    rc[L + t] = (unsigned char)arg;
  }
  __syncthreads();
  for (int s = tid; s < L; s += kAdjNT) {  // pass 3
    T mn = inf_of<T>();
    int arg = 0;
    for (int t = 0; t < L; ++t) {
      const T x = th[(size_t)s * L + t] - q[t];
      if (x < mn) { mn = x; arg = t; }
    }
    rc[2 * L + s] = (unsigned char)arg;
    const T rs = mn - delta;
    ph[s] = rs;
    if constexpr (kComp) comp_update(hu[s], lu[s], ou[s], rs, Uu[s], Ulo[(size_t)si.u * L + s]);
    else Uu[s] = au[s] + mn;
  }
  for (int t = tid; t < L; t += kAdjNT) {
    const T qs = q[t] + delta;
    ph[L + t] = qs;
    if constexpr (kComp) comp_update(hv[t], lv[t], ov[t], qs, Uv[t], Ulo[(size_t)si.v * L + t]);
    else Uv[t] = av[t] + q[t];
  }
}

// Reverse of one matching.  Ub [n][L] adjoints of the unaries, pb [m][2][L]
// of the messages (slot order), thb [m][L][L] accumulated table adjoints.
template <typename T>
__global__ void __launch_bounds__(kAdjNT) k_adj_step(const SlotInfo* __restrict__ slots, int L, int slot_begin,
                                                     const unsigned char* __restrict__ rec, T* __restrict__ Ub,
                                                     T* __restrict__ pb, T* __restrict__ thb) {
  __shared__ T rb[MPLPXX_MAX_LABELS], qb[MPLPXX_MAX_LABELS], bb[MPLPXX_MAX_LABELS], pbv[MPLPXX_MAX_LABELS];
  __shared__ T abu[MPLPXX_MAX_LABELS], abv[MPLPXX_MAX_LABELS];
  __shared__ unsigned char t1[MPLPXX_MAX_LABELS], s2[MPLPXX_MAX_LABELS], t3[MPLPXX_MAX_LABELS];
  const int slot = slot_begin + blockIdx.x;
  const SlotInfo si = slots[slot];
  T* Ubu = Ub + (size_t)si.u * L;
  T* Ubv = Ub + (size_t)si.v * L;
  T* p = pb + (size_t)slot * 2 * L;
  T* g = thb + (size_t)slot * L * L;
  const unsigned char* rc = rec + (size_t)slot * 3 * L;
  const int tid = threadIdx.x;
  for (int i = tid; i < L; i += kAdjNT) {
    t1[i] = rc[i];
    s2[i] = rc[L + i];
    t3[i] = rc[2 * L + i];
    rb[i] = p[i] + Ubu[i];
    qb[i] = p[L + i] + Ubv[i];
    abu[i] = Ubu[i];
    abv[i] = Ubv[i];
  }
  __syncthreads();
  // r = th(s, t3) - q(t3)
  for (int s = tid; s < L; s += kAdjNT) g[(size_t)s * L + t3[s]] += rb[s];
  for (int t = tid; t < L; t += kAdjNT) {
    T acc = qb[t];
    for (int s = 0; s < L; ++s)
      if (t3[s] == t) acc -= rb[s];
    qb[t] = acc;
  }
  __syncthreads();
  // q = th(s2, t) + b(s2)
  for (int t = tid; t < L; t += kAdjNT) g[(size_t)s2[t] * L + t] += qb[t];
  for (int s = tid; s < L; s += kAdjNT) {
    T acc = T(0);
    for (int t = 0; t < L; ++t)
      if (s2[t] == s) acc += qb[t];
    bb[s] = acc;
  }
  __syncthreads();
  // b = (a_u - p) / 2
  for (int s = tid; s < L; s += kAdjNT) {
    abu[s] += T(0.5) * bb[s];
    pbv[s] = -T(0.5) * bb[s];
  }
  __syncthreads();
  // p = th(s, t1) + a_v(t1)
  for (int s = tid; s < L; s += kAdjNT) g[(size_t)s * L + t1[s]] += pbv[s];
  for (int t = tid; t < L; t += kAdjNT) {
    T acc = abv[t];
    for (int s = 0; s < L; ++s)
      if (t1[s] == t) acc += pbv[s];
    abv[t] = acc;
  }
  __syncthreads();
  // a_u = U_u - phi0, a_v = U_v - phi1
  for (int i = tid; i < L; i += kAdjNT) {
    Ubu[i] = abu[i];
    p[i] = -abu[i];
    Ubv[i] = abv[i];
    p[L + i] = -abv[i];
  }
}

// Seed for D_K = sum_u min_s U_u: one-hot at the smallest minimizing label;
// loss partial per node in FP64 (FP32: U + Ulo, exact in FP64).
template <typename T>
__global__ void __launch_bounds__(64) k_adj_seed(const T* __restrict__ U, const T* __restrict__ Ulo, int L,
                                                 T* __restrict__ Ub, double* __restrict__ node_min) {
  const int u = blockIdx.x;
  const int lane = threadIdx.x;
  double best = __builtin_inf();
  int arg = 0x7fffffff;
  for (int s = lane; s < L; s += 64) {
    const size_t i = (size_t)u * L + s;
    const double x = (double)U[i] + (Ulo ? (double)Ulo[i] : 0.0);
    if (x < best) { best = x; arg = s; }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const double ob = __shfl_xor(best, o, 64);
    const int oa = __shfl_xor(arg, o, 64);
    if (ob < best || (ob == best && oa < arg)) { best = ob; arg = oa; }
  }
  for (int s = lane; s < L; s += 64) Ub[(size_t)u * L + s] = (s == arg) ? T(1) : T(0);
  if (lane == 0) node_min[u] = best;
}

template <typename T>
hipError_t launch_step_record(const T* tables, T* phi, T* U, T* Ulo, const SlotInfo* slots, int L, int slot_begin,
                              int count, unsigned char* rec, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_step_record<T>, dim3(count), dim3(kAdjNT), 0, st, tables, phi, U, Ulo, slots, L, slot_begin,
                     rec);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_adj_step(const SlotInfo* slots, int L, int slot_begin, int count, const unsigned char* rec, T* Ub,
                           T* pb, T* thb, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_adj_step<T>, dim3(count), dim3(kAdjNT), 0, st, slots, L, slot_begin, rec, Ub, pb, thb);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_adj_seed(const T* U, const T* Ulo, int n, int L, T* Ub, double* node_min, hipStream_t st) {
  hipLaunchKernelGGL(k_adj_seed<T>, dim3(n), dim3(64), 0, st, U, Ulo, L, Ub, node_min);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Persistent FP64 adjoint (tiles up to 64 labels): one launch per segment of
// the checkpointed run, whose workgroups reverse the segment and, beside it,
// recompute an earlier one with records where the forward kept none, instead
// of one launch per matching.  The forward role and the mailboxes are in
// mailbox64.h; the reverse runs the same slots in the opposite order, its node
// adjoints in a second set of mailboxes.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(64) k_mb64_init(const double* __restrict__ x, unsigned long long* __restrict__ mb,
                                                  int n, int L) {
  for (size_t u = blockIdx.x; u < (size_t)n; u += gridDim.x) {
    for (int s = threadIdx.x; s < L; s += 64) {
      const unsigned long long b = (unsigned long long)__double_as_longlong(x[u * L + s]);
      unsigned long long* w = mb + u * mb64_row_words(L) + 2 * s;
      w[0] = b & 0xffffffffull;
      w[1] = b >> 32;
    }
  }
}
// values back; trace_row: their minimum per node
__global__ void __launch_bounds__(64) k_mb64_fini(double* __restrict__ x, const unsigned long long* __restrict__ mb,
                                                  int n, int L, double* __restrict__ trace_row) {
  for (size_t u = blockIdx.x; u < (size_t)n; u += gridDim.x) {
    double mn = __builtin_inf();
    for (int s = threadIdx.x; s < L; s += 64) {
      const unsigned long long* w = mb + u * mb64_row_words(L) + 2 * s;
      const double v = __longlong_as_double((long long)((w[0] & 0xffffffffull) | (w[1] << 32)));
      x[u * L + s] = v;
      mn = vmin(mn, v);
    }
    if (trace_row) {
      mn = row16_min(mn);
      mn = pair16_min(mn, mn);
      mn = join32_min(mn, mn);
      if (threadIdx.x == 0) trace_row[u] = mn;
    }
  }
}

template <int LT> struct SmemR64 {
  using Mask = typename std::conditional<LT <= 32, unsigned, unsigned long long>::type;
  double ubu[2][LT];
  double ubv[2][LT];
  Mask mask[3][LT];  // labels whose record names this label
  int abort_flag;
};

// Sums over the labels k with idx(k) = this lane's label, in ascending k: the
// first kAhead source lanes are taken out of the mask before the step's values
// arrive, the rest one by one.  (Records spread their indices: of 32 labels
// three or four at most usually name the same one.)
constexpr int kAhead = 4;
template <typename Mask> struct ScatterSum {
  int src[kAhead];
  bool has[kAhead];
  Mask rest;
  __device__ __forceinline__ static int low(Mask m) {
    return sizeof(Mask) == 4 ? __ffs((int)m) - 1 : __ffsll((unsigned long long)m) - 1;
  }
  __device__ __forceinline__ void prepare(Mask m) {
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      has[i] = m != 0;
      src[i] = has[i] ? 4 * low(m) : 0;
      m &= m - 1;
    }
    rest = m;
  }
  // acc +- x(k) for every k of the mask
  template <bool MINUS> __device__ __forceinline__ double run(double acc, double x) const {
    double y[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) y[i] = bperm(x, src[i]);
#pragma unroll
    for (int i = 0; i < kAhead; ++i) acc = has[i] ? (MINUS ? acc - y[i] : acc + y[i]) : acc;
    Mask m = rest;
    while (__any(m != 0)) {
      const double z = bperm(x, m != 0 ? 4 * low(m) : 0);
      acc = m != 0 ? (MINUS ? acc - z : acc + z) : acc;
      m &= m - 1;
    }
    return acc;
  }
};

// Reverse of `seg` recorded iterations (FP64, L <= 64): node adjoints in the
// mailboxes (version = updates of the node already reversed in this
// launch), message adjoints pb (slot order).  One compute wave, lane =
// label; the arithmetic of every adjoint is that of the per-matching reverse
// (same terms, same order).  A step's sums take only the labels whose records
// name this one, found before the step's values arrive (all labels in turn,
// with a compare each, took 2.5 us a matching at 32 labels; 1.28 us now, most
// of it the handoff).  The table adjoints are not accumulated here:
// each reverse step writes its three scatter vectors rb, q-bar and p-bar to
// contrib[it][slot][3L] for k_thb_acc, which adds them in the per-matching
// kernel's order.
template <int LT>
__device__ __forceinline__ void rev64_role(const Rev64Args& a, int first_in, int G_in, SmemR64<LT>& sm) {
  using Mask = typename SmemR64<LT>::Mask;
  const SlotInfo* __restrict__ slots = a.slots;
  const unsigned char* __restrict__ rec = a.rec;
  unsigned long long* __restrict__ mb = a.mb;
  double* __restrict__ pb = a.pb;
  double* __restrict__ contrib = a.contrib;
  const int L = uni(a.L), m = uni(a.m), seg = uni(a.seg);
  const int mbs = mb64_row_words(L);
  const int first = uni(first_in), G = uni(G_in);
  int* err = a.err;
  const long long spin_limit = a.spin_limit;
  const int tid = threadIdx.x;
  const int owned = (m - first + G - 1) / G;
  const int total = owned * seg;
  const size_t rec_it = (size_t)m * 3 * L;
  if (tid >= 64 && tid < kF64NT) {
    // ---- waves 1..3 are idle in this role: they take part in its barriers ----
    for (int q = 0; q < total; ++q) {
      __syncthreads();
      if (sm.abort_flag == q + 1) return;
    }
    return;
  }
  if (tid >= kF64NT) {
    // ---- sync waves ----
    const bool is_u = tid < kF64NT + 64;
    int parity = 0, done = 0, j = owned - 1;
    SlotInfo si = ld_const(slots + first + j * G);
    for (int q = 0; q < total; ++q) {
      const int slot = first + j * G;
      const int nxt = uni(j == 0 ? first + (owned - 1) * G : slot - G);
      const SlotInfo si_next = ld_const(slots + nxt);
      const int node = is_u ? si.u : si.v;
      const int deg = is_u ? si.deg_u : si.deg_v;
      const int pos = is_u ? si.pos_u : si.pos_v;
      const unsigned want = (unsigned)done * (unsigned)deg + (unsigned)(deg - 1 - pos);
      unsigned seen = 0;
      unsigned* dst = reinterpret_cast<unsigned*>(is_u ? sm.ubu[parity] : sm.ubv[parity]);
      if (!mb64_gather<LT>(mb + (size_t)node * mbs, L, want, dst, spin_limit, err, &seen)) {
        if ((tid & 63) == 0) {
          if (ld_dev(err) == 0 || seen != want) report_timeout(err, slot, node, want, seen);
          sm.abort_flag = q + 1;
        }
      }
      __syncthreads();
      if (sm.abort_flag == q + 1) return;
      si = si_next;
      parity ^= 1;
      if (--j < 0) { j = owned - 1; ++done; }
    }
    return;
  }
  // ---- the compute wave: lane = label ----
  const int s = tid;
  const bool real = s < L;
  const int sc = real ? s : 0;
  double p0 = 0.0, p1 = 0.0;
  int t1 = 0, s2 = 0, t3 = 0;
  auto load_step = [&](int slot, int it) __attribute__((always_inline)) {
    const unsigned char* rc = rec + (size_t)it * rec_it + (size_t)slot * 3 * L;
    t1 = rc[sc];
    s2 = rc[L + sc];
    t3 = rc[2 * L + sc];
    p0 = pb[(size_t)slot * 2 * L + sc];
    p1 = pb[(size_t)slot * 2 * L + L + sc];
  };
  int parity = 0, done = 0, j = owned - 1;
  load_step(first + j * G, seg - 1);
  SlotInfo si = ld_const(slots + first + j * G);
  for (int q = 0; q < total; ++q) {
    const int slot = first + j * G;
    const int it = seg - 1 - done;
    const int nxt_slot = uni(j == 0 ? first + (owned - 1) * G : slot - G);
    const SlotInfo si_next = ld_const(slots + nxt_slot);
    // before the step's values are there: who adds to this lane's label
    // (labels past L take no part)
    ScatterSum<Mask> sum3, sum2, sum1;
    if (s < LT) sm.mask[0][s] = sm.mask[1][s] = sm.mask[2][s] = 0;
    wave_sync();
    if (real) {
      const Mask bit = (Mask)1 << s;
      atomicOr(&sm.mask[0][t3], bit);
      atomicOr(&sm.mask[1][s2], bit);
      atomicOr(&sm.mask[2][t1], bit);
    }
    wave_sync();
    sum3.prepare(real ? sm.mask[0][s] : 0);
    sum2.prepare(real ? sm.mask[1][s] : 0);
    sum1.prepare(real ? sm.mask[2][s] : 0);
    const double b0 = p0, b1 = p1;
    __syncthreads();  // the step's node adjoints are in LDS
    if (sm.abort_flag == q + 1) return;
    const double ubu = sm.ubu[parity][sc], ubv = sm.ubv[parity][sc];
    // r = th(s, t3) - q(t3): rb = pb0 + Ub_u, q-bar(t) -= sum of rb(s), t3(s) = t
    const double rb = b0 + ubu;
    const double qb = sum3.template run<true>(b1 + ubv, rb);
    // q = th(s2, t) + b(s2)
    const double bb = sum2.template run<false>(0.0, qb);
    // b = (a_u - p) / 2
    const double abu = ubu + 0.5 * bb;
    const double pbv = -0.5 * bb;
    // p = th(s, t1) + a_v(t1)
    const double abv = sum1.template run<false>(ubv, pbv);
    // a_u = U_u - phi0, a_v = U_v - phi1
    if (real) {
      mb64_put(mb + (size_t)si.u * mbs + 2 * s, abu, (unsigned)done * (unsigned)si.deg_u + (unsigned)(si.deg_u - si.pos_u));
      mb64_put(mb + (size_t)si.v * mbs + 2 * s, abv, (unsigned)done * (unsigned)si.deg_v + (unsigned)(si.deg_v - si.pos_v));
      pb[(size_t)slot * 2 * L + s] = -abu;
      pb[(size_t)slot * 2 * L + L + s] = -abv;
      double* ct = contrib + ((size_t)it * m + slot) * 3 * L;
      ct[s] = rb;
      ct[L + s] = qb;
      ct[2 * L + s] = pbv;
    }
    si = si_next;
    parity ^= 1;
    if (--j < 0) { j = owned - 1; ++done; }
    // (each lane reads back only message adjoints that it stored itself)
    if (q + 1 < total) load_step(nxt_slot, seg - 1 - done);
  }
}

// Workgroups [0, r.grid) run the reverse of one recorded segment, the others
// the recording forward of `f.iters` iterations of another: they share no
// data, so they run side by side on the device.  Each workgroup has kF64NT +
// 128 threads; the reverse uses wave 0 and the two sync waves.
// Segments are queued behind one another without a check between them, and a
// segment whose recording timed out has left records that nobody wrote: the
// launches behind it end at once (failed_before) instead of taking such bytes
// for labels.
template <int LT, bool PHI_LDS>
__global__ void __launch_bounds__(kF64NT + 128) k_adj64(Fwd64Args f, Rev64Args r) {
  __shared__ SmemF64<LT> smf;
  __shared__ SmemR64<LT> smr;
  extern __shared__ __align__(16) double phi_lds64[];
  const int b = blockIdx.x;
  if (b < r.grid) {
    if (b >= r.m || r.seg <= 0 || failed_before(r.err, smr.abort_flag)) return;
    rev64_role<LT>(r, b, r.grid, smr);
  } else {
    const int first = b - r.grid;
    if (first >= f.m || f.iters <= 0 || failed_before(f.err, smf.abort_flag)) return;
    fwd64_role<LT, PHI_LDS, true, false>(f, first, f.grid, smf, phi_lds64);
  }
}
template <int LT, bool PHI_LDS, bool TRACE>
__global__ void __launch_bounds__(kF64NT + 128) k_fwd64(Fwd64Args f) {
  __shared__ SmemF64<LT> smf;
  extern __shared__ __align__(16) double phi_lds64[];
  if ((int)blockIdx.x >= f.m || failed_before(f.err, smf.abort_flag)) return;
  fwd64_role<LT, PHI_LDS, false, TRACE>(f, blockIdx.x, f.grid, smf, phi_lds64);
}

// Table adjoints of one segment: thb[slot] += the reverse steps' scatters,
// iterations descending, within each r (thb(s, t3(s)) += rb(s)), then q
// (thb(s2(t), t) += q-bar(t)), then p (thb(s, t1(s)) += p-bar(s)): the
// order of the per-matching reverse.  One workgroup per slot, the slot's
// table adjoint in LDS.  (After a failed launch there may be no records.)
template <int LT>
__global__ void __launch_bounds__(256) k_thb_acc(double* __restrict__ thb, const unsigned char* __restrict__ rec,
                                                 const double* __restrict__ contrib, int L, int m, int seg,
                                                 const int* __restrict__ err) {
  __shared__ double g[LT * LT];
  if (ld_dev(err) != 0) return;
  const int slot = blockIdx.x;
  const int tid = threadIdx.x;
  double* gt = thb + (size_t)slot * L * L;
  for (int k = tid; k < L * L; k += 256) g[k] = gt[k];
  __syncthreads();
  const size_t rec_it = (size_t)m * 3 * L;
  for (int it = seg - 1; it >= 0; --it) {
    const unsigned char* rc = rec + (size_t)it * rec_it + (size_t)slot * 3 * L;
    const double* ct = contrib + ((size_t)it * m + slot) * 3 * L;
    if (tid < L) g[tid * L + rc[2 * L + tid]] += ct[tid];
    __syncthreads();
    if (tid < L) g[rc[L + tid] * L + tid] += ct[L + tid];
    __syncthreads();
    if (tid < L) g[tid * L + rc[tid]] += ct[2 * L + tid];
    __syncthreads();
  }
  for (int k = tid; k < L * L; k += 256) gt[k] = g[k];
}

hipError_t launch_mb64_init(const double* x, unsigned long long* mb, int n, int L, hipStream_t st) {
  hipLaunchKernelGGL(k_mb64_init, dim3(stride_blocks(n)), dim3(64), 0, st, x, mb, n, L);
  return hipGetLastError();
}
hipError_t launch_mb64_fini(double* x, const unsigned long long* mb, int n, int L, double* trace_row, hipStream_t st) {
  hipLaunchKernelGGL(k_mb64_fini, dim3(stride_blocks(n)), dim3(64), 0, st, x, mb, n, L, trace_row);
  return hipGetLastError();
}

// dynamic LDS for the messages of a forward workgroup's slots, 0 where they
// do not fit (they then stay in memory)
static size_t fwd64_lds(const Fwd64Args& f) {
  if (f.grid <= 0) return 0;
  const size_t bytes = ((size_t)f.m + f.grid - 1) / f.grid * 2 * f.L * sizeof(double);
  return bytes <= kPhiLdsBudget ? bytes : 0;
}
static hipError_t coop(const void* fn, int grid, void** args, size_t lds, hipStream_t st) {
  const hipError_t e = hipLaunchCooperativeKernel(fn, dim3(grid), dim3(kF64NT + 128), args, lds, st);
  if (e != hipSuccess) (void)hipGetLastError();  // (a refused launch: not left for a later launch check)
  return e;
}

template <int LT> static hipError_t fwd64_one(const Fwd64Args& f, hipStream_t st) {
  void* args[] = {(void*)&f};
  const size_t lds = fwd64_lds(f);
  const void* fn = lds ? (f.trace ? (const void*)k_fwd64<LT, true, true> : (const void*)k_fwd64<LT, true, false>)
                       : (f.trace ? (const void*)k_fwd64<LT, false, true> : (const void*)k_fwd64<LT, false, false>);
  return coop(fn, f.grid, args, lds, st);
}
// Tiles of 16, 32, 48 and 64 labels.  In FP64 the passes over the tile's entries
// weigh enough that 48 is worth a tile of its own (microseconds a matching of 60
// nodes, tile of 64 / of 48: 36 labels 2.0 / 1.51, 48 labels 2.05 / 1.56; with
// the adjoint's records 2.8 / 1.8).
hipError_t launch_fwd64(const Fwd64Args& f, hipStream_t st) {
  if (f.m <= 0 || f.iters <= 0 || f.grid <= 0) return hipSuccess;
  if (f.L <= 16) return fwd64_one<16>(f, st);
  if (f.L <= 32) return fwd64_one<32>(f, st);
  if (f.L <= 48) return fwd64_one<48>(f, st);
  if (f.L <= 64) return fwd64_one<64>(f, st);
  return hipErrorInvalidValue;
}

template <int LT>
static hipError_t adj64_one(const Fwd64Args& f, const Rev64Args& r, double* thb, hipStream_t st) {
  void* args[] = {(void*)&f, (void*)&r};
  const size_t lds = fwd64_lds(f);
  const void* fn = lds ? (const void*)k_adj64<LT, true> : (const void*)k_adj64<LT, false>;
  const int grid = r.grid + f.grid;
  if (grid <= 0) return hipSuccess;
  const hipError_t e = coop(fn, grid, args, lds, st);
  if (e != hipSuccess) return e;
  if (r.grid > 0 && r.seg > 0 && r.m > 0) {
    hipLaunchKernelGGL(k_thb_acc<LT>, dim3(r.m), dim3(256), 0, st, thb, r.rec, r.contrib, r.L, r.m, r.seg,
                       r.err);
    return hipGetLastError();
  }
  return hipSuccess;
}
hipError_t launch_adj64(const Fwd64Args& f, const Rev64Args& r, double* thb, hipStream_t st) {
  const int L = f.grid > 0 ? f.L : r.L;
  if (L <= 16) return adj64_one<16>(f, r, thb, st);
  if (L <= 32) return adj64_one<32>(f, r, thb, st);
  if (L <= 48) return adj64_one<48>(f, r, thb, st);
  if (L <= 64) return adj64_one<64>(f, r, thb, st);
  return hipErrorInvalidValue;
}

#define MPLPXX_INST(T)                                                                                        \
  template hipError_t launch_step_record<T>(const T*, T*, T*, T*, const SlotInfo*, int, int, int,            \
                                            unsigned char*, hipStream_t);                                     \
  template hipError_t launch_adj_step<T>(const SlotInfo*, int, int, int, const unsigned char*, T*, T*, T*,    \
                                         hipStream_t);                                                        \
  template hipError_t launch_adj_seed<T>(const T*, const T*, int, int, T*, double*, hipStream_t);
MPLPXX_INST(float)
MPLPXX_INST(double)
#undef MPLPXX_INST

}  // namespace mplpxx
