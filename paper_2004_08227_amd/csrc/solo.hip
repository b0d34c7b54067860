// Small models on one workgroup: every matching has at most 16 edges and at
// most 32 labels, and the messages fit in LDS.
//
// The mailbox engines spend about half of a step on the handoff of a node's
// values from one workgroup to the next through memory.  Here the whole model
// lives in one workgroup: unaries and messages in LDS, one wavefront per edge
// of a matching, one barrier per matching (Sec. 6), no mailboxes and no waits.
// What is left on the chain from one matching to the next is the update
// itself: two LDS reads, a shuffle into the tile's rows and columns, the three
// passes, a shuffle back, the unary update and the LDS writes.
//
// Lane layout.  Per-label vectors are held by half waves: lane 32 side + s
// holds label s of the lower (side 0) or upper (side 1) node, so both nodes'
// unaries, messages and updates take one instruction.  The table is on the 8 x
// 8 lane grid of the wave engine: lane 8 rb + cb holds rows rb B .. and columns
// cb B .., B = LT / 8, LT = 8, 16 or 32; entries outside L x L are +inf.
//
// Every value is formed by the same IEEE operations in the same order as in
// the other engines (one add per table entry, exact minima, centred FP32
// passes and compensated FP32 unaries), so the states agree bit for bit.
//
// Bound: the step's dependent instructions, and above one wave per SIMD the
// instructions its waves issue: 0.42 us a matching at 8 labels and up to four
// edges (1.1 us on the mailbox engine, 1.75 us in FP64), 0.72 us at 16 edges;
// the figures of the whole range stand at solo_fits.
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "solo.h"

namespace mplpxx {

// the lower and the upper half wave's value of x, in the lanes of both
__device__ __forceinline__ void halves(float x, float& lo, float& hi) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  lo = __uint_as_float(r[0]);
  hi = __uint_as_float(r[1]);
}
// minimum over lanes l, l ^ 16
__device__ __forceinline__ float min_x16(float x) { return pair16_min(x, x); }
__device__ __forceinline__ double min_x16(double x) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(x);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
  return vmin(dbl_of(lo[0], hi[0]), dbl_of(lo[1], hi[1]));
}
// minimum over lanes l, l ^ 32
__device__ __forceinline__ float min_x32(float x) { return join32_min(x, x); }
__device__ __forceinline__ double min_x32(double x) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(x);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
  return vmin(dbl_of(lo[0], hi[0]), dbl_of(lo[1], hi[1]));
}

template <typename T, int LT, bool TRACE>
__global__ void __launch_bounds__(64 * solo_max_waves(LT)) k_solo(SoloArgs<T> a, int iters) {
  constexpr bool kComp = std::is_same<T, float>::value;
  constexpr int B = LT / 8;
  // tables are loaded DEPTH matchings ahead (registers bound the ring)
  constexpr int DEPTH = sizeof(T) == 8 && LT == 32 ? 1 : 2;
  constexpr int RING = DEPTH + 1;
  const T kInf = inf_v<T>();
  extern __shared__ __align__(16) unsigned char solo_lds[];
  const int L = a.L, n = a.n, m = a.m, S = a.S;
  const int nL = n * L;
  T* l_hi = reinterpret_cast<T*>(solo_lds);      // [n][L]
  T* l_phi = l_hi + nL;                           // [m][2][L]
  T* l_lo = l_phi + (size_t)m * 2 * L;            // [n][L] (FP32)
  int* l_uv = reinterpret_cast<int*>(l_lo + (kComp ? nL : 0));  // [m] u | v << 16
  int* l_ptr = l_uv + m;                          // [S + 1]
  const int tid = threadIdx.x, nt = blockDim.x;
  for (int i = tid; i < nL; i += nt) {
    l_hi[i] = a.U[i];
    if (kComp) l_lo[i] = a.Ulo[i];
  }
  for (int i = tid; i < m * 2 * L; i += nt) l_phi[i] = a.phi[i];
  for (int i = tid; i < m; i += nt) {
    const SlotInfo si = a.slots[i];
    l_uv[i] = si.u | (si.v << 16);
    if (i == 0 || a.slots[i - 1].step != si.step) l_ptr[si.step] = i;
  }
  if (tid == 0) l_ptr[S] = m;
  __syncthreads();

  const int w = uni(tid >> 6), lane = tid & 63;
  const int side = lane >> 5, s = lane & 31;
  const int sc = s < L ? s : L - 1;
  const bool real = s < L;
  const int rb = lane >> 3, cb = lane & 7;
  // shuffles: label vectors to the tile's rows and columns and back
  int to_row[B], to_col[B];
#pragma unroll
  for (int i = 0; i < B; ++i) {
    to_row[i] = 4 * (rb * B + i);
    to_col[i] = 4 * (32 + cb * B + i);
  }
  const int from_r = 4 * (8 * (sc / B) + sc % B);  // r(s) in lane cb = s % B of its row block
  const int from_q = 4 * (8 * (sc % B) + sc / B);  // q(t) in lane rb = t % B of its column block
  bool row_real[B], col_real[B];
#pragma unroll
  for (int i = 0; i < B; ++i) {
    row_real[i] = rb * B + i < L;
    col_real[i] = cb * B + i < L;
  }
  unsigned at[B];  // this lane's rows of a table
#pragma unroll
  for (int i = 0; i < B; ++i) at[i] = (unsigned)(min(rb * B + i, L - 1) * L);
  auto load_tile = [&](T (&x)[B][B], int slot) __attribute__((always_inline)) {
    const T* tab = a.tables + (size_t)slot * L * L;
#pragma unroll
    for (int i = 0; i < B; ++i)
#pragma unroll
      for (int j = 0; j < B; ++j) x[i][j] = tab[at[i] + min(cb * B + j, L - 1)];
  };
  // this wave's slot in matching k (or any slot: its results are not used)
  auto slot_of = [&](int k) __attribute__((always_inline)) { return uni(min(l_ptr[k] + w, m - 1)); };
  auto wrap = [&](int k) __attribute__((always_inline)) { return k >= S ? k - S : k; };

  const long long total = (long long)iters * S;
  T t0[B][B], t1[B][B], t2[B][B];
  int k = 0, it = 0, ahead = DEPTH % S;  // matching of this step and of the step DEPTH ahead
  load_tile(t0, slot_of(0));
  if (DEPTH == 2) load_tile(t1, slot_of(S > 1 ? 1 : 0));
  int slot = slot_of(0);
  bool active = w < l_ptr[1] - l_ptr[0];

  auto step = [&](T (&xc)[B][B], T (&xp)[B][B]) __attribute__((always_inline)) {
    // before the barrier: what needs no other wave's result
    load_tile(xp, slot_of(ahead));
    const int uv = l_uv[slot];
    const int node = side ? uv >> 16 : uv & 0xffff;
    const int at_node = node * L + sc;
    T* ph = l_phi + (size_t)slot * 2 * L + side * L + sc;
    const T pold = *ph;
    const int kn = wrap(k + 1);
    const int slot_next = slot_of(kn);
    const bool active_next = w < l_ptr[kn + 1] - l_ptr[kn];
    bool last_upd = false;
    if (TRACE) {
      // the node's last update of the iteration leaves its value of the trace
      const SlotInfo si = a.slots[slot];
      last_upd = side ? si.pos_v == si.deg_v - 1 : si.pos_u == si.deg_u - 1;
    }
#pragma unroll
    for (int i = 0; i < B; ++i)
#pragma unroll
      for (int j = 0; j < B; ++j) xc[i][j] = row_real[i] && col_real[j] ? xc[i][j] : kInf;
    __syncthreads();
    if (active) {
      const T hi = l_hi[at_node];
      T lo = T(0), delta = T(0), x;
      if constexpr (kComp) {
        lo = l_lo[at_node];
        T c = row16_min(hi);
        if (LT == 32) c = min_x16(c);
        T cu, cv;
        halves(c, cu, cv);
        delta = T(0.5) * (cu - cv);
        x = ((hi - c) + lo) - pold;
      } else {
        x = hi - pold;
      }
      T au[B], av[B];
#pragma unroll
      for (int i = 0; i < B; ++i) au[i] = bperm(x, to_row[i]);
#pragma unroll
      for (int j = 0; j < B; ++j) av[j] = bperm(x, to_col[j]);
      // pass 1: p(s) = min_t [th(s,t) + a_v(t)], b = (a_u - p) / 2
      T b[B];
#pragma unroll
      for (int i = 0; i < B; ++i) {
        T mn = xc[i][0] + av[0];
#pragma unroll
        for (int j = 1; j < B; ++j) mn = vmin(mn, xc[i][j] + av[j]);
        b[i] = mn;
      }
#pragma unroll
      for (int i = 0; i < B; ++i) b[i] = vmin(b[i], dpp_f<0xB1>(b[i]));
#pragma unroll
      for (int i = 0; i < B; ++i) b[i] = vmin(b[i], dpp_f<0x4E>(b[i]));
#pragma unroll
      for (int i = 0; i < B; ++i) b[i] = vmin(b[i], dpp_f<0x141>(b[i]));
#pragma unroll
      for (int i = 0; i < B; ++i) b[i] = row_real[i] ? T(0.5) * (au[i] - b[i]) : T(0);
      // pass 2: q(t) = min_s [th(s,t) + b(s)]
      T q[B];
#pragma unroll
      for (int j = 0; j < B; ++j) {
        T mn = xc[0][j] + b[0];
#pragma unroll
        for (int i = 1; i < B; ++i) mn = vmin(mn, xc[i][j] + b[i]);
        q[j] = mn;
      }
#pragma unroll
      for (int j = 0; j < B; ++j) q[j] = vmin(q[j], dpp_f<0x128>(q[j]));
#pragma unroll
      for (int j = 0; j < B; ++j) q[j] = min_x16(q[j]);
#pragma unroll
      for (int j = 0; j < B; ++j) q[j] = min_x32(q[j]);
#pragma unroll
      for (int j = 0; j < B; ++j) q[j] = col_real[j] ? q[j] : T(0);
      // pass 3: r(s) = min_t [th(s,t) - q(t)]
      T r[B];
#pragma unroll
      for (int i = 0; i < B; ++i) {
        T mn = xc[i][0] - q[0];
#pragma unroll
        for (int j = 1; j < B; ++j) mn = vmin(mn, xc[i][j] - q[j]);
        r[i] = mn;
      }
#pragma unroll
      for (int i = 0; i < B; ++i) r[i] = vmin(r[i], dpp_f<0xB1>(r[i]));
#pragma unroll
      for (int i = 0; i < B; ++i) r[i] = vmin(r[i], dpp_f<0x4E>(r[i]));
#pragma unroll
      for (int i = 0; i < B; ++i) r[i] = vmin(r[i], dpp_f<0x141>(r[i]));
      // each label's result: one lane of the row or column block offers it
      T rs = r[0], qs = q[0];
#pragma unroll
      for (int i = 1; i < B; ++i) {
        rs = cb % B == i ? r[i] : rs;
        qs = rb % B == i ? q[i] : qs;
      }
      const T fr = bperm(rs, from_r), fq = bperm(qs, from_q);
      T msg, nhi, nlo = T(0);
      if constexpr (kComp) {
        msg = side ? fq + delta : fr - delta;
        comp_update(hi, lo, pold, msg, nhi, nlo);
      } else {
        msg = side ? fq : fr;
        nhi = x + msg;
      }
      if (real) {
        l_hi[at_node] = nhi;
        if (kComp) l_lo[at_node] = nlo;
        *ph = msg;
      }
      if constexpr (TRACE) {
        double mn = real ? (double)nhi + (double)nlo : __builtin_inf();
        mn = row16_min(mn);
        if (LT == 32) mn = min_x16(mn);
        if (last_upd && s == 0) a.trace[(size_t)it * n + node] = mn;
        if constexpr (kComp) {
          // edge term of Eq. (3) after this update, as in the mailbox engine
          const float d0 = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(delta)));
          float em = kInf;
#pragma unroll
          for (int i = 0; i < B; ++i) {
            const float rr = r[i] - d0;
#pragma unroll
            for (int j = 0; j < B; ++j) {
              const float qq = q[j] + d0;
              const float d = xc[i][j] - qq;
              const float e = (d - rr) + two_sum_err(xc[i][j], -qq, d);
              em = row_real[i] && col_real[j] ? vmin(em, e) : em;
            }
          }
          em = col4_min(row16_min(em));
          if (lane == 0) a.trace_e[(size_t)it * m + slot] = em;
        }
      }
    }
    slot = slot_next;
    active = active_next;
    ahead = wrap(ahead + 1);
    k = kn;
    if (k == 0) ++it;
  };
  long long q = 0;
  if (RING == 2) {
    for (; q + 2 <= total; q += 2) {
      step(t0, t1);
      step(t1, t0);
    }
    if (q < total) step(t0, t1);
  } else {
    for (; q + 3 <= total; q += 3) {
      step(t0, t2);
      step(t1, t0);
      step(t2, t1);
    }
    if (q < total) step(t0, t2);
    if (q + 1 < total) step(t1, t0);
  }
  __syncthreads();
  for (int i = tid; i < nL; i += nt) {
    a.U[i] = l_hi[i];
    if (kComp) a.Ulo[i] = l_lo[i];
  }
  for (int i = tid; i < m * 2 * L; i += nt) a.phi[i] = l_phi[i];
}

template <typename T, int LT>
static hipError_t solo_one(const SoloArgs<T>& a, int waves, int iters, size_t lds, hipStream_t st) {
  if (a.trace) hipLaunchKernelGGL((k_solo<T, LT, true>), dim3(1), dim3(64 * waves), lds, st, a, iters);
  else hipLaunchKernelGGL((k_solo<T, LT, false>), dim3(1), dim3(64 * waves), lds, st, a, iters);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_solo(const SoloArgs<T>& a, int max_step, int iters, hipStream_t st) {
  const size_t lds = solo_lds_bytes(a.n, a.L, a.m, a.S, sizeof(T));
  if (a.L <= 8) return solo_one<T, 8>(a, max_step, iters, lds, st);
  if (a.L <= 16) return solo_one<T, 16>(a, max_step, iters, lds, st);
  return solo_one<T, 32>(a, max_step, iters, lds, st);
}
template hipError_t launch_solo<float>(const SoloArgs<float>&, int, int, hipStream_t);
template hipError_t launch_solo<double>(const SoloArgs<double>&, int, int, hipStream_t);

}  // namespace mplpxx
