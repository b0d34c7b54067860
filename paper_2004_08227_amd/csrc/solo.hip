// Small models on one workgroup: every matching has at most 16 edges and at
// most 32 labels, and the messages fit in LDS.
//
// The mailbox engines spend about half of a step on the handoff of a node's
// values from one workgroup to the next through memory.  Here the whole model
// lives in one workgroup: unaries and messages in LDS, one wavefront per edge
// of a matching, one barrier per matching (Sec. 6), no mailboxes and no waits.
// What is left on the chain from one matching to the next is the update
// itself: one LDS round trip, the three passes, the unary update and the LDS
// writes.  Positions and tables of the coming matchings are fetched while the
// update's own reads are on their way.
//
// Lane layout.  The table is on the 8 x 8 lane grid of the wave engine: lane 8 rb
// + cb holds rows rb B .. and columns cb B .., B = LT / 8, LT = 8, 16 or 32;
// entries outside L x L are +inf.  Every lane reads its rows' and its columns'
// labels straight from LDS, and results leave from lanes that hold them anyway:
// row rb B + d from the lane with cb - rb = d (mod 8), d < B, column cb B + j from
// the one with rb - cb = j + 1; with B up to 4 no lane has two.
//
// Every value is formed by the same IEEE operations in the same order as in
// the other engines (one add per table entry, exact minima, centred FP32
// passes and compensated FP32 unaries), so the states agree bit for bit.
//
// Bound: the step's dependent instructions, and above one wave per SIMD the
// instructions its waves issue: 0.36 us a matching at 8 labels and up to four
// edges (0.44 with the vectors shuffled through the lanes, see k_solo_label; 1.1
// us on the mailbox engine), 0.32 us in FP64 (0.42; 1.13), 0.72 us at 16 edges;
// the figures of the whole range stand at solo_fits.
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "solo.h"

namespace mplpxx {

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

// A label's unary in LDS: with its correction (FP32), or alone
struct Unary32 {
  float hi, lo;
};
template <typename T> using SoloUnary = typename std::conditional<std::is_same<T, float>::value, Unary32, double>::type;

template <typename T, int LT, bool TRACE>
__global__ void __launch_bounds__(64 * solo_max_waves(LT)) k_solo(SoloArgs<T> a, int iters) {
  constexpr bool kComp = std::is_same<T, float>::value;
  constexpr int B = LT / 8;
  using E = SoloUnary<T>;
  static_assert(sizeof(E) == 8, "one LDS word pair a label");
  // tables are loaded DEPTH matchings ahead (registers bound the ring)
  constexpr int DEPTH = sizeof(T) == 8 && LT == 32 ? 1 : 2;
  constexpr int RING = DEPTH + 1;
  const T kInf = inf_v<T>();
  extern __shared__ __align__(16) unsigned char solo_lds[];
  const int L = a.L, n = a.n, m = a.m, S = a.S;
  const int nL = n * L;
  // (a tile's worth of zeros behind the unaries and the messages: rows are read whole)
  E* l_u = reinterpret_cast<E*>(solo_lds);                        // [n][L]
  T* l_phi = reinterpret_cast<T*>(l_u + nL + LT);                 // [m][2][L]
  int* l_uv = reinterpret_cast<int*>(l_phi + (size_t)m * 2 * L + LT);  // [m] u L, v L (15 bits) and whether it is the node's last update
  int* l_ptr = l_uv + m;                                          // [S + 1]
  const int tid = threadIdx.x, nt = blockDim.x;
  for (int i = tid; i < nL + LT; i += nt) {
    if constexpr (kComp) l_u[i] = i < nL ? Unary32{a.U[i], a.Ulo[i]} : Unary32{0.0f, 0.0f};
    else l_u[i] = i < nL ? a.U[i] : 0.0;
  }
  for (int i = tid; i < m * 2 * L + LT; i += nt) l_phi[i] = i < m * 2 * L ? a.phi[i] : T(0);
  for (int i = tid; i < m; i += nt) {
    const SlotInfo si = a.slots[i];
    l_uv[i] = (int)((unsigned)(si.u * L) | (si.pos_u == si.deg_u - 1 ? 1u << 15 : 0u) | (unsigned)(si.v * L) << 16 |
                    (si.pos_v == si.deg_v - 1 ? 1u << 31 : 0u));
    if (i == 0 || a.slots[i - 1].step != si.step) l_ptr[si.step] = i;
  }
  if (tid == 0) l_ptr[S] = m;
  __syncthreads();

  const int w = uni(tid >> 6), lane = tid & 63;
  const int rb = lane >> 3, cb = lane & 7;
  bool row_real[B], col_real[B];
#pragma unroll
  for (int i = 0; i < B; ++i) {
    row_real[i] = rb * B + i < L;
    col_real[i] = cb * B + i < L;
  }
  // this lane's output: label out_s of the lower (out_u) or the upper node, its
  // oi-th row or column
  const int diag = (cb - rb) & 7;
  const bool out_u = diag < B;
  const int oi = out_u ? diag : 7 - diag;
  const int out_s = (out_u ? rb : cb) * B + oi;
  const bool out = oi < B && out_s < L;
  // this lane's entries of a table (all tables of a model that fits LDS are far
  // below 4 GB)
  unsigned at[B][B];
#pragma unroll
  for (int i = 0; i < B; ++i)
#pragma unroll
    for (int j = 0; j < B; ++j) at[i][j] = (unsigned)(min(rb * B + i, L - 1) * L + min(cb * B + j, L - 1)) * (unsigned)sizeof(T);
  const unsigned table_bytes = (unsigned)(L * L) * (unsigned)sizeof(T);
  auto load_tile = [&](T (&x)[B][B], int slot) __attribute__((always_inline)) {
    const char* tab = reinterpret_cast<const char*>(a.tables) + (unsigned)slot * table_bytes;
#pragma unroll
    for (int i = 0; i < B; ++i)
#pragma unroll
      for (int j = 0; j < B; ++j) x[i][j] = *reinterpret_cast<const T*>(tab + at[i][j]);
  };
  // this wave's slot in the matching of [p, q) (or any slot: its results are not used)
  auto slot_at = [&](int p) __attribute__((always_inline)) { return uni(min(p + w, m - 1)); };
  auto wrap = [&](int k) __attribute__((always_inline)) { return k >= S ? k - S : k; };

  const long long total = (long long)iters * S;
  T t0[B][B], t1[B][B], t2[B][B];
  // slots and activity of this matching (0) and the next two, and the words that
  // give the third's and the next one's nodes, read one matching ahead
  const int k1 = 1 % S, k2 = 2 % S;
  int k = 0, k3 = 3 % S, it = 0;
  int slot0 = slot_at(l_ptr[0]), slot1 = slot_at(l_ptr[k1]), slot2 = slot_at(l_ptr[k2]);
  bool act0 = w < uni(l_ptr[1] - l_ptr[0]), act1 = w < uni(l_ptr[k1 + 1] - l_ptr[k1]),
       act2 = w < uni(l_ptr[k2 + 1] - l_ptr[k2]);
  unsigned uv = (unsigned)uni(l_uv[slot0]);
  int p3 = l_ptr[k3], e3 = l_ptr[k3 + 1], uv1 = l_uv[slot1];
  load_tile(t0, slot0);
  if (DEPTH == 2) load_tile(t1, slot1);

  auto step = [&](T (&xc)[B][B], T (&xp)[B][B]) __attribute__((always_inline)) {
    __syncthreads();
    const int uL = uv & 0x7fff, vL = (uv >> 16) & 0x7fff;
    int slot3 = 0;
    bool act3 = false;
    unsigned uv_next = 0;
    // the table DEPTH matchings ahead, the positions of the coming matchings,
    // this table's pads
    auto between = [&]() __attribute__((always_inline)) {
      load_tile(xp, DEPTH == 2 ? slot2 : slot1);
      slot3 = slot_at(p3);
      act3 = w < uni(e3 - p3);
      uv_next = (unsigned)uni(uv1);
#pragma unroll
      for (int i = 0; i < B; ++i)
#pragma unroll
        for (int j = 0; j < B; ++j) xc[i][j] = row_real[i] && col_real[j] ? xc[i][j] : kInf;
    };
    if (!act0) {
      between();
    } else {
      // every read of the update first, the rest while they are on their way
      const E* rows = l_u + uL + rb * B;
      const E* cols = l_u + vL + cb * B;
      T* ph = l_phi + (size_t)slot0 * 2 * L;
      E eu[B], ev[B];
      T pu[B], pv[B];
      float hc[B];  // (FP32: the lower node's labels by columns too, so that both references are minima over an octet)
#pragma unroll
      for (int j = 0; j < B; ++j) {
        ev[j] = cols[j];
        if constexpr (kComp) hc[j] = l_u[uL + cb * B + j].hi;
      }
#pragma unroll
      for (int j = 0; j < B; ++j) pv[j] = ph[L + cb * B + j];
#pragma unroll
      for (int i = 0; i < B; ++i) {
        eu[i] = rows[i];
        pu[i] = ph[rb * B + i];
      }
      between();
      T au[B], av[B], delta = T(0);
      if constexpr (kComp) {
        float c_u = kInf, c_v = kInf;
#pragma unroll
        for (int j = 0; j < B; ++j) {
          asm volatile("" : "+v"(hc[j]));  // (read by every lane)
          c_u = vmin(c_u, col_real[j] ? hc[j] : kInf);
          c_v = vmin(c_v, col_real[j] ? ev[j].hi : kInf);
        }
        c_u = vmin(c_u, dpp_f<0xB1>(c_u));
        c_v = vmin(c_v, dpp_f<0xB1>(c_v));
        c_u = vmin(c_u, dpp_f<0x4E>(c_u));
        c_v = vmin(c_v, dpp_f<0x4E>(c_v));
        c_u = vmin(c_u, dpp_f<0x141>(c_u));
        c_v = vmin(c_v, dpp_f<0x141>(c_v));
        delta = T(0.5) * (c_u - c_v);
#pragma unroll
        for (int j = 0; j < B; ++j) av[j] = ((ev[j].hi - c_v) + ev[j].lo) - pv[j];
#pragma unroll
        for (int i = 0; i < B; ++i) au[i] = ((eu[i].hi - c_u) + eu[i].lo) - pu[i];
      } else {
#pragma unroll
        for (int j = 0; j < B; ++j) av[j] = ev[j] - pv[j];
#pragma unroll
        for (int i = 0; i < B; ++i) au[i] = eu[i] - pu[i];
      }
      // this lane's old value and message
      E eo = out_u ? eu[0] : ev[0];
      T po = out_u ? pu[0] : pv[0], xo = out_u ? au[0] : av[0];
#pragma unroll
      for (int i = 1; i < B; ++i) {
        if constexpr (kComp) {
          eo.hi = oi == i ? (out_u ? eu[i].hi : ev[i].hi) : eo.hi;
          eo.lo = oi == i ? (out_u ? eu[i].lo : ev[i].lo) : eo.lo;
          po = oi == i ? (out_u ? pu[i] : pv[i]) : po;
        } else {
          xo = oi == i ? (out_u ? au[i] : av[i]) : xo;
        }
      }
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
#pragma unroll
      for (int i = 0; i < B; ++i) asm volatile("" : "+v"(r[i]));  // (finished by every lane)
      // push back
      T ro = r[0], qo = q[0];
#pragma unroll
      for (int i = 1; i < B; ++i) {
        ro = oi == i ? r[i] : ro;
        qo = oi == i ? q[i] : qo;
      }
      E ne;
      T msg;
      if constexpr (kComp) {
        msg = out_u ? ro - delta : qo + delta;
        comp_update(eo.hi, eo.lo, po, msg, ne.hi, ne.lo);
      } else {
        msg = out_u ? ro : qo;
        ne = xo + msg;
      }
      if (out) {
        l_u[(out_u ? uL : vL) + out_s] = ne;
        ph[(out_u ? 0 : L) + out_s] = msg;
      }
      if constexpr (TRACE) {
        // a node's last update of the iteration leaves its value of the trace
        // (read back by the wave that wrote it; lower node in lanes 0..31)
        if (uv & 0x80008000u) {
          wave_sync();
          const int s = lane & 31, base = lane < 32 ? uL : vL;
          const E e = l_u[base + min(s, L - 1)];
          double mn;
          if constexpr (kComp) mn = (double)e.hi + (double)e.lo;
          else mn = e;
          mn = row16_min(mn);
          if (LT == 32) mn = min_x16(mn);
          if (s == 0 && (uv & (lane < 32 ? 0x8000u : 0x80000000u))) a.trace[(size_t)it * n + base / L] = mn;
        }
        if constexpr (kComp) {
          // edge term of Eq. (3) after this update, as in the mailbox engine
          float em = kInf;
#pragma unroll
          for (int i = 0; i < B; ++i) {
            const float rr = r[i] - delta;
#pragma unroll
            for (int j = 0; j < B; ++j) {
              const float qq = q[j] + delta;
              const float d = xc[i][j] - qq;
              const float e = (d - rr) + two_sum_err(xc[i][j], -qq, d);
              em = row_real[i] && col_real[j] ? vmin(em, e) : em;
            }
          }
          em = col4_min(row16_min(em));
          if (lane == 0) a.trace_e[(size_t)it * m + slot0] = em;
        }
      }
    }
    slot0 = slot1;
    slot1 = slot2;
    slot2 = slot3;
    act0 = act1;
    act1 = act2;
    act2 = act3;
    uv = uv_next;
    k = wrap(k + 1);
    if (k == 0) ++it;
    k3 = wrap(k3 + 1);
    p3 = l_ptr[k3];
    e3 = l_ptr[k3 + 1];
    uv1 = l_uv[slot1];
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
    if constexpr (kComp) {
      a.U[i] = l_u[i].hi;
      a.Ulo[i] = l_u[i].lo;
    } else {
      a.U[i] = l_u[i];
    }
  }
  for (int i = tid; i < m * 2 * L; i += nt) a.phi[i] = l_phi[i];
}

// The same with per-label vectors held by half waves, lane 32 side + s label s of
// the lower (side 0) or upper (side 1) node, and shuffled into the tile's rows
// and columns and back.  Two more LDS round trips a step, but fewer instructions
// where a lane has several rows and FP32 has the references and corrections of
// each.  FP32 above 8 labels runs here for every number of edges: it is the
// better way from two waves a SIMD on, and with fewer a little behind the one
// above (microseconds a matching at 4, 8 and 16 edges, 16 labels: 0.56, 0.66 and
// 0.99 here, 0.51, 0.73 and 1.13 above; 32 labels, 2 edges: 0.86 and 0.95).
// the lower and the upper half wave's value of x, in the lanes of both
__device__ __forceinline__ void halves(float x, float& lo, float& hi) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  lo = __uint_as_float(r[0]);
  hi = __uint_as_float(r[1]);
}
template <typename T, int LT, bool TRACE>
__global__ void __launch_bounds__(64 * solo_max_waves(LT)) k_solo_label(SoloArgs<T> a, int iters) {
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
  const void* f;
  if constexpr (sizeof(T) == 4 && LT > 8)
    f = a.trace ? (const void*)k_solo_label<T, LT, true> : (const void*)k_solo_label<T, LT, false>;
  else
    f = a.trace ? (const void*)k_solo<T, LT, true> : (const void*)k_solo<T, LT, false>;
  SoloArgs<T> args = a;
  void* p[] = {(void*)&args, (void*)&iters};
  return hipLaunchKernel(f, dim3(1), dim3(64 * waves), p, lds, st);
}

template <typename T>
hipError_t launch_solo(const SoloArgs<T>& a, int max_step, int iters, hipStream_t st) {
  const size_t lds = solo_lds_bytes(a.n, a.L, a.m, a.S, sizeof(T)) + solo_lds_pad(a.L, sizeof(T));
  if (a.L <= 8) return solo_one<T, 8>(a, max_step, iters, lds, st);
  if (a.L <= 16) return solo_one<T, 16>(a, max_step, iters, lds, st);
  return solo_one<T, 32>(a, max_step, iters, lds, st);
}
template hipError_t launch_solo<float>(const SoloArgs<float>&, int, int, hipStream_t);
template hipError_t launch_solo<double>(const SoloArgs<double>&, int, int, hipStream_t);

}  // namespace mplpxx
