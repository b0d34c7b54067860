// FP64 mailbox forward (tiles up to 64 labels): the FP32 mailbox engine's
// structure (device_common.h) for doubles, optionally with the argmin records
// the adjoint needs, or with the per-iteration trace.
//
// Mailboxes.  A node's FP64 values (the unaries in the forward, their
// adjoints in the reverse) travel between workgroups as two 64-bit words per
// label, mb[node][label][h]: bits 0..31 hold the low (h = 0) or high (h = 1)
// half of the double, bits 32..63 the number of updates the node has had in
// this launch.  Each word is written and read with one device-scope atomic
// access, so a consumer that sees the version it waits for in both words of
// every label holds the values of that version: no flag, no fence.  (The
// FP32 engines pack value and version into one word the same way.)  A node's
// row fills whole cache lines (mb64_row_words), as in FP32.
//
// Bound: the chain of dependent matchings, as in FP32.  Against the former
// FP64 forward (argmins carried through every minimum, tables loaded after the
// step that used the last ones, divergent stores), microseconds a matching:
// n = 100, L = 16 1.72 -> 1.14, L = 32 2.49 -> 1.33, L = 64 4.82 -> 2.08;
// traces, which ran on release and acquire fences, 4.62 -> 1.13, 5.39 -> 1.33,
// 6.25 -> 2.03.  The records cost nothing at L = 32: they
// are made while the next workgroup of the chain works.
//
// Slots are owned statically: workgroup w runs slots w, w + G, ... in schedule
// order every iteration, so an edge's messages and records never leave one
// workgroup, and every wait is for an update earlier in the order.
#pragma once
#include "device_common.h"

namespace mplpxx {

__device__ __forceinline__ unsigned long long mb64_word(unsigned half, unsigned ver) {
  return ((unsigned long long)ver << 32) | half;
}
__device__ __forceinline__ void mb64_put(unsigned long long* dst, double x, unsigned ver) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(x);
  mb_store(dst, mb64_word((unsigned)b, ver));
  mb_store(dst + 1, mb64_word((unsigned)(b >> 32), ver));
}

// sync wave: poll the 2L words of one node until every one carries `want`,
// then write their payloads to dst (2L 32-bit halves = L doubles).  Every
// lane reloads its words until the whole wave sees the version: no word can
// move past it meanwhile, since this workgroup makes the node's next update
// (lanes past the row read its last word).
template <int LT>
__device__ __forceinline__ bool mb64_gather(const unsigned long long* __restrict__ row, int L, unsigned want,
                                            unsigned* dst, long long spin_limit, const int* err, unsigned* seen_out) {
  const int lane = threadIdx.x & 63;
  constexpr int PER = (2 * LT + 63) / 64;
  unsigned long long val[PER];
  long long spins = 0;
  bool done;
  do {
    bool all = true;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int i = lane + 64 * k;
      val[k] = mb_load(row + (i < 2 * L ? i : 2 * L - 1));
      all &= (unsigned)(val[k] >> 32) == want;
    }
    done = __all(all);
  } while (!done && ++spins <= spin_limit && ((spins & 255) != 0 || ld_dev(err) == 0));
  if (!done) {
    unsigned seen = want;
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if ((unsigned)(val[k] >> 32) != want) seen = (unsigned)(val[k] >> 32);
    for (int o = 32; o >= 1; o >>= 1) seen = min(seen, (unsigned)__shfl_xor((int)seen, o, 64));
    *seen_out = seen;
    return false;
  }
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (lane + 64 * k < 2 * L) dst[lane + 64 * k] = (unsigned)val[k];
  return true;
}

constexpr int kF64NT = 256;  // compute threads of the FP64 mailbox forward

// Start of a workgroup: clears its abort flag; true in every thread if an earlier
// launch has already failed (steps that abort set the flag to 1 or more)
__device__ __forceinline__ bool failed_before(const int* err, int& abort_flag) {
  if (threadIdx.x == 0) abort_flag = ld_dev(err) != 0 ? -1 : 0;
  __syncthreads();
  return abort_flag == -1;
}

template <int LT> struct SmemF64 {
  double hu[2][LT];   // the step's nodes from the sync waves (double buffered)
  double hv[2][LT];
  double red[kF64NT / 64][LT];
  int redi[2][kF64NT / 64][LT];   // REC: each wave's lowest argmin row of a column
  int abort_flag;
};

// column minima over the wave's four row blocks (see col4_min_store)
__device__ __forceinline__ double pair16_min(double a, double b) {
  const unsigned long long x = (unsigned long long)__double_as_longlong(a), y = (unsigned long long)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  return vmin(dbl_of(lo[0], hi[0]), dbl_of(lo[1], hi[1]));
}
__device__ __forceinline__ double join32_min(double a, double b) {
  const unsigned long long x = (unsigned long long)__double_as_longlong(a), y = (unsigned long long)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  return vmin(dbl_of(lo[0], hi[0]), dbl_of(lo[1], hi[1]));
}
template <int BC>
__device__ __forceinline__ void col4_min_store64(const double (&x)[BC], double* red, int cb, int lane) {
  const int k = lane >> 4;
  constexpr int Q = BC / 4 * 4;  // columns in groups of four, then two, then one
#pragma unroll
  for (int g = 0; g < Q; g += 4)
    red[cb * BC + g + k] = join32_min(pair16_min(x[g], x[g + 1]), pair16_min(x[g + 2], x[g + 3]));
  if constexpr (BC - Q == 3) {
    const double f = join32_min(pair16_min(x[Q], x[Q + 1]), pair16_min(x[Q + 2], x[Q + 2]));
    if (lane < 48) red[cb * BC + Q + k] = f;
  } else if constexpr (BC - Q == 2) {
    const double p = pair16_min(x[Q], x[Q + 1]);
    const double f = join32_min(p, p);
    if (lane < 32) red[cb * BC + Q + k] = f;
  } else if constexpr (BC - Q == 1) {
    const double p = pair16_min(x[Q], x[Q]);
    const double f = join32_min(p, p);
    if (lane < 16) red[cb * BC + Q] = f;
  }
}
// lowest index over the 16 lanes of a row, and over the four row blocks
template <int CTRL> __device__ __forceinline__ int dpp_i(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, true);
}
__device__ __forceinline__ int row16_imin(int x) {
  x = min(x, dpp_i<0xB1>(x));
  x = min(x, dpp_i<0x4E>(x));
  x = min(x, dpp_i<0x141>(x));
  return min(x, dpp_i<0x140>(x));
}
__device__ __forceinline__ int col4_imin(int x) {
  auto a = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)x, false, false);
  x = min((int)a[0], (int)a[1]);
  auto b = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)x, false, false);
  return min((int)b[0], (int)b[1]);
}

// Forward of `iters` iterations: the unaries in the mailboxes, the messages in
// LDS or phi (slot order).  Every value is the same IEEE result as in the other
// FP64 kernels (one add per entry, exact minima, the same a_u, a_v), so the
// runs agree bit for bit.
//
// The step's critical path holds minima only.  REC: the argmins of every
// update, rec[it][slot][0..L) = t1, [L..2L) = s2, [2L..3L) = t3 (lowest index
// on ties), are found after the step's results are published, as the lowest
// index whose candidate equals the minimum; s2 needs the waves' row ranges
// joined, which the next step's barriers do for free (its record is written
// one step later).
// Costs near the largest double overflow to infinities and their differences to
// NaN, and then no candidate, or only a padded one, equals the minimum: a record
// is at most L - 1 all the same (the reverse takes it for a label).
template <int LT, bool PHI_LDS, bool REC, bool TRACE>
__device__ __forceinline__ void fwd64_role(const Fwd64Args& a, int first_in, int G_in, SmemF64<LT>& sm, double* phi_lds) {
  constexpr int NT = kF64NT;
  using S = TileShape<double, LT, NT>;
  const double* __restrict__ tables = a.tables;
  unsigned long long* __restrict__ mb = a.mb;
  const SlotInfo* __restrict__ slots = a.slots;
  const int L = uni(a.L), m = uni(a.m), n = uni(a.n), iters = uni(a.iters);
  const int mbs = mb64_row_words(L);
  const int first = uni(first_in), G = uni(G_in);
  int* err = a.err;
  const long long spin_limit = a.spin_limit;
  const int tid = threadIdx.x;
  const int owned = (m - first + G - 1) / G;
  const int total = owned * iters;
  if (PHI_LDS) {
    for (int slot = first, j = 0; slot < m; slot += G, ++j)
      for (int k = tid; k < 2 * L; k += NT + 128) phi_lds[j * 2 * L + k] = a.phi[(size_t)slot * 2 * L + k];
    __syncthreads();
  }
  if (tid >= NT) {
    // ---- sync waves: wait for the step's two nodes ----
    const bool is_u = tid < NT + 64;
    const int lane = tid & 63;
    int parity = 0, it = 0, j = 0;
    bool ok = true;
    SlotInfo si = ld_const(slots + first);
    for (int q = 0; q < total; ++q) {
      const int slot = first + j * G;
      // metadata of the next owned slot, off the dependency chain
      const int nxt = uni(j + 1 == owned ? first : slot + G);
      const SlotInfo si_next = ld_const(slots + nxt);
      const int node = is_u ? si.u : si.v;
      const int pos = is_u ? si.pos_u : si.pos_v;
      const unsigned want = (unsigned)it * (unsigned)(is_u ? si.deg_u : si.deg_v) + (unsigned)pos;
      unsigned seen = 0;
      double* val = is_u ? sm.hu[parity] : sm.hv[parity];
      if (!mb64_gather<LT>(mb + (size_t)node * mbs, L, want, reinterpret_cast<unsigned*>(val), spin_limit, err, &seen)) {
        if (lane == 0) {
          if (ld_dev(err) == 0 || seen != want) report_timeout(err, slot, node, want, seen);
          sm.abort_flag = q + 1;
        }
      }
      __syncthreads();  // the step's nodes are in LDS
      __syncthreads();  // the compute waves' mid-step barrier
      if (sm.abort_flag == q + 1) {
        ok = false;
        break;
      }
      // the first update of a node in iteration it sees its value at the end
      // of iteration it - 1
      if (TRACE && it > 0 && pos == 0) {
        double mn = lane < L ? val[lane] : __builtin_inf();
        mn = row16_min(mn);
        mn = pair16_min(mn, mn);
        mn = join32_min(mn, mn);
        if (lane == 0) a.trace[(size_t)(it - 1) * n + node] = mn;
      }
      si = si_next;
      parity ^= 1;
      if (++j == owned) { j = 0; ++it; }
    }
    if (!ok) return;
    if (REC) __syncthreads();  // (the compute waves' last records)
    if (PHI_LDS) {
      __syncthreads();
      for (int slot = first, j2 = 0; slot < m; slot += G, ++j2)
        for (int k = tid; k < 2 * L; k += NT + 128) a.phi[(size_t)slot * 2 * L + k] = phi_lds[j2 * 2 * L + k];
    }
    return;
  }
  // ---- compute waves ----
  const int rb = tid >> 4, cb = tid & 15, wave = tid >> 6, lane = tid & 63;
  const size_t rec_it = (size_t)m * 3 * L;
  // output lane of this thread: rows by lane cb = i of each row block, columns
  // by the other lanes of each wave (as in the FP32 engine)
  constexpr int VPW = LT / S::W;
  static_assert(VPW <= 4 * (16 - S::BR), "column outputs per wave");
  static_assert(S::BR <= 8, "row outputs in the first half of a row block");
  const bool out_u = cb < S::BR;
  const int out_s = rb * S::BR + cb;
  const int lw = (rb & 3) * (16 - S::BR) + (cb - S::BR);
  const int out_t = wave * VPW + lw;
  const bool outk = out_u ? out_s < L : lw < VPW && out_t < L;
  const int out_i = out_u ? out_s : out_t;
  const int out_ic = out_i < L ? out_i : L - 1;
  unsigned long long* sink = a.sink + (size_t)blockIdx.x * kF64Sink + wave * 64;
  bool row_real[S::BR], col_real[S::BC];
#pragma unroll
  for (int i = 0; i < S::BR; ++i) row_real[i] = rb * S::BR + i < L;
#pragma unroll
  for (int jj = 0; jj < S::BC; ++jj) col_real[jj] = cb * S::BC + jj < L;
  // rows clamped, columns not (the array has a zeroed tail): entries outside
  // L x L become +inf before use
  auto load_tile64 = [&](double (&x)[S::BR][S::BC], int slot) __attribute__((always_inline)) {
    const double* tab = tables + (size_t)slot * L * L;
#pragma unroll
    for (int i = 0; i < S::BR; ++i) {
      const int s = rb * S::BR + i;
      const double* row = tab + (s < L ? s : L - 1) * L + cb * S::BC;
#pragma unroll
      for (int jj = 0; jj < S::BC; ++jj) x[i][jj] = row[jj];
    }
  };
  double pu[S::BR], pv[S::BC], pvo = 0.0;
  auto load_phi64 = [&](int slot, int j) __attribute__((always_inline)) {
    const double* ph = PHI_LDS ? phi_lds + (size_t)j * 2 * L : a.phi + (size_t)slot * 2 * L;
#pragma unroll
    for (int i = 0; i < S::BR; ++i) pu[i] = ph[row_real[i] ? rb * S::BR + i : L - 1];
#pragma unroll
    for (int jj = 0; jj < S::BC; ++jj) pv[jj] = ph[L + (col_real[jj] ? cb * S::BC + jj : L - 1)];
    pvo = ph[L + out_ic];
  };
  // tables are loaded two steps ahead, one where the argmins take the registers
  // (k_adj64 at 64 labels: 5 registers spilled where messages stay in memory, none
  // in LDS; with the candidates kept from the passes and two steps ahead, 142:
  // forward with records of 100 nodes 2.77 us a matching, 2.25 now, backward 4.10,
  // 2.92 now)
  constexpr int DEPTH = REC && LT == 64 ? 1 : 2;
  double t0[S::BR][S::BC], t1[S::BR][S::BC], t2[S::BR][S::BC];
  load_tile64(t0, first);
  if (DEPTH == 2) load_tile64(t1, first + (owned > 1 ? G : 0));
  // (a workgroup that owns one slot reads back the messages it wrote at the
  // previous step: after the next step's first barrier)
  if (owned > 1) load_phi64(first, 0);
  int parity = 0, it = 0, j = 0, jp = DEPTH % owned;
  SlotInfo si = ld_const(slots + first);
  unsigned char* rec_prev = nullptr;  // REC: the s2 record of the previous step
  auto finish_s2 = [&](int par) __attribute__((always_inline)) {
    int s2 = sm.redi[par][0][out_ic];
#pragma unroll
    for (int w = 1; w < S::W; ++w) s2 = min(s2, sm.redi[par][w][out_ic]);
    *(outk && !out_u ? rec_prev + out_i : reinterpret_cast<unsigned char*>(sink)) = (unsigned char)min(s2, L - 1);
  };
  auto step = [&](double (&xc)[S::BR][S::BC], double (&xp)[S::BR][S::BC], int q) __attribute__((always_inline)) -> bool {
    const int slot = first + j * G;
    const int nj = j + 1 == owned ? 0 : j + 1;
    const int nxt = uni(first + nj * G);
    const SlotInfo si_next = ld_const(slots + nxt);
    load_tile64(xp, first + jp * G);
    if (PHI_LDS && owned > 1) load_phi64(slot, j);
    const int node = out_u ? si.u : si.v;
    const unsigned ver = (unsigned)it * (unsigned)(out_u ? si.deg_u : si.deg_v) + (unsigned)(out_u ? si.pos_u : si.pos_v) + 1u;
    unsigned long long* mb_dst = outk ? mb + (size_t)node * mbs + 2 * out_i : sink;
    asm volatile("" ::"v"(mb_dst), "v"(ver));
#pragma unroll
    for (int i = 0; i < S::BR; ++i)
#pragma unroll
      for (int jj = 0; jj < S::BC; ++jj) {
        xc[i][jj] = row_real[i] && col_real[jj] ? xc[i][jj] : __builtin_inf();
        asm volatile("" : "+v"(xc[i][jj]));  // (here, not behind the barrier)
      }
    __syncthreads();  // the step's nodes are in LDS
    if (owned == 1) load_phi64(slot, j);
    double au[S::BR], av[S::BC];
#pragma unroll
    for (int jj = 0; jj < S::BC; ++jj) {
      av[jj] = sm.hv[parity][col_real[jj] ? cb * S::BC + jj : L - 1] - pv[jj];
    }
#pragma unroll
    for (int i = 0; i < S::BR; ++i) au[i] = sm.hu[parity][row_real[i] ? rb * S::BR + i : L - 1] - pu[i];
    double oa = sm.hv[parity][out_ic] - pvo;  // a of this lane's output
    if (out_u) {
      oa = au[0];
#pragma unroll
      for (int i = 1; i < S::BR; ++i)
        if (cb == i) oa = au[i];
    }
    // pass 1: p(s) = min_t [th(s,t) + a_v(t)], b = (a_u - p) / 2
    double pm[S::BR], b[S::BR];
#pragma unroll
    for (int i = 0; i < S::BR; ++i) {
      double mn = xc[i][0] + av[0];
#pragma unroll
      for (int jj = 1; jj < S::BC; ++jj) mn = vmin(mn, xc[i][jj] + av[jj]);
      pm[i] = mn;
    }
    row16_min_n<S::BR>(pm);
#pragma unroll
    for (int i = 0; i < S::BR; ++i) b[i] = row_real[i] ? 0.5 * (au[i] - pm[i]) : 0.0;
    // pass 2: q(t) = min_s [th(s,t) + b(s)]
    double qv[S::BC];
#pragma unroll
    for (int jj = 0; jj < S::BC; ++jj) {
      double mn = xc[0][jj] + b[0];
#pragma unroll
      for (int i = 1; i < S::BR; ++i) mn = vmin(mn, xc[i][jj] + b[i]);
      qv[jj] = mn;
    }
    col4_min_store64<S::BC>(qv, sm.red[wave], cb, lane);
    __syncthreads();  // mid-step barrier
    double part[S::W][S::BC], opart[S::W];
#pragma unroll
    for (int w = 0; w < S::W; ++w) {
#pragma unroll
      for (int jj = 0; jj < S::BC; ++jj) part[w][jj] = sm.red[w][cb * S::BC + jj];
      opart[w] = sm.red[w][out_ic];
    }
    const int aborted = sm.abort_flag;
    __builtin_amdgcn_sched_barrier(0);
    if (aborted == q + 1) return false;
    double oq = opart[0];
#pragma unroll
    for (int w = 1; w < S::W; ++w) oq = vmin(oq, opart[w]);
#pragma unroll
    for (int jj = 0; jj < S::BC; ++jj) {
      double mn = part[0][jj];
#pragma unroll
      for (int w = 1; w < S::W; ++w) mn = vmin(mn, part[w][jj]);
      qv[jj] = col_real[jj] ? mn : 0.0;
    }
    // pass 3: r(s) = min_t [th(s,t) - q(t)]; only lane cb = i of a row block
    // needs row i's minimum (see the FP32 engine)
    double r[S::BR];
#pragma unroll
    for (int i = 0; i < S::BR; ++i) {
      double mn = xc[i][0] - qv[0];
#pragma unroll
      for (int jj = 1; jj < S::BC; ++jj) mn = vmin(mn, xc[i][jj] - qv[jj]);
      r[i] = mn;
    }
    row16_min_n<S::BR, 3>(r);
    const int half_row = cb < 8 ? cb : 15 - cb;
    double sel = r[0];
#pragma unroll
    for (int i = 1; i < S::BR; ++i) sel = half_row == i ? r[i] : sel;
    sel = vmin(sel, dpp_f<0x140>(sel));
    // push back: U_u = a_u + r, phi[0] = r; U_v = a_v + q, phi[1] = q
    const double omsg = out_u ? sel : oq;
    mb64_put(mb_dst, oa + omsg, ver);
    if (PHI_LDS) {
      if (outk) phi_lds[(size_t)j * 2 * L + (out_u ? 0 : L) + out_i] = omsg;
    } else {
      *(outk ? a.phi + (size_t)slot * 2 * L + (out_u ? 0 : L) + out_i : reinterpret_cast<double*>(sink + 8)) = omsg;
    }
    if constexpr (REC) {
      // argmins, after everything another workgroup waits for
      if (rec_prev) finish_s2(parity ^ 1);
      if constexpr (LT > 32) {
        // (the candidates are formed anew: kept from the passes, they would
        // not fit the registers beside the tiles)
#pragma unroll
        for (int jj = 0; jj < S::BC; ++jj) asm volatile("" : "+v"(av[jj]), "+v"(qv[jj]));
#pragma unroll
        for (int i = 0; i < S::BR; ++i) asm volatile("" : "+v"(b[i]));
      }
      int a1 = 255, a3 = 255;
#pragma unroll
      for (int i = 0; i < S::BR; ++i) {
        int k1 = 255, k3 = 255;
        const double rf = vmin(r[i], dpp_f<0x140>(r[i]));
#pragma unroll
        for (int jj = S::BC - 1; jj >= 0; --jj) {
          k1 = xc[i][jj] + av[jj] == pm[i] ? cb * S::BC + jj : k1;
          k3 = xc[i][jj] - qv[jj] == rf ? cb * S::BC + jj : k3;
        }
        k1 = row16_imin(k1);
        k3 = row16_imin(k3);
        a1 = cb == i ? k1 : a1;
        a3 = cb == i ? k3 : a3;
      }
#pragma unroll
      for (int jj = 0; jj < S::BC; ++jj) {
        int k2 = 255;
#pragma unroll
        for (int i = S::BR - 1; i >= 0; --i) k2 = xc[i][jj] + b[i] == qv[jj] ? rb * S::BR + i : k2;
        k2 = col4_imin(k2);
        if (lane < 16) sm.redi[parity][wave][cb * S::BC + jj] = k2;
      }
      unsigned char* rc = a.rec + (size_t)it * rec_it + (size_t)slot * 3 * L;
      unsigned char* sk = reinterpret_cast<unsigned char*>(sink + 16);
      *(outk && out_u ? rc + out_i : sk) = (unsigned char)min(a1, L - 1);
      *(outk && out_u ? rc + 2 * L + out_i : sk) = (unsigned char)min(a3, L - 1);
      rec_prev = rc + L;
    }
    if (!PHI_LDS && owned > 1 && q + 1 < total) load_phi64(nxt, nj);
    si = si_next;
    parity ^= 1;
    j = nj;
    if (j == 0) ++it;
    if (++jp == owned) jp = 0;
    return true;
  };
  int q = 0;
  if (DEPTH == 2) {
    for (; q + 3 <= total; q += 3) {
      if (!step(t0, t2, q)) return;
      if (!step(t1, t0, q + 1)) return;
      if (!step(t2, t1, q + 2)) return;
    }
    if (q < total && !step(t0, t2, q)) return;
    if (q + 1 < total && !step(t1, t0, q + 1)) return;
  } else {
    for (; q + 2 <= total; q += 2) {
      if (!step(t0, t1, q)) return;
      if (!step(t1, t0, q + 1)) return;
    }
    if (q < total && !step(t0, t1, q)) return;
  }
  if (REC) {
    __syncthreads();
    finish_s2(parity ^ 1);
  }
  if (PHI_LDS) {
    __syncthreads();
    for (int slot = first, j2 = 0; slot < m; slot += G, ++j2)
      for (int k = tid; k < 2 * L; k += NT + 128) a.phi[(size_t)slot * 2 * L + k] = phi_lds[j2 * 2 * L + k];
  }
}

}  // namespace mplpxx
