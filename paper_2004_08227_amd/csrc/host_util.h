// Host-side helpers shared by the solver and batch runtimes.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <string>

#include "common.h"

namespace mplpxx {

// text of the last failure on the calling thread (mplpxx_last_error)
inline thread_local std::string g_last_error;

// Records the failure's text.  It also takes the HIP runtime's last error,
// which a failed runtime call leaves set: left there, the next launch check
// of a later call (hipGetLastError after a launch) would report it again.
inline int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_last_error = buf;
  (void)hipGetLastError();
  return code;
}

#define HIP_TRY(expr)                                                                                       \
  do {                                                                                                      \
    hipError_t e_ = (expr);                                                                                 \
    if (e_ != hipSuccess) {                                                                                 \
      if (e_ == hipErrorOutOfMemory) return ::mplpxx::fail(MPLPXX_ENOMEM, "%s: %s", #expr, hipGetErrorString(e_)); \
      return ::mplpxx::fail(MPLPXX_EDEVICE, "%s: %s", #expr, hipGetErrorString(e_));                       \
    }                                                                                                       \
  } while (0)

// Truncated linear parameters (w, tau) per edge: finite, w >= 0, tau >= 0,
// and the costs fl(w * tau), fl(w * d) within the FP32 cost bound.
inline int check_trunc_linear_params(const float* prm, int64_t m) {
  for (int64_t e = 0; e < m; ++e) {
    const float w = prm[2 * e], tau = prm[2 * e + 1];
    if (!(w >= 0.0f && tau >= 0.0f && std::isfinite(w) && std::isfinite(tau)))
      return fail(MPLPXX_EINVAL, "edge %lld: truncated linear costs need finite w >= 0 and tau >= 0", (long long)e);
    if (!(w * tau <= (float)MPLPXX_F32_MAX_COST) || !(w * (float)MPLPXX_MAX_LABELS <= (float)MPLPXX_F32_MAX_COST))
      return fail(MPLPXX_EINVAL, "edge %lld: truncated linear cost above %g", (long long)e, MPLPXX_F32_MAX_COST);
  }
  return MPLPXX_OK;
}

// Truncated quadratic parameters (w, tau) per edge: finite, w >= 0, tau >= 0,
// and every entry fl(w * min(d^2, tau)) within the FP32 cost bound.
inline int check_trunc_quad_params(const float* prm, int64_t m) {
  const float dmax = (float)((MPLPXX_MAX_LABELS - 1) * (MPLPXX_MAX_LABELS - 1));
  for (int64_t e = 0; e < m; ++e) {
    const float w = prm[2 * e], tau = prm[2 * e + 1];
    if (!(w >= 0.0f && tau >= 0.0f && std::isfinite(w) && std::isfinite(tau)))
      return fail(MPLPXX_EINVAL, "edge %lld: truncated quadratic costs need finite w >= 0 and tau >= 0", (long long)e);
    if (!(w * (tau < dmax ? tau : dmax) <= (float)MPLPXX_F32_MAX_COST))
      return fail(MPLPXX_EINVAL, "edge %lld: truncated quadratic cost above %g", (long long)e, MPLPXX_F32_MAX_COST);
  }
  return MPLPXX_OK;
}

// parameter check of a structured cost kind (Potts weights are checked as
// costs by the caller)
inline int check_structured_params(int kind, const float* prm, int64_t m) {
  if (kind == MPLPXX_COST_TRUNC_LINEAR) return check_trunc_linear_params(prm, m);
  if (kind == MPLPXX_COST_TRUNC_QUAD) return check_trunc_quad_params(prm, m);
  return MPLPXX_OK;
}
inline bool known_cost_kind(int kind) {
  return kind == MPLPXX_COST_POTTS || kind == MPLPXX_COST_TRUNC_LINEAR || kind == MPLPXX_COST_TRUNC_QUAD;
}

// Mailbox engines: messages of a workgroup's slots kept in LDS up to this
// size
constexpr size_t kPhiLdsBudget = 96 * 1024;

// Workgroups of the mailbox engines.
//  * A matching with more edges than there are compute units: one workgroup
//    per edge of it as far as they fit (`per_cu` on each compute unit), so a
//    workgroup runs about one update per matching instead of several one
//    after another.
//  * Otherwise two per edge of the largest matching, at most one per compute
//    unit: while one workgroup updates its edge, the one that owns the edge of
//    the next matching has its table and waits.  Workgroups beyond that only
//    poll the same mailboxes and delay the stores into them; with one per edge
//    a workgroup's own preparation of its next step joins the chain.
//    Microseconds a matching with one, two and 256 / (edges of a matching)
//    workgroups per edge: n = 33, L = 11 1.22 / 1.27 / 1.52; n = 61, L = 21
//    1.32 / 1.31 / 1.45; n = 200, L = 64 1.60 / 1.36 / 1.37; n = 40, L = 100
//    2.89 / 2.36 / 2.57.
//    More where the messages of a workgroup's slots would not fit in LDS
//    otherwise.
template <typename F>
inline int mb_default_grid(int max_step, int num_cus, long long m, int L, const F& per_cu, size_t esz = sizeof(float)) {
  if (max_step > num_cus) return std::max(num_cus, std::min(max_step, per_cu() * num_cus));
  const long long slots_in_lds = (long long)(kPhiLdsBudget / (2 * esz * L));
  const long long fit = (m + slots_in_lds - 1) / slots_in_lds;
  return (int)std::min<long long>(num_cus, std::max<long long>(2ll * max_step, fit));
}

// `k` iterations of a mailbox engine on `grid` workgroups, f(done, c) for the next
// c of them: in as few launches as a workgroup can count its updates of in 31 bits
// (a state passes from one launch to the next bit for bit).
template <typename F> inline hipError_t in_launches(int k, long long m, int grid, const F& f) {
  const long long owned = (m + grid - 1) / grid;
  const int most = (int)std::max(1ll, (1ll << 30) / std::max(1ll, owned));
  hipError_t e = hipSuccess;
  for (int done = 0, c; done < k && e == hipSuccess; done += c) {
    c = std::min(most, k - done);
    e = f(done, c);
  }
  return e;
}

// messages of at least this size are put into the caller's edge order on the
// device when a state is read (figures at mplpxx_get_state)
constexpr size_t kExportOnDevice = 1 << 20;

// device workspaces of calls on a handle stay with it up to this size, larger ones
// are given back when the call ends
constexpr size_t kKeepWorkspace = (size_t)96 << 20;
template <typename T> inline void give_back_large(T*& p, size_t bytes) {
  if (!p || bytes <= kKeepWorkspace) return;
  (void)hipFree(p);
  p = nullptr;
}

// smallest register tile (16, 32, 64, 128) holding L labels
inline int next_tile(int L) {
  int lt = 16;
  while (lt < L) lt *= 2;
  return lt;
}

}  // namespace mplpxx
