// The FP32 mailbox engine keeping the messages of every iteration (mb_kernel.h),
// for bounds and labellings per iteration: `iters` iterations in one launch,
// each result also stored to its iteration's copy, behind everything that
// another workgroup waits for.
#include "host_util.h"
#include "mb_kernel.h"

namespace mplpxx {

static size_t snap_lds(int m, int L, int grid) { return ((size_t)m + grid - 1) / grid * 2 * L * sizeof(float); }
// (the default way of the engine up to 64 labels; other models run one
// iteration a launch, with a copy after each)
bool mb_snap_fits(int m, int L, int grid) {
  return L <= 64 && grid > 0 && m / grid >= 4 && snap_lds(m, L, grid) <= kPhiLdsBudget;
}

template <int LT>
static hipError_t mb_snap_one(const HsArgs<float>& a, unsigned long long* mb, int grid, int iters, hipStream_t st) {
  void* args[] = {(void*)&a, (void*)&mb, (void*)&iters};
  const void* f =
      a.L == LT ? (const void*)k_persistent_mb<LT, 256, true, true, false, true, 2, kCostDense, MPLPXX_RULE_H, true>
                : (const void*)k_persistent_mb<LT, 256, true, false, false, true, 2, kCostDense, MPLPXX_RULE_H, true>;
  const hipError_t e =
      hipLaunchCooperativeKernel(f, dim3(a.wgs.launch), dim3(256 + 128), args, snap_lds(a.m, a.L, grid) + kPhiLdsTail, st);
  if (e != hipSuccess) (void)hipGetLastError();  // (a refused launch: not left for a later launch check)
  return e;
}

hipError_t launch_mb_snap(const HsArgs<float>& a, unsigned long long* mb, int grid, int iters, hipStream_t st) {
  if (!mb_snap_fits(a.m, a.L, grid) || !a.snap) return hipErrorInvalidValue;
  if (a.L <= 16) return mb_snap_one<16>(a, mb, grid, iters, st);
  if (a.L <= 32) return mb_snap_one<32>(a, mb, grid, iters, st);
  return mb_snap_one<64>(a, mb, grid, iters, st);
}

}  // namespace mplpxx
