// The FP32 mailbox engine's kernel (device_common.h's mb_run on one model) and
// its tiles of 80, 96 and 112 labels.
#pragma once
#include "device_common.h"

namespace mplpxx {

// LDS behind the last slot's messages: whole tile rows are read (mb_run)
constexpr size_t kPhiLdsTail = 128 * sizeof(float);

// Label counts that run on a tile of their own multiple of 16 instead of the
// next power of two.  The update's passes run over every entry of the tile: one
// of 80 has 25/64 of the entries of one of 128, and its registers hold without
// spills.  Microseconds a matching on complete graphs of 40 nodes, tile of 128
// / own tile: 65 labels 2.33 / 1.66, 80 2.33 / 1.62, 96 2.33 / 1.74, 100
// 2.34 / 2.00, 112 2.33 / 1.92.  (A tile of 48 gains nothing over 64: at 40
// labels 1.41 / 1.57, at 48 1.41 / 1.39.)
constexpr bool mb_odd_tile(int L) { return L > 64 && L <= 112; }
// the kernel of such a tile, for occupancy queries
const void* mb_odd_kernel(int L);
// (four compute waves, dense tables, (H), no trace; a.wgs is set)
hipError_t launch_mb_odd(const HsArgs<float>& a, unsigned long long* mb, int grid, int iters, int phi_in_lds,
                         size_t dyn_lds, hipStream_t st);

template <int LT, int NT, bool PHI_LDS, bool FULL, bool TRACE, bool PHI_FAR, int DEPTH = (LT <= 64 ? 2 : 1),
          int KIND = kCostDense, int RULE = MPLPXX_RULE_H, bool SNAP = false>
__global__ void __launch_bounds__(NT + 128) k_persistent_mb(HsArgs<float> a, unsigned long long* __restrict__ mb,
                                                            int iters) {
  __shared__ SmemMB<LT, NT> sm;
  extern __shared__ float phi_lds[];
  const int tid = threadIdx.x;
  const int L = FULL ? LT : a.L;
  const int G = a.wgs.G, wg = wg_logical(a.wgs, blockIdx.x);
  if (wg >= G || wg >= a.m) return;
  if (tid == 0) sm.abort_flag = 0;
  if (PHI_LDS) {
    for (int slot = wg, j = 0; slot < a.m; slot += G, ++j)
      for (int k = tid; k < 2 * L; k += NT + 128) phi_lds[j * 2 * L + k] = a.phi[(size_t)slot * 2 * L + k];
  }
  __syncthreads();
  MbView v{a.tables, a.phi, mb, a.slots, a.deg, a.trace, a.trace_e, a.stamps, L, a.m, a.n, nullptr, nullptr,
           a.sink + (size_t)wg * (NT + 128), a.mbs, a.snap};
  if (!mb_run<LT, NT, PHI_LDS, FULL, TRACE, false, PHI_FAR, DEPTH, KIND, RULE, SNAP>(v, wg, G, iters, sm, phi_lds,
                                                                               a.spin_limit, a.err))
    return;
  __syncthreads();
  if (PHI_LDS) {
    for (int slot = wg, j = 0; slot < a.m; slot += G, ++j)
      for (int k = tid; k < 2 * L; k += NT + 128) a.phi[(size_t)slot * 2 * L + k] = phi_lds[j * 2 * L + k];
  }
}

}  // namespace mplpxx
