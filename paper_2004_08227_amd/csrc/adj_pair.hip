// The adjoint forward of an FP32 handle: its FP32 run beside the FP64 run that
// is differentiated.
//
// Both runs are chains of dependent matchings that leave most of the chip idle
// (a matching of a complete graph of n nodes has n / 2 edges) and they share
// nothing but the graph, so one launch gives each a part of the workgroups:
// [0, f.grid) the FP64 forward (mailbox64.h), the rest the FP32 engine
// (device_common.h), every workgroup on a compute unit of its own.  The launch
// takes as long as the FP64 run, the longer of the two.  (The FP32 run's own
// time, clk: complement of its first workgroup's start and its last one's end on
// the device's clock.)  Milliseconds of a
// forward of 10 iterations with two checkpoints, in turn / side by side: 40
// nodes of 16 labels 1.12 / 0.68, 100 of 32 2.85 / 1.63, 100 of 64 5.17 / 4.07,
// 200 of 32 5.45 / 3.20, 256 of 16 6.17 / 3.33.
#include <algorithm>

#include "device_common.h"
#include "host_util.h"
#include "mailbox64.h"
#include "mb_kernel.h"

namespace mplpxx {

static_assert(kPairNT == kF64NT, "both roles have workgroups of one size");

template <int LT, bool REC>
__global__ void __launch_bounds__(kF64NT + 128) k_adj_pair(Fwd64Args f, HsArgs<float> a,
                                                           unsigned long long* __restrict__ mb, int grid32,
                                                           unsigned long long* __restrict__ clk) {
  constexpr int NT = kF64NT;
  __shared__ SmemF64<LT> smf;
  constexpr int LT32 = LT <= 32 ? LT : 64;
  __shared__ SmemMB<LT32, NT> sm;
  extern __shared__ __align__(16) double pair_lds[];
  const int tid = threadIdx.x;
  const int b = blockIdx.x;
  if (b < f.grid) {
    if (failed_before(f.err, smf.abort_flag)) return;
    fwd64_role<LT, true, REC, false>(f, b, f.grid, smf, pair_lds);
    return;
  }
  if (failed_before(a.err, sm.abort_flag)) return;
  if (tid == 0) atomicMax(clk, ~(unsigned long long)wall_clock64());
  const int first = b - f.grid;
  const int L = a.L;
  float* phi_lds = reinterpret_cast<float*>(pair_lds);
  for (int slot = first, j = 0; slot < a.m; slot += grid32, ++j)
    for (int k = tid; k < 2 * L; k += NT + 128) phi_lds[j * 2 * L + k] = a.phi[(size_t)slot * 2 * L + k];
  __syncthreads();
  MbView v{a.tables, a.phi, mb, a.slots, a.deg, nullptr, nullptr, nullptr, L, a.m, a.n, nullptr, nullptr,
           a.sink + (size_t)first * (NT + 128), a.mbs};
  if (!mb_run<LT32, NT, true, false, false, false, true, 2, kCostDense, MPLPXX_RULE_H>(v, first, grid32, f.iters, sm,
                                                                                      phi_lds, a.spin_limit, a.err))
    return;
  __syncthreads();
  for (int slot = first, j = 0; slot < a.m; slot += grid32, ++j)
    for (int k = tid; k < 2 * L; k += NT + 128) a.phi[(size_t)slot * 2 * L + k] = phi_lds[j * 2 * L + k];
  if (tid == 0) atomicMax(clk + 1, (unsigned long long)wall_clock64());
}

template <int LT>
static hipError_t adj_pair_one(const Fwd64Args& f, const HsArgs<float>& a, unsigned long long* mb, int grid32,
                               unsigned long long* clk, size_t lds, hipStream_t st) {
  void* args[] = {(void*)&f, (void*)&a, (void*)&mb, (void*)&grid32, (void*)&clk};
  const void* fn = f.rec ? (const void*)k_adj_pair<LT, true> : (const void*)k_adj_pair<LT, false>;
  const hipError_t e = hipLaunchCooperativeKernel(fn, dim3(f.grid + grid32), dim3(kF64NT + 128), args, lds, st);
  if (e != hipSuccess) (void)hipGetLastError();  // (a refused launch: not left for a later launch check)
  return e;
}

// Messages of both roles stay in LDS, and the FP32 run's are read two steps
// ahead.
static size_t pair_lds64(int m, int L, int grid) { return ((size_t)m + grid - 1) / grid * 2 * L * sizeof(double); }
static size_t pair_lds32(int m, int L, int grid) { return ((size_t)m + grid - 1) / grid * 2 * L * sizeof(float); }
bool adj_pair_fits(int m, int L, int grid64, int grid32) {
  return L <= 64 && grid64 > 0 && grid32 > 0 && m / grid32 >= 4 && m >= grid64 &&
         pair_lds64(m, L, grid64) <= kPhiLdsBudget && pair_lds32(m, L, grid32) <= kPhiLdsBudget;
}

hipError_t launch_adj_pair(const Fwd64Args& f, const HsArgs<float>& a, unsigned long long* mb, int grid32,
                           unsigned long long* clk, hipStream_t st) {
  if (f.L != a.L || f.m != a.m || f.iters <= 0 || !adj_pair_fits(f.m, f.L, f.grid, grid32)) return hipErrorInvalidValue;
  const size_t lds = std::max(pair_lds64(f.m, f.L, f.grid), pair_lds32(f.m, f.L, grid32) + kPhiLdsTail);
  if (f.L <= 16) return adj_pair_one<16>(f, a, mb, grid32, clk, lds, st);
  if (f.L <= 32) return adj_pair_one<32>(f, a, mb, grid32, clk, lds, st);
  if (f.L <= 48) return adj_pair_one<48>(f, a, mb, grid32, clk, lds, st);
  return adj_pair_one<64>(f, a, mb, grid32, clk, lds, st);
}

}  // namespace mplpxx
