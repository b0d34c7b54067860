// The FP32 mailbox engine on tiles that are no power of two (mb_kernel.h).
#include "mb_kernel.h"

namespace mplpxx {

// tables two steps ahead where the ring of three tiles leaves registers for
// the rest
template <int LT> constexpr int odd_depth() { return LT <= 96 ? 2 : 1; }

template <int LT>
static hipError_t mb_odd_one(const HsArgs<float>& a, unsigned long long* mb, int grid, int iters, int phi_in_lds,
                             size_t dyn_lds, hipStream_t st) {
  constexpr int D = odd_depth<LT>();
  const bool full = a.L == LT;
  // messages prefetched with the tables when every workgroup owns enough slots
  const bool far = (a.m / grid) >= D + 2;
  void* args[] = {(void*)&a, (void*)&mb, (void*)&iters};
#define MPLPXX_G(P, F, A) (const void*)k_persistent_mb<LT, 256, P, F, false, A, D>
  const void* f = phi_in_lds ? (full ? (far ? MPLPXX_G(true, true, true) : MPLPXX_G(true, true, false))
                                     : (far ? MPLPXX_G(true, false, true) : MPLPXX_G(true, false, false)))
                             : (full ? (far ? MPLPXX_G(false, true, true) : MPLPXX_G(false, true, false))
                                     : (far ? MPLPXX_G(false, false, true) : MPLPXX_G(false, false, false)));
#undef MPLPXX_G
  const hipError_t e = hipLaunchCooperativeKernel(f, dim3(a.wgs.launch), dim3(256 + 128), args, dyn_lds, st);
  if (e != hipSuccess) (void)hipGetLastError();  // (a refused launch: not left for a later launch check)
  return e;
}

const void* mb_odd_kernel(int L) {
  switch ((L + 15) / 16) {
    case 5: return (const void*)k_persistent_mb<80, 256, false, false, false, true, odd_depth<80>()>;
    case 6: return (const void*)k_persistent_mb<96, 256, false, false, false, true, odd_depth<96>()>;
    default: return (const void*)k_persistent_mb<112, 256, false, false, false, true, odd_depth<112>()>;
  }
}

hipError_t launch_mb_odd(const HsArgs<float>& a, unsigned long long* mb, int grid, int iters, int phi_in_lds,
                         size_t dyn_lds, hipStream_t st) {
  switch ((a.L + 15) / 16) {
    case 5: return mb_odd_one<80>(a, mb, grid, iters, phi_in_lds, dyn_lds, st);
    case 6: return mb_odd_one<96>(a, mb, grid, iters, phi_in_lds, dyn_lds, st);
    case 7: return mb_odd_one<112>(a, mb, grid, iters, phi_in_lds, dyn_lds, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mplpxx
