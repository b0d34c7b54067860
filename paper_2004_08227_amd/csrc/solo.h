// Host interface of the one-workgroup engine for small models (solo.hip).
#pragma once
#include "common.h"

namespace mplpxx {

template <typename T> struct SoloArgs {
  const T* tables;        // [m][L][L] slot order
  T* phi;                 // [m][2][L] slot order
  T* U;                   // [n][L]
  T* Ulo;                 // [n][L] (FP32)
  const SlotInfo* slots;  // [m]
  double* trace;          // [iters][n] node minima after each iteration, or null
  float* trace_e;         // [iters][m] edge terms (FP32 traces)
  int L, m, n, S;
};

// LDS of the launch: unaries, messages, node pairs, matching offsets
inline size_t solo_lds_bytes(int n, int L, int m, int S, size_t esz) {
  return ((size_t)n * L * (esz == 4 ? 2 : 1) + (size_t)m * 2 * L) * esz + ((size_t)m + S + 1) * sizeof(int);
}
constexpr size_t kSoloLds = 144 * 1024;
// behind the unaries and the messages (whole tile rows are read); beside the limit
inline size_t solo_lds_pad(int L, size_t esz) { return (size_t)(L <= 8 ? 8 : L <= 16 ? 16 : 32) * (8 + esz); }
// waves a workgroup can have (more registers for the 32-label tile)
constexpr int solo_max_waves(int LT) { return LT == 32 ? 4 : 16; }

// Whether the model runs on one workgroup: its state fits in LDS, and one wave
// per edge of its largest matching gives a shorter step than the mailbox
// engines.  The step grows with the waves a SIMD has to issue for, the mailbox
// step does not (microseconds a matching, one workgroup / mailboxes, at 2, 8
// and 16 edges a matching):
//   FP32, L = 8   0.35 / 1.18   0.47 / 1.11   0.72 / 1.07
//   FP32, L = 16  0.51 / 1.07   0.66 / 1.12   0.99 / 1.08
//   FP32, L = 32  0.86 / 1.16   1.73 / 1.14
//   FP32 traces, L = 8   0.54 / 1.29   0.65 / 1.27   0.93 / 1.21
//   FP32 traces, L = 16  0.84 / 1.23   1.18 / 1.37   1.65 / 1.34
//   FP64, L = 8   0.32 / 1.13   0.41 / 1.13   0.61 / 1.13
//   FP64, L = 16  0.45 / 1.14   0.72 / 1.14   0.94 / 1.14 (12 edges)  1.14
//   FP64, L = 32  1.05 / 1.31   1.16 / 1.31 (3 edges)   1.92 / 1.31
//   FP64 traces, L = 16  0.52 / 1.13   0.76 / 1.13   0.97 / 1.11 (12 edges)
//   FP64 traces, L = 32  1.12 / 1.31   1.65 / 1.31 (4 edges)
inline bool solo_fits(int n, int L, int m, int S, int max_step, size_t esz, bool trace) {
  if (m < 1 || n > 32767 || L > 32 || solo_lds_bytes(n, L, m, S, esz) > kSoloLds) return false;
  if (L <= 8) return max_step <= 16;
  if (L <= 16) return max_step <= (esz == 8 ? 12 : trace ? 8 : 16);
  return max_step <= (esz == 8 ? (trace ? 2 : 3) : (trace ? 0 : 2));
}

// one workgroup of max_step waves (solo_fits holds)
template <typename T> hipError_t launch_solo(const SoloArgs<T>& a, int max_step, int iters, hipStream_t st);

}  // namespace mplpxx
