// Internal declarations shared by the host runtime and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/mplpxx.h"

namespace mplpxx {

// Workgroups of a launch over `count` items that takes them at a grid stride: a
// launch's threads are a 32-bit number, and 2^20 workgroups are far more than run
// at once.
constexpr unsigned kMaxBlocks = 1u << 20;
inline unsigned stride_blocks(size_t count) { return count < kMaxBlocks ? (unsigned)count : kMaxBlocks; }

enum { ENGINE_AUTO = 0, ENGINE_STEP = 1, ENGINE_PERSISTENT = 2 };

// Pairwise cost of a model: a dense L x L table per edge, or a structured
// cost given by a few parameters per edge (MPLPXX_COST_* of the header):
// Potts w [s != t] (1 parameter: w), truncated linear w min(|s - t|, tau)
// and truncated quadratic w min((s - t)^2, tau) (2 parameters: w, tau).  The
// parameters of slot i sit at tables[i * cost_params(kind)].
constexpr int kCostDense = 0;
__host__ __device__ constexpr int cost_params(int kind) {
  return kind == MPLPXX_COST_TRUNC_LINEAR || kind == MPLPXX_COST_TRUNC_QUAD ? 2 : 1;
}
// fl(w * min(d, tau)) for a distance term d that is exact in FP32: the
// entry of the expanded table of the truncated kinds
__host__ __device__ inline float truncated_cost(float w, float tau, float d) { return w * (d < tau ? d : tau); }
// th(s, t) of a structured cost from its parameters (the expanded table)
__host__ __device__ inline float structured_cost(int kind, const float* prm, int s, int t) {
  if (kind == MPLPXX_COST_TRUNC_LINEAR || kind == MPLPXX_COST_TRUNC_QUAD) {
    const float d = (float)(s > t ? s - t : t - s);
    return truncated_cost(prm[0], prm[1], kind == MPLPXX_COST_TRUNC_QUAD ? d * d : d);
  }
  return s == t ? 0.0f : prm[0];
}

// timestamps per slot: 4 in normal builds; a diagnostics build
// (-DMPLPXX_FINE_STAMPS=1) records 4 more points inside the edge update
#ifndef MPLPXX_FINE_STAMPS
#define MPLPXX_FINE_STAMPS 0
#endif
constexpr int kStampStride = MPLPXX_FINE_STAMPS ? 8 : 4;

// One entry per schedule slot (slot i = i-th edge of the schedule queue).
// Elements allocated (zeroed) past the end of every tables and messages
// array: the FP32 engines load whole tile rows without clamping the column
// index, so a row of a table (or of a slot's messages) may read up to LT
// elements into whatever follows it.
constexpr size_t kTailPad = 256;

struct SlotInfo {
  int e;       // index of the edge in the caller's edge list
  int u, v;    // its nodes, u < v
  int pos_u;   // number of edges of u that precede this one in the queue
  int pos_v;   // same for v
  int deg_u;   // degree of u (updates of u per iteration)
  int deg_v;   // degree of v
  int step;    // index of its matching in the schedule
};

// Words of one node's row of mailboxes: whole 128-byte lines.  Rows of L words
// share lines wherever L is no multiple of 16, and the polls of one node's
// waiters then delay the stores of another node's producer.  Microseconds a
// matching with rows of L words and of whole lines (complete graphs): n = 33,
// L = 11 1.27 -> 1.15; n = 61, L = 21 1.31 -> 1.21; n = 200, L = 60 1.55 ->
// 1.43; multiples of 16 the same.
__host__ __device__ constexpr int mb_row_words(int L) { return (L + 15) / 16 * 16; }

// ---------------------------------------------------------------------------
// Which compute die a workgroup of the FP32 mailbox engine runs on.
//
// The dispatcher hands workgroups to the 8 dies (XCDs) in turn.  In the schedule
// of a complete graph a node moves from one position of the matching to a
// neighbouring one, so with positions dealt out like that every handoff crosses
// dies; with blocks of neighbouring positions on one die only those at the
// blocks' ends do (a handoff takes 0.31 to 0.35 us within a die, 0.40 to 0.54
// between dies).  Positions are the slots of a matching; the map needs all
// matchings to have the same number `ms` of them and G to be a multiple of it, and
// leaves the slots that logical workgroup w owns (w, w + G, ...) as they are.
// Workgroups beyond a die's last position leave at once.  Were workgroups dealt
// out differently, only the gain would be lost.
//
// Microseconds a matching, in turn / in blocks, complete graphs of n nodes and L
// labels: n = 40, L = 24 1.20 / 1.13; 61, 21 1.22 / 1.13; 100, 9 1.11 / 1.07; 100, 32
// 1.19 / 1.08; 150, 50 1.40 / 1.33; 160, 64 1.33 / 1.28; 200, 16 1.09 / 1.06; 200, 56
// 1.39 / 1.34; 120, 16 alone no gain, 1.075 / 1.088.  Tables beyond the 256 MB of the
// last-level cache come from HBM in every iteration, and there the blocks are
// slower: 200, 64 (326 MB) 1.342 / 1.363.  FP64 runs were within 1.5 % either way
// and keep the plain order.
// ---------------------------------------------------------------------------
struct WgMap {
  int G;       // logical workgroups
  int launch;  // workgroups of the launch
  int ms;      // positions of a matching (0: logical = launched)
};
constexpr int kDies = 8;
constexpr size_t kLastLevelCache = (size_t)256 << 20;
// even: all matchings have `ms` slots; cap: most workgroups of the launch
inline WgMap wg_map(int G, int ms, bool even, size_t table_bytes, int cap) {
  if (even && ms >= kDies && G % ms == 0 && table_bytes <= kLastLevelCache) {
    const int launch = kDies * ((ms + kDies - 1) / kDies) * (G / ms);
    if (launch <= cap) return WgMap{G, launch, ms};
  }
  return WgMap{G, G, 0};
}
// logical workgroup of launched workgroup b (G: none)
__host__ __device__ inline int wg_logical(const WgMap& w, int b) {
  if (w.ms == 0) return b;
  const int d = w.G / w.ms, die = b % kDies, i = b / kDies;
  const int p = die * w.ms / kDies + i / d;
  return p < (die + 1) * w.ms / kDies ? i % d * w.ms + p : w.G;
}

template <typename T> struct HsArgs {
  const T* tables;        // [m][L][L] slot order, read-only (Potts models: [m] weights)
  T* phi;                 // [m][2][L] slot order
  T* U;                   // [n][L]
  T* Ulo;                 // [n][L] FP32 only: bf16 correction of U (U = U + Ulo), else null
  const SlotInfo* slots;  // [m]
  const int* deg;         // [n]
  int* ver;               // [n] per-node update counters (persistent engine)
  int* err;               // device error word
  double* trace;          // [iters][n] per-node minima after the node's last update, or null
  float* trace_e;         // [iters][m][W] FP32 mailbox engine: per-wave minima of the edge terms, or null
  long long* stamps;      // [m][4] wall-clock stamps of the last iteration, or null
  unsigned long long* sink;  // FP32 mailbox engine: [grid][NT + 128] scratch words
  int L, m, n;
  int mbs;                // FP32 mailbox engine: words from one node's mailbox row to the next
  float* snap;            // [iters][m][2][L] messages of every iteration (launch_mb_snap)
  WgMap wgs;              // FP32 mailbox engine: the launch's workgroups
  long long spin_limit;
};

// ---------------------------------------------------------------------------
// Batched engine: many independent FP32 models in one persistent launch.
// ---------------------------------------------------------------------------
struct BatchModel {
  long long table_off;  // floats into the concatenated tables
  long long phi_off;    // floats into the concatenated messages
  long long u_off;      // entries into U / unaries (n*L per model)
  long long mb_off;     // words into the mailboxes (n * mb_row_words(L) per model)
  int slot_off;         // first slot of the model in the concatenated SlotInfo
  int node_off;         // first node of the model (degrees, node maps)
  int n, L, m, lt;      // sizes and register tile (16, 32, 64 or 128)
  int csr_off;          // first node_ptr entry (n+1 per model)
  int inc_off;          // first incidence entry (2m per model)
  int potts;            // cost kind (0 dense; MPLPXX_COST_*: parameters per slot at table_off + slot * cost_params)
};
struct BatchTask {
  int model;   // which model
  int first;   // first slot of the model this workgroup owns
  int stride;  // team size: the workgroup owns slots first, first+stride, ...
  int lds;     // 1: a whole model whose unaries live in this workgroup's LDS for the launch
};
struct BatchArgs {
  const float* tables;
  float* phi;
  unsigned long long* mb;
  const SlotInfo* slots;
  const int* deg;
  const BatchModel* models;
  const BatchTask* tasks;
  const int* task_ptr;    // [G+1] task range of each logical workgroup
  int* ticket;            // [0] start-order counter, [1] queue head (both zeroed before each launch)
  int qbegin, qlen;       // tasks[qbegin, qbegin + qlen): single-workgroup tasks taken in order by free workgroups
  unsigned long long* sink;  // scratch words of the workgroups (stores of lanes without an output)
  long long* wg_time;        // [grid][2] start and end clock of each logical workgroup
  int* err;
  long long spin_limit;
};
hipError_t launch_batch(const BatchArgs& b, int max_lt, int grid, int iters, size_t dyn_lds, hipStream_t st);
int batch_blocks_per_cu(int max_lt, size_t dyn_lds);
size_t batch_lds_limit(int max_lt);
// LDS-resident unaries of one model in the batched engine: n*L hi values
// (FP32), then, from this byte offset, n*L bf16 corrections
__host__ __device__ inline size_t lds_lo_offset(int n, int L) { return ((size_t)n * L * 4 + 15) / 16 * 16; }
__host__ __device__ inline size_t lds_model_bytes(int n, int L) { return lds_lo_offset(n, L) + (size_t)n * L * 2; }
hipError_t launch_u_to_mb(const float* U, const float* Ulo, unsigned long long* mb, const BatchModel* models,
                          const int* node_model, int total_nodes, hipStream_t st);
hipError_t launch_mb_to_u(float* U, float* Ulo, const unsigned long long* mb, const BatchModel* models,
                          const int* node_model, int total_nodes, hipStream_t st);
hipError_t launch_batch_dual(const float* unaries, const float* tables, const float* phi, const BatchModel* models,
                             const int* node_model, const int* slot_model, const int* node_ptr, const int* inc,
                             int total_nodes, int total_slots, int count, double* node_min, double* edge_min,
                             double* out, hipStream_t st);

// adjoint (adjoint.hip)
template <typename T>
hipError_t launch_step_record(const T* tables, T* phi, T* U, T* Ulo, const SlotInfo* slots, int L, int slot_begin,
                              int count, unsigned char* rec, hipStream_t st);
template <typename T>
hipError_t launch_adj_step(const SlotInfo* slots, int L, int slot_begin, int count, const unsigned char* rec, T* Ub,
                           T* pb, T* thb, hipStream_t st);
template <typename T>
hipError_t launch_adj_seed(const T* U, const T* Ulo, int n, int L, T* Ub, double* node_min, hipStream_t st);
// FP64 mailbox engine, L <= 64 (mailbox64.h, adjoint.hip): values in mailboxes
// of two tagged 64-bit words per label, a node's row filling whole cache lines
__host__ __device__ constexpr int mb64_row_words(int L) { return (2 * L + 15) / 16 * 16; }
struct Fwd64Args {
  const double* tables;
  double* phi;
  unsigned long long* mb;    // [n][mb64_row_words(L)]
  const SlotInfo* slots;
  int L, m, n, iters;
  unsigned char* rec;        // [iters][m][3][L] argmin records, or null
  double* trace;             // [iters][n] node minima (the last row by launch_mb64_fini), or null
  unsigned long long* sink;  // [kF64Sink per workgroup of the launch] scratch words
  int* err;
  long long spin_limit;
  int grid;                  // workgroups of this role (0: none)
};
// Reverse of `seg` recorded iterations
struct Rev64Args {
  const SlotInfo* slots;
  int L, m, seg;
  const unsigned char* rec;
  unsigned long long* mb;    // node adjoints
  double* pb;                // [m][2][L] message adjoints
  double* contrib;           // [seg][m][3][L] scatter vectors for the table adjoints
  int* err;
  long long spin_limit;
  int grid;                  // workgroups of this role (0: none)
};
constexpr int kF64Sink = 256;
hipError_t launch_mb64_init(const double* x, unsigned long long* mb, int n, int L, hipStream_t st);
hipError_t launch_mb64_fini(double* x, const unsigned long long* mb, int n, int L, double* trace_row, hipStream_t st);
// the forward alone (no records; `trace` if given)
hipError_t launch_fwd64(const Fwd64Args& f, hipStream_t st);
// one launch: the reverse of a recorded segment beside the recording forward
// of another (either may have no workgroups), then the reversed segment's
// table adjoints
hipError_t launch_adj64(const Fwd64Args& f, const Rev64Args& r, double* thb, hipStream_t st);

// one launch: f.iters iterations of the FP64 forward beside as many of the FP32
// mailbox engine on `grid32` workgroups (adj_pair.hip); adj_pair_fits: whether
// these grids can be launched so; clk: two zeroed words that give the FP32 run's time
constexpr int kPairNT = 256;  // compute threads of each role
bool adj_pair_fits(int m, int L, int grid64, int grid32);
hipError_t launch_adj_pair(const Fwd64Args& f, const HsArgs<float>& a, unsigned long long* mb, int grid32,
                           unsigned long long* clk, hipStream_t st);

int max_blocks_per_cu_mb(int LT, int NT, int L, bool traces);
// the (M) and (U) updates on the per-matching engine (rules.hip); rule 1 = M, 2 = U
template <typename T>
hipError_t launch_step_rule(const HsArgs<T>& a, int rule, int LT, int NT, int slot_begin, int count, hipStream_t st);
template <typename T>
hipError_t launch_handshake(const HsArgs<T>& a, int engine, int LT, int NT, int slot_begin, int count, int grid,
                            int iters, hipStream_t st);
template <typename T> int max_blocks_per_cu(int LT, int NT);
// FP32 persistent engine with tagged mailboxes
// prefetch: steps the tables are loaded ahead (0 the default: 2 for tiles up
// to 64, 1 for 128; 1: one step, for tiles up to 64 without a trace)
// kind: a structured cost (MPLPXX_COST_*, NT = 256, LT <= 64) whose tiles
// are formed from the slots' parameters
// rule: MPLPXX_RULE_H, or MPLPXX_RULE_M / _U (dense tables, NT = 256, no trace)
hipError_t launch_persistent_mb(const HsArgs<float>& a, unsigned long long* mb, int LT, int NT, int grid, int iters,
                                int phi_in_lds, size_t dyn_lds, hipStream_t st, int prefetch = 0, int kind = 0,
                                int rule = 0);
// the same for Potts models (one weight per slot, L <= 64; potts_mb.h)
int max_blocks_per_cu_mb_potts(int kind);
hipError_t launch_persistent_mb_potts(const HsArgs<float>& a, unsigned long long* mb, int grid, int iters,
                                      int phi_in_lds, size_t dyn_lds, hipStream_t st, int kind = MPLPXX_COST_POTTS);
// the same on `grid` workgroups, the messages of every iteration kept in a.snap
// (mb_snap.hip); mb_snap_fits: whether this model can
bool mb_snap_fits(int m, int L, int grid);
hipError_t launch_mb_snap(const HsArgs<float>& a, unsigned long long* mb, int grid, int iters, hipStream_t st);
// (mbs: words of a node's mailbox row)
hipError_t launch_mb_init(const float* U, const float* Ulo, unsigned long long* mb, int n, int L, int mbs,
                          hipStream_t st);
hipError_t launch_mb_fini(float* U, float* Ulo, const unsigned long long* mb, int n, int L, int mbs, double* trace_row,
                          hipStream_t st);

// dual bound, traces, decode (dual.hip); states: of so many message arrays one
// after another, with as many outputs and scratch terms
template <typename T>
hipError_t launch_dual(const T* unaries, const T* tables, const T* phi, const int* node_ptr, const int* inc, int n,
                       int L, int m, double* node_min, double* edge_min, double* out, hipStream_t st, int potts = 0,
                       int states = 1);
template <typename T>
hipError_t launch_trace_nodes(const T* U, const T* Ulo, int n, int L, double* row, hipStream_t st);
template <typename T>
hipError_t launch_trace_edges(const T* tables, const T* phi, int m, int L, float* out, hipStream_t st);
template <typename T>
hipError_t launch_trace_sum(double* trace_nodes, const float* trace_e, int m, int W, const T* U, const int* deg, int n,
                            int L, int iters, double* out,
                            hipStream_t st);
// (ticket: one int of scratch; node_e [n], edge_e [m]: the energy's terms;
// err, spin_limit: bound of the waits for labels, as in the engines)
template <typename T>
hipError_t launch_decode(const T* unaries, const T* tables, const T* phi, const SlotInfo* slots, const int* node_ptr,
                         const int* inc, int n, int L, int m, int* labels, int* ticket, double* node_e, double* edge_e,
                         double* energy, int* err, long long spin_limit, hipStream_t st, int potts = 0, int states = 1);
template <typename T>
hipError_t launch_check_finite(const T* p, size_t count, int* flag, hipStream_t st);
template <typename S, typename D>
hipError_t launch_pack_tables(const S* src, D* dst, const int* slot_edge, const int* slot_flip, int m, int L,
                              hipStream_t st);
template <typename T>
hipError_t launch_phi_by_edge(const T* phi_slot, const int* slot_of_edge, int m, int L, T* out, hipStream_t st);
hipError_t launch_fill_int(int* p, int value, size_t count, hipStream_t st);
hipError_t launch_convert(const float* src, double* dst, size_t count, hipStream_t st);
hipError_t launch_convert(const double* src, float* dst, size_t count, hipStream_t st);

}  // namespace mplpxx
