// Device-side argument block and the launchers of the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "lqsgd_plan.h"

namespace lqsgd {

// Passed by value to every kernel (lands in the kernarg segment, read with
// scalar loads).  All pointers are device pointers.
struct DevArgs {
  const LayerDesc* layers;
  const VecDesc* vecs;
  const float* const* grads;   // W * n_all gradient tensors (fp32, or bfloat16 behind the same pointer type if g_bf16)
  float* const* ghat;          // n_all optional outputs (entries may be null), or null
  float* E;                    // residual / M = G + E, per worker
  float* Ppart;                // sweep-0 partial products, per worker
  float* Ppre;                 // P_w before Gram-Schmidt
  float* Porth;                // P_w after Gram-Schmidt
  float* orth_part;            // [2][L*W][ceil(max_rows/256)][RP] slice partials of the many-workgroup Gram-Schmidt
  unsigned long long* orth_table;      // [2][L*W][ceil(max_rows/256)][RP] tagged partials of its one-launch form
  // Cholesky-QR form of the tall Gram-Schmidt (rank pads >= 8; null if the context has none; at rank pad 64 and fewer than 8
  // slices chol_part and chol_redo lie in Qpart, whose planes are dead while Gram-Schmidt runs):
  unsigned long long* chol_table;      // [L*W][ceil(max_rows/256) + 1][NE] tagged Gram matrices of the slices, their total last
  float* chol_part;            // [L*W][ceil(max_rows/256)][NE] the same matrices in plain memory, for the form of three launches: of the
  float* chol_part2;           // first pass, and of the second
  int* chol_redo;              // [L*W] bit 0 raised for a pair that has to be done column by column, bit 1 of the first word for any
  int* status;                 // pinned host word the kernels raise when a bounded device-side wait expires
  float* Pbar;                 // aggregated P (shared)
  float* Qpart;                // sweep-1 partial products, per worker
  float* Qw;                   // Q_w
  float* Qbar;                 // aggregated Q = warm-start Q (shared)
  float* Pop; float* Qop;      // the factors as the sweeps read them, rows of rank_pad ranks: Pbar / Qbar, or zero-padded copies (padded)
  uint8_t* magP; uint8_t* sgnP; float* scaleP;   // packets of the P exchange
  uint8_t* magQ; uint8_t* sgnQ; float* scaleQ;   // packets of the Q exchange
  const float* thrP; const float* levP;           // quantiser tables for b_p
  const float* thrQ; const float* levQ;           // ... and b_q
  float* vmean;
  int64_t m_stride, p_stride, q_stride, ppart_stride, qpart_stride;
  int64_t magp_stride, sgnp_stride, magq_stride, sgnq_stride;
  int32_t W, L, n_all, bits_p, bits_q;
  int32_t rank_pad;            // Plan::RP
  int32_t padded;              // Plan::padded: Pop / Qop are copies, written by the exchange beside Pbar / Qbar
  float alpha;                 // log scale of Eq. (5)
  int32_t quant_fast;          // alpha is such that the hardware log2 finds a code to within one level
  float qscale_p, qscale_q;    // (2^b - 1) / log2(1 + alpha) for b_p, b_q
  int32_t slices;              // slices of 256 rows of one worker's factors (Plan::slices)
  int32_t agg_first;           // aggregate-first order: scaleP is an atomic-max accumulator (sweep 0 zeroes it)
  int32_t orth_shared;         // the Gram-Schmidt kernels run once per layer, in place on the plane at Ppart + p_off
  int32_t g_bf16;              // the gradient tensors hold bfloat16 values (G-hat / parameters stay fp32)
  int32_t update;              // G-hat outputs are parameters to update: w <- w - eta G-hat
  int32_t nt_store;            // sweep 0 streams the residual slabs: non-temporal loads of E and stores of M (the launchers pick the kernels built that way)
  int32_t nt_fused;            // the same for sweep 0 with the deferred residual on the matrix cores
  int32_t by_blocks;           // sweep 0 by blocks per wavefront, not by rounds.  Rank pad 16, of 64 columns: 1 with the deferred
                               // residual, 2 with and without.  Rank pad 32, of 32 columns: 1 without it, 2 with and without
  float eta;
};

enum ExchangeMode { kQuantOnly = 0, kMeanOnly = 1, kFused = 2 };

// The device function the calling thread's most recent launcher call has launched, with its
// template arguments, as a profiler's kernel list names it (namespaces and parameters left out).
const char* last_launched_kernel();

// Each launcher enqueues one kernel on `s` and returns hipGetLastError().
// `reverse` walks the work list backwards: consecutive sweeps alternate direction so that
// each one starts on the data the previous one touched last (still in the memory-side cache).
// fuse_residual: the buffer E holds last iteration's M and the residual update
// E = M - P-bar Q-bar^T is applied on the fly (see add_project_kernel).
// narrow_rows (Plan::narrow_rows): as many wavefronts as the registers allow, see kTwoPerCu.
hipError_t launch_add_project(int RP, const DevArgs& a, const Tile* tiles, int ntiles, int fuse_residual, int narrow_rows, int reverse,
                              hipStream_t s);
// What a context keeps for the one-launch (cooperative) Gram-Schmidt of tall factors.
struct CoopState {
  unsigned long long epoch = 0;   // launches made so far: makes the tags in `a.orth_table` unique
  int capacity = -1;              // workgroups of that kernel that fit the context's device at once (-1: not asked yet)
  int chol_capacity = -1;         // the same for the Cholesky-QR kernel
  unsigned max_polls = 0;         // bound of a device-side wait; 0 = the default (about a second), not set from outside
};
// Entries of the r x r Gram matrix that the slices of a factor exchange at rank pad RP (NE above); 0 if
// the Cholesky-QR form does not exist at that pad.
int chol_entries(int RP);
// coop: NULL disables the one-launch forms.
// *copied: whether the launch has written the padded copy Pop of an aggregate (orth_shared) too, where there is one.
// plane_rows: Plan::plane_rows, or max_rows where there is one plane.
hipError_t launch_orth(int RP, int max_rows, int max_rank, int64_t plane_rows, const DevArgs& a, CoopState* coop, bool* copied, hipStream_t s);
hipError_t launch_exchange(int mode, int phase, const DevArgs& a, const XTile* tiles, int ntiles, hipStream_t s);
// Sweep 1 also runs the plain mean of the 1-D tensors (nvtiles extra workgroups).  Layers whose
// items cover all their rows (LayerDesc::direct_q) get Q_w and its absmax from this sweep itself.
hipError_t launch_back_project(int RP, const DevArgs& a, const Tile* tiles, int ntiles, const VTile* vtiles, int nvtiles,
                               int reverse, hipStream_t s);
// The same sweep on the matrix cores (rank pad 32 or 64; tiles are row block x 512-column group).
hipError_t launch_back_project_mfma(int RP, const DevArgs& a, const Tile* tiles, int ntiles, const VTile* vtiles, int nvtiles,
                                    int reverse, hipStream_t s);
// phase 1: Q_w from sweep 1's row-block planes; phase 0: the raw P_w from sweep 0's column-segment
// planes (aggregate-first order, where the exchange comes before Gram-Schmidt).
hipError_t launch_reduce_q(int phase, const DevArgs& a, const RTile* tiles, int ntiles, hipStream_t s);
// mode: 0 = residual for all workers, 1 = residual + G-hat, 2 = G-hat only (tiles of worker 0).
hipError_t launch_residual(int RP, int mode, const DevArgs& a, const Tile* tiles, int ntiles, int narrow_rows, int reverse, hipStream_t s);

// Refreshes the copy a.Pop (which = 0) or a.Qop (which = 1) from the tightly packed factor (the exchange writes both at once;
// this is for a factor that came another way).
hipError_t launch_pad_factor(int RP, int which, const DevArgs& a, hipStream_t s);

// The per-GPU blocks of the entry point that allocates nothing, scratch and operand copies: device addresses of
// those of `device`, which must be the current device on the first call for it.
hipError_t static_scratch(int device, void** scratch, void** operands, void** grams);
// Clears `bytes` (a multiple of 16) at the 16-byte aligned device address p with a kernel.
hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s);

// Writes n device pointers to the device table dst, in the order of the stream (kPointerBatch of them per launch).
constexpr int kPointerBatch = 448;       // 3.5 KB of kernel arguments
hipError_t launch_write_pointers(const void** dst, const void* const* src, size_t n, hipStream_t s);

// Sweeps 0 and 2 on the matrix cores (rank pad 16, 32 or 64), over the work list of
// sweep 0 (32-row items, at rank pad 64 of 64 rows).  mode: 0 = M = G + E and P partials, 1 = the same with the deferred
// residual applied on the fly, 2 = residual, 3 = residual + G-hat, 4 = G-hat only, over a list of its own (Plan::tilesAG).
// two: Plan::twoA, 0 for that list.
hipError_t launch_mfma_sweep(int RP, int mode, const DevArgs& a, const Tile* tiles, int ntiles, int two, int reverse, hipStream_t s);

}  // namespace lqsgd
