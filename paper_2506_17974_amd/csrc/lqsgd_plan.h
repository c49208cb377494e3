// Host-side planning for the LQ-SGD compressor: layer table, buffer layout in
// HBM and the flattened work lists of every kernel.  Pure C++ (no HIP calls),
// so it can be exercised on a machine without a GPU.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "lqsgd.h"

namespace lqsgd {

constexpr int kWave = 64;
constexpr int kRowsPerGroup = 8;   // rows a wavefront carries through one column pass of sweep 0
constexpr int kGhatCols = 256;     // columns of an item of the G-hat pass on the matrix cores
constexpr int kMfmaCols = 512;     // columns one workgroup of the matrix-core sweep 1 covers (4 waves x 4 strips x 32)
constexpr int kXGroup = 8;         // elements one lane quantises / packs (b bytes + 1 sign byte)
constexpr int kXBlockGroups = 32;  // groups of 8 elements one exchange workgroup covers
constexpr int kFactorSlack = 64;   // readable floats after the last row of every factor buffer (loaders of ranks below their pad overrun)

// Device memory of the entry point that allocates nothing (lqsgd_step_static), per GPU.
#ifndef LQSGD_STATIC_SCRATCH_BYTES
#define LQSGD_STATIC_SCRATCH_BYTES (32u << 20)
#endif
// ... and of the padded operand copies (Plan::padded) and the residual sweep's items where that block has no room left.  Where the layers' ranks
// are more than half their register pad, the copies are at most twice what the block already holds of the same factors.
#ifndef LQSGD_STATIC_OPERAND_BYTES
#define LQSGD_STATIC_OPERAND_BYTES (64u << 20)
#endif
// ... and of the second-pass Gram matrices of tall factors.  The first-pass ones, which are as many, lie in the first block: a
// configuration that this block had no room for has been refused before.
#ifndef LQSGD_STATIC_GRAM_BYTES
#define LQSGD_STATIC_GRAM_BYTES LQSGD_STATIC_SCRATCH_BYTES
#endif
static_assert(LQSGD_STATIC_GRAM_BYTES >= LQSGD_STATIC_SCRATCH_BYTES, "second-pass Gram matrices");

// One matrix layer as the kernels see it.  Offsets are in elements (floats)
// from the start of a per-worker slab unless they say bytes.
struct LayerDesc {
  int32_t rows, cols, r, kind;  // kind of rows: 0 = cols % 4 == 0 (16-byte aligned), 1 = not, 2 = not and at most 64 columns
  int32_t segw, nseg;           // sweep 0: column segment width (multiple of 256) and count
  int32_t rbb, nrb;             // sweep 1: rows per row block and count
  int32_t bcw;                  // sweep 1 on the vector units: columns of a chunk, 256 or (one per lane) 64
  int32_t gidx;                 // position in the caller's tensor list
  int32_t np_el, nq_el;         // rows*r, cols*r
  int32_t np_pad, nq_pad;       // the same rounded up to 16 elements (stride of the partial planes)
  int32_t direct_q;             // sweep 1 covers all rows in one block and writes Q_w (and its absmax) itself: no partial planes, no reduce
  int32_t slice0;               // slices of 256 rows in the layers before (Gram-Schmidt by slices)
  int64_t pop_off, qop_off;     // into the factors the sweeps read: copies with rows padded to RP ranks (Plan::padded), or p_off / q_off
  int64_t m_off;                // into E / M          (worker stride m_stride)
  int64_t p_off;                // into rows x r slabs (worker stride p_stride)
  int64_t q_off;                // into cols x r slabs (worker stride q_stride)
  int64_t ppart_off;            // nseg planes of np_pad (worker stride ppart_stride)
  int64_t qpart_off;            // nrb planes of nq_pad  (worker stride qpart_stride)
  int64_t magp_off, sgnp_off;   // bytes (worker strides magp_stride, sgnp_stride)
  int64_t magq_off, sgnq_off;   // bytes
};

struct VecDesc {
  int32_t len, gidx;
  int64_t off;                  // into the vmean buffer
};

// Work item of a streaming sweep.  lw = layer * W + worker.
// sweep 0: one wavefront; rows [row0, row0+nrows), column segment `aux`.
// sweep 1: one workgroup; rows [row0, row0+nrows), column chunk `aux` (LayerDesc::bcw wide).  Sweep 2: the same, 256 wide.
struct Tile {
  int32_t lw, row0, nrows, aux;
};
struct XTile {   // exchange kernels: kXBlockGroups groups of 8 elements starting at group grp0 of `layer`
  int32_t layer, grp0;
};
struct RTile {   // reduce_q: n elements of (layer, worker) starting at el0 (n <= 8192, el0 a multiple of 1024)
  int32_t lw, el0, n;
};
struct VTile {   // vector_mean: 1024 elements of vector `vec` starting at el0
  int32_t vec, el0;
};

struct Plan {
  lqsgd_config cfg{};
  int32_t n_all = 0;            // tensors in the caller's list
  int32_t W = 0, L = 0, V = 0;  // workers, matrix layers, vector layers
  int32_t RP = 0;               // register rank: smallest of 1, 2, 4, .. 64 >= max layer rank
  int32_t max_rows = 0;         // largest row count of a matrix layer
  int32_t max_rank = 0;         // largest effective rank of a matrix layer
  int32_t slices = 0;           // slices of 256 rows of all matrix layers
  int64_t plane_rows = 0;       // largest rows * nseg of a matrix layer: what Gram-Schmidt adds up of one factor
  bool mfma = false;            // sweep 1 runs on the matrix cores (rank pads 32 and 64)
  bool mfma_a = false;          // sweeps 0 and 2 run on the matrix cores (rank pad >= 16): 32-row work items, 64 rows at rank pad 64
  std::vector<LayerDesc> layers;
  std::vector<VecDesc> vecs;
  std::vector<int32_t> kind_of;    // per caller index: >= 0 matrix index, < 0 -(vector index) - 1
  std::vector<Tile> tilesA, tilesB;
  std::vector<Tile> tilesR;        // residual sweep of the vector path: row block x 256 columns, all workers
  std::vector<Tile> tilesAG;       // G-hat pass of the matrix-core path: worker 0, a block of rows x kGhatCols
  int32_t twoA = 0;                // rank pad 64: items of more than 32 rows, the first ones of tilesA
  std::vector<Tile> tilesBM;       // sweep 1 on the matrix cores (rank pads 32 and 64): row block x 512-column group
  std::vector<Tile> tilesG;        // one pass over every layer of worker 0 (G-hat only): row block x 256 columns
  std::vector<XTile> tilesXP, tilesXQ;
  std::vector<RTile> tilesRQ;
  int64_t spared_rq = 0;           // ... of layers of one row block at rank pads 32 and 64, which need none; block_bytes() counts them
  std::vector<RTile> tilesRP;      // aggregate-first order: reduce of the P partials (1024 elements each)
  bool agg_first = false;          // LQSGD_FLAG_AGGREGATE_FIRST
  bool narrow_rows = false;        // most elements are in layers of fewer than 256 columns
  // Some layer has fewer ranks than the register pad: the sweeps then read P-bar and Q-bar from copies
  // whose rows are padded with zeros to RP ranks (aligned rows, no rank tests in the loops);
  // ppad_total / qpad_total floats.
  bool padded = false;
  int64_t ppad_total = 0, qpad_total = 0;
  std::vector<VTile> tilesV;
  int64_t m_stride = 0, p_stride = 0, q_stride = 0, ppart_stride = 0, qpart_stride = 0;
  int64_t magp_stride = 0, sgnp_stride = 0, magq_stride = 0, sgnq_stride = 0, v_total = 0;
  int64_t device_bytes = 0, wire_bytes = 0, matrix_elements = 0;
  std::string err;

  // Returns LQSGD_OK or a negative status with `err` set.
  int build(const lqsgd_config* cfg, const lqsgd_layer* layers, int32_t n_layers);

  // Bytes of a caller-provided block that hold everything but the padded operand copies and the residual sweep's items (an
  // upper bound).
  int64_t block_bytes() const;

 private:
  int build_split(const lqsgd_config* cfg, const lqsgd_layer* layers, int32_t n_layers, bool fine);
  bool fine_split = false;         // sweeps 0 / 1 at rank pads 32 and 64: shorter segments or lower row blocks than usual
};

// Quantiser tables of Section 4.1 for one bit width, computed in double and
// rounded to fp32: thr[k] = decision threshold between levels k and k+1 in the
// normalised magnitude u = |x|/s, k < 2^b - 1; lev[k] = dequantised magnitude
// of level k, k < 2^b.
void quantiser_tables(int bits, double alpha, std::vector<float>& thr, std::vector<float>& lev);

// Rank pad 64: a work item of sweep 0 is 64 rows, and the kernels of 32 rows run two workgroups on it, or one where it has no more
// than 32 rows.  The items of two come first in the list (`two` of them), so that no workgroup is launched without rows: empty ones
// in between, a place per CU and in turn over the dies and their shader engines, left most of the chip idle (64 layers of 32 x 2048,
// r = 50, W = 8: G-hat pass 45 us with an empty workgroup beside each, 28 without, eager residual 240 and 140).
struct HalfItem { int item, half; };
constexpr HalfItem half_item(int block, int two) { return block < 2 * two ? HalfItem{block >> 1, block & 1} : HalfItem{block - two, 0}; }

inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

}  // namespace lqsgd
