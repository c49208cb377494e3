// Host-side planning: validation, HBM layout, work lists.  No HIP calls.
#include "lqsgd_plan.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>

namespace lqsgd {

namespace {

// Work-list sizes below have measured defaults.  Only a build with -DLQSGD_TUNING (for sweeps of
// these sizes) lets an environment variable override them; the normal build reads no environment.
int64_t env_i64(const char* name, int64_t dflt) {
#ifdef LQSGD_TUNING
  const char* s = std::getenv(name);
  if (!s || !*s) return dflt;
  char* end = nullptr;
  long long v = std::strtoll(s, &end, 10);
  return (end && *end == 0 && v > 0) ? (int64_t)v : dflt;
#else
  (void)name;
  return dflt;
#endif
}

int pad_rank(int r) {
  int p = 1;
  while (p < r) p <<= 1;
  return p;
}

}  // namespace

void quantiser_tables(int bits, double alpha, std::vector<float>& thr, std::vector<float>& lev) {
  thr.clear();
  lev.clear();
  if (bits <= 0) return;
  const int lv = (1 << bits) - 1;
  const double l1a = std::log1p(alpha);
  // Eq. (6) at the level q = k/lv, and at the midpoint between two levels.
  for (int k = 0; k <= lv; ++k) lev.push_back((float)(std::expm1((double)k / lv * l1a) / alpha));
  for (int k = 0; k < lv; ++k) thr.push_back((float)(std::expm1((k + 0.5) / lv * l1a) / alpha));
  lev[lv] = 1.0f;   // (1+alpha)^1 - 1 = alpha exactly: the top level is the scale itself
}

int64_t Plan::block_bytes() const {
  auto granules = [](int64_t bytes) { return round_up(std::max<int64_t>(1, bytes), 256); };
  const int64_t w = W, l = std::max(L, 1), slack = kFactorSlack, slices = (max_rows + 255) / 256;
  int64_t n = 0;
  n += granules(4 * (w * ppart_stride + slack)) + granules(4 * (w * qpart_stride + slack));
  n += 2 * granules(4 * (w * p_stride + slack)) + granules(4 * (p_stride + slack)) + granules(4 * (w * q_stride + slack));
  n += granules(4 * 2 * w * l * slices * RP);
  if (slices >= 8 && RP >= 8) n += granules(4 * w * l * slices * RP * RP) + granules(4 * w * l);
  n += granules(w * magp_stride) + granules(w * sgnp_stride) + granules(w * magq_stride) + granules(w * sgnq_stride);
  n += 2 * granules(4 * w * l) + granules(4 * v_total) + granules(8 * w * n_all) + granules(8 * (int64_t)n_all);
  n += granules(sizeof(LayerDesc) * L) + granules(sizeof(VecDesc) * V) + 4 * granules(4 * 256);
  n += granules(sizeof(Tile) * tilesA.size()) + granules(sizeof(Tile) * tilesB.size()) + granules(sizeof(Tile) * tilesBM.size());
  n += granules(sizeof(XTile) * tilesXP.size()) + granules(sizeof(XTile) * tilesXQ.size());
  n += granules(sizeof(RTile) * (tilesRQ.size() + spared_rq)) + granules(sizeof(RTile) * tilesRP.size()) + granules(sizeof(VTile) * tilesV.size());
  return n;
}

// The finer splits (small sets at rank pads 32 and 64; rows of more than 64 columns that are no multiple of four) have up to
// four times the partial planes.  A set that fits the block of the entry point that allocates nothing only without them goes
// without: that entry point's results are the context's to the last bit, the split decides their order of sums, and so both
// take the same one.
int Plan::build(const lqsgd_config* c, const lqsgd_layer* ls, int32_t n_layers) {
  const int rc = build_split(c, ls, n_layers, true);
  if (rc || !fine_split || block_bytes() <= LQSGD_STATIC_SCRATCH_BYTES) return rc;
  const int rc2 = build_split(c, ls, n_layers, false);
  if (rc2 || block_bytes() <= LQSGD_STATIC_SCRATCH_BYTES) return rc2;
  return build_split(c, ls, n_layers, true);     // it does not fit either way
}

int Plan::build_split(const lqsgd_config* c, const lqsgd_layer* ls, int32_t n_layers, bool fine) {
  char buf[256];
  if (!c || !ls) { err = "NULL config or layer list"; return LQSGD_EINVAL; }
  if (n_layers < 1) { err = "n_layers must be >= 1"; return LQSGD_EINVAL; }
  if (c->rank < 1 || c->rank > LQSGD_MAX_RANK) {
    std::snprintf(buf, sizeof buf, "rank %d outside 1..%d", c->rank, LQSGD_MAX_RANK);
    err = buf;
    return c->rank < 1 ? LQSGD_EINVAL : LQSGD_EUNSUPPORTED;
  }
  if (c->bits_p < 0 || c->bits_p > 8 || c->bits_q < 0 || c->bits_q > 8) {
    err = "bits_p / bits_q must be 0 (off) or 1..8";
    return LQSGD_EINVAL;
  }
  if (c->workers < 1 || c->workers > LQSGD_MAX_WORKERS) {
    std::snprintf(buf, sizeof buf, "workers %d outside 1..%d", c->workers, LQSGD_MAX_WORKERS);
    err = buf;
    return LQSGD_EINVAL;
  }
  if (!(c->alpha > 0.0f) || !std::isfinite(c->alpha)) { err = "alpha must be finite and > 0"; return LQSGD_EINVAL; }
  if (c->flags & ~(LQSGD_FLAG_EAGER_RESIDUAL | LQSGD_FLAG_AGGREGATE_FIRST | LQSGD_FLAG_BF16_GRADIENTS | LQSGD_FLAG_NO_COOPERATIVE_LAUNCH)) { err = "unknown config flags"; return LQSGD_EINVAL; }
  agg_first = (c->flags & LQSGD_FLAG_AGGREGATE_FIRST) != 0;
  cfg = *c;
  W = c->workers;
  n_all = n_layers;
  layers.clear(); vecs.clear(); kind_of.clear();
  tilesA.clear(); tilesAG.clear(); tilesB.clear(); tilesBM.clear(); tilesG.clear(); tilesR.clear(); tilesXP.clear(); tilesXQ.clear(); tilesRQ.clear(); tilesRP.clear(); tilesV.clear();

  int max_r = 1;
  max_rows = 0;
  slices = 0;
  plane_rows = 0;
  spared_rq = 0;
  matrix_elements = 0;
  for (int i = 0; i < n_layers; ++i) {
    const lqsgd_layer& l = ls[i];
    if (l.rows < 1 || l.cols < 1) {
      std::snprintf(buf, sizeof buf, "layer %d: rows and cols must be >= 1", i);
      err = buf;
      return LQSGD_ESHAPE;
    }
    if ((int64_t)l.rows * l.cols >= ((int64_t)1 << 31)) {
      std::snprintf(buf, sizeof buf, "layer %d: rows*cols must be < 2^31", i);
      err = buf;
      return LQSGD_ESHAPE;
    }
    if (l.flags & ~LQSGD_LAYER_VECTOR) {
      std::snprintf(buf, sizeof buf, "layer %d: unknown flags", i);
      err = buf;
      return LQSGD_EINVAL;
    }
    if (l.flags & LQSGD_LAYER_VECTOR) {
      if (l.cols != 1) {
        std::snprintf(buf, sizeof buf, "layer %d: a VECTOR layer needs cols == 1", i);
        err = buf;
        return LQSGD_ESHAPE;
      }
      VecDesc v{};
      v.len = l.rows;
      v.gidx = i;
      kind_of.push_back(-(int32_t)vecs.size() - 1);
      vecs.push_back(v);
    } else {
      LayerDesc d{};
      d.rows = l.rows;
      d.cols = l.cols;
      d.r = std::min(c->rank, std::min(l.rows, l.cols));
      d.kind = l.cols % 4 == 0 ? 0 : l.cols > kWave ? 1 : 2;
      d.gidx = i;
      d.np_el = d.rows * d.r;
      d.nq_el = d.cols * d.r;
      d.np_pad = (int32_t)round_up(d.np_el, 16);
      d.nq_pad = (int32_t)round_up(d.nq_el, 16);
      max_r = std::max(max_r, d.r);
      max_rows = std::max(max_rows, d.rows);
      d.slice0 = slices;
      slices += (d.rows + 255) / 256;
      matrix_elements += (int64_t)d.rows * d.cols;
      kind_of.push_back((int32_t)layers.size());
      layers.push_back(d);
    }
  }
  L = (int32_t)layers.size();
  V = (int32_t)vecs.size();
  RP = pad_rank(max_r);
  max_rank = max_r;
  mfma_a = RP >= 16;
  mfma = RP >= 32;                  // measured: at rank pad 16 the vector kernel is still faster

  // ---- tile sizes --------------------------------------------------------
  // A launch wants several times 256 CUs x 16 wavefronts of work items, each
  // long enough to amortise its set-up; huge jobs get larger items so that the
  // work lists stay small.
  const int64_t total = matrix_elements * W;
  const int64_t tgtA = env_i64("LQSGD_TILE_A", std::min<int64_t>(131072, std::max<int64_t>(2048, total / 49152)));
  const int64_t tgtB = env_i64("LQSGD_TILE_B", std::min<int64_t>(524288, std::max<int64_t>(16384, total / 2730)));   // (floor: small CNN set, sweep 1 17.1 -> 14.7 us against 8192)
  // The residual sweep has no sums to carry down its columns, so its items are lower than sweep 1's (which take a layer's
  // whole height where they can): 8 rows per wavefront, more only where the list would pass 131072 items.  With sweep 1's
  // items a wavefront goes through up to 128 rows in rounds of 8: 240 x 309 .. 1628 x 28, W = 7 44 -> 9 us, ResNet-18 set,
  // W = 8 136 -> 113 us (115 / 120 / 128 with 16384 / 32768 / 65536 elements).
  const int64_t tgtR = env_i64("LQSGD_TILE_R", std::min<int64_t>(tgtB, std::max<int64_t>(8192, total / 131072)));
  // the G-hat-only pass covers one worker's worth of elements: smaller items keep its grid wide
  const int64_t tgtG = env_i64("LQSGD_TILE_G", std::min<int64_t>(tgtB, std::max<int64_t>(4096, matrix_elements / 2730)));
  // column segments: at most 1024 columns (2048 at rank pad 32, where fewer, longer segments save
  // more in partial planes and Gram-Schmidt input than they cost in sweep 0; 1024 there too where a small set would have
  // fewer than four items of 32 rows per CU.  Sweep 0, Gram-Schmidt and G-hat pass together, microseconds at 2048 / 1024: ragged
  // set at r = 20 120 / 110, 1024 x 2048, W = 4, r = 32 121 / 104, 2 x 2048^2, W = 1, r = 64 265 / 236, 4096^2, W = 1, r = 32
  // 155 / 157)
  auto mfma_items = [&](int64_t rows, int64_t cols) {
    int64_t n = 0;
    for (const LayerDesc& d : layers) n += W * ((d.rows + rows - 1) / rows) * ((d.cols + cols - 1) / cols);
    return n;
  };
  const bool seg_fine = mfma && fine && mfma_items(32, 2048) < 1024;
  const int64_t segmax4 = env_i64("LQSGD_SEGMAX", mfma && !seg_fine ? 2048 : 1024);
  // Row blocks of the matrix-core sweep 1: 256 rows at least, 128 where that leaves CUs without two items, 64 where 128 leaves
  // CUs without any.  Sweep 1 and its reduce, microseconds at 256 / 128 / 64 rows: 4 x 512^2, W = 2, r = 32 (16 items of 256 rows)
  // 37 / 26 / 21; 2 x 2048^2, W = 1, r = 64 (64) 59 / 42 / 37; 1024 x 2048, W = 4, r = 32 (64) 39 / 30 / 27; 4096^2, W = 1, r = 32
  // (128) 41 / 34 / 40; 4 x 1024^2, W = 4, r = 32 (128) 43 / 35 / 39; 2048^2, W = 4, r = 50 (128) 62 / 48 / 56; ragged set at
  // r = 20 (132 items of 256, 248 of 128) 44 / 33 / 32; the ResNet-18 set at r = 32 (1794) sweep 1 85 / 90 at 256 / 128.
  const int64_t rbm_min = !mfma || !fine || mfma_items(256, kMfmaCols) >= 512 ? 256 : mfma_items(128, kMfmaCols) >= 256 ? 128 : 64;
  fine_split = seg_fine || rbm_min < 256;

  // sweep 0's column segments, and the items it would have with one group of rows in each
  constexpr int cw = kWave * 4;                          // columns of a wavefront's pass over a row
  const int rowgrp = RP == 64 ? 64 : mfma_a ? 32 : kRowsPerGroup;   // a matrix-core item is one 32-row tile, at rank pad 64 two
  int64_t items0 = 0, narrow = 0;
  auto cut = [&](LayerDesc& d, int64_t segmax) {
    const int nseg = (int)((d.cols + segmax - 1) / segmax);
    d.segw = (int32_t)round_up((d.cols + nseg - 1) / nseg, cw);
    d.nseg = (d.cols + d.segw - 1) / d.segw;
  };
  for (LayerDesc& d : layers) {
    cut(d, round_up(segmax4, cw));
    items0 += (int64_t)W * ((d.rows + rowgrp - 1) / rowgrp) * d.nseg;
    if (d.cols < cw) narrow += (int64_t)d.rows * d.cols;
  }
  narrow_rows = 2 * narrow > matrix_elements;
  // Sets with less than one item per SIMD wait for a single wavefront's passes: rows that are no multiple of four, whose last
  // group takes the longest, then have one pass per segment (240 x 309, r = 7, W = 7, sweep 0 13.3 -> 10.4 us; 128 x 1001, r = 8,
  // W = 4 16.2 -> 10.4).
  if (!mfma_a && items0 < 1024)
    for (LayerDesc& d : layers)
      if (d.kind == 1) cut(d, cw);
  // the residual sweep's items likewise, 32 rows each; layers of at most 64 columns take up to four times as many rows where
  // the list is long (1000000 x 16 at r = 4, W = 8 1097 us with 32 rows and three wavefronts a SIMD, 680 with 128 and what the
  // registers allow)
  int64_t itemsR = 0;
  for (const LayerDesc& d : layers) itemsR += (int64_t)W * ((d.rows + 31) / 32) * ((d.cols + cw - 1) / cw);

  // Sweep 1 on the vector units: rows of a row block (rows of one column per lane count 64 columns: 4 x (100000 x 21) at r = 4,
  // W = 8, sweep 1 91 us and reduce 17 with 384 rows, 184 and 50 with 96).
  auto row_block = [&](const LayerDesc& d) {
    const int64_t rowcols = d.kind == 2 || (d.kind == 1 && !fine) ? kWave : cw;
    const int64_t rbb = std::max<int64_t>(4, round_up(std::max<int64_t>(1, tgtB / rowcols), 4));
    // Layers of moderate height take one row block per column chunk: sweep 1 then writes Q_w itself
    // (no partial planes, no reduce pass for this layer), and measured on the ResNet-18-shaped set
    // it streams as fast with 512-row items as with 128-row ones (63 us either way).
    // Not where that would leave the launch with too few items: at most four times the size the
    // work list aims for (a 1024-row layer of a small set keeps its row blocks).
    if (!mfma && (int64_t)d.rows * rowcols <= env_i64("LQSGD_DIRECT_Q_MAX", 262144) && d.rows <= 4 * rbb) return (int32_t)round_up(d.rows, 4);
    const int64_t r = std::min<int64_t>(rbb, round_up(d.rows, 4)), n = (d.rows + r - 1) / r;
    // equal blocks: 8192 rows in blocks of 1536 would end in a block of 512
    return (int32_t)std::min<int64_t>(r, round_up((d.rows + n - 1) / n, 4));
  };
  // Its items in chunks of 256 columns.  Sets with fewer than CUs take rows that are no multiple of four in chunks of 64, one
  // column per lane: the same sums on four times the workgroups (240 x 309, r = 7, W = 7 26.0 -> 11.0 us; 300 x 515, r = 3, W = 1
  // 10.8 -> 7.5; 1000 x 1002, r = 12, W = 2 14.5 -> 8.9).
  int64_t items1 = 0;
  for (const LayerDesc& d : layers) items1 += (int64_t)W * ((d.rows + row_block(d) - 1) / row_block(d)) * ((d.cols + cw - 1) / cw);

  int64_t m_acc = 0, p_acc = 0, q_acc = 0, pp_acc = 0, qp_acc = 0;
  int64_t mp_acc = 0, sp_acc = 0, mq_acc = 0, sq_acc = 0;
  int64_t ppd_acc = 0, qpd_acc = 0;
  padded = false;
  wire_bytes = 0;
  // the reduce passes: items of 1024 .. 8192 elements, as large as still leaves about 512 of them
  // (one atomic maximum per item on a cell per (layer, worker); several loads in flight per thread)
  auto reduce_chunk = [&](bool q) {
    int64_t total = 0;
    for (const LayerDesc& d : layers) total += q ? d.nq_el : d.np_el;
    return (int32_t)(1024 * std::min<int64_t>(8, std::max<int64_t>(1, total * W / (1024 * 512))));
  };
  const int32_t rq_chunk = reduce_chunk(true), rp_chunk = reduce_chunk(false);
  // Rows of an item of the G-hat pass on the matrix cores: 32 where that leaves few items for a CU, as many as save operand reads
  // where there are plenty (us at 32 / 64 / 128 rows: 100 x 300, 20 of them, r = 50, 160 items of 32 rows, 8.8 / 11.4 / 16.5; 1024^2, 6 of
  // them, r = 64, 768 15.0 / 16.5 / 17.6; ResNet-18 set, 1360, r = 50 25.8 / 22.3 / 25.9, r = 32 16.0 / 14.2 / 16.5; 11008 x 4096,
  // 5504, r = 32 44.8 / 38.1 / 36.7; 8192^2, 8192, r = 64 108 / 88 / 86; rank pad 16 reads half as much: ResNet-18 set 12.4 / 13.1 /
  // 12.9, 8192^2 43 / 45 / 48).
  auto ghat_items = [&](int64_t rows) {
    int64_t n = 0;
    for (const LayerDesc& d : layers) n += ((d.rows + rows - 1) / rows) * ((d.cols + kGhatCols - 1) / kGhatCols);
    return n;
  };
  const int32_t rows_g = (int32_t)env_i64("LQSGD_TILE_AG", RP <= 16 || ghat_items(32) < 1024 ? 32 : ghat_items(64) < 2048 ? 64 : 128);
  for (int li = 0; li < L; ++li) {
    LayerDesc& d = layers[li];
    // Groups of rows per item.  Counted in whole passes of 256 columns, a row of 21 costs a pass like one of 256, and a
    // wavefront that takes a dozen groups of such rows one after the other is what a small set waits for (1210 x 21 at
    // r = 7 45 -> 14 us).  With many times as many items as the chip holds wavefronts it is the set-up of an item that
    // counts, and the elements decide (1000000 x 16 at r = 4, W = 8: one group 1560 us, 4 groups 1110, 20 groups 1030;
    // 4 x (100000 x 16) 630 / 450 / 430): one group per 16384 items in between.
    auto groups = [&](int64_t width) {
      const int64_t e = (int64_t)rowgrp * width;
      return std::max<int64_t>(1, (tgtA + e / 2) / e);
    };
    int64_t ng = 1;
    if (!mfma_a) {
      const int64_t lo = groups(std::min<int64_t>(d.segw, round_up(d.cols, cw))), hi = groups(std::min(d.segw, d.cols));
      ng = std::min(hi, std::max(lo, items0 / 16384));
    }
    const int32_t trows = (int32_t)std::min<int64_t>(round_up(d.rows, rowgrp), ng * rowgrp);

    const int32_t rbb_v = row_block(d), nrb_v = (d.rows + rbb_v - 1) / rbb_v;
    d.bcw = d.kind == 2 || (d.kind == 1 && (!fine || items1 < 256)) ? kWave : cw;
    fine_split |= !mfma && d.kind == 1;
    // the partial planes of Q belong to whichever kernel runs sweep 1
    if (mfma) {
      const int64_t rbm = env_i64("LQSGD_TILE_BM", std::min<int64_t>(2048, std::max<int64_t>(rbm_min, total / (49152 * 16))));
      d.rbb = (int32_t)std::min<int64_t>(round_up(rbm, 2), round_up(d.rows, 2));
    } else {
      d.rbb = rbb_v;
    }
    d.nrb = (d.rows + d.rbb - 1) / d.rbb;
    d.direct_q = d.nrb == 1 ? 1 : 0;
    const int nchunk = (d.cols + cw - 1) / cw, nchunk_b = (d.cols + d.bcw - 1) / d.bcw;

    d.m_off = m_acc;   m_acc += round_up((int64_t)d.rows * d.cols, 64);
    d.p_off = p_acc;   p_acc += round_up(d.np_el, 64);
    d.q_off = q_acc;   q_acc += round_up(d.nq_el, 64);
    d.ppart_off = pp_acc; pp_acc += (int64_t)d.nseg * d.np_pad;
    plane_rows = std::max(plane_rows, (int64_t)d.rows * d.nseg);
    d.qpart_off = qp_acc; qp_acc += d.direct_q && !mfma ? 0 : (int64_t)d.nrb * d.nq_pad;   // no partial planes where sweep 1 stores Q_w itself.  Rank pads 32 and 64 keep their room: it is part of block_bytes(), by which build() chooses a set's split, and its sums with it; at pad 64 Gram matrices lie there besides
    d.pop_off = ppd_acc; ppd_acc += round_up((int64_t)d.rows * RP, 64);
    d.qop_off = qpd_acc; qpd_acc += round_up((int64_t)d.cols * RP, 64);
    if (d.r < RP) padded = true;
    const int64_t gp = (d.np_el + kXGroup - 1) / kXGroup, gq = (d.nq_el + kXGroup - 1) / kXGroup;
    d.magp_off = mp_acc; mp_acc += round_up(gp * std::max(1, cfg.bits_p), 16);
    d.sgnp_off = sp_acc; sp_acc += round_up(gp, 16);
    d.magq_off = mq_acc; mq_acc += round_up(gq * std::max(1, cfg.bits_q), 16);
    d.sgnq_off = sq_acc; sq_acc += round_up(gq, 16);

    wire_bytes += cfg.bits_p ? ((int64_t)d.np_el * cfg.bits_p + 7) / 8 + gp + 4 : 4 * (int64_t)d.np_el;
    wire_bytes += cfg.bits_q ? ((int64_t)d.nq_el * cfg.bits_q + 7) / 8 + gq + 4 : 4 * (int64_t)d.nq_el;

    for (int w = 0; w < W; ++w) {
      const int32_t lw = li * W + w;
      for (int32_t row0 = 0; row0 < d.rows; row0 += trows)
        for (int32_t s = 0; s < d.nseg; ++s) {
          tilesA.push_back(Tile{lw, row0, std::min(trows, d.rows - row0), s});
        }
      for (int32_t rb = 0; rb < nrb_v; ++rb)
        for (int32_t ch = 0; ch < nchunk_b; ++ch)
          tilesB.push_back(Tile{lw, rb * rbb_v, std::min(rbb_v, d.rows - rb * rbb_v), ch});
      if (!mfma_a) {
        const int64_t rr = std::max<int64_t>(1, tgtR / cw) * (d.cols > kWave ? 1 : std::min<int64_t>(4, std::max<int64_t>(1, itemsR / 16384)));
        const int32_t rbr = (int32_t)std::min<int64_t>(round_up(rr, 4), round_up(d.rows, 4));
        for (int32_t row0 = 0; row0 < d.rows; row0 += rbr)
          for (int32_t ch = 0; ch < nchunk; ++ch)
            tilesR.push_back(Tile{lw, row0, std::min(rbr, d.rows - row0), ch});
      }
      for (int32_t row0 = 0; w == 0 && mfma_a && row0 < d.rows; row0 += rows_g)
        for (int32_t s = 0; s * kGhatCols < d.cols; ++s) tilesAG.push_back(Tile{lw, row0, std::min(rows_g, d.rows - row0), s});
      if (w == 0) {
        const int32_t rbg = (int32_t)std::min<int64_t>(round_up(std::max<int64_t>(1, tgtG / (d.kind == 2 ? kWave : cw)), 4), round_up(d.rows, 4));
        for (int32_t row0 = 0; row0 < d.rows; row0 += rbg)
          for (int32_t ch = 0; ch < nchunk; ++ch)
            tilesG.push_back(Tile{lw, row0, std::min(rbg, d.rows - row0), ch});
      }
      if (mfma)
        for (int32_t rb = 0; rb < d.nrb; ++rb)
          for (int32_t cg = 0; cg < (d.cols + kMfmaCols - 1) / kMfmaCols; ++cg)
            tilesBM.push_back(Tile{lw, rb * d.rbb, std::min(d.rbb, d.rows - rb * d.rbb), cg});
      if (d.direct_q && mfma) spared_rq += (d.nq_el + rq_chunk - 1) / rq_chunk;
      if (!d.direct_q)
        for (int32_t e = 0; e < d.nq_el; e += rq_chunk) tilesRQ.push_back(RTile{lw, e, std::min(rq_chunk, d.nq_el - e)});
      if (agg_first)
        for (int32_t e = 0; e < d.np_el; e += rp_chunk) tilesRP.push_back(RTile{lw, e, std::min(rp_chunk, d.np_el - e)});
    }
    for (int32_t g = 0; g < gp; g += kXBlockGroups) tilesXP.push_back(XTile{li, g});
    for (int32_t g = 0; g < gq; g += kXBlockGroups) tilesXQ.push_back(XTile{li, g});
  }
  // Rank pads 32 and 64: few workgroups fit a CU there and an item can take a tenth of the launch, so that the widest go first and
  // the last ones are short (sweep 0 forwards, as it runs there with the deferred residual, us, in the layers' order / sorted: ragged
  // set, r = 20, W = 4 50 / 44; ResNet-18 set, W = 8, r = 50 271 / 260, r = 32 215 / 211).  Items of more than 32 rows before the
  // others (HalfItem).
  twoA = 0;
  if (mfma) {
    auto two = [](const Tile& t) { return t.nrows > 32; };
    auto width = [&](const Tile& t) {
      const LayerDesc& d = layers[t.lw / W];
      return std::min(d.segw, d.cols - t.aux * d.segw);
    };
    std::stable_sort(tilesA.begin(), tilesA.end(), [&](const Tile& x, const Tile& y) {
      return two(x) != two(y) ? two(x) : width(x) > width(y);
    });
    twoA = (int32_t)std::count_if(tilesA.begin(), tilesA.end(), two);
  }

  m_stride = round_up(m_acc, 64);
  p_stride = round_up(p_acc, 64);
  q_stride = round_up(q_acc, 64);
  ppart_stride = round_up(pp_acc, 64);
  qpart_stride = round_up(qp_acc, 64);
  magp_stride = round_up(mp_acc, 64);
  sgnp_stride = round_up(sp_acc, 64);
  magq_stride = round_up(mq_acc, 64);
  sgnq_stride = round_up(sq_acc, 64);
  if (!padded)
    for (LayerDesc& d : layers) { d.pop_off = d.p_off; d.qop_off = d.q_off; }
  ppad_total = padded ? ppd_acc : 0;
  qpad_total = padded ? qpd_acc : 0;

  int64_t v_acc = 0;
  for (int vi = 0; vi < V; ++vi) {
    vecs[vi].off = v_acc;
    for (int32_t e = 0; e < vecs[vi].len; e += 1024) tilesV.push_back(VTile{vi, e});
    v_acc += round_up(vecs[vi].len, 64);
  }
  v_total = v_acc;

  const int64_t tile_bytes = (int64_t)(tilesA.size() + tilesAG.size() + tilesR.size() + tilesB.size() + tilesBM.size() + tilesG.size()) * sizeof(Tile) +
                             (int64_t)(tilesXP.size() + tilesXQ.size()) * sizeof(XTile) +
                             (int64_t)(tilesRQ.size() + tilesRP.size()) * sizeof(RTile) + (int64_t)tilesV.size() * sizeof(VTile);
  device_bytes = 4 * ((int64_t)W * (m_stride + 2 * p_stride + q_stride + ppart_stride + qpart_stride) +
                      p_stride + q_stride + ppad_total + qpad_total + v_total + 2 * (int64_t)W * std::max(L, 1) +
                      6 * (int64_t)W * std::max(L, 1) * ((max_rows + 255) / 256) * RP) +
                 (int64_t)W * (magp_stride + sgnp_stride + magq_stride + sgnq_stride) + tile_bytes +
                 (int64_t)L * sizeof(LayerDesc) + (int64_t)V * sizeof(VecDesc) +
                 (int64_t)(W + 1) * n_all * 8 + 4 * 4 * 256;
  if (tilesA.size() > 0x7fffffff / 4 || tilesB.size() > 0x7fffffffu) {
    err = "work list too long";
    return LQSGD_EUNSUPPORTED;
  }
  return LQSGD_OK;
}

}  // namespace lqsgd
