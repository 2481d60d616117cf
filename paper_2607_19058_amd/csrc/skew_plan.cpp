// skew_plan.cpp -- host-only planning of a descriptor table: validation, the tier
// state each tensor keeps (Fig. 1; Sec. 3 "The tiers"), the state size of Eq. 2
// (plus the exact v of vectors, Table 6), the tile grids and the work-item lists.
// No HIP calls: this runs without a GPU.
#include <algorithm>
#include <climits>
#include <cmath>
#include <utility>

#include "skew_internal.h"

namespace skew {

static int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Row-band pass: zcw 512-column chunks per row, nseg of them per wave, so wpr = ceil(zcw /
// nseg) <= 8 waves share a row and rpi = 8 / wpr rows are side by side. One chunk per wave
// only for rows of one chunk; two up to 16 chunks; three without momentum up to 24, and where two
// leave more of the waves idle (3, 5, 6, 9 to 12 chunks: a slot of either costs the same; pass over
// 3.65e8 elements in rows of 2730 / 2765 / 1031 columns: 215 / 242 / 312 us with two, 181 / 208 /
// 260 with three); else four. A block is rpi * zrb rows, zrb (rows per group) as many as the registers hold: two
// blocks (bf16 gradient, and fp32 momentum where kept) beside the band's double sums.
// zrb = 0: no row band.
// Rows of fewer than 8 columns: a matrix of up to kNarrowRows of them takes the tiled passes (step of 100
// matrices of 64 x 3: 55 us tiled, 59 by row bands; of 64 slices of 64 x 7: 64, 69). Their fold and
// update sums go over the partials of every 128 rows: longer ones take row bands (16384 x 4: 100 us
// tiled, 62 by row bands; 1e6 x 5: 4210, 739; 2^25 x 1: 193 ms, 16.8).
constexpr int64_t kNarrowRows = 2048;
constexpr int64_t kMaxMomChunks = 21, kFewRows = 8;
struct RowBandShape {
  int64_t zcw, nseg, rpi, zrb;
};
static RowBandShape rowband_shape(int64_t n, int64_t m, int64_t ld, bool momentum, bool compact) {
  RowBandShape r;
  r.zcw = ceil_div(m, kChunk);
  r.nseg = r.zcw <= 1 ? 1 : (r.zcw <= 2 * kZWaves ? 2 : (!momentum && r.zcw <= 3 * kZWaves ? 3 : 4));
  auto busy = [&](int64_t nseg) {   // chunks summed per pass of the work-group, of 8 * nseg that it could
    const int64_t w = ceil_div(r.zcw, nseg);
    return w > kZWaves ? 0.0 : (double)(kZWaves / w * r.zcw) / (double)(kZWaves * nseg);
  };
  if (!momentum && r.nseg == 2 && busy(3) > busy(2)) r.nseg = 3;
  const int64_t wpr = ceil_div(r.zcw, r.nseg);
  r.rpi = wpr <= kZWaves ? kZWaves / wpr : 0;
  r.zrb = zrows_per_group((int)r.nseg, momentum, 0);
  // rows too long for the work-group, or so far apart that the byte offsets of a block (of the mode
  // with the longest blocks) pass 31 bits, take the tiled passes
  if (r.rpi < 1 || ld > 0x7FFFFFFF / 2 / (r.rpi * zrows_per_group_max((int)r.nseg, momentum)))
    r.zrb = 0;
  if (m < kZMinCols && n <= kNarrowRows && !compact) r.zrb = 0;
  // up to 8 rows of more than 21 chunks with momentum: a work-group per row leaves the chip idler than
  // tiles do (4 x 16384 in the gradient-norm mode: 47 us tiled, 54 by row bands; 12 rows: equal)
  if (momentum && r.zcw > kMaxMomChunks && n <= kFewRows) r.zrb = 0;
  return r;
}

// A row of a few columns takes a wave as long as one of a whole chunk, and counts as one in the band
// size (bands of 2048 rows whatever the width would be 64 waits for memory one after the other)
constexpr int64_t kZMinRowCost = 128;
static int64_t row_cost(int64_t m) { return m < kZMinCols ? kZMinRowCost : m; }

// Rows per band for bands of about `band_elems` elements (fewer with momentum, whose elements
// take kMomCost times as long): whole blocks, at most kZMaxBandRows
constexpr double kMomCost = 3.3;
static int64_t band_rows(const RowBandShape &r, int64_t m, bool momentum, int64_t band_elems,
                         double mom_cost = kMomCost) {
  const int64_t rows_block = r.rpi * r.zrb;
  const int64_t e = momentum ? (int64_t)((double)band_elems / mom_cost) : band_elems;
  const int64_t rows = ceil_div(std::max<int64_t>(1, e / row_cost(m)), rows_block) * rows_block;
  return std::min<int64_t>(rows, kZMaxBandRows / rows_block * rows_block);
}

// Row-band size: the one with the least estimated time of the row-band pass and its fold. A
// work-group fills a compute unit, so the bands run in rounds of kCus: many small bands waste
// less of the last round, and fill the chip when the table is small; each costs its start and
// end (kBandUs) and a row of column partials that the fold reads back (kFoldBytesPerUs for both).
// Measured on one MI355X: 1.07e-4 us per element and compute unit (3.3 times that with
// momentum), 3 us per band, 4 TB/s. 1.1e9 elements in bands of 2^21 / 2^20 / 2^19: 2.2, 4.4 and
// 8.75 rounds, 724 / 608 / 561 us for the pass and 24 / 27 / 42 us for the fold. The partials stay
// below 256 MiB or 1/40 of the gradients.
constexpr double kCus = 256.0, kElemUs = 1.07e-4, kBandUs = 3.0, kFoldBytesPerUs = 2.0e6,
                 kFoldMaxBytes = 268435456.0;
static int64_t choose_band_elems(const skew_tensor_desc *d, int n, double max_bytes = HUGE_VAL) {
  struct Shape {
    RowBandShape r;
    int64_t n, m;
    bool mom;
    double count;
  };
  double grad_bytes = 0.0;
  std::vector<Shape> shapes;   // the distinct shapes (runs of the table), counted
  double cost = 0.0;
  for (int i = 0; i < n; i++) {
    const skew_tensor_desc &x = d[i];
    if (x.ndim == 1 || x.rows <= 0 || x.cols <= 0 || (x.ndim == 3 && x.batch <= 0)) continue;
    if (x.tier == SKEW_TIER_ROUTER && !(x.state_flags & SKEW_STATE_FACTORED)) continue;
    const bool mom = x.tier == SKEW_TIER_BACKBONE || (x.state_flags & SKEW_STATE_MOMENTUM) != 0;
    const RowBandShape r = rowband_shape(x.rows, x.cols, x.ld, mom, false);
    if (r.zrb < 1) continue;
    const double E = x.ndim == 3 ? (double)x.batch : 1.0;
    cost += E * (double)x.rows * (double)row_cost(x.cols) * (mom ? kMomCost : 1.0) * kElemUs;
    grad_bytes += E * (double)x.rows * (double)x.cols * 2.0;
    bool found = false;
    for (size_t j = shapes.size(); j-- > 0 && j + 8 >= shapes.size() && !found;) {
      Shape &s = shapes[j];
      if (s.n == x.rows && s.m == x.cols && s.mom == mom && s.r.zrb == r.zrb) {
        s.count += E;
        found = true;
      }
    }
    if (!found) shapes.push_back({r, x.rows, x.cols, mom, E});
  }
  int64_t best = kZBandElems;
  double best_us = HUGE_VAL;
  for (int step = 0;; step++) {
    const int64_t b = (int64_t)((double)kZBandElems * std::exp2(-step / 8.0));
    if (b < kZMinBandElems) break;
    double bands = 0.0, bytes = 0.0;
    for (const Shape &s : shapes) {
      const double nb = s.count * (double)ceil_div(s.n, band_rows(s.r, s.m, s.mom, b));
      bands += nb;
      bytes += nb * 16.0 * (double)s.m;
    }
    if (bands <= 0.0 || (step > 0 && bytes > std::min(max_bytes, std::max(kFoldMaxBytes, grad_bytes / 40.0))))
      break;
    const double us = std::ceil(bands / kCus) * (cost / bands + kBandUs) + bytes / kFoldBytesPerUs;
    if (us < best_us) {
      best_us = us;
      best = b;
    }
  }
  return best;
}

// Elements per update tile: kTileElems, or fewer where the table would not fill the chip with
// them (four work-groups of the update pass fit a compute unit: kTileCount is two rounds), down to
// kMinTileElems (a work-group of the pass takes 2048 elements at a time, and starts each tile
// with its column factors). Update pass at tiles of 2^16 / 2^13 / 2^12 / 2^11 elements: 4.5e6
// elements 39 / 18 / 21 / 29 us; 5.0e7 odd-width ones 142 us at 2^16, 110 at 2^14, 129 at 2^13.
constexpr int64_t kMinTileElems = 1 << 13, kTileCount = 2048;
// Tiles of the tiled passes: a tile costs a row of column partials and the column factors of the update
// sums, and two work-groups of pass 1 fit a compute unit, so kWideTileCount of them are enough
// (counted over the tensors of those passes alone). Step of one 20000-column matrix at tiles of
// 2^16 / 2^14 / 2^13 elements: 3.4e7 elements 148 / 194 / - us; 1.7e7 96 / - / 117; 8e6 (2^15) 70 / - / 79.
constexpr int64_t kWideTileCount = 256;
static bool tiled(const skew_tensor_desc &x) {   // a factored matrix that the row-band pass does not take
  const bool mom = x.tier == SKEW_TIER_BACKBONE || (x.state_flags & SKEW_STATE_MOMENTUM) != 0;
  return x.ndim != 1 && (x.tier != SKEW_TIER_ROUTER || (x.state_flags & SKEW_STATE_FACTORED) != 0) &&
         rowband_shape(x.rows, x.cols, x.ld, mom, false).zrb < 1;
}
static int64_t choose_tile_elems(const skew_tensor_desc *d, int n, bool wide) {
  const double count = (double)(wide ? kWideTileCount : kTileCount);
  double total = 0.0;
  for (int i = 0; i < n; i++)
    if (d[i].rows > 0 && d[i].cols > 0 && (!wide || tiled(d[i])))
      total += (double)d[i].rows * (double)d[i].cols * (d[i].ndim == 3 ? (double)std::max<int64_t>(d[i].batch, 0) : 1.0);
  int64_t t = kTileElems;
  while (t > kMinTileElems && total < (double)t * count) t >>= 1;
  return t;
}

// (the longest bands with momentum: 2.2e6 elements)
constexpr double kLeastMomCost = 1.9;
// What trades workspace for time: elements per row band and per tile, and (`compact` unset) padded
// column partials, flat exact-moment tensors and tiles for short narrow matrices; `least`: nothing else
// fits
struct PlanSize {
  int64_t band_elems, tile_elems, wide_tile_elems;
  bool compact, least;
};
static int plan_sized(const skew_tensor_desc *d, int n, const PlanSize &size, Plan *out) {
  const int64_t band_elems = size.band_elems;
  const bool compact = size.compact;
  const double mom_cost = size.least ? kLeastMomCost : kMomCost;
  Plan p;
  // descriptors -> sub-tensors: a stacked (ndim 3) descriptor of E matrices becomes E
  // sub-tensors (one per slice, factored on its own, Sec. 3 footnote) that share one clip
  // factor; every other descriptor is one sub-tensor
  p.desc_sub0.assign((size_t)n, 0);
  p.desc_nsub.assign((size_t)n, 1);
  int64_t nsub = 0;
  for (int i = 0; i < n; i++) {
    const skew_tensor_desc &x = d[i];
    if (x.tier < SKEW_TIER_BACKBONE || x.tier > SKEW_TIER_ROUTER) return SKEW_EINVAL;
    if (x.ndim < 1 || x.ndim > 3) return SKEW_EINVAL;
    if ((x.state_flags & ~(uint32_t)(SKEW_STATE_MOMENTUM | SKEW_STATE_FACTORED | SKEW_STATE_FP32)) != 0)
      return SKEW_EINVAL;
    if (x.ndim == 3 ? x.batch < 0 : (x.batch != 0 && x.batch != 1)) return SKEW_EINVAL;
    const int64_t E = (x.ndim == 3 && x.batch > 1) ? x.batch : 1;
    if (E > INT32_MAX / 4) return SKEW_EINVAL;
    p.desc_sub0[(size_t)i] = (int32_t)nsub;
    p.desc_nsub[(size_t)i] = (int32_t)E;
    nsub += E;
    if (nsub > INT32_MAX / 4) return SKEW_EINVAL;
  }
  p.t.resize((size_t)nsub);
  size_t st = 0;        // state bytes
  size_t ws_part = 0;   // partial-sum bytes (offsets relative to the partial region)
  int64_t items_total = 0;
  for (int di = 0; di < n; di++) {
  const skew_tensor_desc &x = d[di];
  const int32_t sub0 = p.desc_sub0[(size_t)di], E = p.desc_nsub[(size_t)di];
  for (int32_t e = 0; e < E; e++) {
    const int i = sub0 + e;   // the sub-tensor
    TensorPlan &tp = p.t[(size_t)i];
    tp.desc = di;
    tp.grp0 = sub0;
    tp.ngrp = E;
    if (x.rows < 0 || x.cols < 0) return SKEW_EINVAL;
    if (x.rows > 0 && x.cols > INT64_MAX / x.rows) return SKEW_EINVAL;
    const int64_t N = (x.ndim == 3 && x.batch == 0) ? 0 : x.rows * x.cols;
    if (N > 0 && E > INT64_MAX / N) return SKEW_EINVAL;
    tp.tier = x.tier;
    tp.N = N;
    tp.idx0 = (int64_t)e * N;   // the slice's first element in the stacked tensor
    if (x.ndim == 1) {
      if (N > 0 && x.rows != 1 && x.cols != 1) return SKEW_EINVAL;
      tp.n = N > 0 ? 1 : 0;
      tp.m = N;
      tp.ld = N;
    } else {
      if (x.ld < x.cols || x.ld < 1) return SKEW_EINVAL;
      if (x.rows > 0 && x.ld > INT64_MAX / x.rows / E) return SKEW_EINVAL;
      tp.n = x.rows;
      tp.m = x.cols;
      tp.ld = x.ld;
    }
    tp.empty = (N == 0);
    // tiers (Fig. 1) and their variants (Table 3): momentum in the backbone or on request;
    // the exact second moment for vectors and router matrices unless factoring is requested
    const bool factor_router = (x.state_flags & SKEW_STATE_FACTORED) != 0;
    tp.kind = ((x.tier == SKEW_TIER_ROUTER && !factor_router) || x.ndim == 1) ? kExact : kFactored;
    tp.momentum = (x.tier == SKEW_TIER_BACKBONE || (x.state_flags & SKEW_STATE_MOMENTUM) != 0) ? 1 : 0;
    tp.fp32 = (x.state_flags & SKEW_STATE_FP32) != 0 ? 1 : 0;
    if (tp.fp32 && tp.kind != kExact) return SKEW_EINVAL;   // float32 masters: exact-moment tensors
    if (tp.empty) continue;
    // exact-moment tensors are elementwise: where the rows follow each other they are taken as rows
    // of 2048 elements, or as one row (a 2048 x 128 router would leave three lanes of four idle) while
    // its tiles of one row of 2048 are not too many for a launch (2^32 threads: 2^34 elements)
    constexpr int64_t kRow = kChunk * kMaxCw, kMaxOneRow = int64_t(1) << 31;
    if (tp.kind == kExact && tp.ld == tp.m && !compact && (N % kRow == 0 || N <= kMaxOneRow)) {
      tp.n = N % kRow == 0 ? N / kRow : 1;
      tp.m = tp.ld = N / tp.n;
    }

    // state slices: one contiguous array per descriptor (slice e at e times the slice)
    if (e == 0) {
      if (tp.momentum) { tp.off_m = st; st = align_up(st + (size_t)E * N * 4); }
      if (tp.kind == kExact) { tp.off_v = st; st = align_up(st + (size_t)E * N * 4); }
      if (tp.kind == kFactored) {
        tp.off_r = st; st = align_up(st + (size_t)E * tp.n * 4);
        tp.off_c = st; st = align_up(st + (size_t)E * tp.m * 4);
      }
    } else {
      const TensorPlan &t0 = p.t[(size_t)sub0];
      if (tp.momentum) tp.off_m = t0.off_m + (size_t)e * N * 4;
      if (tp.kind == kExact) tp.off_v = t0.off_v + (size_t)e * N * 4;
      if (tp.kind == kFactored) {
        tp.off_r = t0.off_r + (size_t)e * tp.n * 4;
        tp.off_c = t0.off_c + (size_t)e * tp.m * 4;
      }
    }

    // tile grid: tr rows x (512 * cw) columns, about kTileElems elements; cw in {1, 2, 4}
    // so that the four waves of a work-group map onto (chunk, row) pairs statically. The widest
    // strip that fits; a narrower one when the last strip would leave more than 1/16 of the
    // row's width in idle lanes (1536 columns: 512 of 2048; 11008: 1280 of 12288)
    tp.cw = tp.m > 2 * kChunk ? 4 : (tp.m > kChunk ? 2 : 1);
    {
      auto waste = [&](int64_t cw) { return ceil_div(tp.m, (int64_t)kChunk * cw) * kChunk * cw - tp.m; };
      if (16 * waste(tp.cw) > tp.m)
        for (int32_t cw = tp.cw / 2; cw >= 1; cw /= 2)
          if (waste(cw) < waste(tp.cw)) tp.cw = cw;
    }
    const int64_t tc = (int64_t)kChunk * tp.cw;
    // the row-band pass (see rowband_shape)
    const RowBandShape rbs = rowband_shape(tp.n, tp.m, tp.ld, tp.momentum != 0, compact);
    const int64_t zcw = rbs.zcw, nseg = rbs.nseg, rpi = rbs.rpi, zrb = rbs.zrb;
    tp.zpath = (tp.kind == kFactored && rpi > 0 && zrb >= 1) ? 1 : 0;
    // (where workspace is shortest: few rows of more than kMaxMomChunks chunks with momentum, whose tiles
    // keep fewer rows of column partials than the two of each band: half the workspace for 42 x 13259)
    if (tp.zpath && size.least && tp.momentum && zcw > kMaxMomChunks &&
        ceil_div(tp.n, std::max<int64_t>(1, size.wide_tile_elems / tc)) <
            2 * ceil_div(tp.n, band_rows(rbs, tp.m, true, band_elems, mom_cost)))
      tp.zpath = 0;
    // (exact-moment tensors take a quarter of that: their element-by-element path is the
    // slowest per element, and their few tiles would otherwise finish last)
    const int64_t tile_elems = tp.kind == kFactored && !tp.zpath ? size.wide_tile_elems : size.tile_elems;
    tp.tr = std::max<int64_t>(1, tile_elems / tc / (tp.kind == kExact ? 4 : 1));
    const int64_t ntc = ceil_div(tp.m, tc), ntr = ceil_div(tp.n, tp.tr);
    if (ntc * ntr > INT32_MAX / 2 / kSub) return SKEW_EINVAL;   // tile * kSub + part fits an int32
    tp.ntc = (int32_t)ntc;
    tp.ntr = (int32_t)ntr;
    const int64_t tiles = ntc * ntr;

    tp.off_ssum = ws_part; ws_part = align_up(ws_part + (size_t)tiles * kSub * 8);
    tp.off_qsum = ws_part; ws_part = align_up(ws_part + (size_t)tiles * kSub * 8);
    tp.off_sc = ws_part; ws_part = align_up(ws_part + sizeof(TensorScalars));
    if (e == 0) p.clip.push_back({i, 0});   // one clip item per group (its first slice)
    if (E > 1) p.clip_slices.push_back({i, 0});
    // Column partials of successive bands lie 256 bytes off a multiple of 4 KiB: the fold reads a few
    // columns of every band, which at a power of two distance all fall on the same memory channels
    tp.ldp = tp.m + (!compact && tp.m % 512 == 0 ? 32 : 0);
    if (tp.zpath) {
      tp.zcw = (int32_t)zcw;
      tp.nseg = (int32_t)nseg;
      tp.zrpi = (int32_t)rpi;
      tp.zrb = (int32_t)zrb;
      tp.zrows = band_rows(rbs, tp.m, tp.momentum != 0, band_elems, mom_cost);
      const int64_t nzb = ceil_div(tp.n, tp.zrows), nfc = ceil_div(tp.m, kFold);
      if (nzb > INT32_MAX / 2 || nfc > INT32_MAX / 2) return SKEW_EINVAL;
      tp.nzb = (int32_t)nzb;
      tp.nfr = 0;
      tp.nfc = (int32_t)nfc;
      tp.off_colpart = ws_part; ws_part = align_up(ws_part + (size_t)nzb * tp.ldp * 8);
      tp.off_zpart = ws_part; ws_part = align_up(ws_part + (size_t)nzb * tp.ldp * 8);
      tp.off_ainv = ws_part; ws_part = align_up(ws_part + (size_t)tp.n * 8);
      tp.off_bst = ws_part; ws_part = align_up(ws_part + (size_t)nzb * sizeof(BandStats));
      tp.off_cst = ws_part; ws_part = align_up(ws_part + (size_t)nfc * sizeof(ColStats));
      const int64_t nzr = ceil_div(tp.n, kFold);   // row chunks of the gradient-norm mode's fold
      if (nzr > INT32_MAX / 4) return SKEW_EINVAL;
      tp.off_rsum = ws_part; ws_part = align_up(ws_part + (size_t)nzr * 8);
      for (int32_t k = 0; k < tp.nzb; k++) p.z.push_back({i, k});
      // fold items: the column chunks, then runs of kZMaxBandRows rows, whose repeated factors are
      // counted (no more of them than bands: each has a band's statistics to write to; one alone is
      // left to the first column chunk)
      const int64_t nrd = tp.n > kZMaxBandRows ? ceil_div(tp.n, kZMaxBandRows) : 0;
      for (int32_t k = 0; k < (int32_t)nrd + tp.nfc; k++) p.fold.push_back({i, k});
      for (int32_t k = 0; k < (int32_t)nzr + tp.nfc; k++) p.fold_rows.push_back({i, k});
      items_total += nzb + nfc + nrd + nzr + nfc;
    } else if (tp.kind == kFactored) {
      const int64_t nfr = ceil_div(tp.n, kFold), nfc = ceil_div(tp.m, kFold);
      if (nfr + nfc > INT32_MAX / 2) return SKEW_EINVAL;
      tp.nfr = (int32_t)nfr;
      tp.nfc = (int32_t)nfc;
      tp.off_rowpart = ws_part; ws_part = align_up(ws_part + (size_t)ntc * tp.n * 8);
      tp.off_colpart = ws_part; ws_part = align_up(ws_part + (size_t)ntr * tp.ldp * 8);
      tp.off_ainv = ws_part; ws_part = align_up(ws_part + (size_t)tp.n * 8);
      tp.off_rsum = ws_part; ws_part = align_up(ws_part + (size_t)nfr * 8);
      tp.off_cst = ws_part; ws_part = align_up(ws_part + (size_t)(nfr + nfc) * sizeof(ColStats));
      for (int32_t k = 0; k < tp.ntr * tp.ntc; k++) p.p1.push_back({i, k});
      for (int32_t k = 0; k < tp.nfr + tp.nfc; k++) p.fold.push_back({i, k});
      for (int32_t k = 0; k < tp.nfr + tp.nfc; k++) p.fold_rows.push_back({i, k});
      items_total += tiles + 2 * (nfr + nfc);
    }
    if (!tp.zpath) {
      for (int32_t k = 0; k < tp.ntr * tp.ntc * kSub; k++) p.p2.push_back({i, k});   // tile * kSub + part
      items_total += tiles * kSub;
    }
    for (int32_t k = 0; k < tp.ntr * tp.ntc; k++) p.p3.push_back({i, k});
    items_total += tiles;
    if (items_total > INT32_MAX / 2) return SKEW_EINVAL;
  }
  }
  const int nt = (int)p.t.size();   // sub-tensors: the device table's entries
  // update-pass and update-sum items: tiles that take longest go first, so that they do not
  // finish last: the exact second moment's element-by-element path, and matrices narrower
  // than a 512-column strip (idle lanes)
  {
    auto slow = [&](const Item &it) {
      const TensorPlan &tp = p.t[(size_t)it.tensor];
      return tp.kind == kExact || tp.m < 512;
    };
    auto order = [&](std::vector<Item> &v) {
      std::stable_sort(v.begin(), v.end(), [&](const Item &a, const Item &b) { return slow(a) && !slow(b); });
    };
    order(p.p3);
    order(p.p2);
    // row bands: those with momentum, which take longest, first; each of the kernel's bodies together
    auto body = [&](const Item &it) {
      const TensorPlan &tp = p.t[(size_t)it.tensor];
      return std::make_pair(!tp.momentum, tp.nseg == 3 ? 5 : tp.nseg);
    };
    std::stable_sort(p.z.begin(), p.z.end(), [&](const Item &a, const Item &b) { return body(a) < body(b); });
  }
  p.state_bytes = st;
  // workspace: [device tensor table][items p1|z|fold|p2|p3|clip][re-check lists][partials]
  size_t ws = 0;
  p.off_table = ws; ws = align_up(ws + sizeof(DevTensor) * (size_t)std::max(nt, 1));
  // the item lists as the device keeps them
  p.off_items = ws;
  ws = align_up(ws + sizeof(Item) * (p.p1.size() + p.z.size() + p.fold.size() + p.p2.size() + p.p3.size() +
                                     p.clip.size() + p.clip_slices.size() + p.fold_rows.size() + 1));
  p.off_lists = ws;
  ws = align_up(ws + sizeof(RecheckLists) + sizeof(int32_t) * 2 * (size_t)std::max(nt, 1));
  p.off_gscale = ws;
  ws = align_up(ws + sizeof(float));
  p.off_gsq = ws;
  ws = align_up(ws + sizeof(double) * (size_t)std::max(nt, 1));
  auto shift = [ws](size_t &off) {
    if (off != SIZE_MAX) off += ws;
  };
  for (auto &tp : p.t) {
    if (tp.empty) continue;
    for (size_t *o : {&tp.off_ssum, &tp.off_qsum, &tp.off_sc, &tp.off_rowpart, &tp.off_colpart, &tp.off_ainv,
                      &tp.off_rsum, &tp.off_zpart, &tp.off_bst, &tp.off_cst})
      shift(*o);
  }
  p.ws_bytes = ws + ws_part;
  *out = std::move(p);
  return SKEW_OK;
}

int plan_build(const skew_tensor_desc *d, int n, Plan *out) {
  if (n < 0 || (n > 0 && d == nullptr) || out == nullptr) return SKEW_EINVAL;
  return plan_sized(d, n, {choose_band_elems(d, n), choose_tile_elems(d, n, false), choose_tile_elems(d, n, true), false, false}, out);
}

// Most of a large table's workspace are the row bands' column partials: the band size is chosen again with
// fewer bytes for them until the plan fits, up to bands of kZBandElems elements (at last also with
// momentum, or about)
int plan_build_within(const skew_tensor_desc *d, int n, size_t limit, Plan *out) {
  int rc = plan_build(d, n, out);
  double bytes = (double)limit;   // for the column partials
  for (bool last = false; rc == SKEW_OK && out->ws_bytes > limit && !last;) {
    last = bytes <= 0.0;
    const int64_t band = last ? kZBandElems : choose_band_elems(d, n, bytes);
    rc = plan_sized(d, n, {band, kTileElems, kTileElems, true, last}, out);
    bytes = band >= kZBandElems ? 0.0 : bytes - std::max((double)out->ws_bytes - (double)limit, (double)limit / 16);
  }
  return rc;
}

}  // namespace skew
