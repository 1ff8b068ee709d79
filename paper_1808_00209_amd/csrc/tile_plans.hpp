// Launch plans of the matrix-core conv kernels and the many-row FC kernel: which
// shapes they take and how they cut them.  Pure functions of the sizes, on the
// host, so that a plan can be looked at (and its bounds checked) without a GPU.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "conv_geom.hpp"

namespace bnn {

constexpr int kCUs = 256;  // compute units of the chip

// --------------------------------------------- general conv (bconv_mfma.hip)

// Launch plan of the matrix-core conv for a geometry: words per lane and
// iteration (vw), filter tiles per wave (tf), K split (ks), weights through
// LDS (lds), late threshold staging (late), C not a multiple of 64 (tail),
// and whether prepared weights pay (prep).
struct GeneralConvPlan {
  int vw, tf, ks;
  bool lds, late, tail, short8, prep;
  int iters;       // iterations of 2 vw words over the window
  int64_t groups;  // 64-pixel groups
};

inline GeneralConvPlan plan_general_conv(const ConvGeom& g, bool pool, int lds_weights,
                                         int late_thresholds) {
  GeneralConvPlan p;
  const int64_t items = pool ? 4 * int64_t{g.N} * g.Hp * g.Wp : int64_t{g.N} * g.Ho * g.Wo;
  const int64_t groups = (items + 63) / 64;
  const int64_t ftiles = (g.F + 31) / 32;
  // Words per lane, row and iteration: 8-word chunks (128-bit loads) where
  // the channels allow, which halves the vector-memory instructions per MFMA
  // (the texture-address unit is the busiest unit of the small grids), but
  // not when that leaves fewer than 8 iterations to split.
  // C not a multiple of 64: the loop walks Cc >= Cw words per tap, whole
  // chunks of 2 VW words, with the words past Cw zeroed and every word
  // loaded on its own (bconv_mfma32_kernel, TAIL).  VW is the largest of 4,
  // 2, 1 whose padding stays within 1/8 of the row.
  p.tail = g.C % 64 != 0;
  int vw = g.Cw % 8 == 0 ? 4 : g.Cw % 4 == 0 ? 2 : 1;
  // Windows of at most 4 eight-word chunks (K <= 1024 bits, e.g. FC layers
  // of 1024 inputs) on grids too small to fill the chip keep 8-word chunks
  // and no K split: there the split's LDS reduction costs more than it
  // hides (1024 -> 1024 and 1024 -> 10 at 64 rows: 4.15 and 4.30 us against
  // 4.42 and 4.57 us with 2-word chunks split 4 ways).
  const int chunks8 = g.KH * g.KW * (g.Cw / 8);
  p.short8 = !p.tail && vw == 4 && chunks8 <= 4 && groups * ftiles < 1024;
  if (vw == 4 && chunks8 < 8 && !p.short8) vw = 2;
  // Option lds_weights = 1 asks for the LDS-weights kernel wherever no K
  // split is used; it takes chunks of at most 2 words.
  if (lds_weights == 1 && vw == 4) vw = 2;
  if (p.tail) {
    vw = 1;
    for (int t = 4; t >= 2 && vw == 1; t /= 2)
      if (((g.Cw + 2 * t - 1) / (2 * t) * (2 * t) - g.Cw) * 8 <= g.Cw) vw = t;
  }
  p.vw = vw;
  const int Cc = (g.Cw + 2 * vw - 1) / (2 * vw) * (2 * vw);
  const int iters = g.KH * g.KW * (Cc / (2 * vw));
  p.iters = iters;
  p.groups = groups;

  // Tile shape and K split: 64-filter wave tiles down to ~1 wave per SIMD
  // (1024 waves), then 32-filter tiles with a K split over up to 4 waves
  // until there are ~1 (8-word chunks) or ~2 (smaller chunks) waves per
  // SIMD, keeping at least 2 iterations per wave.  Splitting 8 ways never
  // beat 4 (the LDS reduction then costs more than it hides).  With 2-word
  // chunks, grids of >= 4096 64-filter tiles stage the weights through LDS
  // (5-20 % faster there, slower on smaller grids); 8-word chunks without
  // staging were as fast or faster wherever the channels allow them.  All
  // measured on every layer shape of the networks here.
  int tf = 2, ks = 1;
  if (g.F % 64 != 0 || groups * (g.F / 64) < 1024) {
    tf = 1;
    const int64_t target = vw == 4 ? 1024 : 2048;
    while (!p.short8 && ks < 4 && groups * ftiles * ks < target && iters >= 4 * ks) ks *= 2;
  }
  bool lds = lds_weights == -1 ? vw <= 2 && tf == 2 && groups * (g.F / 64) >= 4096
                                    : lds_weights == 1;
  if (ks > 1 || vw == 4) lds = false;
  if (p.tail) {
    tf = 1;
    lds = false;
    if (ks > 4) ks = 4;
  }
  p.tf = tf;
  p.ks = ks;
  p.lds = lds;
  // Thresholds staged after the main loop on grids of at most 2 waves per
  // SIMD (2048 waves) with 32-filter tiles, at kernel start otherwise, where
  // the accumulators can then start from them (16x16x128 -> 256 and
  // 16x16x256 -> 256 pool at batch 64: 5.98 / 7.50 us early against
  // 6.25 / 7.94 us late; 8x8x256 -> 512 with 32-filter tiles: 6.11 us late,
  // 6.22 us early).  Option late_thresholds overrides.
  const int64_t waves = (groups + 3) / 4 * 4 * ((g.F + 32 * tf - 1) / (32 * tf));
  p.late = p.tail || (late_thresholds == -1 ? waves <= 2048 && tf == 1
                                                 : late_thresholds == 1);
  // Prepared weights where they pay (graph-timed on every conv shape of the
  // networks here): 32-filter tiles, where a wave's vector-ALU work per MFMA
  // then drops from 12 to 8 instructions (8x8x512 -> 512 pool at batch 64:
  // 9.7 -> 8.2 us; 8x8x256 -> 512: 6.6 -> 6.0 us), and rows of at most 2
  // words.  With 64-filter tiles over 256 or more channels the prepared
  // operands' registers cost a wave per SIMD (180 against 154 VGPRs) and
  // 4x the weight bytes through L1: 56x56x256 -> 256 took 54 us packed and
  // 60-65 us prepared.  Rows of 4 words without LDS staging also pay
  // (16x16x128 -> 256 at batch 64: 6.3 -> 5.9 us); with LDS staging the
  // packed words are expanded once per block, which prepared operands
  // cannot match (48x48x128 -> 128 pool at batch 256: 48 against 54 us).
  p.prep = tf == 1 || g.Cw <= 2 || (g.Cw <= 4 && !lds);
  return p;
}

// Estimated time of the general conv in microseconds at default options, for
// C not a multiple of 64, fitted (non-negative least squares on relative
// errors) to graph-timed runs of 8000 random shapes (32 to 600 channels, 33 to
// 512 filters, 1 to 30 taps, 4 to 300 us; half of the estimates within 6 %,
// nine in ten within 16 %): a start, then per pass the latency of a wave's
// k-steps, what its vector instructions and MFMAs take from its SIMD (more
// where rows of a multiple of 32 bytes meet in the same cache banks), and the
// sums' bytes.  prep: with prepared weights.
inline double general_conv_us(const ConvGeom& g, bool sums, bool bits, bool prep) {
  struct Cost {
    double start, latency, step, wave, row32, split;
  };
  static constexpr Cost kPacked[3] = {{3.16, 0.142, 0.132, 0.278, 0.026, 0.10},
                                      {3.34, 0.083, 0.096, 0.472, 0.041, 0.02},
                                      {3.76, 0.078, 0.076, 1.010, 0.050, 0.00}};
  static constexpr Cost kPrepared[3] = {{3.07, 0.110, 0.096, 0.278, 0, 0.13},
                                        {3.32, 0.041, 0.074, 0.348, 0, 0.10},
                                        {3.24, 0.037, 0.055, 0.533, 0, 0.00}};
  const bool row32 = g.KH * g.KW * g.Cw % 8 == 0;
  // odd pooled sizes with sums: one pass for the sums, one for the bits
  const bool two = g.pool == 2 && sums && ((g.Ho & 1) || (g.Wo & 1));
  double us = 0;
  for (int pass = 0; pass < (two && bits ? 2 : 1); ++pass) {
    const bool pool = g.pool == 2 && !(two && pass == 0), s = sums && pass == 0;
    const GeneralConvPlan p = plan_general_conv(g, pool, -1, -1);
    const bool pr = prep && p.prep;
    const int v = p.vw == 4 ? 2 : p.vw - 1;
    const Cost& c = pr ? kPrepared[v] : kPacked[v];
    const int64_t fy = (g.F + 32 * p.tf - 1) / (32 * p.tf);
    const int64_t pixel_waves = p.ks == 1 ? (p.groups + 3) / 4 * 4 : p.groups * p.ks;
    const double waves = static_cast<double>(pixel_waves * fy) / 1024;  // per SIMD
    const double steps = static_cast<double>(p.iters) * p.vw / p.ks;
    us += c.start + c.latency * steps +
          waves * (steps * (c.step + (row32 ? c.row32 : 0)) + c.wave + (p.ks > 1 ? c.split : 0));
    if (s) {
      const double mb = 4e-6 * g.N * g.Ho * g.Wo * g.F;
      us += 1.7 + mb * (g.F % 4 ? 0.58 : 0.17);
    }
  }
  return us;
}

// ------------------------------------------- staged-tile conv (bconv_tile.hip)

// LDS words per pixel of a wave's 64 sums (16-byte aligned, odd in 16s).
constexpr int kConvTileSumStride = 68;

// K-steps per tap and chunk (ks), chunks, log2 of the waves along the filters
// (wfl), filter groups (fgs), strips of Ws item columns, LDS bytes; ok when
// the kernel takes the shape.
struct ConvTilePlan {
  bool ok;
  double cost;
  int ks, nchunk, wfl, RS, Ws, cols;
  int64_t strips, items, units, fgs;  // units: of 32 pixels per wave, all strips
  size_t lds;
  int64_t ups;                        // units per strip
  int32_t H, W, N, Ho, Wo, Hw, Ww;
};

// Smallest grids worth it, in units times filter groups (conv_tile_pays).
constexpr int64_t kConvTileUnits = 2048, kConvTileTailUnits = 256;
constexpr size_t kConvTileLds = 79 * 1024;  // dynamic LDS per block: two blocks per CU

inline ConvTilePlan plan_conv_tile(const ConvGeom& g, bool sums) {
  ConvTilePlan p = {};
  const bool pool = g.pool == 2;
  // A 1x1 conv has no neighbours: its pixels are rows of one column, so that
  // a block stages only its own pixels.
  const bool flat = g.KH == 1 && g.KW == 1 && g.pad == 0 && !pool;
  p.N = flat ? 1 : g.N;
  p.H = flat ? g.N * g.H * g.W : g.H;
  p.W = flat ? 1 : g.W;
  p.Ho = flat ? p.H : g.Ho;
  p.Wo = flat ? 1 : g.Wo;
  // pooling windows: whole ones, or with sums wanted also those cut by an
  // odd edge, so that every pixel is covered
  p.Hw = pool ? (sums ? (p.Ho + 1) / 2 : p.Ho / 2) : p.Ho;
  p.Ww = pool ? (sums ? (p.Wo + 1) / 2 : p.Wo / 2) : p.Wo;
  const int rh = pool ? 2 : 1;
  const int skip = std::max(p.H + 2 * g.pad - rh * p.Hw, 0);
  // Waves along the filters (4, 2 or 1, the rest along the pixels), channel
  // chunk and strip width: the cheapest in estimated cycles.  Per full run and
  // wave: its MFMAs (32 cycles, 1.25 times that with the loop's other work),
  // the staging's vector instructions (about 30 + 8 ks per word half, 4 cycles
  // each) and about 4500 cycles of start, barriers and epilogue; times the
  // runs, padded filters and columns included.
  for (int wfl = 2; wfl >= 0; --wfl) {
    const int64_t fgs = (g.F + (64 << wfl) - 1) / (64 << wfl);
    const int unit = (4 >> wfl) * 32;
    const int per = 4 * unit / (rh * rh);  // grid items of a run
    bool fits = false;
    // Chunks of at most 8 words, smaller ones where the staged rows do not
    // fit (of the sizes that cut Cw into as many chunks, the smallest).
    int ks = (g.Cw + 2 * ((g.Cw + 7) / 8) - 1) / (2 * ((g.Cw + 7) / 8));
    for (; !fits && ks >= 1; --ks) {
      const int nchunk = (g.Cw + 2 * ks - 1) / (2 * ks);
      if (ks > 1 && (g.Cw + 2 * ks - 3) / (2 * ks - 2) == nchunk) continue;
      const int ps = 2 * ks + 1;
      const double mfma = 1.25 * 32 * 2 * 4 * g.KH * g.KW * ks;
      // Strip widths worth a look: wider than a run only stages more columns,
      // and a run touches at least two item rows, which have to fit.  From
      // there down every width that some number of strips has, above 32 in
      // steps of an eighth, so that a plan takes about as long on a wide map
      // as on a small one (0.9 us at 56 columns, 2.4 us at 1024 and at
      // 262144, where a step per strip took 11 us and 2.1 ms).
      const int fit = static_cast<int>(kConvTileLds / 16) / (ps * (2 * rh + g.KH - 1));
      for (int w = std::min({p.Ww, per, (fit - (g.KW - 1)) / rh}); w >= 1;) {
        const int strips = (p.Ww + w - 1) / w;
        if (strips > 1 && p.Ww / strips < 4) break;
        const int Ws = (p.Ww + strips - 1) / strips;
        w = Ws > 32 ? Ws - Ws / 8 : Ws - 1;
        // Virtual rows a run may touch: item rows spanned, the window height,
        // and the rows skipped at each image boundary crossed.
        const int span = 1 + (per - 1 + Ws - 1) / Ws;
        const int cross = (span - 1 + p.Hw - 1) / p.Hw;
        const int rows = rh * span + g.KH - 1 + cross * skip;
        const int cols = rh * Ws + g.KW - 1;
        int RS = cols * ps;
        // Pooled tiles: a row stride of 4 mod 8 entries puts the two rows of a
        // window on different banks.
        if (pool) RS += ((4 - RS % 8) + 8) % 8;
        size_t lds = static_cast<size_t>(rows) * RS * 16;
        if (sums) lds = std::max(lds, size_t{4} * 32 * kConvTileSumStride * 4);
        if (lds > kConvTileLds) continue;
        fits = true;
        const int64_t items = int64_t{rh * rh} * p.N * p.Hw * Ws;
        const int64_t ups = (items + unit - 1) / unit;
        const double cost = static_cast<double>(fgs * strips * ups) / 4 *
                            (nchunk * (mfma + rows * cols / 128.0 * (30 + 8 * ks) * 4) + 4500);
        if (p.ok && cost >= p.cost) continue;
        p.ok = true;
        p.cost = cost;
        p.wfl = wfl;
        p.fgs = fgs;
        p.ks = ks;
        p.nchunk = nchunk;
        p.Ws = Ws;
        p.strips = strips;
        p.RS = RS;
        p.lds = lds;
        p.cols = cols;
        p.items = items;
        p.ups = ups;
        p.units = strips * ups;
      }
    }
  }
  return p;
}
// The runs of an XCD's units: `full` of 4 units, as many rounds of one per
// block slot as there are whole ones, then runs of `last` units that give
// every slot an even share.
struct ConvTileRuns {
  int64_t slots, per_xcd, full, last, rest;
};

inline ConvTileRuns conv_tile_runs(const ConvTilePlan& p) {
  ConvTileRuns r;
  r.slots = std::max<int64_t>(512 / p.fgs / 8, 1);  // per XCD and filter group
  r.per_xcd = (p.units + 7) / 8;
  r.full = r.per_xcd / (4 * r.slots) * r.slots;
  r.rest = r.per_xcd - 4 * r.full;
  // (runs of 2 units, two to a compute unit, take as long as half as many
  // full ones, one to a compute unit)
  const int64_t even = r.rest ? (r.rest + r.slots - 1) / r.slots : 1;
  r.last = even == 2 && r.full > 0 ? 4 : even;
  return r;
}

// Virtual rows that a run of `units` units may touch.
inline int conv_tile_rows(const ConvGeom& g, const ConvTilePlan& p, int units) {
  const int rh = g.pool == 2 ? 2 : 1;
  const int per = std::max(units * (4 >> p.wfl) * 32 / (rh * rh), 1);
  const int span = 1 + (per - 1 + p.Ws - 1) / p.Ws;
  const int cross = (span - 1 + p.Hw - 1) / p.Hw;
  return rh * span + g.KH - 1 + cross * std::max(p.H + 2 * g.pad - rh * p.Hw, 0);
}

// Estimated time of the staged-tile conv in microseconds, C not a multiple of
// 64, fitted like general_conv_us and as close: rounds of runs, each its
// start, its taps' and chunks' latencies, the staging's vector instructions
// and its units' MFMAs (which take four times as long with two blocks on a
// compute unit as with one: the last round of at most 256 blocks), then the
// sums.  The 4-k-step form spills registers, most of all with sums.
inline double conv_tile_us(const ConvGeom& g, const ConvTilePlan& p, bool sums) {
  const ConvTileRuns r = conv_tile_runs(p);
  const double full = static_cast<double>(r.full / r.slots);
  const int last = r.rest ? static_cast<int>(r.last) : 0;
  const bool paired = r.rest && (r.rest + r.last - 1) / r.last * p.fgs * 8 > 256;
  const int taps = g.KH * g.KW, steps = taps * p.ks * p.nchunk;
  const double rounds = full + (last ? 1 : 0);
  const double staged = full * conv_tile_rows(g, p, 4) * p.cols / 128.0 +
                        (last ? conv_tile_rows(g, p, last) * p.cols / 128.0 : 0);
  const double units2 = 4 * full + (paired ? last : 0), units1 = paired ? 0 : last;
  const double units = units2 + 0.4 * units1;
  double us = 2.25 + rounds * (1.58 + p.nchunk * (0.88 + 0.145 * taps)) +
              staged * p.nchunk * p.ks * 0.08 + steps * (0.058 * units2 + 0.015 * units1);
  if (taps * g.Cw % 8 == 0 && p.ks <= 2) us += 0.010 * units * steps;  // rows of 32 bytes
  if (p.ks == 4) us += 0.012 * units * steps;
  if (sums) {
    const double mb = 4e-6 * g.N * g.Ho * g.Wo * g.F;
    us += 2.03 + mb * ((g.F % 4 ? 0.31 : 0.129) + (p.ks == 4 ? 0.078 : 0));
  }
  // (chunks of one k-step: the loop's start and end outweigh it)
  return p.ks == 1 && p.nchunk >= 3 ? 1.2 * us : us;
}

// Where this kernel is the faster one.  prep: the general kernel would get
// prepared weights.
inline bool conv_tile_pays(const ConvGeom& g, bool sums, bool bits, bool prep,
                           const ConvTilePlan& p) {
  if (!p.ok || p.fgs > 64) return false;
  const int taps = g.KH * g.KW, steps = taps * p.ks;
  // C not a multiple of 64: the general kernel loads word by word and pads in
  // its loop, which this one avoids on large grids (160 -> 256, 5x5 at 19 x
  // 64 x 64: 108 -> 47 us) and does not on small ones, at padded row lengths
  // or against prepared weights (49 -> 414 3x4 at 12 x 29 x 59: 13.0 us there,
  // 15.1 here; 459 -> 256 3x3 at 28 x 45 x 12, prepared: 12.8 and 18.5; 195 ->
  // 256 1x1 at 194 x 13 x 15 with sums: 16.7 and 19.4): the smaller estimate,
  // less a margin where the estimates favour this kernel too often (even
  // windows, whose filters' words collide in the caches, 1x1 and prepared
  // weights).
  if (g.C % 64 != 0) {
    if (p.units * p.fgs < kConvTileTailUnits) return false;
    const double margin =
        (taps == 1 ? 0.92 : taps % 2 == 0 ? 0.85 : 1.0) * (prep ? 0.95 : 1.0);
    return conv_tile_us(g, p, sums) < margin * general_conv_us(g, sums, bits, prep);
  }
  // Otherwise: a neighbourhood to stage for, one channel chunk (two halve the
  // work per staging: 512 -> 512 at 28 x 28 x 34 ran 8 % slower here), at
  // least 9 k-steps per run's pixel (18 when pooling: 64 -> 256 pooled 3 %
  // slower, 64 -> 128 without pooling the same to 10 % faster), at least two
  // waves along the filters of which at most 1/8 is padding, and a full run
  // for every block slot (smaller grids are faster with the general kernel's
  // K split).  Bits of windows of a multiple of 4 taps, whose filters' rows
  // are a multiple of 32 bytes, only at 192 channels or from 48 k-steps on (64
  // -> 128 4x4 at 141 x 55 x 105: 50.7 us there, 65.5 here; 256 -> 512 2x2 at
  // 5 x 38 x 586: 28.0 and 32.1; with sums this kernel is the faster one).
  if (!sums && taps % 4 == 0 && g.C != 192 && steps < 48) return false;
  const int64_t units = p.units * p.fgs;
  // (Just past a full round of 2048 units the second one's runs of one unit, on
  // more than one block per compute unit, take most of a full run's time: 128
  // -> 256 at 32 x 26 x 98, 2548 units, 14.9 us there, 17.2 here.  On one block
  // per compute unit they do not (256 -> 512 pooled at 256 x 12 x 12, 2304
  // units, 20.4 and 17.7), and from 512 units on they are runs of 4 on fewer
  // blocks (256 -> 256 from 2560 units 0.83 to 0.92 of the time); at 64
  // channels a run's start weighs more.  Sums gain more than that, but at 256
  // channels, and so do 192 channels.)
  if (g.F % 64 == 0 && g.C != 192 && (!sums || g.C == 256) && units > 2304 &&
      units < (g.C == 64 ? 3072 : 2560))
    return false;
  return p.nchunk == 1 && steps >= (g.pool == 2 ? 18 : 9) && p.wfl >= 1 &&
         8 * p.fgs * (64 << p.wfl) <= 9 * int64_t{g.F} && units >= kConvTileUnits;
}

// Whether the staged-tile kernel takes the conv, and how.  What can be told
// without a plan comes first (a plan takes 1 to 3 us of host time).
inline bool conv_tile_plan(const ConvGeom& g, bool sums, bool bits, bool prep, ConvTilePlan* p) {
  // (With 32 filters half of every wave's would be padding; a 1x1 conv has
  // nothing to stage for unless its rows are ragged, and it lost there too
  // when pooled (96 -> 192 at 64 x 64 x 120: 26 -> 31 us) or of several chunks
  // (4100 -> 1000 at 4096 rows: 22 -> 44 us).)
  const bool ragged = g.C % 64 != 0, one = g.KH * g.KW == 1;
  if (g.F <= 32 || (one && (!ragged || g.pool == 2)) || ((!ragged || one) && g.Cw > 8))
    return false;
  // (the k-steps of one chunk: conv_tile_pays)
  if (!ragged && g.KH * g.KW * (g.Cw / 2) < (g.pool == 2 ? 18 : 9)) return false;
  // (units x filter groups, padding aside, are the outputs / 8192)
  const int64_t outputs = int64_t{g.N} * (g.Ho + 1) * (g.Wo + 1) * ((g.F + 63) / 64 * 64);
  if (outputs / 8192 < (ragged ? kConvTileTailUnits : kConvTileUnits) * 2 / 3) return false;
  *p = plan_conv_tile(g, sums);
  return conv_tile_pays(g, sums, bits, prep, *p);
}

// ------------------------------------------------ many-row FC (bfc_tile.hip)

constexpr int kFcTileRows = 128;  // data rows per block, at most

// log2 of the waves along the outputs, 32-row tiles per wave, and the grid in
// tiles.
struct FcTilePlan {
  int wfl, pt;
  int64_t output_tiles, row_tiles;
};

// Whether the many-row kernel takes an FC layer / GEMM, and how.
inline bool fc_tile_plan(int64_t M, int64_t N, int64_t K, bool sums, bool bits, FcTilePlan* p) {
  const int64_t Kw = (K + 31) / 32;
  if (K < 1024 || K >= (1 << 22) || M * Kw * 4 >= (int64_t{1} << 31) - 4096 ||
      N * Kw * 4 >= (int64_t{1} << 31) - 4096)
    return false;
  // Grids of more than 1024 32 x 32 tiles, where the FC kernel's 2 x 2 form
  // needs a second round of workgroups (graph-timed, bits: 1100 x 8192 -> 1024
  // 19.3 us there, 17.5 here; 1024 x 1024 -> 1024, one round, 4.6 and 6.2);
  // where N is not a multiple of 64, more than 2048, below which the conv
  // kernel is as fast (2048 x 4096 -> 1000 9.7 us there, 11.3 here; 4096 x
  // 4100 -> 1000 22.4 and 15.3).
  const int64_t t32 = ((M + 31) / 32) * ((N + 31) / 32);
  if (t32 <= (N % 64 == 0 ? 1024 : 2048)) return false;
  // Sums alone are as fast there up to 2048 tiles at the row lengths that the
  // FC kernel splits evenly (262 x 2048 -> 4096 8.2 us there, 8.7 here; 4096
  // bits 11.5 and 11.9, 1280 bits 7.5 and 6.7; with bits too 9.2 and 9.0).
  if (!bits && t32 <= 2048 && (K == 1024 || K == 2048 || K == 4096)) return false;
  // Up to 32 outputs, where at least half of a wave's 64 are padding, only
  // where the conv kernel cannot take the rows in whole 256-bit chunks, and
  // then long ones (bits, 66000 rows: 4096 -> 32 15.6 us there, 19.4 here; 1030
  // -> 32 7.5 and 10.6; 5000 -> 32 26.9 and 23.7, -> 4 20.6 and 22.2; 16000 -> 16
  // 61.8 and 54.6).
  if (N <= 32 && (K % 256 == 0 || (K < 8192 && (K % 64 == 0 || N <= 16 || (!sums && K < 4096)))))
    return false;
  // Tile: 4 waves as 1 << wfl along the outputs (64 each) and the rest along
  // the rows (32 PT each, at most 128 in all), by the estimated time: rounds of
  // two blocks per compute unit, each its chunks' MFMAs (8 PT per chunk and
  // wave, at about 38 / 44 / 60 cycles for PT = 4 / 2 / 1, whose weight
  // expansion serves fewer MFMAs; at least the latency of a chunk) plus about
  // 7000 cycles.
  const int64_t chunks = (Kw + 7) / 8;
  double best = 0;
  p->wfl = -1;
  for (int wfl = 0; wfl <= 2; ++wfl) {
    for (int pt = 4; pt >= 1; pt /= 2) {
      const int wp = 4 >> wfl;
      if (wp * pt * 32 > kFcTileRows) continue;
      const int64_t tiles = ((N + (64 << wfl) - 1) / (64 << wfl)) *
                            ((M + wp * pt * 32 - 1) / (wp * pt * 32));
      // one block or two per compute unit
      const double one = 8 * pt * (pt == 4 ? 38 : pt == 2 ? 44 : 60);
      const double per = tiles <= kCUs ? std::max(one, 700.0) : std::max(1.9 * one, 1000.0);
      const double cost = static_cast<double>((tiles + 2 * kCUs - 1) / (2 * kCUs)) *
                          (chunks * per + 7000);
      if (p->wfl < 0 || cost < best) {
        best = cost;
        p->wfl = wfl;
        p->pt = pt;
      }
    }
  }
  const int64_t rows = (4 >> p->wfl) * p->pt * 32;
  p->output_tiles = (N + (64 << p->wfl) - 1) / (64 << p->wfl);
  p->row_tiles = (M + rows - 1) / rows;
  return true;
}

// --------------------------------------------------- 1x1 conv (bconv_1x1.hip)

constexpr int kConv1x1Pixels = 256;  // pixels per block

// Groups that the F filters are split into, for `blocks` blocks of pixels: one
// block takes all of them, or a half or quarter (at least 4 chunks of 64)
// where the finer grid's last round is that much fuller, at about 2 % per
// extra group for the operands built again.  56 x 56 x 256 -> 1024 at
// batch 64 is 3.06 whole-row blocks per compute unit, of which some took a
// fourth: 34.1 us, 29.6 in quarters.
inline int conv1x1_groups(int64_t blocks, int F) {
  int groups = 1;
  double best = 0;
  for (int n = 1; n <= 4 && F % (64 * n) == 0 && (n == 1 || F / n >= 256); n *= 2) {
    const double cost = static_cast<double>((blocks * n + kCUs - 1) / kCUs) / n *
                        (1 + 0.02 * (n - 1));
    if (n == 1 || cost < best) {
      best = cost;
      groups = n;
    }
  }
  return groups;
}

}  // namespace bnn
