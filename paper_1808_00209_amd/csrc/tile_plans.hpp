// Launch plans of the tile kernels: which shapes they take and how they cut
// them.  Pure functions of the sizes, on the host, so that a plan can be
// looked at (and its bounds checked) without a GPU.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "conv_geom.hpp"

namespace bnn {

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
// Where the staged-tile kernel is the faster one (graph-timed against the general kernel
// over 140 random shapes, 2 to 250 images, 32 to 512 channels and filters, 1x1
// to 5x5).
inline bool conv_tile_pays(const ConvGeom& g, const ConvTilePlan& p) {
  if (!p.ok || p.fgs > 64) return false;
  // C not a multiple of 64: the general kernel loads word by word and pads in
  // its loop (x1.04 to x2.4 here from 256 units on; 160 -> 256, 5x5 at 19 x 64
  // x 64: 108 -> 47 us).
  if (g.C % 64 != 0) return p.units * p.fgs >= kConvTileTailUnits;
  // Otherwise: a neighbourhood to stage for, one channel chunk (two halve the
  // work per staging: 512 -> 512 at 28 x 28 x 34 ran 8 % slower here), at
  // least 9 k-steps per run's pixel (18 when pooling: 64 -> 256 pooled 3 %
  // slower, 64 -> 128 without pooling 9 % faster), at least two waves along
  // the filters of which at most 1/8 is padding, and a full run for every
  // block slot (smaller grids are faster with the general kernel's K split).
  const int steps = g.KH * g.KW * p.ks;
  return p.nchunk == 1 && steps >= (g.pool == 2 ? 18 : 9) && p.wfl >= 1 &&
         8 * p.fgs * (64 << p.wfl) <= 9 * int64_t{g.F} && p.units * p.fgs >= kConvTileUnits;
}

// Whether the staged-tile kernel takes the conv, and how.  What can be told
// without a plan comes first (a plan takes 1 to 3 us of host time).
inline bool conv_tile_plan(const ConvGeom& g, bool sums, ConvTilePlan* p) {
  // (With 32 filters half of every wave's would be padding; a 1x1 conv has
  // nothing to stage for unless its rows are ragged, and it lost there too
  // when pooled (96 -> 192 at 64 x 64 x 120: 26 -> 31 us) or of several chunks
  // (4100 -> 1000 at 4096 rows: 22 -> 44 us).)
  const bool ragged = g.C % 64 != 0, one = g.KH * g.KW == 1;
  if (g.F <= 32 || (one && (!ragged || g.pool == 2)) || ((!ragged || one) && g.Cw > 8)) return false;
  // (the k-steps of one chunk: conv_tile_pays)
  if (!ragged && g.KH * g.KW * (g.Cw / 2) < (g.pool == 2 ? 18 : 9)) return false;
  // (units x filter groups, padding aside, are the outputs / 8192)
  const int64_t outputs = int64_t{g.N} * (g.Ho + 1) * (g.Wo + 1) * ((g.F + 63) / 64 * 64);
  if (outputs / 8192 < (ragged ? kConvTileTailUnits : kConvTileUnits) * 2 / 3) return false;
  *p = plan_conv_tile(g, sums);
  return conv_tile_pays(g, *p);
}

}  // namespace bnn
