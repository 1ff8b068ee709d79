// Binary convolution on the fp4 matrix cores with the input staged once per
// run of pixels (Eq. 3 and Eq. 4 with the threshold / flip / OR-pool epilogue
// of bnn_bconv2d; sums as well as bits).
//
// The general kernel (bconv_mfma.hip) loads and expands both operands of
// every k-step in every wave: 8-13 vector instructions per MFMA at 4 cycles
// each beside the MFMA's 32, and an image word is expanded once per tap,
// filter tile and wave.  Here a block stages the input rows that a run of
// output pixels touches in LDS, each word already expanded to its fp4 operand
// (16 bytes), once; every tap of up to 256 filters then reads activation
// operands straight from LDS.  A wave computes 64 filters x 32 PT pixels
// (PT up to 4): per k-step 2 weight operands (packed words, expanded in
// registers) serve 2 PT MFMAs.
//
// The map is cut into strips of Ws columns (as few staged pixels per output
// pixel as the shape allows: a run of 128 pixels touches 8 rows of 58 columns
// at 56 x 56 in one strip, 13 of 16 in four).  Within a strip, pixels are
// taken in raster order over the whole batch (2x2 windows in raster order when
// pooling), so a run may span images and only a strip's last one is partial.
// Rows are numbered virtually: image n's padded rows are n Hv .. n Hv + Hv -
// 1, Hv = H + 2 pad, and output row i of image n reads virtual rows n Hv + i
// .. n Hv + i + KH - 1; a block stages the virtual rows from its first pixel's
// window to its last one's.  Channels are taken in chunks of 2 KS words;
// positions past C are stored as fp4 0.0, so their products vanish whatever
// the weight words hold there.
//
// A block takes a run of 4 units (32 pixels per wave along the pixels), two
// blocks per compute unit; the runs of the grid's last round are shorter, as
// many as it takes to give every compute unit an even share (56 x 56 x 256 at
// batch 64 is 6.1 full runs per compute unit: with full runs only, a few
// took 7).
#include <type_traits>

#include "fastdiv.hpp"
#include "fp32_split.hpp"
#include "fp4_expand.hpp"
#include "kernels.hpp"
#include "lane_ops.hpp"
#include "tile_plans.hpp"

namespace bnn {
namespace {

constexpr uint32_t kOutOfRange = 0x80000000u;  // raw buffer loads read 0 there
constexpr int kRsrcWord3 = 0x00020000;
constexpr int kNT = 256;

struct TileArgs {
  const uint32_t* in;
  const uint32_t* w;
  const int32_t* thr;
  const uint32_t* flip;
  int32_t* sums;
  uint32_t* bits;
  int32_t H, W, Cw, F, Fw, KH, KW, pad;
  int32_t Ho, Wo;      // outputs before pooling
  int32_t Hw;          // item grid rows per image: pooling windows, or pixels
  int32_t Ws;          // item columns per strip
  int32_t Hp, Wp;      // stored bits
  int32_t items;       // pixels of a strip (4 per window when pooling)
  int32_t Hv, vrows;   // virtual rows per image / in all
  int32_t cols;        // staged columns of a strip
  int32_t RS;          // LDS entries per staged row
  int32_t step_row, step_col;  // kNT / 2 pixels on in the staged rows
  int32_t K, nchunk, pool;
  int32_t wfl;         // log2 of the waves along the filters
  int32_t fstride;     // words per filter
  uint32_t tmask_c;    // valid bits of a pixel's last word
  int32_t in_bytes, w_bytes;
  FastDiv31 div_w, div_h, div_cols, div_hv, div_f, div_t;
  int32_t units;       // units of 32 wp pixels (wp: waves along the pixels), all strips
  int32_t nfull, last; // per XCD: runs of 4 units; then runs of `last` units
  int32_t xcd_units;   // units per XCD
};

// Image, item grid position and output pixel; jw and j count from the
// strip's first column.
struct Pix {
  int n, iw, jw, i, j;
};

__device__ __forceinline__ Pix decode(const TileArgs& a, int item) {
  const uint32_t m = static_cast<uint32_t>(item);
  const uint32_t p = a.pool ? m >> 2 : m;
  const uint32_t t = fdiv(p, a.div_w);
  Pix r;
  r.jw = static_cast<int>(p - t * a.div_w.d);
  r.n = static_cast<int>(fdiv(t, a.div_h));
  r.iw = static_cast<int>(t - r.n * a.div_h.d);
  r.i = a.pool ? 2 * r.iw + static_cast<int>((m >> 1) & 1) : r.iw;
  r.j = a.pool ? 2 * r.jw + static_cast<int>(m & 1) : r.jw;
  return r;
}

// KS consecutive words at any 4-byte alignment.
template <int KS>
__device__ __forceinline__ void load_words(uint32_t (&v)[KS], __amdgpu_buffer_rsrc_t r,
                                           uint32_t voff, uint32_t soff) {
  if constexpr (KS == 4) {
    const auto t = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = t[i];
  } else if constexpr (KS == 3) {
    const auto t = __builtin_amdgcn_raw_buffer_load_b96(r, voff, soff, 0);
#pragma unroll
    for (int i = 0; i < 3; ++i) v[i] = t[i];
  } else if constexpr (KS == 2) {
    const auto t = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
    v[0] = t[0];
    v[1] = t[1];
  } else {
    v[0] = __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0);
  }
}

// KS: k-steps (of 64 bits) per tap and channel chunk; lane half h feeds words
// h KS .. h KS + KS - 1 of the chunk in both operands, so a lane's weight
// words of a tap are one load.  SUMS: int32 sums wanted (bits too when
// a.bits).  TAIL: C is not 64 KS nchunk.
template <int KS, bool SUMS, bool TAIL>
__global__ __launch_bounds__(kNT, 2) void bconv_tile_kernel(TileArgs a) {
  constexpr int CW = 2 * KS;
  constexpr int PS = CW + 1;              // LDS entries per staged pixel (odd: no conflicts)
  constexpr int PD = KS == 4 ? 3 : KS == 3 ? 2 : 4;  // taps of weight words in flight
  constexpr int UB = 2;                   // staging loads in flight per thread
  extern __shared__ v4i act[];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, c = lane & 31;
  // Block b runs on XCD b mod 8: an XCD's blocks take neighbouring runs in
  // order (first its full ones), and the blocks of a run's filter groups
  // follow each other.
  const uint32_t bt = blockIdx.x >> 3;
  const int q = static_cast<int>(fdiv(bt, a.div_f));
  const int fg = static_cast<int>(bt) - q * static_cast<int>(a.div_f.d);
  int u = static_cast<int>(blockIdx.x & 7) * a.xcd_units +
          (q < a.nfull ? 4 * q : 4 * a.nfull + (q - a.nfull) * a.last);
  const int u_end = min(u + (q < a.nfull ? 4 : a.last),
                        min(a.units, (static_cast<int>(blockIdx.x & 7) + 1) * a.xcd_units));
  const int wfi = wave & ((1 << a.wfl) - 1), wpi = wave >> a.wfl;
  const int wp = 4 >> a.wfl;              // waves along the pixels
  const int f0 = (fg << (6 + a.wfl)) + wfi * 64;  // wave's first filter
  const int rs = a.pool ? 2 : 1;

  const __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint32_t*>(a.in), 0, a.in_bytes, kRsrcWord3);
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint32_t*>(a.w), 0, a.w_bytes, kRsrcWord3);
  // (thresholds and flips through buffers of length 0 when absent: no branch
  // that would wait for them here)
  const __amdgpu_buffer_rsrc_t rthr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int32_t*>(a.thr), 0, !SUMS || a.bits ? a.F * 4 : 0, kRsrcWord3);
  const __amdgpu_buffer_rsrc_t rflip = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint32_t*>(a.flip), 0, a.flip ? a.Fw * 4 : 0, kRsrcWord3);
  const int wi = f0 / 32 + h;             // this lane half's output word

  // This thread's first staged pixel (word halves tid, tid + kNT, ...).
  const uint32_t srow = fdiv(static_cast<uint32_t>(tid) >> 1, a.div_cols);
  const int scol = static_cast<int>((static_cast<uint32_t>(tid) >> 1) - srow * a.div_cols.d);
  const uint32_t smask = __builtin_amdgcn_readfirstlane(0x88888888u);
  uint32_t vfill;
  asm("v_mov_b32 %0, 0x22222222" : "=v"(vfill));

  // Weight words of the next PD taps, in flight.
  const int taps = a.KH * a.KW;
  uint32_t woff[2];
#pragma unroll
  for (int tf = 0; tf < 2; ++tf)
    woff[tf] = (static_cast<uint32_t>(f0 + 32 * tf + c) * a.fstride + h * KS) * 4;
  uint32_t wr[PD][2][KS];
  auto load_w = [&](uint32_t (&ww)[2][KS], int tap, int ch) {
    const uint32_t so = static_cast<uint32_t>((min(tap, taps - 1) * a.Cw + ch * CW) * 4);
#pragma unroll
    for (int tf = 0; tf < 2; ++tf) load_words<KS>(ww[tf], rw, woff[tf], so);
  };
  int32_t thv[2];
  uint32_t fl;

  // The run of PT units from unit u on (within one strip).
  auto do_run = [&](auto ptc) {
    constexpr int PT = decltype(ptc)::value;
    const int strip = static_cast<int>(fdiv(static_cast<uint32_t>(u), a.div_t));
    const int js0 = strip * a.Ws;  // the strip's first item column
    const int p0 = (u - strip * static_cast<int>(a.div_t.d)) * 32 * wp;
    const Pix first = decode(a, min(p0, a.items - 1));
    const Pix end = decode(a, min(p0 + PT * 32 * wp, a.items) - 1);
    const int v0 = first.n * a.Hv + rs * first.iw;  // staged virtual rows
    const int rows = end.n * a.Hv + rs * end.iw + (rs - 1) - v0 + a.KH;
    const int halves = rows * a.cols * 2;  // word halves (KS words) to stage
    // Staging: thread t takes word halves t, t + kNT, ... (KS words each;
    // pixels outside the image read the pad word 0), UB loads in flight,
    // skipped by the waves past the end.
    uint32_t row, xw[UB][KS];
    int col, dst[UB];
    auto stage_load = [&](int base, int ch) {
#pragma unroll
      for (int b = 0; b < UB; ++b) {
        if (base + b * kNT >= halves) break;
        const uint32_t v = static_cast<uint32_t>(v0) + row;
        const uint32_t n = fdiv(v, a.div_hv);
        const int y = static_cast<int>(v - n * a.div_hv.d) - a.pad;
        const int x = col + rs * js0 - a.pad;
        const bool ok = static_cast<unsigned>(y) < static_cast<unsigned>(a.H) &&
                        static_cast<unsigned>(x) < static_cast<unsigned>(a.W) &&
                        static_cast<int>(v) < a.vrows;
        // (unsigned: near 2 GiB of input, the bytes past the last pixel's row)
        const uint32_t off =
            4u * static_cast<uint32_t>(((static_cast<int>(n) * a.H + y) * a.W + x) * a.Cw +
                                       ch * CW + (tid & 1) * KS);
        load_words<KS>(xw[b], rin, ok ? off : kOutOfRange, 0u);
        dst[b] = static_cast<int>(row) * a.RS + col * PS + (tid & 1) * KS;
        row += a.step_row;  // kNT / 2 pixels on
        col += a.step_col;
        if (col >= a.cols) {
          col -= a.cols;
          ++row;
        }
      }
    };
    auto stage_store = [&](int base, int ch) {
#pragma unroll
      for (int b = 0; b < UB; ++b) {
        if (base + b * kNT >= halves) break;
        v8i x[KS];
        if constexpr (TAIL) {
          const int w0 = ch * CW + (tid & 1) * KS;
#pragma unroll
          for (int s = 0; s < KS; ++s) {
            const uint32_t vm = w0 + s < a.Cw - 1 ? ~0u : (w0 + s == a.Cw - 1 ? a.tmask_c : 0u);
            const v8i e = expand_fp4(xw[b][s] & vm, smask, 0u);
            const v8i f = expand_fp4(vm, smask, 0u);
#pragma unroll
            for (int r = 0; r < 4; ++r)
              x[s][r] = static_cast<int>(static_cast<uint32_t>(e[r]) |
                                         (static_cast<uint32_t>(f[r]) >> 2));
          }
        } else {
#pragma unroll
          for (int s = 0; s + 1 < KS; s += 2)
            expand_pair(xw[b][s], xw[b][s + 1], smask, vfill, x[s], x[s + 1]);
          if constexpr (KS & 1) x[KS - 1] = expand_fp4(xw[b][KS - 1], smask, vfill);
        }
        if (base + b * kNT + lane < halves) {
#pragma unroll
          for (int s = 0; s < KS; ++s) act[dst[b] + s] = v4i{x[s][0], x[s][1], x[s][2], x[s][3]};
        }
      }
    };
    // The order of the first loads: the input (needed first), the weights,
    // then what only the epilogue and the start values need.
    row = srow;
    col = scol;
    stage_load(wave * 64, 0);
#pragma unroll
    for (int d = 0; d < PD; ++d) load_w(wr[d], d, 0);
    // Thresholds and flip word (offsets past F or Fw read 0 and are masked).
#pragma unroll
    for (int tf = 0; tf < 2; ++tf)
      thv[tf] = static_cast<int32_t>(
          __builtin_amdgcn_raw_buffer_load_b32(rthr, (f0 + 32 * tf + c) * 4, 0, 0));
    fl = __builtin_amdgcn_raw_buffer_load_b32(rflip, wi * 4, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    v16f acc[2][PT];
    // Adds 0.5 - thr to every sum (thr clamped to [-K-1, K+1], which keeps
    // the comparison since |S| <= K), so that its sign is set exactly when S <
    // thr: one bf16 MFMA per tile, A a filter's value as three bf16 parts
    // (exact: half-integers below 2^23), B ones.  (Copies from LDS took 16 PT
    // vector instructions per filter tile.)
    auto add_thresholds = [&]() {
      const uint16_t ones[8] = {kBf16One, kBf16One, kBf16One, kBf16One,
                                kBf16One, kBf16One, kBf16One, kBf16One};
      v4i b = __builtin_bit_cast(v4i, bf16x8(ones));
#pragma unroll
      for (int tf = 0; tf < 2; ++tf) {
        const Split3 sp = split3(
            h == 0 ? 0.5f - static_cast<float>(min(max(thv[tf], -a.K - 1), a.K + 1)) : 0.0f);
        const uint16_t parts[8] = {bf16_bits(sp.p0), bf16_bits(sp.p1), bf16_bits(sp.p2), kBf16Zero,
                                   kBf16Zero, kBf16Zero, kBf16Zero, kBf16Zero};
#pragma unroll
        for (int pt = 0; pt < PT; ++pt) {
          asm volatile("" : "+v"(b));  // (else one product and 16 PT moves again)
          acc[tf][pt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              bf16x8(parts), __builtin_bit_cast(v8bf, b), acc[tf][pt], 0, 0, 0);
        }
      }
    };
    // This lane's window origins (unit pt of the run: 32 pixels per wave).
    int abase[PT];
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) {
      const Pix p = decode(a, min(p0 + (pt * wp + wpi) * 32 + c, a.items - 1));
      abase[pt] = (p.n * a.Hv + p.i - v0) * a.RS + p.j * PS + h * KS;
    }
    for (int ch = 0; ch < a.nchunk; ++ch) {
      if (ch > 0) __syncthreads();  // every wave is done with the last chunk
      if (ch > 0) {
        row = srow;
        col = scol;
        stage_load(wave * 64, ch);
      }
      for (int base = wave * 64; base < halves; base += UB * kNT) {
        if (base != wave * 64) stage_load(base, ch);
        stage_store(base, ch);
      }
      __syncthreads();
      if (ch == 0) {
#pragma unroll
        for (int tf = 0; tf < 2; ++tf)
#pragma unroll
          for (int pt = 0; pt < PT; ++pt) acc[tf][pt] = v16f{};
        if constexpr (!SUMS) add_thresholds();
      }

      // The taps, one k-step of 2 PT MFMAs at a time.  After each MFMA come a
      // few instructions for the next k-step: its weight words' expansion (up
      // to 4 vector instructions hide behind an MFMA; in one clump before the
      // MFMAs they do not), and, once both filter tiles have used a pixel
      // tile's operand, that tile's next one from LDS.  Weight words are
      // loaded PD taps ahead.  The scheduling barriers keep this in place.
      int toff = 0, tnext = 0, kw = 0;
      v4i B[PT];
      v4i A[2][2];  // [ring][filter tile]
      auto expand_op = [&](v4i (&x)[2], uint32_t w, int tf, int k) {
        if (k == 0)
          x[tf][0] = static_cast<int>(and_or(w << 3, smask, vfill));
        else if (k == 1)
          x[tf][1] = static_cast<int>(and_or(w << 2, smask, vfill));
        else if (k == 2)
          x[tf][2] = static_cast<int>(and_or(w << 1, smask, vfill));
        else
          x[tf][3] = static_cast<int>(and_or(w, smask, vfill));
      };
      auto tap = [&](int t, auto dc) {
        constexpr int d = decltype(dc)::value;
        tnext = toff + PS;
        if (++kw == a.KW) {
          kw = 0;
          tnext += a.RS - a.KW * PS;
        }
        if (t + 1 == taps) tnext = toff;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          const int ring = (d * KS + s) & 1;
          const int dn = s + 1 < KS ? d : (d + 1) % PD, sn = s + 1 < KS ? s + 1 : 0;
          // tap t's words are all expanded: load those PD taps on
          if (s == KS - 1) load_w(wr[d], t + PD, ch);
#pragma unroll
          for (int m = 0; m < 2 * PT; ++m) {
            const int pt = m / 2, tf = m % 2;
            const v4i x = A[ring][tf], b = B[pt];
            acc[tf][pt] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                v8i{x[0], x[1], x[2], x[3], 0, 0, 0, 0}, v8i{b[0], b[1], b[2], b[3], 0, 0, 0, 0},
                acc[tf][pt], 4, 4, 0, 127, 0, 127);
#pragma unroll
            for (int o = m * 8 / (2 * PT); o < (m + 1) * 8 / (2 * PT); ++o)
              expand_op(A[ring ^ 1], wr[dn][o / 4][sn], o / 4, o % 4);
            if (tf == 1) B[pt] = act[abase[pt] + (s + 1 < KS ? toff + s + 1 : tnext)];
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        toff = tnext;
      };
      static_assert((PD * KS) % 2 == 0, "the ring returns after PD taps");
#pragma unroll
      for (int pt = 0; pt < PT; ++pt) B[pt] = act[abase[pt]];
#pragma unroll
      for (int o = 0; o < 8; ++o) expand_op(A[0], wr[0][o / 4][0], o / 4, o % 4);
      int t = 0;
      for (; t + PD <= taps; t += PD) {
        tap(t, std::integral_constant<int, 0>{});
        tap(t + 1, std::integral_constant<int, 1>{});
        if constexpr (PD > 2) tap(t + 2, std::integral_constant<int, 2 % PD>{});
        if constexpr (PD > 3) tap(t + 3, std::integral_constant<int, 3 % PD>{});
      }
      if (t < taps) tap(t, std::integral_constant<int, 0>{});
      if constexpr (PD > 2)
        if (t + 1 < taps) tap(t + 1, std::integral_constant<int, 1>{});
      if constexpr (PD > 3)
        if (t + 2 < taps) tap(t + 2, std::integral_constant<int, 2 % PD>{});
      if (ch + 1 < a.nchunk) {
#pragma unroll
        for (int d = 0; d < PD; ++d) load_w(wr[d], d, ch + 1);
      }
    }

    if constexpr (SUMS) {
      // A wave's 64 x 32 sums go through LDS (all waves must be done with the
      // staged tile) so that a pixel's are stored as two contiguous runs (8
      // lanes x 16 bytes each), its position decoded once for both (a pass per
      // 32 filters: 50 x 50 x 160 -> 200 pooled at batch 7 13.8 us, 12.8 here; 56 x
      // 56 x 256 -> 256 at batch 64 73.1, 70.0).
      __syncthreads();
      constexpr int TS = kConvTileSumStride;
      int32_t* ts = reinterpret_cast<int32_t*>(act) + wave * (32 * TS);
      const int f = f0 + 4 * (lane & 7);
#pragma unroll
      for (int pt = 0; pt < PT; ++pt) {
#pragma unroll
        for (int tf = 0; tf < 2; ++tf)
#pragma unroll
          for (int g = 0; g < 4; ++g)
            *reinterpret_cast<int4*>(&ts[c * TS + 32 * tf + 8 * g + 4 * h]) =
                int4{static_cast<int>(acc[tf][pt][4 * g]), static_cast<int>(acc[tf][pt][4 * g + 1]),
                     static_cast<int>(acc[tf][pt][4 * g + 2]),
                     static_cast<int>(acc[tf][pt][4 * g + 3])};
#pragma unroll 2
        for (int r = 0; r < 4; ++r) {
          const int prow = 8 * r + (lane >> 3);
          const int item = p0 + (pt * wp + wpi) * 32 + prow;
          const Pix p = decode(a, min(item, a.items - 1));
          const int j = p.j + rs * js0;
          int32_t* dst = a.sums + (static_cast<size_t>(p.n * a.Ho + p.i) * a.Wo + j) * a.F + f;
          const int4 v[2] = {*reinterpret_cast<const int4*>(&ts[prow * TS + 4 * (lane & 7)]),
                             *reinterpret_cast<const int4*>(&ts[prow * TS + 32 + 4 * (lane & 7)])};
          if (item < a.items && p.i < a.Ho && j < a.Wo) {
#pragma unroll
            for (int tf = 0; tf < 2; ++tf) {
              const int ft = f + 32 * tf;
              if ((a.F & 3) == 0) {
                if (ft < a.F) *reinterpret_cast<int4*>(dst + 32 * tf) = v[tf];
              } else {
                if (ft < a.F) dst[32 * tf] = v[tf].x;
                if (ft + 1 < a.F) dst[32 * tf + 1] = v[tf].y;
                if (ft + 2 < a.F) dst[32 * tf + 2] = v[tf].z;
                if (ft + 3 < a.F) dst[32 * tf + 3] = v[tf].w;
              }
            }
          }
        }
      }
    }
    if (!SUMS || a.bits) {
      if constexpr (SUMS) add_thresholds();
      const uint32_t fm = wi == a.Fw - 1 ? tail_mask(a.F) : ~0u;
#pragma unroll
      for (int pt = 0; pt < PT; ++pt) {
        // one v_permlane32_swap of the two filter tiles' words leaves lane
        // half h with the whole word of tile h; output bit = sign xor ~flip
        const auto sw = __builtin_amdgcn_permlane32_swap(sign_word(acc[0][pt], h),
                                                         sign_word(acc[1][pt], h), false, false);
        uint32_t wd = ((sw[0] | sw[1]) ^ ~fl) & fm;
        if (a.pool) wd = or_quad(wd);
        const int item = p0 + (pt * wp + wpi) * 32 + c;
        const Pix p = decode(a, min(item, a.items - 1));
        const int jw = p.jw + js0;
        // (item grid rows and columns past Hp, Wp: odd edges of pooled sums, a
        // strip's columns past the image)
        if (item < a.items && wi < a.Fw && (!a.pool || (c & 3) == 0) && p.iw < a.Hp && jw < a.Wp)
          a.bits[(static_cast<size_t>(p.n * a.Hp + p.iw) * a.Wp + jw) * a.Fw + wi] = wd;
      }
    }
    u += PT;
    if (u < u_end) __syncthreads();  // (the next strip's first units: rare)
  };
  while (u < u_end) {
    const int left = static_cast<int>(a.div_t.d) -
                     (u - static_cast<int>(fdiv(static_cast<uint32_t>(u), a.div_t)) *
                              static_cast<int>(a.div_t.d));
    const int n = min(u_end - u, left);
    if (n >= 4)
      do_run(std::integral_constant<int, 4>{});
    else if (n == 3)
      do_run(std::integral_constant<int, 3>{});
    else if (n == 2)
      do_run(std::integral_constant<int, 2>{});
    else
      do_run(std::integral_constant<int, 1>{});
  }
}

template <int KS>
void launch_ks(const TileArgs& a, bool tail, unsigned grid, size_t lds, hipStream_t s) {
  if (a.sums && tail)
    bconv_tile_kernel<KS, true, true><<<grid, kNT, lds, s>>>(a);
  else if (a.sums)
    bconv_tile_kernel<KS, true, false><<<grid, kNT, lds, s>>>(a);
  else if (tail)
    bconv_tile_kernel<KS, false, true><<<grid, kNT, lds, s>>>(a);
  else
    bconv_tile_kernel<KS, false, false><<<grid, kNT, lds, s>>>(a);
}

}  // namespace

bool launch_bconv_tile(const ConvGeom& g, const uint32_t* in, const uint32_t* w,
                       const int32_t* thr, const uint32_t* flip, int32_t* sums, uint32_t* bits,
                       bool prepared, hipStream_t s, hipError_t* err) {
  // The options pick variants of the general kernel.
  const bnn_options& o = options();
  if (o.xcd_order != 1 || o.lds_weights != -1 || o.late_thresholds != -1) return false;
  ConvTilePlan p;
  if (!conv_tile_plan(g, sums != nullptr, bits != nullptr, prepared, &p)) return false;
  TileArgs a;
  a.in = in;
  a.w = w;
  a.thr = thr;
  a.flip = flip;
  a.sums = sums;
  a.bits = bits;
  a.H = p.H;
  a.W = p.W;
  a.Cw = g.Cw;
  a.F = g.F;
  a.Fw = g.Fw;
  a.KH = g.KH;
  a.KW = g.KW;
  a.pad = g.pad;
  a.Ho = p.Ho;
  a.Wo = p.Wo;
  a.Hw = p.Hw;
  a.pool = g.pool == 2;
  a.Hp = a.pool ? p.Ho / 2 : p.Ho;
  a.Wp = a.pool ? p.Wo / 2 : p.Wo;
  a.items = static_cast<int32_t>(p.items);
  a.Hv = p.H + 2 * g.pad;
  a.vrows = p.N * a.Hv;
  a.cols = p.cols;
  a.Ws = p.Ws;
  a.RS = p.RS;
  a.step_row = kNT / 2 / a.cols;
  a.step_col = kNT / 2 % a.cols;
  a.K = g.KH * g.KW * g.C;
  a.nchunk = p.nchunk;
  a.wfl = p.wfl;
  a.fstride = g.KH * g.KW * g.Cw;
  a.tmask_c = tail_mask(g.C);
  a.in_bytes = static_cast<int32_t>(static_cast<int64_t>(g.N) * g.H * g.W * g.Cw * 4);
  a.w_bytes = static_cast<int32_t>(static_cast<int64_t>(g.F) * a.fstride * 4);
  a.div_w = make_fastdiv31(static_cast<uint32_t>(p.Ws));
  a.div_t = make_fastdiv31(static_cast<uint32_t>(p.ups));
  a.div_h = make_fastdiv31(static_cast<uint32_t>(p.Hw));
  a.div_cols = make_fastdiv31(static_cast<uint32_t>(a.cols));
  a.div_hv = make_fastdiv31(static_cast<uint32_t>(a.Hv));
  a.div_f = make_fastdiv31(static_cast<uint32_t>(p.fgs));
  a.units = static_cast<int32_t>(p.units);
  const ConvTileRuns r = conv_tile_runs(p);
  a.nfull = static_cast<int32_t>(r.full);
  a.last = static_cast<int32_t>(r.last);
  a.xcd_units = static_cast<int32_t>(r.per_xcd);
  const unsigned grid =
      static_cast<unsigned>(8 * p.fgs * (r.full + (r.rest + r.last - 1) / r.last));
  const bool tail = g.C != 64 * p.ks * p.nchunk;
  switch (p.ks) {
    case 1: launch_ks<1>(a, tail, grid, p.lds, s); break;
    case 2: launch_ks<2>(a, tail, grid, p.lds, s); break;
    case 3: launch_ks<3>(a, tail, grid, p.lds, s); break;
    default: launch_ks<4>(a, tail, grid, p.lds, s); break;
  }
  *err = hipGetLastError();
  return true;
}

}  // namespace bnn
