// Binary 1x1 conv with short windows (Eq. 4 with a single tap, K = C = 64,
// 128 or 256 bits) on the fp4 matrix cores, for large pixel counts.
//
// With K <= 256 a 32 x 32 output tile is only 1..4 MFMA k-steps deep, so in
// the general conv kernel a wave spends more on its pixel operands, its
// set-up and its epilogue than on the matrix cores.  Here a wave keeps the
// fp4 operands of its 64 pixels in registers, expanded once, and walks all
// filters in chunks of 64: per chunk it expands only the chunk's weights
// (prefetched one chunk ahead), runs 4 KS MFMAs and puts the chunk's two
// output words per pixel into the wave's LDS copy of its 64 output rows.  At
// the end the wave writes those rows out whole: consecutive lanes store
// consecutive 8-byte pieces of adjacent rows, where storing each word
// straight from its lane touched 64 rows per instruction, 4 bytes each (the
// stores then took about 40 % of the kernel).  Where whole rows per block
// would leave the last round of blocks nearly empty, a block takes a half or a
// quarter of the filters.  The block's thresholds (as 0.5 - thr, the
// accumulators' start value) and flip words are staged in LDS once.
#include <stdint.h>

#include "fastdiv.hpp"
#include "fp4_expand.hpp"
#include "kernels.hpp"
#include "tile_plans.hpp"

namespace bnn {
namespace {

constexpr int kPix = kConv1x1Pixels;  // pixels per block: 4 waves x 64
constexpr int kMaxF = 1024;  // LDS: output rows 34 KB + thresholds 4 KB at F = 1024

struct B1Args {
  const uint32_t* in;    // [M, Cw]
  const uint32_t* w;     // [F, Cw]
  const int32_t* thr;    // [F]
  const uint32_t* flip;  // [Fw] or null
  uint32_t* bits;        // [M, Fw]
  int32_t M, F, Fw, K;
  int32_t fpb;           // filters per block
  FastDiv31 div_g;       // filter groups
};

// KS consecutive words of a row: one 128-, 64- or 32-bit load.
template <int KS>
__device__ __forceinline__ void load_words(const uint32_t* p, uint32_t (&v)[KS]) {
  if constexpr (KS == 4) {
    const uint4 t = *reinterpret_cast<const uint4*>(p);
    v[0] = t.x;
    v[1] = t.y;
    v[2] = t.z;
    v[3] = t.w;
  } else if constexpr (KS == 2) {
    const uint2 t = *reinterpret_cast<const uint2*>(p);
    v[0] = t.x;
    v[1] = t.y;
  } else {
    v[0] = p[0];
  }
}

// KS = k-steps of 64 bits = Cw / 2.  Lane (h, c) feeds words h KS .. h KS +
// KS - 1 of its operand row, in both operands (the same permutation of the
// window's bit positions on both sides leaves every dot product unchanged):
// k-step s pairs word s of lane half 0 with word KS + s of lane half 1.
template <int KS>
__global__ __launch_bounds__(256) void bconv1x1_kernel(B1Args a) {
  constexpr int CW = 2 * KS;
  __shared__ float thl[kMaxF];
  __shared__ uint32_t nfl[kMaxF / 32];
  // The wave's output rows: 64 rows of fpb / 32 words at that stride + 2 (8-byte
  // aligned; an odd half-stride spreads a column over the banks).
  extern __shared__ uint32_t ostage[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = lane >> 5, c = lane & 31;
  // Block b runs on XCD b mod 8; the filter groups of a pixel block follow
  // each other on one XCD, whose L2 then holds its rows whole.
  const uint32_t k = blockIdx.x >> 3;
  const uint32_t pb = fdiv(k, a.div_g);
  const int fb = static_cast<int>(k - pb * a.div_g.d) * a.fpb;  // first filter
  const int p0 = static_cast<int>(8 * pb + (blockIdx.x & 7)) * kPix + wave * 64;
  const int ow = a.fpb / 32;  // words per row of this block
  const int os = ow + 2;
  uint32_t* orow = ostage + wave * 64 * os;

  // Pixel words and the first chunk's weight words, then the thresholds
  // (clamped to [-K-1, K+1], which keeps every comparison since |S| <= K).
  uint32_t xw[2][KS];
  bool pv[2];
#pragma unroll
  for (int tp = 0; tp < 2; ++tp) {
    const int p = p0 + 32 * tp + c;
    pv[tp] = p < a.M;
    load_words<KS>(a.in + static_cast<size_t>(pv[tp] ? p : a.M - 1) * CW + h * KS, xw[tp]);
  }
  // Row 8 g + 4 h' + r of a weight tile (g, r < 4) holds filter 16 h' + 4 g + r:
  // a lane half's 16 results are then 16 consecutive filters.
  const int wrow = 16 * ((c >> 2) & 1) + 4 * (c >> 3) + (c & 3);
  uint32_t wa[2][KS], wb[2][KS];
#pragma unroll
  for (int tf = 0; tf < 2; ++tf)
    load_words<KS>(a.w + static_cast<size_t>(fb + 32 * tf + wrow) * CW + h * KS, wa[tf]);
  for (int f = threadIdx.x; f < a.fpb; f += 256)
    thl[f] = 0.5f - static_cast<float>(min(max(a.thr[fb + f], -a.K - 1), a.K + 1));
  for (int i = threadIdx.x; i < ow; i += 256) nfl[i] = ~(a.flip ? a.flip[fb / 32 + i] : 0u);

  const uint32_t smask = __builtin_amdgcn_readfirstlane(0x88888888u);
  uint32_t vfill;
  asm("v_mov_b32 %0, 0x22222222" : "=v"(vfill));
  v8i B[2][KS];
#pragma unroll
  for (int tp = 0; tp < 2; ++tp) expand_words<KS>(xw[tp], smask, vfill, B[tp]);
  __syncthreads();

  // One chunk of 64 filters: expand its weights, prefetch the next chunk's,
  // MFMAs from 0.5 - thr, then the sign bits.  Register e of lane (h, c)
  // ends as S - thr + 0.5 of filter f0 + 32 tf + 16 h + e at pixel c of tile
  // tp; its sign bit is the complement of the output bit.  16 v_alignbit
  // collect them (with the filters in row order, nibble by nibble, it took 21
  // instructions), and one v_permlane32_swap of the two filter tiles' halves
  // leaves lane half h with both halves of tile h's word.
  const int nch = a.fpb / 64;
  auto chunk = [&](int ch, const uint32_t (&cw)[2][KS], uint32_t (&nw)[2][KS]) {
    const int f0 = 64 * ch;
    v8i A[2][KS];
#pragma unroll
    for (int tf = 0; tf < 2; ++tf) expand_words<KS>(cw[tf], smask, vfill, A[tf]);
    if (ch + 1 < nch) {
#pragma unroll
      for (int tf = 0; tf < 2; ++tf)
        load_words<KS>(a.w + static_cast<size_t>(fb + f0 + 64 + 32 * tf + wrow) * CW + h * KS,
                       nw[tf]);
    }
    v16f acc[2][2];
#pragma unroll
    for (int tf = 0; tf < 2; ++tf) {
      v16f t;
#pragma unroll
      for (int e = 0; e < 16; ++e) t[e] = thl[f0 + 32 * tf + 16 * h + e];
      acc[tf][0] = t;
      acc[tf][1] = t;
    }
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int tf = 0; tf < 2; ++tf)
#pragma unroll
        for (int tp = 0; tp < 2; ++tp)
          acc[tf][tp] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
              A[tf][s], B[tp][s], acc[tf][tp], 4, 4, 0, 127, 0, 127);
    const uint32_t fx = nfl[f0 / 32 + h];
#pragma unroll
    for (int tp = 0; tp < 2; ++tp) {
      uint32_t wd[2];
#pragma unroll
      for (int tf = 0; tf < 2; ++tf) {
        wd[tf] = 0u;
#pragma unroll
        for (int e = 0; e < 16; ++e)
          wd[tf] = __builtin_amdgcn_alignbit(wd[tf], __float_as_uint(acc[tf][tp][e]), 31);
      }
      const auto sw = __builtin_amdgcn_permlane32_swap(wd[0], wd[1], false, false);
      orow[(32 * tp + c) * os + f0 / 32 + h] = ((sw[0] << 16) | sw[1]) ^ fx;
    }
  };
  // Two chunks per trip, so the two weight register sets keep fixed names.
  for (int ch = 0; ch < nch; ch += 2) {
    chunk(ch, wa, wb);
    if (ch + 1 < nch) chunk(ch + 1, wb, wa);
  }
  __syncthreads();

  // Rows out: hw = fpb / 64 pieces of 8 bytes per row, rpi whole rows per
  // store instruction (lanes past rpi * hw idle), rows p0 .. p0 + 63 being
  // adjacent in memory.
  const int hw = ow / 2;
  const int rpi = 64 / hw;
  const int r0 = lane / hw, q = lane - r0 * hw;
  if (r0 < rpi) {
    for (int r = r0; r < 64; r += rpi) {
      if (p0 + r >= a.M) break;
      const uint2 v = *reinterpret_cast<const uint2*>(&orow[r * os + 2 * q]);
      *reinterpret_cast<uint2*>(&a.bits[static_cast<size_t>(p0 + r) * a.Fw + fb / 32 + 2 * q]) = v;
    }
  }
}

}  // namespace

bool bconv1x1_supported(const ConvGeom& g, bool sums) {
  const int64_t M = static_cast<int64_t>(g.N) * g.H * g.W;
  // C = 64, 128 or 256: 1, 2 or 4 k-steps, the instantiated variants (the
  // launcher maps Cw = 2 / 4 / 8 onto them and nothing else).
  return !sums && g.KH == 1 && g.KW == 1 && g.pad == 0 && g.pool == 0 &&
         (g.C == 64 || g.C == 128 || g.C == 256) && g.F % 64 == 0 && g.F <= kMaxF && M >= 256 * kPix &&
         M * g.Fw < (int64_t{1} << 31);
}

hipError_t launch_bconv1x1(const ConvGeom& g, const uint32_t* in, const uint32_t* w,
                           const int32_t* thr, const uint32_t* flip, uint32_t* bits,
                           hipStream_t s) {
  B1Args a;
  a.in = in;
  a.w = w;
  a.thr = thr;
  a.flip = flip;
  a.bits = bits;
  a.M = static_cast<int32_t>(static_cast<int64_t>(g.N) * g.H * g.W);
  a.F = g.F;
  a.Fw = g.Fw;
  a.K = g.C;
  const int64_t pb = (int64_t{a.M} + kPix - 1) / kPix;
  const int groups = conv1x1_groups(pb, g.F);
  a.fpb = g.F / groups;
  a.div_g = make_fastdiv31(static_cast<uint32_t>(groups));
  const unsigned blocks = static_cast<unsigned>((pb + 7) / 8 * 8 * groups);
  const size_t lds = static_cast<size_t>(4 * 64) * (a.fpb / 32 + 2) * sizeof(uint32_t);
  switch (g.Cw) {
    case 2: bconv1x1_kernel<1><<<blocks, 256, lds, s>>>(a); break;
    case 4: bconv1x1_kernel<2><<<blocks, 256, lds, s>>>(a); break;
    case 8: bconv1x1_kernel<4><<<blocks, 256, lds, s>>>(a); break;
    default: return hipErrorInvalidValue;  // not reachable: bconv1x1_supported
  }
  return hipGetLastError();
}

}  // namespace bnn
