// Sign-to-bits packing (Eq. 1 and Eq. 2 of the paper with B = 32; input
// thresholding sign(X + T) of Sec. II-C).  Value i of a group of 32 goes to
// bit 31 - i, bit = ((x + offset) > 0) computed in fp32, tail bits 0.
//
// HBM-bound: 4 bytes read per value, 1/8 byte written.  Two mappings:
//  * D >= 32: 8 lanes per output word, 4 consecutive values each (one 16-byte
//    load), 8 words in flight per lane group.
//  * D < 32 (one word per row, e.g. RGB input with D = 3): one lane per row,
//    reading its D values; consecutive lanes read consecutive rows.
#include "fastdiv.hpp"
#include "kernels.hpp"

namespace bnn {
namespace {

constexpr int kBlock = 256;
constexpr int kDepth = 8;                 // words per 8-lane group
constexpr int kWaveWords = 8 * kDepth;    // consecutive words a wave packs

// Four consecutive floats at 4-byte alignment: rows of any D start anywhere,
// and a 16-byte load needs only dword alignment on this target.
struct __attribute__((packed, aligned(4))) F4 {
  float v[4];
};

// OR over the 8 lanes 8k .. 8k + 7: DPP quad permutes (lane ^ 1, lane ^ 2),
// then row_half_mirror (lane 7 - i of the same 8).
__device__ __forceinline__ uint32_t or8(uint32_t x) {
  x |= static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0xB1, 0xF, 0xF, false));
  x |= static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x4E, 0xF, 0xF, false));
  x |= static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x141, 0xF, 0xF, false));
  return x;
}

// A wave packs kWaveWords consecutive words of the flat [rows][Dw] output:
// lane group g = lane / 8 takes words 8 i + g (i < kDepth), each of its lanes
// 4 of the word's 32 values, and after the OR over the group lane 8 g + i
// keeps word 8 i + g, so the wave's stores cover kWaveWords contiguous words.
// Bound by HBM reads; with one 4-byte load per lane and one word per 32 lanes
// (the form before) too few bytes were in flight: 51.4 M values with an
// offset took 83-104 us (2.0-2.5 TB/s), 36.6 us here (5.8 TB/s).
// OFF: whether there is an offset.
template <bool OFF>
__global__ __launch_bounds__(kBlock) void pack_words_kernel(
    const float* __restrict__ x, const float* __restrict__ offset,
    uint32_t total_words, uint32_t D, FastDiv div_dw, uint32_t* __restrict__ out) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t w0 = (blockIdx.x * (kBlock / 64) + threadIdx.x / 64) * kWaveWords;
  const uint32_t g = lane >> 3, q = 4 * (lane & 7);
  // Values past D of a short last word: the load moves back to the row's
  // last four values, and the bits move up by as much, so no load sits
  // behind a branch.
  F4 v[kDepth], o[OFF ? kDepth : 1];
  uint32_t up[kDepth];
#pragma unroll
  for (int i = 0; i < kDepth; ++i) {
    const uint32_t word = min(w0 + 8 * i + g, total_words - 1);
    const uint32_t r = fdiv(word, div_dw);
    const uint32_t d = (word - r * div_dw.d) * 32 + q;
    const uint32_t dl = min(d, D - 4);
    up[i] = min(d - dl, 4u);
    v[i] = *reinterpret_cast<const F4*>(x + static_cast<uint64_t>(r) * D + dl);
    if constexpr (OFF) o[i] = *reinterpret_cast<const F4*>(offset + dl);
  }
  uint32_t mine = 0;
#pragma unroll
  for (int i = 0; i < kDepth; ++i) {
    uint32_t nib = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float t = OFF ? v[i].v[e] + o[i].v[e] : v[i].v[e];
      nib |= static_cast<uint32_t>(t > 0.0f) << (3 - e);
    }
    nib = (nib << up[i]) & 15u;
    const uint32_t word = or8(nib << (28 - q));
    if ((lane & 7) == static_cast<uint32_t>(i)) mine = word;
  }
  const uint32_t word = w0 + 8 * (lane & 7) + g;
  if (word < total_words) out[word] = mine;
}

__global__ __launch_bounds__(kBlock) void pack_rows_kernel(
    const float* __restrict__ x, const float* __restrict__ offset,
    uint64_t rows, uint32_t D, uint32_t* __restrict__ out) {
  const uint64_t r = static_cast<uint64_t>(blockIdx.x) * kBlock + threadIdx.x;
  if (r >= rows) return;
  const float* xr = x + r * D;
  uint32_t v = 0;
  for (uint32_t d = 0; d < D; ++d) {
    float t = xr[d];
    if (offset) t = t + offset[d];
    v |= static_cast<uint32_t>(t > 0.0f) << (31 - d);
  }
  out[r] = v;
}

}  // namespace

hipError_t launch_pack_bits(const float* x, const float* offset, int64_t rows,
                            int64_t D, uint32_t* out, hipStream_t s) {
  if (D < 32) {
    const uint64_t blocks = (static_cast<uint64_t>(rows) + kBlock - 1) / kBlock;
    pack_rows_kernel<<<dim3(static_cast<uint32_t>(blocks)), dim3(kBlock), 0, s>>>(
        x, offset, static_cast<uint64_t>(rows), static_cast<uint32_t>(D), out);
  } else {
    const int64_t Dw = words_of(D);
    const int64_t words = rows * Dw;
    const int64_t per_block = (kBlock / 64) * kWaveWords;
    const dim3 grid(static_cast<uint32_t>((words + per_block - 1) / per_block));
    if (offset)
      pack_words_kernel<true><<<grid, dim3(kBlock), 0, s>>>(
          x, offset, static_cast<uint32_t>(words), static_cast<uint32_t>(D),
          make_fastdiv(static_cast<uint32_t>(Dw)), out);
    else
      pack_words_kernel<false><<<grid, dim3(kBlock), 0, s>>>(
          x, nullptr, static_cast<uint32_t>(words), static_cast<uint32_t>(D),
          make_fastdiv(static_cast<uint32_t>(Dw)), out);
  }
  return hipGetLastError();
}

}  // namespace bnn
