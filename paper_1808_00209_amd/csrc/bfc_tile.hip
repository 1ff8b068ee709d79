// Binary FC layer / GEMM (Sec. III-B, Eq. 4) at many rows: S[m][n] = sum_k
// a[m][k] b[n][k] over +-1 values, with the threshold / flip epilogue of
// bnn_bgemm, on the fp4 matrix cores.
//
// The FC kernel (bfc_gemm.hip) gives each wave one 32 x 32 tile and expands
// both of its operands: 11 vector instructions at 4 cycles each and two LDS
// reads for every MFMA of 32 cycles.  Here a workgroup of 4 waves computes up
// to 256 outputs x 128 rows, a wave 64 outputs x 32 PT rows: per k-step two
// weight operands (expanded in registers from packed words) and PT data
// operands serve 2 PT MFMAs.  The data rows are staged in LDS, expanded once per
// workgroup, 256 bits of each at a time in two buffers: while one chunk's
// MFMAs run, the next one's words (loaded a chunk earlier) are expanded into
// the other, a few vector instructions after each MFMA (up to 4 hide behind
// it), and one barrier separates the chunks.  Two workgroups share a compute
// unit, so that one's MFMAs cover the other's barriers (one of 8 waves: 61
// against 57 us).  Words and bits past K are staged as fp4 0.0, so their
// products vanish whatever the weight words hold there.
// 4096 x 8192 -> 4096, bits: 133 us in the FC kernel, 50 us here (5.5e15
// operations a second; the matrix cores are busy 86 % of the waves' cycles,
// at a clock that drops to about 1.5 GHz).
#include <type_traits>

#include "fastdiv.hpp"
#include "fp32_split.hpp"
#include "fp4_expand.hpp"
#include "kernels.hpp"
#include "lane_ops.hpp"
#include "tile_plans.hpp"

namespace bnn {
namespace {

constexpr int kNT = 256;
constexpr int kKS = 4;             // k-steps (64 bits) per chunk
constexpr int kPS = 2 * kKS + 1;   // LDS entries per staged row (odd: no conflicts)
constexpr int kRows = kFcTileRows;  // data rows per block, at most (staged, used or not)
constexpr int kSumStride = 36;     // LDS words per row of a sums tile
constexpr int kRsrcWord3 = 0x00020000;

struct BtArgs {
  const uint32_t* A;      // [M][Kw]
  const uint32_t* B;      // [N][Kw]
  const int32_t* thr;     // [N] or null
  const uint32_t* flip;   // [Nw] or null
  int32_t* sums;          // [M][N] or null
  uint32_t* bits;         // [M][Nw] or null
  int32_t M, N, Nw, Kw, K;
  int32_t chunks;         // of 8 words
  uint32_t tmask;         // valid bits of word Kw - 1
  int32_t wfl;            // log2 of the waves along the outputs
  int32_t a_bytes, b_bytes;
  int32_t rt;             // row tiles
  FastDiv31 div_g, div_r; // tiles per group of 4 row tiles; rows of the last group
};

__device__ __forceinline__ v4i load4(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}

// PT: 32-row tiles per wave.  Lane half h feeds words 4 h .. 4 h + 3 of a
// chunk in both operands, one 16-byte load per row and half.
template <int PT, bool SUMS>
__global__ __launch_bounds__(kNT, 2) void bfc_tile_kernel(BtArgs a) {
  constexpr int kRing = PT == 4 ? 2 : 4;  // chunks of words in flight
  extern __shared__ v4i act[];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, c = lane & 31;
  // Block b runs on XCD b mod 8: an XCD takes consecutive tiles, ordered in
  // groups of 4 row tiles with the row varying fastest, so that its L2 serves
  // each row and each weight row to several blocks.
  const uint32_t t = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const uint32_t grp = fdiv(t, a.div_g);
  const uint32_t in = t - grp * a.div_g.d;
  const bool full = static_cast<int>(4 * grp + 4) <= a.rt;
  const uint32_t ft = full ? in >> 2 : fdiv(in, a.div_r);
  const uint32_t rt = 4 * grp + (full ? in & 3 : in - ft * a.div_r.d);
  const int wp = 4 >> a.wfl;
  const int wfi = wave & ((1 << a.wfl) - 1), wpi = wave >> a.wfl;
  const int f0 = (static_cast<int>(ft) << (6 + a.wfl)) + wfi * 64;  // wave's first output
  const int m00 = static_cast<int>(rt) * wp * PT * 32;              // block's first row
  constexpr int buf1 = kRows * kPS;  // second LDS buffer
  const int wi = f0 / 32 + h;  // this lane half's output word

  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint32_t*>(a.A), 0, a.a_bytes, kRsrcWord3);
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint32_t*>(a.B), 0, a.b_bytes, kRsrcWord3);
  const __amdgpu_buffer_rsrc_t rthr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int32_t*>(a.thr), 0, !SUMS || a.bits ? a.N * 4 : 0, kRsrcWord3);
  const __amdgpu_buffer_rsrc_t rflip = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint32_t*>(a.flip), 0, a.flip ? a.Nw * 4 : 0, kRsrcWord3);
  const uint32_t smask = __builtin_amdgcn_readfirstlane(0x88888888u);
  uint32_t vfill;
  asm("v_mov_b32 %0, 0x22222222" : "=v"(vfill));

  // Staging: thread t takes half t % 2 (4 words) of row t / 2 of every chunk
  // (rows past M repeat row M - 1; the buffers hold kRows rows, used or not,
  // so that no branch cuts the loop).
  const uint32_t aoff =
      (static_cast<uint32_t>(min(m00 + (tid >> 1), a.M - 1)) * a.Kw + 4 * (tid & 1)) * 4;
  const int sdst = (tid >> 1) * kPS + 4 * (tid & 1);
  const int whole = a.K >> 8;  // chunks of 256 valid bits
  // Word s of the thread's half of chunk ch, expanded into LDS.  MASK: the
  // chunk may hold words or bits past K (or lie past it altogether).
  auto stage_word = [&](const v4i& x, int ch, int s, int buf, auto mc) {
    const uint32_t w = static_cast<uint32_t>(x[s]);
    v4i e;
    if constexpr (!decltype(mc)::value) {
      e[0] = static_cast<int>(and_or(w << 3, smask, vfill));
      e[1] = static_cast<int>(and_or(w << 2, smask, vfill));
      e[2] = static_cast<int>(and_or(w << 1, smask, vfill));
      e[3] = static_cast<int>(and_or(w, smask, vfill));
    } else {
      const int wi0 = 8 * ch + 4 * (tid & 1) + s;
      const uint32_t vm = wi0 < a.Kw - 1 ? ~0u : (wi0 == a.Kw - 1 ? a.tmask : 0u);
      const v8i p = expand_fp4(w & vm, smask, 0u), q = expand_fp4(vm, smask, 0u);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        e[r] = static_cast<int>(static_cast<uint32_t>(p[r]) | (static_cast<uint32_t>(q[r]) >> 2));
    }
    act[buf + sdst + s] = e;
  };

  uint32_t woff[2];
#pragma unroll
  for (int tf = 0; tf < 2; ++tf)
    woff[tf] = (static_cast<uint32_t>(f0 + 32 * tf + c) * a.Kw + 4 * h) * 4;
  v4i xr[kRing], wr[kRing][2];  // words of the next kRing chunks, in flight
  auto load_x = [&](int r, int ch) { xr[r] = load4(ra, aoff, static_cast<uint32_t>(ch) * 32); };
  auto load_w = [&](int r, int ch) {
#pragma unroll
    for (int tf = 0; tf < 2; ++tf) wr[r][tf] = load4(rb, woff[tf], static_cast<uint32_t>(ch) * 32);
  };
  const int nch = a.chunks;
#pragma unroll
  for (int r = 0; r < kRing; ++r) {
    load_x(r, min(r, nch - 1));
    load_w(r, min(r, nch - 1));
  }
  int32_t thv[2];
#pragma unroll
  for (int tf = 0; tf < 2; ++tf)
    thv[tf] = static_cast<int32_t>(
        __builtin_amdgcn_raw_buffer_load_b32(rthr, (f0 + 32 * tf + c) * 4, 0, 0));
  const uint32_t fl = __builtin_amdgcn_raw_buffer_load_b32(rflip, wi * 4, 0, 0);

  int abase[PT];
#pragma unroll
  for (int pt = 0; pt < PT; ++pt) abase[pt] = ((wpi * PT + pt) * 32 + c) * kPS + 4 * h;
#pragma unroll
  for (int s = 0; s < kKS; ++s) stage_word(xr[0], 0, s, 0, std::true_type{});
  load_x(0, min(kRing, nch - 1));
  __syncthreads();

  v16f acc[2][PT];
  // Adds 0.5 - thr to every sum (thr clamped to [-K-1, K+1], which keeps the
  // comparison since |S| <= K): one bf16 MFMA per tile, A an output's value as
  // three bf16 parts (exact: half-integers below 2^23), B ones.
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
        asm volatile("" : "+v"(b));  // (else one product and 16 PT moves)
        acc[tf][pt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            bf16x8(parts), __builtin_bit_cast(v8bf, b), acc[tf][pt], 0, 0, 0);
      }
    }
  };
#pragma unroll
  for (int tf = 0; tf < 2; ++tf)
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) acc[tf][pt] = v16f{};
  if constexpr (!SUMS) add_thresholds();

  // Activation operands: with few row tiles a k-step is shorter than an LDS
  // read takes, so a whole chunk's are read at its start; with four, each is
  // read again as soon as both filter tiles have used it.
  constexpr int NB = PT == 4 ? 1 : kKS;
  v4i B[NB][PT], A[2][2];  // A: [ring][filter tile]
  auto expand_op = [&](v4i (&x)[2], int w, int tf, int k) {
    const uint32_t u = static_cast<uint32_t>(w);
    x[tf][k] = static_cast<int>(and_or(k == 3 ? u : u << (3 - k), smask, vfill));
  };
#pragma unroll
  for (int o = 0; o < 8; ++o) expand_op(A[0], wr[0][o / 4][0], o / 4, o % 4);

  // Chunk ch (ring slot r) from LDS buffer `buf`; stages chunk ch + 1 (its
  // words in the next slot) into `obuf`, loads the words of kRing chunks on.
  auto chunk = [&](int ch, auto rc, int buf, int obuf, auto mc) {
    constexpr int r = decltype(rc)::value;
    constexpr int r1 = (r + 1) % kRing;
#pragma unroll
    for (int s = 0; s < NB; ++s)
#pragma unroll
      for (int pt = 0; pt < PT; ++pt) B[s][pt] = act[buf + abase[pt] + s];
#pragma unroll
    for (int s = 0; s < kKS; ++s) {
      const int ring = s & 1;
      const int rn = s + 1 < kKS ? r : r1, sn = s + 1 < kKS ? s + 1 : 0;
      if (s == kKS - 1) load_w(r, min(ch + kRing, nch - 1));
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 0; m < 2 * PT; ++m) {
        const int pt = m / 2, tf = m % 2;
        const v4i x = A[ring][tf], b = B[s % NB][pt];
        acc[tf][pt] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
            v8i{x[0], x[1], x[2], x[3], 0, 0, 0, 0}, v8i{b[0], b[1], b[2], b[3], 0, 0, 0, 0},
            acc[tf][pt], 4, 4, 0, 127, 0, 127);
#pragma unroll
        for (int o = m * 8 / (2 * PT); o < (m + 1) * 8 / (2 * PT); ++o)
          expand_op(A[ring ^ 1], wr[rn][o / 4][sn], o / 4, o % 4);
        if (NB == 1 && tf == 1 && s + 1 < kKS) B[0][pt] = act[buf + abase[pt] + s + 1];
        __builtin_amdgcn_sched_barrier(0);
      }
      stage_word(xr[r1], ch + 1, s, obuf, mc);
    }
    load_x(r1, min(ch + 1 + kRing, nch - 1));
    __syncthreads();
  };
  // (kRing chunks per trip: LDS buffers and ring slots keep fixed names)
  auto trip = [&](int ch, auto mc) {
    constexpr bool mask = decltype(mc)::value;
    chunk(ch, std::integral_constant<int, 0>{}, 0, buf1, mc);
    if (mask && ch + 1 >= nch) return;
    chunk(ch + 1, std::integral_constant<int, 1>{}, buf1, 0, mc);
    if constexpr (kRing == 4) {
      if (mask && ch + 2 >= nch) return;
      chunk(ch + 2, std::integral_constant<int, 2 % kRing>{}, 0, buf1, mc);
      if (mask && ch + 3 >= nch) return;
      chunk(ch + 3, std::integral_constant<int, 3 % kRing>{}, buf1, 0, mc);
    }
  };
  int ch = 0;
  for (; ch + kRing < whole; ch += kRing) trip(ch, std::false_type{});
  for (; ch < nch; ch += kRing) trip(ch, std::true_type{});

  if constexpr (SUMS) {
    // A wave's 32 x 32 tile goes through LDS so that a row's 32 sums are
    // stored as one contiguous run (8 lanes x 16 bytes).
    int32_t* ts = reinterpret_cast<int32_t*>(act) + wave * (32 * kSumStride);
#pragma unroll
    for (int pt = 0; pt < PT; ++pt)
#pragma unroll
      for (int tf = 0; tf < 2; ++tf) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<int4*>(&ts[c * kSumStride + 8 * g + 4 * h]) =
              int4{static_cast<int>(acc[tf][pt][4 * g]), static_cast<int>(acc[tf][pt][4 * g + 1]),
                   static_cast<int>(acc[tf][pt][4 * g + 2]),
                   static_cast<int>(acc[tf][pt][4 * g + 3])};
        const int f = f0 + 32 * tf + 4 * (lane & 7);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = 8 * q + (lane >> 3);
          const int m = m00 + (wpi * PT + pt) * 32 + row;
          const int4 v = *reinterpret_cast<const int4*>(&ts[row * kSumStride + 4 * (lane & 7)]);
          if (m < a.M) {
            int32_t* dst = a.sums + static_cast<size_t>(m) * a.N + f;
            if ((a.N & 3) == 0) {
              if (f < a.N) *reinterpret_cast<int4*>(dst) = v;
            } else {
              if (f < a.N) dst[0] = v.x;
              if (f + 1 < a.N) dst[1] = v.y;
              if (f + 2 < a.N) dst[2] = v.z;
              if (f + 3 < a.N) dst[3] = v.w;
            }
          }
        }
      }
  }
  if (!SUMS || a.bits) {
    if constexpr (SUMS) add_thresholds();
    const uint32_t fm = wi == a.Nw - 1 ? tail_mask(a.N) : ~0u;
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) {
      // one v_permlane32_swap of the two output tiles' words leaves lane half
      // h with the whole word of tile h; output bit = sign xor ~flip
      const auto sw = __builtin_amdgcn_permlane32_swap(sign_word(acc[0][pt], h),
                                                       sign_word(acc[1][pt], h), false, false);
      const int m = m00 + (wpi * PT + pt) * 32 + c;
      if (m < a.M && wi < a.Nw)
        a.bits[static_cast<size_t>(m) * a.Nw + wi] = ((sw[0] | sw[1]) ^ ~fl) & fm;
    }
  }
}

template <int PT>
void launch_pt(const BtArgs& a, unsigned grid, size_t lds, hipStream_t s) {
  if (a.sums)
    bfc_tile_kernel<PT, true><<<grid, kNT, lds, s>>>(a);
  else
    bfc_tile_kernel<PT, false><<<grid, kNT, lds, s>>>(a);
}

}  // namespace

bool launch_bfc_tile(int64_t M, int64_t N, int64_t K, const uint32_t* A, const uint32_t* B,
                     const int32_t* thr, const uint32_t* flip, int32_t* sums, uint32_t* bits,
                     hipStream_t s, hipError_t* err) {
  FcTilePlan p;
  if (!fc_tile_plan(M, N, K, sums != nullptr, bits != nullptr, &p)) return false;
  const int64_t Kw = (K + 31) / 32;
  BtArgs a;
  a.A = A;
  a.B = B;
  a.thr = thr;
  a.flip = flip;
  a.sums = sums;
  a.bits = bits;
  a.M = static_cast<int32_t>(M);
  a.N = static_cast<int32_t>(N);
  a.Nw = static_cast<int32_t>((N + 31) / 32);
  a.Kw = static_cast<int32_t>(Kw);
  a.K = static_cast<int32_t>(K);
  a.chunks = static_cast<int32_t>((Kw + 7) / 8);
  a.tmask = tail_mask(K);
  a.wfl = p.wfl;
  a.a_bytes = static_cast<int32_t>(M * Kw * 4);
  a.b_bytes = static_cast<int32_t>(N * Kw * 4);
  a.rt = static_cast<int32_t>(p.row_tiles);
  a.div_g = make_fastdiv31(static_cast<uint32_t>(4 * p.output_tiles));
  a.div_r = make_fastdiv31(static_cast<uint32_t>(p.row_tiles % 4 ? p.row_tiles % 4 : 4));
  const unsigned grid = static_cast<unsigned>((p.output_tiles * p.row_tiles + 7) / 8 * 8);
  constexpr size_t lds = size_t{2} * kRows * kPS * 16;
  static_assert(lds >= 4 * 32 * kSumStride * 4, "the sums tiles fit");
  switch (p.pt) {
    case 4: launch_pt<4>(a, grid, lds, s); break;
    case 2: launch_pt<2>(a, grid, lds, s); break;
    default: launch_pt<1>(a, grid, lds, s); break;
  }
  *err = hipGetLastError();
  return true;
}

}  // namespace bnn
