"""The launch plans of csrc/tile_plans.hpp (host code, no HIP) as a small
shared library built with the host compiler: which kernel variant a shape
gets, without a GPU."""
import ctypes
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1808_00209_amd", "csrc")

SHIM = r"""
#include <chrono>
#include "tile_plans.hpp"
using namespace bnn;

static ConvGeom geom(const int32_t* v) {
  ConvGeom g = {v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[8]};
  g.Cw = (g.C + 31) / 32;
  g.Fw = (g.F + 31) / 32;
  g.Ho = g.H + 2 * g.pad - g.KH + 1;
  g.Wo = g.W + 2 * g.pad - g.KW + 1;
  g.Hp = g.pool ? g.Ho / 2 : g.Ho;
  g.Wp = g.pool ? g.Wo / 2 : g.Wo;
  return g;
}

static void fill(const ConvTilePlan& p, int64_t* o) {
  const int64_t v[] = {p.ok, p.ks, p.nchunk, p.wfl, p.Ws, p.strips, p.RS, p.cols, p.items,
                       p.ups, p.units, p.fgs, (int64_t)p.lds, p.H, p.W, p.N, p.Ho, p.Wo, p.Hw, p.Ww};
  for (unsigned i = 0; i < sizeof(v) / sizeof(v[0]); ++i) o[i] = v[i];
}

// The cheapest plan, whether or not the shape goes to the kernel.
extern "C" void conv_tile_cheapest(const int32_t* shape, int sums, int64_t* o) {
  fill(plan_conv_tile(geom(shape), sums != 0), o);
}

// 1 where the staged-tile kernel takes the shape.
extern "C" int conv_tile_takes(const int32_t* shape, int sums, int bits, int prep, int64_t* o) {
  ConvTilePlan p = {};
  const bool r = conv_tile_plan(geom(shape), sums != 0, bits != 0, prep != 0, &p);
  fill(p, o);
  return r;
}

extern "C" int fc_tile_takes(int64_t M, int64_t K, int64_t N, int sums, int bits, int64_t* o) {
  FcTilePlan p = {};
  const bool r = fc_tile_plan(M, N, K, sums != 0, bits != 0, &p);
  const int64_t v[] = {p.wfl, p.pt, p.output_tiles, p.row_tiles};
  for (int i = 0; i < 4; ++i) o[i] = v[i];
  return r;
}

extern "C" int conv1x1_groups_of(int64_t pixels, int F) {
  return conv1x1_groups((pixels + kConv1x1Pixels - 1) / kConv1x1Pixels, F);
}

// Least host time of a decision, in microseconds.
extern "C" double conv_tile_host_us(const int32_t* shape, int sums, int reps) {
  const ConvGeom g = geom(shape);
  double best = 1e30;
  for (int i = 0; i < reps; ++i) {
    const auto t0 = std::chrono::steady_clock::now();
    ConvTilePlan p = {};
    volatile bool r = conv_tile_plan(g, sums != 0, true, false, &p);
    (void)r;
    const auto t1 = std::chrono::steady_clock::now();
    best = std::min(best, std::chrono::duration<double, std::micro>(t1 - t0).count());
  }
  return best;
}
"""

FIELDS = ("ok ks nchunk wfl Ws strips RS cols items ups units fgs lds H W N Ho Wo Hw Ww").split()


@functools.lru_cache(maxsize=None)
def lib():
    with tempfile.TemporaryDirectory(prefix="tile_plans_") as d:
        src, so = os.path.join(d, "shim.cpp"), os.path.join(d, "shim.so")
        with open(src, "w") as f:
            f.write(SHIM)
        subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, src, "-o", so],
                       check=True)
        h = ctypes.CDLL(so)
    h.conv_tile_host_us.restype = ctypes.c_double
    return h


def _shape(N, H, W, C, F, KH, KW, pad, pool):
    return (ctypes.c_int32 * 9)(N, H, W, C, F, KH, KW, pad, pool)


def _dict(o):
    return dict(zip(FIELDS, o))


def cheapest(shape, sums):
    o = (ctypes.c_int64 * 20)()
    lib().conv_tile_cheapest(_shape(*shape), int(sums), o)
    return _dict(o)


def conv_tile(shape, sums, bits=True, prepared=False):
    """The plan with which the staged-tile kernel takes (N, H, W, C, F, KH, KW,
    pad, pool), or None where another kernel does."""
    o = (ctypes.c_int64 * 20)()
    takes = lib().conv_tile_takes(_shape(*shape), int(sums), int(bits), int(prepared), o)
    return _dict(o) if takes else None


def conv_tile_host_us(shape, sums, reps=50):
    return lib().conv_tile_host_us(_shape(*shape), int(sums), reps)


def fc_tile(M, K, N, sums, bits):
    """The plan with which the many-row FC kernel takes M x K -> N, or None."""
    o = (ctypes.c_int64 * 4)()
    i64 = ctypes.c_int64
    takes = lib().fc_tile_takes(i64(M), i64(K), i64(N), int(sums), int(bits), o)
    return dict(zip(("wfl", "pt", "output_tiles", "row_tiles"), o)) if takes else None


def conv1x1_groups(pixels, F):
    """Filter groups of the 1x1 kernel (C = 64, 128 or 256, at least 65536 pixels)."""
    return lib().conv1x1_groups_of(ctypes.c_int64(pixels), int(F))
