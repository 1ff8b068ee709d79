"""The staged-tile conv kernel where it can go wrong.  TAKEN holds shapes that
its rule takes, with the k-steps per tap, channel chunks and log2 of the waves
along the filters that the plan gives them (asserted, so that a change of the
rule cannot empty the test): every k-step count with and without a channel tail
and with and without sums, one and several chunks, filter counts around a
wave's 64 and not a multiple of 4, square and other windows, odd pooled sizes,
runs that span images and strips, whole rounds and short runs, LDS tiles above
64 KB.  CASES are shapes on both sides of the rule.  The reference is the
vector-ALU kernel, itself checked against the oracle, on the same packed
inputs (tail bits garbled); every word and sum is compared."""
import pytest
import torch

import tile_plans
from paper_1808_00209_amd import bnn

pytestmark = pytest.mark.gpu

TAKEN = [
    # (N, H, W, C, F, KH, KW, pad, pool), sums, bits, k-steps, chunks, log2 waves
    ((7, 45, 61, 160, 200, 3, 3, 1, 2), 1, 1, 3, 1, 2),
    ((64, 17, 17, 200, 128, 3, 3, 1, 0), 0, 1, 4, 1, 1),
    ((120, 24, 24, 128, 256, 3, 3, 1, 0), 0, 1, 2, 1, 2),
    ((64, 56, 56, 256, 256, 3, 3, 1, 2), 1, 1, 4, 1, 2),
    ((19, 57, 56, 33, 33, 5, 2, 0, 2), 1, 0, 1, 1, 0),
    ((24, 60, 5, 33, 130, 3, 3, 2, 2), 1, 0, 1, 1, 0),
    ((26, 38, 38, 32, 33, 5, 2, 2, 2), 1, 1, 1, 1, 0),
    ((31, 44, 53, 33, 33, 5, 2, 2, 2), 1, 0, 1, 1, 0),
    ((40, 16, 46, 32, 33, 3, 3, 2, 2), 1, 0, 1, 1, 0),
    ((40, 48, 24, 33, 33, 1, 3, 2, 2), 1, 0, 1, 1, 0),
    ((42, 41, 58, 32, 33, 1, 3, 2, 2), 0, 1, 1, 1, 0),
    ((44, 3, 1441, 33, 40, 3, 4, 2, 2), 1, 0, 1, 1, 0),
    ((44, 5, 43, 32, 130, 1, 3, 1, 2), 1, 0, 1, 1, 0),
    ((47, 40, 65, 32, 33, 5, 2, 2, 2), 0, 1, 1, 1, 0),
    ((50, 16, 54, 33, 33, 3, 3, 2, 2), 0, 1, 1, 1, 0),
    ((51, 54, 40, 32, 40, 5, 2, 2, 2), 0, 1, 1, 1, 0),
    ((58, 53, 70, 33, 33, 1, 1, 0, 0), 0, 1, 1, 1, 0),
    ((60, 3, 69, 50, 40, 1, 3, 2, 2), 1, 1, 1, 1, 0),
    ((62, 15, 39, 33, 33, 5, 5, 2, 2), 1, 1, 1, 1, 0),
    ((64, 21, 43, 33, 33, 3, 3, 1, 2), 0, 1, 1, 1, 0),
    ((82, 34, 14, 33, 33, 3, 3, 2, 2), 1, 1, 1, 1, 0),
    ((87, 10, 40, 32, 33, 5, 5, 2, 0), 1, 0, 1, 1, 0),
    ((91, 22, 3, 32, 150, 3, 3, 2, 2), 1, 1, 1, 1, 0),
    ((91, 58, 13, 33, 33, 5, 2, 2, 2), 1, 1, 1, 1, 0),
    ((93, 34, 29, 32, 33, 1, 3, 2, 2), 0, 1, 1, 1, 0),
    ((101, 3, 77, 33, 33, 3, 3, 2, 2), 1, 0, 1, 1, 0),
    ((104, 38, 14, 32, 33, 5, 2, 2, 0), 1, 1, 1, 1, 0),
    ((107, 9, 6, 32, 130, 1, 3, 2, 2), 1, 1, 1, 1, 0),
    ((109, 53, 7, 32, 33, 5, 2, 2, 2), 1, 0, 1, 1, 0),
    ((111, 38, 20, 32, 33, 5, 2, 1, 2), 1, 0, 1, 1, 0),
    ((112, 3, 78, 33, 40, 5, 2, 2, 2), 1, 1, 1, 1, 0),
    ((117, 22, 9, 33, 40, 1, 3, 2, 2), 1, 1, 1, 1, 0),
    ((11, 5, 390, 33, 70, 3, 4, 2, 0), 1, 1, 1, 1, 1),
    ((29, 31, 78, 32, 70, 5, 2, 2, 2), 0, 1, 1, 1, 1),
    ((51, 49, 5, 32, 70, 3, 3, 2, 2), 1, 1, 1, 1, 1),
    ((76, 39, 4, 32, 70, 3, 3, 2, 2), 1, 0, 1, 1, 1),
    ((85, 4, 29, 32, 70, 1, 3, 2, 2), 1, 0, 1, 1, 1),
    ((86, 23, 10, 33, 65, 1, 3, 2, 2), 1, 0, 1, 1, 1),
    ((113, 39, 17, 32, 65, 5, 2, 0, 2), 0, 1, 1, 1, 1),
    ((119, 4, 38, 33, 65, 3, 1, 2, 2), 1, 1, 1, 1, 1),
    ((34, 39, 55, 64, 256, 2, 5, 0, 0), 0, 1, 1, 1, 2),
    ((45, 30, 55, 33, 200, 3, 3, 0, 2), 0, 1, 1, 1, 2),
    ((94, 10, 61, 64, 256, 3, 3, 2, 0), 1, 0, 1, 1, 2),
    ((105, 5, 13, 300, 300, 5, 2, 2, 2), 1, 1, 1, 5, 0),
    ((90, 55, 5, 70, 65, 3, 1, 2, 2), 0, 1, 2, 1, 1),
    ((93, 4, 54, 70, 65, 1, 3, 2, 2), 0, 1, 2, 1, 1),
    ((94, 8, 30, 70, 65, 3, 1, 2, 2), 0, 1, 2, 1, 1),
    ((110, 33, 38, 70, 70, 1, 1, 0, 0), 1, 1, 2, 1, 1),
    ((98, 21, 12, 128, 512, 2, 3, 2, 0), 0, 1, 2, 1, 2),
    ((102, 3, 70, 128, 512, 2, 3, 2, 0), 1, 1, 2, 1, 2),
    ((75, 48, 61, 224, 33, 3, 1, 0, 2), 0, 1, 2, 2, 0),
    ((72, 59, 5, 500, 33, 5, 2, 2, 2), 1, 1, 2, 4, 0),
    ((44, 3, 52, 700, 150, 3, 3, 2, 2), 1, 1, 2, 6, 0),
    ((87, 15, 34, 700, 33, 3, 3, 2, 2), 0, 1, 2, 6, 0),
    ((46, 7, 64, 192, 512, 1, 3, 2, 0), 0, 1, 3, 1, 2),
    ((59, 13, 73, 192, 256, 1, 3, 2, 0), 1, 1, 3, 1, 2),
    ((87, 8, 25, 300, 256, 1, 4, 1, 2), 1, 1, 3, 2, 2),
    ((37, 5, 1455, 500, 33, 1, 3, 2, 2), 0, 1, 3, 3, 0),
    ((83, 11, 49, 700, 33, 3, 1, 2, 0), 0, 1, 3, 4, 0),
    ((83, 20, 48, 200, 96, 2, 3, 0, 2), 0, 1, 4, 1, 1),
    ((47, 3, 457, 256, 256, 3, 1, 2, 0), 0, 1, 4, 1, 2),
    ((56, 11, 78, 256, 256, 1, 4, 2, 0), 1, 0, 4, 1, 2),
    ((56, 3, 19, 700, 512, 2, 5, 2, 2), 1, 0, 4, 3, 2),
]

CASES = [
    # N, H, W, C, F, k, pad, pool
    (3, 40, 40, 32, 96, 3, 1, 0),      # one word per tap, 2-word chunk
    (2, 64, 64, 33, 64, 3, 1, 2),      # a masked second word
    (7, 45, 61, 160, 200, 3, 1, 2),    # 5 words as 3 k-steps, odd sizes
    (9, 23, 29, 100, 130, 3, 0, 0),    # no padding, 4 words, partial waves
    (40, 7, 7, 96, 512, 3, 1, 0),      # runs span several 7x7 images
    (30, 7, 9, 224, 65, 3, 1, 2),      # odd maps pooled, 4 k-steps with a tail
    (5, 31, 33, 300, 70, 3, 1, 0),     # two channel chunks
    (2, 30, 50, 70, 40, 5, 2, 2),      # 5x5, one filter wave
    (64, 17, 17, 200, 128, 1, 0, 0),   # 1x1: pixels as rows of one column
    (64, 17, 17, 200, 128, 1, 0, 2),   # 1x1 pooled
    (1, 3, 1400, 96, 64, 3, 1, 0),     # a wide map: many strips
    (120, 24, 24, 128, 256, 3, 1, 0),  # whole chunks, full rounds and a short one
    (130, 23, 25, 128, 256, 3, 1, 2),  # the same, odd sizes pooled
    (64, 28, 28, 256, 256, 3, 1, 2),   # 4 k-steps per tap
    (56, 32, 40, 192, 128, 3, 1, 0),   # 3 k-steps per tap, two pixel waves
]


def _words(g, *shape):
    return torch.randint(-2 ** 31, 2 ** 31, shape, generator=g, device="cuda",
                         dtype=torch.int64).to(torch.int32)


def _thresholds(g, F, K):
    r = 2 * int(K ** 0.5)
    thr = torch.randint(-r, r + 1, (F,), generator=g, device="cuda").to(torch.int32)
    thr[0], thr[-1] = 2 ** 31 - 1, -2 ** 31
    return thr


@pytest.mark.parametrize("case", TAKEN, ids=[str(c[:3]) for c in TAKEN])
def test_taken_shapes_match_the_vector_kernel(case):
    shape, sums, bits, ks, nchunk, wfl = case
    plan = tile_plans.conv_tile(shape, sums, bits)
    assert plan is not None and (plan["ks"], plan["nchunk"], plan["wfl"]) == (ks, nchunk, wfl)
    N, H, W, C, F, KH, KW, pad, pool = shape
    g = torch.Generator(device="cuda").manual_seed(sum(shape))
    x, w = _words(g, N, H, W, bnn.words(C)), _words(g, F, KH, KW, bnn.words(C))
    thr, flip = _thresholds(g, F, KH * KW * C), _words(g, bnn.words(F))
    desc = bnn.conv_desc(N, H, W, C, F, KH, KW, 1, pad, pool)
    want = dict(want_sums=bool(sums), want_bits=bool(bits))
    got = bnn.bnn_bconv2d(desc, x, w, thr, flip, **want)
    with bnn.options(algo=bnn.ALGO_VALU):
        ref = bnn.bnn_bconv2d(desc, x, w, thr, flip, **want)
    for a, b in zip(got, ref):
        assert (a is None) == (b is None)
        if a is not None:
            assert torch.equal(a, b)


@pytest.mark.parametrize("case", CASES, ids=[str(c) for c in CASES])
@pytest.mark.parametrize("sums,bits", [(False, True), (True, True), (True, False)])
def test_tile_conv_matches_the_vector_kernel(case, sums, bits):
    N, H, W, C, F, k, pad, pool = case
    g = torch.Generator(device="cuda").manual_seed(hash(case) % 2 ** 31)
    x = _words(g, N, H, W, bnn.words(C))
    w = _words(g, F, k, k, bnn.words(C))
    r = 2 * int((k * k * C) ** 0.5)
    thr = torch.randint(-r, r + 1, (F,), generator=g, device="cuda").to(torch.int32)
    thr[0], thr[-1] = 2 ** 31 - 1, -2 ** 31
    flip = _words(g, bnn.words(F))
    desc = bnn.conv_desc(N, H, W, C, F, k, k, 1, pad, pool)
    got = bnn.bnn_bconv2d(desc, x, w, thr, flip, want_sums=sums, want_bits=bits)
    with bnn.options(algo=bnn.ALGO_VALU):
        ref = bnn.bnn_bconv2d(desc, x, w, thr, flip, want_sums=sums, want_bits=bits)
    for a, b in zip(got, ref):
        assert (a is None) == (b is None)
        if a is not None:
            assert torch.equal(a, b)
    if bits and not sums:  # no flips
        got = bnn.bnn_bconv2d(desc, x, w, thr, None, want_sums=False)
        with bnn.options(algo=bnn.ALGO_VALU):
            ref = bnn.bnn_bconv2d(desc, x, w, thr, None, want_sums=False)
        assert torch.equal(got[1], ref[1])


def test_input_of_almost_2_gib():
    """Byte offsets up to 2^31: the last image's rows and the tail words past
    them (96 channels, 12 bytes per pixel).  Only the ends are compared: the
    reference runs on the first and last images alone."""
    N, H, W, C, F = 43690, 64, 64, 96, 33
    assert 2 ** 31 - 2 ** 17 < N * H * W * 12 < 2 ** 31
    assert tile_plans.conv_tile((N, H, W, C, F, 3, 3, 1, 0), False)
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.empty(N, H, W, 3, dtype=torch.int32, device="cuda")
    for n in range(0, N, 4370):
        x[n:n + 4370] = _words(g, *x[n:n + 4370].shape)
    w, thr, flip = _words(g, F, 3, 3, 3), _thresholds(g, F, 9 * C), _words(g, 2)
    got = bnn.bnn_bconv2d(bnn.conv_desc(N, H, W, C, F, 3, 3, 1, 1, 0), x, w, thr, flip,
                          want_sums=False)[1]
    with bnn.options(algo=bnn.ALGO_VALU):
        for part in (slice(0, 4), slice(N - 4, N)):
            ref = bnn.bnn_bconv2d(bnn.conv_desc(4, H, W, C, F, 3, 3, 1, 1, 0),
                                  x[part].contiguous(), w, thr, flip, want_sums=False)[1]
            assert torch.equal(got[part], ref)
