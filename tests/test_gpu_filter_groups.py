"""Layers whose filters are split over blocks or groups, where the split can go
wrong: the real-valued first layer with an odd number of 64-filter groups (two
to a block on large grids), ragged filter counts beside its contiguous sum
stores, and 1x1 layers whose blocks take a half or a quarter of the filters.
The reference is the vector-ALU kernel, itself checked against the oracle; the
first layer's inputs lie on a 2^-8 grid, so its fp32 sums are exact in any
order and every sum and word must agree."""
import pytest
import torch

import tile_plans
from paper_1808_00209_amd import bnn

pytestmark = pytest.mark.gpu

FCONV = [
    # N, H, W, C, F, pool
    (32, 64, 64, 3, 192, 0), (32, 64, 64, 1, 320, 2), (32, 62, 63, 3, 160, 2),
    (32, 64, 64, 3, 128, 0), (3, 23, 45, 3, 70, 0), (2, 17, 33, 1, 36, 2), (1, 9, 31, 3, 192, 2),
]
CONV1 = [
    # N, H, W, C, F, filter groups: at least 65536 pixels, in blocks of 256.
    # 259 blocks, the last one a single pixel
    (1, 257, 257, 256, 1024, 4), (1, 257, 257, 128, 1024, 4), (1, 257, 257, 64, 512, 2),
    # 529, 527 and 519 blocks, partial last ones
    (2, 261, 259, 64, 1024, 4), (1, 311, 433, 256, 768, 2), (1, 401, 331, 128, 512, 2),
    # whole last blocks; all filters per block
    (3, 256, 257, 256, 512, 2), (1, 256, 256, 64, 1024, 1), (1, 257, 257, 256, 192, 1),
    # a pixel fewer than the kernel's smallest grid: another kernel
    (1, 257, 255, 256, 1024, 0),
]


def _words(g, *shape):
    return torch.randint(-2 ** 31, 2 ** 31, shape, generator=g, device="cuda",
                         dtype=torch.int64).to(torch.int32)


def _same(call):
    got = call()
    with bnn.options(algo=bnn.ALGO_VALU):
        ref = call()
    for a, b in zip(got, ref):
        assert (a is None) == (b is None)
        if a is not None:
            assert torch.equal(a, b)


@pytest.mark.parametrize("case", FCONV, ids=[str(c) for c in FCONV])
@pytest.mark.parametrize("sums,bits", [(False, True), (True, True), (True, False)])
def test_first_layer_filter_groups(case, sums, bits):
    N, H, W, C, F, pool = case
    g = torch.Generator(device="cuda").manual_seed(H * W + F)
    x = torch.randint(-1024, 1025, (N, H, W, C), generator=g, device="cuda").float() / 256
    w = _words(g, F, 3, 3, bnn.words(C))
    thr = torch.randint(-12, 13, (F,), generator=g, device="cuda").to(torch.int32)
    flip = _words(g, bnn.words(F))
    desc = bnn.conv_desc(N, H, W, C, F, 3, 3, 1, 1, pool)
    _same(lambda: bnn.bnn_fconv2d_binw(desc, x, w, thr, flip, want_sums=sums, want_bits=bits))


@pytest.mark.parametrize("case", CONV1, ids=[str(c) for c in CONV1])
def test_1x1_filter_groups(case):
    N, H, W, C, F, groups = case
    if groups:
        assert N * H * W >= 65536 and tile_plans.conv1x1_groups(N * H * W, F) == groups
    g = torch.Generator(device="cuda").manual_seed(H * W + C + F)
    x, w = _words(g, N, H, W, bnn.words(C)), _words(g, F, 1, 1, bnn.words(C))
    thr = torch.randint(-20, 21, (F,), generator=g, device="cuda").to(torch.int32)
    thr[0], thr[-1] = 2 ** 31 - 1, -2 ** 31
    flip = _words(g, bnn.words(F))
    desc = bnn.conv_desc(N, H, W, C, F, 1, 1, 1, 0, 0)
    _same(lambda: bnn.bnn_bconv2d(desc, x, w, thr, flip, want_sums=False))


@pytest.mark.parametrize("case", [(2, 24, 40, 3, 64, 0), (2, 24, 40, 1, 70, 2),
                                  (32, 64, 64, 3, 128, 0)], ids=str)
@pytest.mark.parametrize("sums", [False, True])
def test_first_layer_nan_sums_give_bit_0_before_flip(case, sums):
    """S >= thr is false for a NaN sum whatever its sign bit: windows that hold
    a NaN give the same bits as the vector-ALU kernel's comparison."""
    N, H, W, C, F, pool = case
    g = torch.Generator(device="cuda").manual_seed(H * W + F)
    x = torch.randint(-1024, 1025, (N, H, W, C), generator=g, device="cuda").float() / 256
    x[0, 5, 7, 0] = float("nan")
    x.view(torch.int32)[-1, 9, 31, C - 1] = -0x400000  # a NaN with the sign bit set
    w = _words(g, F, 3, 3, bnn.words(C))
    thr = torch.randint(-12, 13, (F,), generator=g, device="cuda").to(torch.int32)
    flip = _words(g, bnn.words(F))
    desc = bnn.conv_desc(N, H, W, C, F, 3, 3, 1, 1, pool)
    got = bnn.bnn_fconv2d_binw(desc, x, w, thr, flip, want_sums=sums)
    with bnn.options(algo=bnn.ALGO_VALU):
        ref = bnn.bnn_fconv2d_binw(desc, x, w, thr, flip, want_sums=sums)
    assert torch.equal(got[1], ref[1])
    if sums:
        assert torch.equal(got[0].isnan(), ref[0].isnan()) and bool(got[0].isnan().any())
