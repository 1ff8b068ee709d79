"""The staged-tile conv kernel where it can go wrong: every k-step count per
tap (C = 32 .. 256, odd word counts, tail bits), one and several channel
chunks, filter counts around the 64-filter waves, runs that span images and
strips, odd pooled sizes with sums, and the last round's short runs.  The
reference is the vector-ALU kernel, itself checked against the oracle, on the
same packed inputs (tail bits garbled); every word and sum is compared."""
import pytest
import torch

from paper_1808_00209_amd import bnn

pytestmark = pytest.mark.gpu

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
