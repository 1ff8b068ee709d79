"""The binding's own output sizes are those of bnn_conv_output_dims, and
descriptors it refuses raise the same errors (CPU only)."""
import itertools

import pytest

from paper_1808_00209_amd import bnn


def _both(d):
    out = []
    for f in (bnn._output_dims, bnn.bnn_conv_output_dims):
        try:
            out.append(f(d))
        except bnn.BnnError as e:
            out.append((e.status, str(e)))
    return out


@pytest.mark.parametrize("KH,KW", [(1, 1), (3, 3), (5, 2), (7, 130), (0, 3)])
@pytest.mark.parametrize("stride", [1, 2])
def test_output_dims_agree(KH, KW, stride):
    for H, W, pad, pool, N, C, F in itertools.product(
            (0, 1, 2, 7, 40000), (1, 3, 8), (-1, 0, 2), (0, 2, 1), (0, 1, 70000), (0, 3, 5000),
            (1, 20000)):
        a, b = _both(bnn.conv_desc(N, H, W, C, F, KH, KW, stride, pad, pool))
        assert a == b
