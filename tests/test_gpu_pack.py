"""bnn_pack_bits where its wave covers ragged rows and a partial last wave:
the words must be those of the oracle at every row length from one word up,
for any 4-byte aligned base pointer (a wave packs 64 words, a lane 4 values)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1808_00209_amd import bnn
from paper_1808_00209_amd.device import to_device, words_u32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,D", [(1, 32), (64, 32), (65, 33), (300, 36), (129, 63), (7, 2048),
                                    (257, 94), (513, 256), (3, 18431)])
@pytest.mark.parametrize("shift", [0, 1, 3])
@pytest.mark.parametrize("with_offset", [False, True])
def test_pack_rows_at_any_alignment(rows, D, shift, with_offset):
    rng = np.random.default_rng(rows * 31 + D)
    x = rng.standard_normal((rows, D)).astype(np.float32)
    off = (np.round(rng.standard_normal(D) * 4) / 4).astype(np.float32) if with_offset else None
    if with_offset:
        x[0] = -off  # ties: x + T == 0 gives bit 0
    x[-1, -1] = np.nan
    x[0, 0] = np.inf
    buf = torch.empty(rows * D + shift, device="cuda")
    xd = buf[shift:].view(rows, D)
    xd.copy_(to_device(x))
    offd = None
    if with_offset:
        obuf = torch.empty(D + shift, device="cuda")
        offd = obuf[shift:]
        offd.copy_(to_device(off))
    got = words_u32(bnn.bnn_pack_bits(xd, offd))
    v = x if off is None else x + off
    ref = oracle.pack_eq2(np.where(v > 0, 1, -1).astype(np.int8))  # NaN -> -1
    assert np.array_equal(got, ref)
