"""The many-row FC kernel where it can go wrong: K at and around whole chunks
of 256 bits (tail bits garbled), 4 to 34 chunks, row and output counts around
the tiles of every wave arrangement.  The reference is the vector-ALU kernel,
itself checked against the oracle, on the same packed inputs; every word and
sum is compared."""
import pytest
import torch

from paper_1808_00209_amd import bnn

pytestmark = pytest.mark.gpu

CASES = [
    # M, K, N
    (1057, 1024, 1024), (1057, 1025, 1088), (1088, 1311, 1024), (2049, 2047, 1100),
    (1300, 4100, 1653), (3001, 1280, 1001), (1100, 8448, 1024), (300, 1536, 4096),
    (9000, 1100, 192), (17000, 1792, 64), (35000, 1024, 64), (129, 1300, 16384),
    (4096, 2304, 2049), (70000, 1030, 33),
]


def _words(g, *shape):
    return torch.randint(-2 ** 31, 2 ** 31, shape, generator=g, device="cuda",
                         dtype=torch.int64).to(torch.int32)


@pytest.mark.parametrize("case", CASES, ids=[str(c) for c in CASES])
@pytest.mark.parametrize("sums,bits", [(False, True), (True, True), (True, False)])
def test_fc_tile_matches_the_vector_kernel(case, sums, bits):
    M, K, N = case
    g = torch.Generator(device="cuda").manual_seed(M + K + N)
    A, B = _words(g, M, bnn.words(K)), _words(g, N, bnn.words(K))
    r = 2 * int(K ** 0.5)
    thr = torch.randint(-r, r + 1, (N,), generator=g, device="cuda").to(torch.int32)
    thr[0], thr[-1] = 2 ** 31 - 1, -2 ** 31
    flip = _words(g, bnn.words(N)) if not sums or bits else None
    got = bnn.bnn_bgemm(A, B, K, thr, flip, want_sums=sums, want_bits=bits)
    with bnn.options(algo=bnn.ALGO_VALU):
        ref = bnn.bnn_bgemm(A, B, K, thr, flip, want_sums=sums, want_bits=bits)
    for a, b in zip(got, ref):
        assert (a is None) == (b is None)
        if a is not None:
            assert torch.equal(a, b)
