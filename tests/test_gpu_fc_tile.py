"""The many-row FC kernel where it can go wrong.  TAKEN holds every wave
arrangement (log2 of the waves along the outputs, 32-row tiles per wave) with
the one that the launcher picks asserted: K off whole chunks of 256 bits (tail
bits garbled), ragged row and output counts, sums, bits or both.  CASES has K at
and around whole chunks, 4 to 34 of them.  The reference is the vector-ALU
kernel, itself checked against the oracle, on the same packed inputs; every
word and sum is compared."""
import pytest
import torch

import tile_plans
from paper_1808_00209_amd import bnn

pytestmark = pytest.mark.gpu

TAKEN = [
    # M, K, N, sums, bits, log2 of the waves along the outputs, row tiles
    (17310, 1197, 64, 1, 1, 0, 1), (33, 1208, 30784, 0, 1, 1, 1), (23354, 1066, 67, 0, 1, 1, 2),
    (1090, 1500, 2060, 1, 0, 1, 2), (6, 1400, 52160, 1, 1, 2, 1), (34, 1055, 33221, 1, 1, 2, 2),
    (2100, 1030, 2050, 0, 1, 2, 4), (2111, 1290, 4100, 1, 1, 2, 4), (4090, 2081, 2050, 0, 1, 2, 4),
    (4001, 5003, 4096, 0, 1, 2, 4), (1500, 1100, 4095, 1, 0, 2, 4), (530, 2079, 8190, 1, 1, 2, 4),
    (270, 1055, 16001, 0, 1, 2, 4), (70000, 5000, 20, 0, 1, 0, 1), (66000, 8200, 7, 1, 1, 0, 1),
]
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


def _same(A, B, K, thr, flip, sums, bits):
    got = bnn.bnn_bgemm(A, B, K, thr, flip, want_sums=bool(sums), want_bits=bool(bits))
    with bnn.options(algo=bnn.ALGO_VALU):
        ref = bnn.bnn_bgemm(A, B, K, thr, flip, want_sums=bool(sums), want_bits=bool(bits))
    for a, b in zip(got, ref):
        assert (a is None) == (b is None)
        if a is not None:
            assert torch.equal(a, b)


def _thresholds(g, N, K):
    r = 2 * int(K ** 0.5)
    thr = torch.randint(-r, r + 1, (N,), generator=g, device="cuda").to(torch.int32)
    thr[0], thr[-1] = 2 ** 31 - 1, -2 ** 31
    return thr


@pytest.mark.parametrize("case", TAKEN, ids=[str(c[:3]) for c in TAKEN])
def test_every_wave_arrangement(case):
    M, K, N, sums, bits, wfl, pt = case
    plan = tile_plans.fc_tile(M, K, N, sums, bits)
    assert plan is not None and (plan["wfl"], plan["pt"]) == (wfl, pt)
    g = torch.Generator(device="cuda").manual_seed(M + K + N)
    _same(_words(g, M, bnn.words(K)), _words(g, N, bnn.words(K)), K, _thresholds(g, N, K),
          _words(g, bnn.words(N)), sums, bits)


@pytest.mark.parametrize("M,K,N", [(4161700, 4100, 64), (33, 16000, 1 << 20)],
                         ids=["rows", "weights"])
def test_operand_of_almost_2_gib(M, K, N):
    """Byte offsets up to 2^31 of the data rows or the weight rows."""
    assert 2 ** 31 - 2 ** 26 < max(M, N) * bnn.words(K) * 4 < 2 ** 31 - 4096
    assert tile_plans.fc_tile(M, K, N, False, True)
    g = torch.Generator(device="cuda").manual_seed(4)
    ops = []
    for n in (M, N):
        t = torch.empty(n, bnn.words(K), dtype=torch.int32, device="cuda")
        for i in range(0, n, 1 << 18):
            t[i:i + (1 << 18)] = _words(g, *t[i:i + (1 << 18)].shape)
        ops.append(t)
    _same(*ops, K, _thresholds(g, N, K), _words(g, bnn.words(N)), False, True)


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
