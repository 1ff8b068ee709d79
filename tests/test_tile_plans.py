"""The plans of the tile kernels, on the host (CPU only).  The staged-tile conv's
does not cost more on a wide map, no run of it reads or stages outside the LDS
tile, for any window (square or not), pooled or not, with and without sums; and
both kernels are taken where they measured faster than the others."""
import random

import numpy as np
import pytest

import tile_plans


@pytest.mark.parametrize("W", [1024, 8192, 65536, 262144])
@pytest.mark.parametrize("C,k,pool", [(96, 3, 0), (128, 3, 2), (1000, 5, 0)])
def test_plan_costs_the_same_on_wide_maps(W, C, k, pool):
    # (a step per strip count took 10 times as long at 1024 columns and 1700
    # times at 262144; the bound leaves room for a busy host)
    small = tile_plans.conv_tile_host_us((1024 * 1024 // 56 // 56, 56, 56, C, 128, k, k, 1, pool), 0)
    wide = tile_plans.conv_tile_host_us((max(1, 1024 * 1024 // 8 // W), 8, W, C, 128, k, k, 1, pool), 0)
    assert wide < 6 * small + 1, (wide, small)


def _shapes():
    rng = random.Random(7)
    out = [(7, 45, 61, 160, 200, 3, 3, 1, 2), (3, 9, 1500, 96, 64, 3, 3, 1, 0),
           (5, 7, 9, 64, 128, 1, 4, 0, 2), (2, 1, 70, 96, 64, 1, 3, 1, 0)]
    while len(out) < 400:
        KH, KW = rng.randint(1, 6), rng.randint(1, 5)
        H, W = rng.randint(1, 40), rng.choice([rng.randint(1, 40), rng.randint(41, 400)])
        s = (rng.randint(1, 9), H, W, rng.choice([32, 64, 100, 256, rng.randint(33, 700)]),
             rng.randint(33, 300), KH, KW, rng.randint(0, 2), rng.choice([0, 2]))
        if H + 2 * s[7] - KH >= 1 and W + 2 * s[7] - KW >= 1:
            out.append(s)
    return out


def _item(p, pool, item):
    """Image, grid row and output row / column (from the strip's first) of items."""
    w = item // 4 if pool else item
    t, jw = w // p["Ws"], w % p["Ws"]
    n, iw = t // p["Hw"], t % p["Hw"]
    return (n, iw, 2 * iw + item // 2 % 2, 2 * jw + item % 2) if pool else (n, iw, iw, jw)


@pytest.mark.parametrize("sums", [False, True])
def test_runs_stay_inside_their_lds_tile(sums):
    """Every run of 1 to 4 units a block may take: the staged rows fit the LDS
    the plan asks for, and every window of every pixel lies in the staged rows
    and columns; the strips cover each output pixel once."""
    planned = 0
    for shape in _shapes():
        p = tile_plans.cheapest(shape, sums)
        if not p["ok"]:
            continue
        planned += 1
        N, H, W, C, F, KH, KW, pad, pool = shape
        pool = pool == 2
        rs, wp = (2 if pool else 1), 4 >> p["wfl"]
        Hv, ps, unit = p["H"] + 2 * pad, 2 * p["ks"] + 1, 32 * (4 >> p["wfl"])
        assert p["lds"] <= 79 * 1024 and p["cols"] == rs * p["Ws"] + KW - 1
        assert p["RS"] >= p["cols"] * ps and p["ups"] * unit >= p["items"]
        n, iw, i, j = _item(p, pool, np.arange(p["items"]))
        for u in range(p["ups"]):
            for units in range(1, min(4, p["ups"] - u) + 1):
                a, b = u * unit, min((u + units) * unit, p["items"])
                if a >= p["items"]:
                    continue
                v0 = n[a] * Hv + rs * iw[a]
                rows = n[b - 1] * Hv + rs * iw[b - 1] + rs - 1 - v0 + KH
                assert ((rows - 1) * p["RS"] + p["cols"] * ps) * 16 <= p["lds"], (shape, u, units)
                r = n[a:b] * Hv + i[a:b] - v0
                assert r.min() >= 0 and r.max() + KH <= rows, (shape, u, units)
        assert j.max() + KW <= p["cols"]
        # coverage: strip s, column js0 + j; pixels outside the map are dropped
        seen = np.zeros((p["N"], p["Ho"], p["Wo"]), int)
        for s in range(p["strips"]):
            col = j + rs * s * p["Ws"]
            ok = (i < p["Ho"]) & (col < p["Wo"])
            np.add.at(seen, (n[ok], i[ok], col[ok]), 1)
        cut = seen if sums or not pool else seen[:, :p["Ho"] // 2 * 2, :p["Wo"] // 2 * 2]
        assert cut.min() == 1 and seen.max() == 1, shape
        assert wp * 32 == unit
    assert planned > 300


# Graph-timed on one card: the general kernel's time and the staged-tile
# kernel's, in microseconds.  (N, H, W, C, F, KH, KW, pad, pool), sums, bits,
# prepared weights, general, staged tile.
MEASURED = [
    ((93, 54, 49, 64, 256, 3, 4, 1, 0), 0, 1, 0, 30.8, 36.8),
    ((21, 24, 434, 64, 512, 4, 4, 2, 0), 0, 1, 0, 66.1, 83.6),
    ((171, 51, 9, 64, 512, 4, 4, 0, 0), 0, 1, 1, 19.8, 23.4),
    ((32, 26, 98, 128, 256, 3, 3, 1, 0), 0, 1, 0, 14.9, 17.2),
    ((77, 6, 18, 41, 203, 1, 1, 0, 0), 0, 1, 0, 3.8, 4.4),
    ((67, 39, 14, 204, 64, 1, 1, 0, 0), 1, 0, 0, 8.0, 9.4),
    ((2, 53, 40, 208, 512, 1, 1, 0, 0), 0, 1, 1, 4.7, 5.6),
    ((11, 31, 31, 249, 256, 1, 1, 0, 0), 1, 0, 1, 7.9, 9.4),
    ((113, 39, 33, 96, 64, 2, 1, 0, 2), 0, 1, 0, 6.5, 7.9),
    ((99, 48, 5, 491, 65, 1, 2, 0, 0), 1, 0, 0, 9.9, 12.4),
    ((13, 60, 30, 238, 128, 1, 3, 0, 0), 0, 1, 1, 5.4, 6.7),
    ((66, 16, 12, 467, 256, 5, 2, 0, 0), 1, 1, 1, 17.0, 20.8),
    ((60, 29, 11, 274, 156, 3, 3, 0, 2), 0, 1, 0, 11.6, 14.5),
    ((48, 14, 14, 277, 512, 5, 5, 0, 0), 1, 0, 0, 37.5, 49.2),
    ((6, 44, 53, 325, 242, 5, 5, 0, 2), 0, 1, 1, 23.4, 29.4),
    ((28, 45, 12, 459, 256, 3, 3, 1, 0), 0, 1, 1, 12.8, 18.5),
    ((147, 10, 43, 192, 512, 1, 7, 0, 0), 0, 1, 0, 26.0, 18.9),
    ((100, 24, 56, 192, 256, 5, 2, 1, 2), 1, 0, 0, 64.1, 41.1),
    ((81, 24, 56, 256, 470, 3, 3, 1, 2), 0, 1, 0, 66.0, 46.2),
    ((64, 56, 56, 256, 256, 3, 3, 1, 0), 0, 1, 1, 48.4, 41.9),
    ((256, 12, 12, 256, 512, 3, 3, 1, 2), 0, 1, 1, 20.4, 17.7),
    ((163, 35, 35, 256, 256, 3, 3, 1, 2), 1, 1, 0, 127.6, 81.0),
    ((116, 61, 61, 64, 473, 3, 3, 0, 0), 0, 1, 1, 107.6, 76.3),
    ((58, 48, 33, 128, 512, 3, 3, 1, 2), 1, 0, 1, 71.8, 46.0),
    ((7, 45, 61, 160, 200, 3, 3, 1, 2), 1, 1, 0, 29.8, 13.7),
    ((173, 12, 12, 255, 256, 1, 1, 0, 0), 0, 1, 0, 9.9, 6.6),
    ((49, 33, 33, 121, 285, 1, 1, 0, 0), 1, 0, 0, 50.3, 33.7),
    ((18, 19, 452, 150, 512, 1, 1, 0, 0), 0, 1, 1, 30.1, 21.9),
    ((30, 37, 16, 215, 512, 1, 7, 0, 0), 0, 1, 0, 18.6, 10.0),
    ((68, 12, 12, 204, 512, 3, 4, 1, 0), 0, 1, 1, 20.8, 12.6),
    ((105, 7, 55, 294, 64, 3, 4, 0, 2), 1, 1, 1, 24.9, 15.4),
    ((238, 37, 32, 180, 54, 5, 5, 2, 2), 0, 1, 0, 88.0, 43.9),
    ((169, 56, 15, 300, 64, 5, 5, 2, 2), 0, 1, 1, 69.6, 41.2),
]


@pytest.mark.parametrize("case", MEASURED, ids=[str(c[:4]) for c in MEASURED])
def test_the_faster_conv_kernel_is_taken(case):
    shape, sums, bits, prepared, general, tile = case
    assert (tile_plans.conv_tile(shape, sums, bits, prepared) is not None) == (tile < general)


# The same for the many-row FC kernel: M, K, N, sums, bits, the FC or conv
# kernel's time and the many-row kernel's.
MEASURED_FC = [
    (66000, 1024, 10, 0, 1, 7.2, 8.9), (150000, 1024, 32, 0, 1, 12.7, 14.2),
    (66000, 4096, 32, 0, 1, 15.6, 19.4), (66000, 4096, 32, 1, 1, 19.0, 22.0),
    (66000, 4096, 10, 1, 0, 15.5, 20.3), (66000, 1030, 32, 0, 1, 7.5, 10.6),
    (66000, 5000, 4, 0, 1, 20.6, 22.2), (66000, 5000, 32, 0, 1, 26.9, 23.7),
    (66000, 5000, 32, 1, 1, 30.4, 25.7), (66000, 16000, 16, 0, 1, 61.8, 54.6),
    (66000, 4096, 48, 0, 1, 20.9, 20.4), (66000, 5000, 33, 0, 1, 32.2, 23.8),
    (262, 2048, 4096, 1, 0, 8.2, 8.7), (262, 2048, 4096, 1, 1, 9.2, 9.0),
    (262, 4096, 4096, 1, 0, 11.5, 11.9), (262, 1280, 4096, 1, 0, 7.5, 6.7),
    (1100, 8192, 1024, 0, 1, 19.3, 17.5), (1024, 1024, 1024, 0, 1, 4.6, 6.2),
    (2048, 4096, 1000, 0, 1, 9.7, 11.3), (4096, 4100, 1000, 0, 1, 22.4, 15.3),
    (4096, 8192, 4096, 0, 1, 133.0, 50.0),
]


@pytest.mark.parametrize("case", MEASURED_FC, ids=[str(c[:3]) for c in MEASURED_FC])
def test_the_faster_fc_kernel_is_taken(case):
    M, K, N, sums, bits, other, tile = case
    assert (tile_plans.fc_tile(M, K, N, sums, bits) is not None) == (tile < other)
