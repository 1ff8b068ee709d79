"""The workloads whose time is tracked, each through the public binding.

A case names a family of calls and its sizes.  ``listed()`` are the fixed
points; ``draw(rng)`` gives another point of the same ranges:

  forward  one bnn_forward of a whole net (the CIFAR-shaped net with a
           real-valued first layer, the vehicle-shaped net with thresholded
           RGB input, Table II's 5x5 net under its three input
           binarizations), 1 to 256 images: what a classifier runs
  conv     one binary conv layer of a deeper net (1x1, 3x3 or 5x5, 32 to 512
           channels, odd ones among them, maps of 7 to 64 pixels a side),
           bits only as inside a net, or with int32 sums as for fitting
           thresholds
  gemm     one binary FC layer / GEMM, 2 to 4096 rows, 1024 to 16384 bits
  fconv    the real-valued first layer on its own, fp32 images of 24 to 224
           pixels a side
  pack     packing fp32 activations into bits

Everything is drawn from the seed on the GPU.  Binary tensors are i.i.d.
Bernoulli(0.5) bits (packed words are uniform 32-bit words; the tail bits of
a short last word are arbitrary, as the interface allows).  Thresholds are
uniform on [-2 ceil(sqrt K), 2 ceil(sqrt K)], which keeps bits near balanced
through deep chains, as after BatchNorm.
"""
import math

import torch

from paper_1808_00209_amd import bnn

DEV = "cuda"
PAPER_INPUTS = {"paper_rgb": "threshold", "paper_gray": "gray", "paper_lbp": "lbp"}


# ------------------------------------------------------------------ cases ---
def listed():
    return [
        # One image at a time: the latency of a small classifier.
        dict(name="forward_cifar_b1", family="forward", net="cifar", batch=1),
        # The usual serving batch of the benchmark's flagship net.
        dict(name="forward_cifar_b64", family="forward", net="cifar", batch=64),
        # Throughput on larger images: 96x96 RGB, a large batch.
        dict(name="forward_vehicle_b256", family="forward", net="vehicle", batch=256),
        # Table II's 5x5 net with local binary patterns, an odd batch.
        dict(name="forward_lbp_b100", family="forward", net="paper_lbp", batch=100),
        # A mid-network 3x3 layer of a large net, bits to bits.
        dict(name="conv3_56_256_b64", family="conv", N=64, H=56, W=56, C=256, F=256, k=3, pad=1,
             pool=0, sums=False, bits=True, prepared=True),
        # A bottleneck's widening 1x1 layer.
        dict(name="conv1_56_256_1024_b64", family="conv", N=64, H=56, W=56, C=256, F=1024, k=1,
             pad=0, pool=0, sums=False, bits=True, prepared=False),
        # Ragged sizes, sums kept beside the bits (threshold fitting).
        dict(name="conv3_ragged_sums", family="conv", N=7, H=45, W=61, C=160, F=200, k=3, pad=1,
             pool=2, sums=True, bits=True, prepared=False),
        # The FC GEMM of the benchmark, int32 sums and bits.
        dict(name="gemm_256_4096_4096", family="gemm", M=256, K=4096, N=4096, sums=True, bits=True),
        # A small FC layer with a ragged row and output count.
        dict(name="gemm_100_4100_1000", family="gemm", M=100, K=4100, N=1000, sums=False,
             bits=True),
        # Many rows: an FC layer over a large batch.
        dict(name="gemm_4096_8192_4096", family="gemm", M=4096, K=8192, N=4096, sums=False,
             bits=True),
        # The real-valued first layer on its own, sums and bits.
        dict(name="fconv_112_b32", family="fconv", N=32, H=112, W=112, C=3, F=64, k=3, pad=1,
             pool=0, sums=True, bits=True),
        # Binarizing a layer's fp32 activations.
        dict(name="pack_64x56x56x256", family="pack", rows=64 * 56 * 56, D=256, offset=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["forward", "conv", "conv", "gemm", "gemm", "fconv", "pack"])
    if family == "forward":
        return dict(family=family, net=rng.choice(["cifar", "vehicle"] + sorted(PAPER_INPUTS)),
                    batch=_log(rng, 1, 256))
    if family == "conv":
        k = rng.choice([1, 3, 3, 5])
        C = rng.choice([64, 128, 256, 512, rng.randint(32, 512)])
        F = rng.choice([64, 128, 256, 512, rng.randint(32, 512)])
        H, W = _log(rng, 7, 64), _log(rng, 7, 64)
        if rng.random() < 0.5:
            W = H
        most = 64 * 56 * 56 * 256 * 9 * 256  # the listed 3x3 layer's bit products
        N = min(_log(rng, 1, 64), max(1, most // (H * W * F * k * k * C)))
        sums = rng.random() < 0.3
        return dict(family=family, N=N, H=H, W=W, C=C, F=F, k=k, pad=k // 2,
                    pool=rng.choice([0, 2]), sums=sums, bits=not sums or rng.random() < 0.7,
                    prepared=rng.random() < 0.5)
    if family == "gemm":
        M = _log(rng, 2, 4096)
        K = rng.choice([1024, 2048, 4096, 8192, _log(rng, 1024, 16384)])
        N = rng.choice([1024, 4096, _log(rng, 10, 4096)])
        if M * N * K > 4096 * 4096 * 8192:
            K = 8192
        sums = rng.random() < 0.4
        return dict(family=family, M=M, K=K, N=N, sums=sums, bits=not sums or rng.random() < 0.5)
    if family == "fconv":
        H = _log(rng, 24, 224)
        N = min(_log(rng, 1, 64), max(1, 32 * 112 * 112 // (H * H)))
        sums = rng.random() < 0.5
        return dict(family=family, N=N, H=H, W=H, C=rng.choice([1, 3]), F=rng.choice([32, 64, 128]),
                    k=3, pad=1, pool=rng.choice([0, 2]), sums=sums,
                    bits=not sums or rng.random() < 0.5)
    D = rng.choice([64, 256, 512, 8192, _log(rng, 33, 18432)])
    return dict(family=family, rows=max(1, _log(rng, 1 << 20, 64 * 56 * 56 * 256) // D), D=D,
                offset=rng.random() < 0.5)


# ----------------------------------------------------------------- inputs ---
def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _words(g, *shape):
    """Uniform 32-bit words (int32 storage)."""
    return torch.randint(-2 ** 31, 2 ** 31, shape, generator=g, device=DEV,
                         dtype=torch.int64).to(torch.int32)


def _thresholds(g, n, K):
    r = 2 * math.isqrt(K - 1) + 2
    return torch.randint(-r, r + 1, (n,), generator=g, device=DEV, dtype=torch.int64).to(torch.int32)


def _conv(g, C, F, k=3, pad=1, pool=0, kind=bnn.LAYER_BCONV):
    return dict(kind=kind, C=C, F=F, KH=k, KW=k, stride=1, pad=pad, pool=pool,
                w=_words(g, F, k, k, bnn.words(C)), thr=_thresholds(g, F, k * k * C),
                flip=_words(g, bnn.words(F)))


def _fc(g, K, N, logits=False):
    d = dict(kind=bnn.LAYER_BFC_LOGITS if logits else bnn.LAYER_BFC, K=K, N=N,
             w=_words(g, N, bnn.words(K)))
    if not logits:
        d.update(thr=_thresholds(g, N, K), flip=_words(g, bnn.words(N)))
    return d


def _offsets(g, n):
    return -torch.randint(64, 192, (n,), generator=g, device=DEV).to(torch.float32)


def _net(case, seed):
    """Layers (with packed weights), image size and input images of a net."""
    g = _generator(seed)
    batch, net = case["batch"], case["net"]
    if net == "cifar":
        size = 32
        layers = [_conv(g, 3, 128, kind=bnn.LAYER_FCONV_BINW), _conv(g, 128, 128, pool=2),
                  _conv(g, 128, 256), _conv(g, 256, 256, pool=2), _conv(g, 256, 512),
                  _conv(g, 512, 512, pool=2), _fc(g, 8192, 1024), _fc(g, 1024, 1024),
                  _fc(g, 1024, 10, logits=True)]
        # Normalised images on a 2^-16 grid: the first layer's sums are exact.
        x = torch.randn(batch, size, size, 3, generator=g, device=DEV)
        x = (x * 65536).round().clamp(-8 * 65536 + 1, 8 * 65536 - 1) / 65536
        return layers, size, x
    size = 96
    x = torch.randint(0, 256, (batch, size, size, 3), generator=g, device=DEV).to(torch.float32)
    if net == "vehicle":
        layers = [dict(kind=bnn.LAYER_INPUT_THRESHOLD, C=3, offset=_offsets(g, 3)),
                  _conv(g, 3, 64), _conv(g, 64, 64, pool=2), _conv(g, 64, 128),
                  _conv(g, 128, 128, pool=2), _conv(g, 128, 256), _conv(g, 256, 256, pool=2),
                  _conv(g, 256, 512, pool=2), _fc(g, 18432, 1024), _fc(g, 1024, 4, logits=True)]
        return layers, size, x
    mode = PAPER_INPUTS[net]
    first = {"threshold": lambda: dict(kind=bnn.LAYER_INPUT_THRESHOLD, C=3, offset=_offsets(g, 3)),
             "gray": lambda: dict(kind=bnn.LAYER_INPUT_GRAY, C=3, offset=_offsets(g, 1)),
             "lbp": lambda: dict(kind=bnn.LAYER_INPUT_LBP, C=3)}[mode]()
    layers = [first, _conv(g, 1 if mode == "gray" else 3, 32, k=5, pad=2, pool=2),
              _conv(g, 32, 32, k=5, pad=2, pool=2), _fc(g, 18432, 100), _fc(g, 100, 100),
              _fc(g, 100, 4, logits=True)]
    return layers, size, x


def _layer_inputs(case, seed):
    """Tensors of a single-layer case."""
    g = _generator(seed)
    if case["family"] == "pack":
        x = torch.randn(case["rows"], case["D"], generator=g, device=DEV)
        off = torch.randn(case["D"], generator=g, device=DEV) if case["offset"] else None
        return dict(x=x, offset=off)
    if case["family"] == "gemm":
        kw = bnn.words(case["K"])
        return dict(x=_words(g, case["M"], kw), w=_words(g, case["N"], kw),
                    thr=_thresholds(g, case["N"], case["K"]), flip=_words(g, bnn.words(case["N"])))
    d = _conv(g, case["C"], case["F"], k=case["k"])
    shape = (case["N"], case["H"], case["W"])
    if case["family"] == "fconv":
        x = torch.randn(*shape, case["C"], generator=g, device=DEV)
    else:
        x = _words(g, *shape, bnn.words(case["C"]))
    return dict(x=x, w=d["w"], thr=d["thr"], flip=d["flip"])


def prepare(case, seed):
    if case["family"] == "forward":
        layers, size, x = _net(case, seed)
        for d in layers:  # conv weights in the kernels' operand form, once per net
            if d["kind"] == bnn.LAYER_BCONV:
                d["wprep"] = bnn.bnn_prepare_weights(d["w"], d["F"], d["KH"], d["KW"], d["C"])
        net = bnn.Network(layers, size, size, 3)
        return dict(case=case, net=net, x=x, ws=net.alloc_workspace(case["batch"]))
    s = dict(case=case, **_layer_inputs(case, seed))
    if case["family"] in ("conv", "fconv"):
        s["desc"] = bnn.conv_desc(case["N"], case["H"], case["W"], case["C"], case["F"],
                                  case["k"], case["k"], 1, case["pad"], case["pool"])
    if case.get("prepared"):
        s["wprep"] = bnn.bnn_prepare_weights(s["w"], case["F"], case["k"], case["k"], case["C"])
    return s


def run(s):
    case = s["case"]
    family = case["family"]
    if family == "forward":
        return bnn.bnn_forward(s["net"], s["x"], s["ws"])
    if family == "pack":
        return bnn.bnn_pack_bits(s["x"], s["offset"])
    want = dict(want_sums=case["sums"], want_bits=case["bits"])
    if family == "gemm":
        return bnn.bnn_bgemm(s["x"], s["w"], case["K"], s["thr"], s["flip"], **want)
    if family == "fconv":
        return bnn.bnn_fconv2d_binw(s["desc"], s["x"], s["w"], s["thr"], s["flip"], **want)
    if case["prepared"]:
        return bnn.bnn_bconv2d_prepared(s["desc"], s["x"], s["w"], s["wprep"], s["thr"], s["flip"],
                                        **want)
    return bnn.bnn_bconv2d(s["desc"], s["x"], s["w"], s["thr"], s["flip"], **want)


# ------------------------------------------------------------------- work ---
def _conv_work(N, H, W, C, F, k, pad, pool, in_bytes, sums, bits):
    Ho, Wo = H + 2 * pad - k + 1, W + 2 * pad - k + 1
    out = N * Ho * Wo * F * 4 if sums else 0
    if bits:
        Hp, Wp = (Ho // 2, Wo // 2) if pool else (Ho, Wo)
        out += N * Hp * Wp * bnn.words(F) * 4
    wts = F * k * k * bnn.words(C) * 4 + F * 4 + bnn.words(F) * 4
    return in_bytes + wts + out, 2 * N * Ho * Wo * F * k * k * C


_NET_LAYERS = {  # (C, F, map side, kernel) of the convs, (K, N) of the FC layers
    "cifar": (32, [(3, 128, 32, 3), (128, 128, 32, 3), (128, 256, 16, 3), (256, 256, 16, 3),
                   (256, 512, 8, 3), (512, 512, 8, 3)], [(8192, 1024), (1024, 1024), (1024, 10)]),
    "vehicle": (96, [(3, 64, 96, 3), (64, 64, 96, 3), (64, 128, 48, 3), (128, 128, 48, 3),
                     (128, 256, 24, 3), (256, 256, 24, 3), (256, 512, 12, 3)],
                [(18432, 1024), (1024, 4)]),
    "paper": (96, [(3, 32, 96, 5), (32, 32, 48, 5)], [(18432, 100), (100, 100), (100, 4)]),
}


def work(case):
    family = case["family"]
    if family == "forward":
        size, convs, fcs = _NET_LAYERS[case["net"].split("_")[0]]
        batch = case["batch"]
        # The images, every layer's weights once and the logits; the bits
        # between layers need not leave the chip.
        b, f = batch * size * size * 3 * 4 + batch * fcs[-1][1] * 4, 0
        for C, F, side, k in convs:
            C = 1 if case["net"] == "paper_gray" and C == 3 else C
            b += F * k * k * bnn.words(C) * 4
            f += 2 * batch * side * side * F * k * k * C
        for K, N in fcs:
            b += N * bnn.words(K) * 4
            f += 2 * batch * K * N
        return {"bytes": b, "flops": f}
    if family == "pack":
        n = case["rows"] * case["D"]
        return {"bytes": 4 * n + 4 * case["rows"] * bnn.words(case["D"]),
                "flops": n * (2 if case["offset"] else 1)}
    if family == "gemm":
        M, K, N = case["M"], case["K"], case["N"]
        b = (M + N) * bnn.words(K) * 4 + N * 4 + bnn.words(N) * 4
        b += (M * N * 4 if case["sums"] else 0) + (M * bnn.words(N) * 4 if case["bits"] else 0)
        return {"bytes": b, "flops": 2 * M * N * K}
    per_pixel = case["C"] * 4 if family == "fconv" else bnn.words(case["C"]) * 4
    b, f = _conv_work(case["N"], case["H"], case["W"], case["C"], case["F"], case["k"],
                      case["pad"], case["pool"], case["N"] * case["H"] * case["W"] * per_pixel,
                      case["sums"], case["bits"])
    return {"bytes": b, "flops": f}


def tolerance(case):
    if case["family"] == "fconv":
        # fp32 sums of at most 27 products in any order; a bit may differ
        # where a sum lies within that rounding of its integer threshold.
        return {"rel": 2.5e-7, "differ": 1e-5}
    return "exact"  # packed bits and integer sums


# ------------------------------------------------------------ exact results ---
def _pm1(words, n):
    """Packed words [..., W] -> +-1.0 [..., n] in 64 bits."""
    sh = torch.arange(31, -1, -1, device=words.device, dtype=torch.int32)
    bits = (words.unsqueeze(-1) >> sh) & 1
    return bits.flatten(-2)[..., :n].double() * 2 - 1


def _pack(bits):
    """Booleans [..., n] -> packed words [..., ceil(n / 32)]."""
    n = bits.shape[-1]
    b = torch.nn.functional.pad(bits.to(torch.int64), (0, -n % 32)).unflatten(-1, (-1, 32))
    sh = torch.arange(31, -1, -1, device=bits.device, dtype=torch.int64)
    w = (b << sh).sum(-1)
    return (w - ((w >> 31) << 32)).to(torch.int32)


def _sums(x, w, k, pad, pad_value):
    """Window sums [N, Ho, Wo, F] of x [N, H, W, C] with w [F, k, k, C]."""
    xp = torch.nn.functional.pad(x, (0, 0, pad, pad, pad, pad), value=pad_value)
    N, Hq, Wq, C = xp.shape
    Ho, Wo = Hq - k + 1, Wq - k + 1
    out = torch.zeros(N * Ho * Wo, w.shape[0], dtype=torch.float64, device=x.device)
    for i in range(k):
        for j in range(k):
            tap = xp[:, i:i + Ho, j:j + Wo].reshape(-1, C)
            out += tap @ w[:, i, j].t().contiguous()
    return out.view(N, Ho, Wo, -1)


def _bits(S, d):
    flip = _pm1(d["flip"], S.shape[-1]) > 0
    return (S >= d["thr"].double()) ^ flip


def _pool(b):
    H, W = b.shape[1] // 2 * 2, b.shape[2] // 2 * 2
    return (b[:, 0:H:2, 0:W:2] | b[:, 1:H:2, 0:W:2] | b[:, 0:H:2, 1:W:2] | b[:, 1:H:2, 1:W:2])


def _gray(x):
    # The luma is defined in fp32, each product and sum rounded on its own.
    return (x[..., 0] * 0.299 + x[..., 1] * 0.587) + x[..., 2] * 0.114


def _input_bits(d, x):
    if d["kind"] == bnn.LAYER_INPUT_THRESHOLD:
        return x + d["offset"] > 0
    g = _gray(x)
    if d["kind"] == bnn.LAYER_INPUT_GRAY:
        return (g + d["offset"][0] > 0).unsqueeze(-1)
    H, W = g.shape[1:]
    gp = torch.nn.functional.pad(g, (1, 1, 1, 1), value=-1.0)
    return torch.stack([gp[:, 1 + di:1 + di + H, 1 + dj:1 + dj + W] > g
                        for di, dj in ((-1, -1), (0, 1), (1, -1))], -1)


def _exact_logits(case, seed):
    layers, _, x = _net(case, seed)
    v = x.double()
    for d in layers:
        kind = d["kind"]
        if kind in (bnn.LAYER_INPUT_THRESHOLD, bnn.LAYER_INPUT_GRAY, bnn.LAYER_INPUT_LBP):
            v = _input_bits(d, x).double() * 2 - 1
        elif kind in (bnn.LAYER_FCONV_BINW, bnn.LAYER_BCONV):
            real = kind == bnn.LAYER_FCONV_BINW
            b = _bits(_sums(v, _pm1(d["w"], d["C"]), d["KH"], d["pad"], 0.0 if real else -1.0), d)
            v = (_pool(b) if d["pool"] else b).double() * 2 - 1
        else:
            S = v.reshape(case["batch"], -1) @ _pm1(d["w"], d["K"]).t().contiguous()
            if kind == bnn.LAYER_BFC_LOGITS:
                return S.to(torch.int32)
            v = _bits(S, d).double() * 2 - 1


def exact(case, seed):
    family = case["family"]
    if family == "forward":
        return _exact_logits(case, seed)
    s = _layer_inputs(case, seed)
    if family == "pack":
        # The offset is added in fp32 by definition.
        x = s["x"] if s["offset"] is None else s["x"] + s["offset"]
        return _pack(x > 0)
    if family == "gemm":
        S = _pm1(s["x"], case["K"]) @ _pm1(s["w"], case["K"]).t().contiguous()
    else:
        x = s["x"].double() if family == "fconv" else _pm1(s["x"], case["C"])
        S = _sums(x, _pm1(s["w"], case["C"]), case["k"], case["pad"],
                  0.0 if family == "fconv" else -1.0)
    b = None
    if case["bits"]:
        b = _bits(S, s)
        b = _pack(_pool(b) if case.get("pool") else b)
    if not case["sums"]:
        return None, b
    return (S if family == "fconv" else S.to(torch.int32)), b
