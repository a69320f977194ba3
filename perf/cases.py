"""The work that a user of this library has it do, as cases that can be timed and compared.

A case is one layer of a network under training: the three calls of a convolution with a compressed saved
input ("step": forward + compress, weight and data gradient, and the bias gradient where the layer has a bias),
the weight gradient alone ("dw"), the pooling of an activation alone ("compress"), or a batch normalisation that
compresses at the producer, forward and backward ("norm").  Layers come from the lists of synth.py (ResNet-18 on
CIFAR- and ImageNet-sized maps, ResNet-50, the deep small maps, the single fp32 layer) and from the odd shapes of
the tests.  Inputs follow the recipe of synth.py: post-ReLU activations, normal gradients, Kaiming weights.
"""
import math

import torch

from paper_2409_11902_amd import binding as B

DEV = "cuda:0"
ALGO = {"inflate": B.DW_INFLATE, "auto": B.DW_AUTO}


def _step(name, N, C, K, H, W, R, stride, k, dtype="bf16", bias=0, algo="inflate"):
    return dict(name=name, op="step", N=N, C=C, K=K, H=H, W=W, R=R, stride=stride, k=k, dtype=dtype, bias=bias, algo=algo)


def listed():
    return [
        # the deep small-map pair that the benchmark's headline step is made of: 14 x 14 is the largest
        # matrix-core work of the lists, 7 x 7 has odd maps and ragged pooling tiles
        _step("step 3x3 512-512@14 b256", 256, 512, 512, 14, 14, 3, 1, 2),
        _step("step 3x3 512-512@7 b256", 256, 512, 512, 7, 7, 3, 1, 2),
        # ResNet-18 on ImageNet: the first stage with the coarser tile, and a strided layer kept uncompressed
        _step("step 3x3 64-64@56 b128 k4", 128, 64, 64, 56, 56, 3, 1, 4),
        _step("step 3x3s2 128-256@28 b128 k1", 128, 128, 256, 28, 28, 3, 2, 1),
        # ResNet-50 bottlenecks: the reduction of a wide map and the expansion of an odd one
        _step("step 1x1 256-64@56 b64", 64, 256, 64, 56, 56, 1, 1, 2),
        _step("step 1x1 512-2048@7 b64", 64, 512, 2048, 7, 7, 1, 1, 2),
        # the CIFAR-sized network's last stage: many channels, hardly any pixels
        _step("step 3x3 512-512@4 b128", 128, 512, 512, 4, 4, 3, 1, 2),
        # the small layer in single precision, with a bias: latency and launches count
        _step("step fp32 3x3 16-16@32 b8", 8, 16, 16, 32, 32, 3, 1, 2, dtype="f32", bias=1),
        # nothing divides anything: channels, maps and batch as a pruned network on cropped images has them
        _step("step 3x3 72-100@27x30 b24", 24, 72, 100, 27, 30, 3, 1, 2, bias=1),
        # a weight gradient alone (frozen or first trained layer: no data gradient), the library choosing the form
        dict(name="dw 3x3 256-256@14 b128 auto", op="dw", N=128, C=256, K=256, H=14, W=14, R=3, stride=1, k=2, dtype="bf16",
             bias=0, algo="auto"),
        # pooling of the largest activation of the ResNet-50 list, for callers with a producer of their own
        dict(name="compress 256@56 b64", op="compress", N=64, C=256, H=56, W=56, k=2, dtype="bf16"),
        # batch normalisation with compression at the producer, forward and backward
        dict(name="norm 512@28 b64", op="norm", N=64, C=512, H=28, W=28, k=2, dtype="bf16"),
    ]


# no drawn case costs more than the largest listed one
MAX_FLOPS, MAX_BYTES = 7.0e11, 1.2e8


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng):
    c = _log_int(rng, 16, 2048)
    return c if rng.random() < 0.4 else max(16, (c + 8) // 16 * 16)


def draw(rng):
    op = rng.choice(["step"] * 7 + ["dw", "compress", "norm"])
    H = _log_int(rng, 4, 56)
    W = H if rng.random() < 0.6 else _log_int(rng, 4, 56)
    c = dict(op=op, N=_log_int(rng, 1, 256), C=_channels(rng), H=H, W=W, k=rng.choice([1, 2, 2, 4]), dtype="bf16")
    if op in ("compress", "norm"):
        c["k"] = rng.choice([2, 2, 4])
        while c["N"] * c["C"] * H * W * 2 > MAX_BYTES:
            c["N"] = max(1, c["N"] // 2)
            if c["N"] == 1:
                c["C"] = max(16, c["C"] // 2)
        return c
    c.update(K=_channels(rng), R=rng.choice([1, 3, 3]), stride=rng.choice([1, 1, 1, 2]), bias=rng.choice([0, 0, 1]), algo="inflate")
    if op == "dw":
        c["algo"] = "auto"
    limit = MAX_FLOPS
    if op == "step" and rng.random() < 0.15:
        # single precision serves small layers and checks, not the large lists
        c.update(dtype="f32", C=min(c["C"], 64), K=min(c["K"], 64))
        limit = 2e9
    while c["C"] * c["K"] * c["R"] ** 2 > 512 * 512 * 9:
        c["C" if c["C"] >= c["K"] else "K"] //= 2
    while work(c)["flops"] > limit or c["N"] * max(c["C"], c["K"]) * H * W * 2 > MAX_BYTES:
        if c["N"] > 1:
            c["N"] //= 2
        else:
            c["C" if c["C"] >= c["K"] else "K"] //= 2
    return c


def _elem(case):
    return 4 if case["dtype"] == "f32" else 2


def _out(case, n):
    return (n + 2 * (case["R"] // 2) - case["R"]) // case["stride"] + 1


def work(case):
    N, C, H, W, e = case["N"], case["C"], case["H"], case["W"], _elem(case)
    k = case["k"]
    x, z = N * C * H * W, N * C * -(-H // k) * -(-W // k)
    if case["op"] == "compress":
        return {"bytes": (x + z) * e, "flops": x}
    if case["op"] == "norm":
        # forward: Y in, X', Z' and Z_in out; backward: Z_in and dY in, dX out, the parameters beside them
        return {"bytes": (2 * x + 2 * z) * e + (2 * x + z) * e + 7 * C * 4, "flops": 12 * x}
    K, R = case["K"], case["R"]
    y, w = N * K * _out(case, H) * _out(case, W), K * C * R * R
    gemm = 2 * y * C * R * R
    if case["op"] == "dw":
        return {"bytes": (z + y) * e + w * 4, "flops": gemm}
    # forward: X, W in, Y, Z out; backward: Z, W, dY in, dW (float), dX out; b and db where there is a bias
    nbytes = (x + w + y + z) * e + (z + w + y + x) * e + w * 4
    return {"bytes": nbytes + case["bias"] * K * (e + 4), "flops": 3 * gemm}


# Measured against exact(): 32-bit results 1e-7 to 4e-7, stated ten times wider for sums up to the drawn lengths;
# bfloat16 results 1.7e-3 (the rounding of one store), a gradient from a rounded record 1.4e-3 to 2.7e-3.
# "max": one unit in the last place of bfloat16 is at most 2^-7 of the value.
def tolerance(case):
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 1e-4}
    return {"rel": 7e-3, "max": 2e-2}


def _inputs(case, seed):
    """Seeded inputs of the layer, rounded to the storage type."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    td = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    N, C, H, W = (case[n] for n in ("N", "C", "H", "W"))

    def normal(*shape, std=1.0):
        return torch.randn(*shape, generator=g, device=DEV).mul_(std)

    if case["op"] == "compress":
        return {"X": normal(N, C, H, W).relu_().to(td)}
    if case["op"] == "norm":
        # a convolution's output: every channel with a mean and spread of its own; the statistics are the caller's
        y = (normal(N, C, H, W) * (0.5 + torch.rand(1, C, 1, 1, generator=g, device=DEV)) + normal(1, C, 1, 1, std=0.5)).to(td)
        mean = y.float().mean(dim=(0, 2, 3))
        invstd = (y.float().var(dim=(0, 2, 3), unbiased=False) + 1e-5).rsqrt()
        gamma, beta = 1 + normal(C, std=0.1), normal(C, std=0.1)
        return {"Y": y, "mean": mean, "invstd": invstd, "gamma": gamma, "beta": beta, "dY": normal(N, C, H, W).to(td)}
    K, R = case["K"], case["R"]
    t = {"X": normal(N, C, H, W).relu_().to(td), "W": normal(K, C, R, R, std=math.sqrt(2.0 / (C * R * R))).to(td),
         "dY": normal(N, K, _out(case, H), _out(case, W)).to(td)}
    if case["bias"]:
        t["b"] = normal(K, std=0.1).to(td)
    return t


def _desc(case):
    R = case.get("R", 1)
    return B.make_desc(case["N"], case["C"], case.get("K", case["C"]), case["H"], case["W"], R, R, case.get("stride", 1),
                       case.get("stride", 1), R // 2, R // 2, case["k"], case["k"], dtype=B.F32 if case["dtype"] == "f32" else B.BF16,
                       has_bias=case.get("bias", 0), dw_algo=ALGO[case.get("algo", "inflate")])


def _scratch(d, *ops):
    n = max(B.cac_workspace_size(d, op) for op in ops)
    return torch.empty((n + 15) // 16 * 16, dtype=torch.uint8, device=DEV) if n else None


def prepare(case, seed):
    s = {"op": case["op"], "d": _desc(case), **_inputs(case, seed)}
    d = s["d"]
    hp, wp, _, _ = B.cac_pooled_shape(d)
    first = s["Y"] if case["op"] == "norm" else s["X"]
    td = first.dtype

    def out(*shape, dtype=td):
        return torch.empty(*shape, dtype=dtype, device=DEV)

    s["Z"] = out(case["N"], case["C"], hp, wp)
    if case["op"] == "compress":
        return s
    if case["op"] == "norm":
        s["scale"] = s["gamma"] * s["invstd"]
        s["shift"] = s["beta"] - s["mean"] * s["scale"]
        s.update(Xn=torch.empty_like(first), Zn=torch.empty_like(s["Z"]), dX=torch.empty_like(first),
                 dgamma=torch.empty_like(s["gamma"]), dbeta=torch.empty_like(s["beta"]), ws=_scratch(d, B.OP_BN_BWD))
        return s
    s["dW"] = out(*s["W"].shape, dtype=torch.float32)
    if case["op"] == "dw":
        B.cac_compress(d, s.pop("X"), s["Z"])  # the record that the forward pass has left
        s["ws"] = _scratch(d, B.OP_BWD_WEIGHT_COMPRESSED)
        return s
    s.update(Yo=torch.empty_like(s["dY"]), dX=torch.empty_like(first), ws=_scratch(d, B.OP_FWD_AND_COMPRESS, B.OP_BWD_WEIGHT_AND_DATA))
    if case["bias"]:
        s["db"] = out(case["K"], dtype=torch.float32)
    return s


def run(s):
    d = s["d"]
    if s["op"] == "compress":
        B.cac_compress(d, s["X"], s["Z"])
        return {"Z": s["Z"]}
    if s["op"] == "norm":
        B.cac_bn_relu_fwd_compress(d, s["Y"], s["scale"], s["shift"], s["Xn"], s["Zn"], s["Z"])
        B.cac_bn_bwd_compressed(d, s["Z"], s["dY"], s["mean"], s["invstd"], s["gamma"], s["dgamma"], s["dbeta"], s["dX"], s["ws"])
        return {"X": s["Xn"], "Z": s["Zn"], "Zin": s["Z"], "dgamma": s["dgamma"], "dbeta": s["dbeta"], "dX": s["dX"]}
    if s["op"] == "dw":
        B.conv_bwd_weight_compressed(d, s["Z"], s["dY"], s["dW"], s["ws"])
        return {"dW": s["dW"]}
    B.conv_fwd_and_compress(d, s["X"], s["W"], s.get("b"), s["Yo"], s["Z"], s["ws"])
    B.conv_bwd_weight_and_data(d, s["Z"], s["W"], s["dY"], s["dW"], s["dX"], s["ws"])
    r = {"Y": s["Yo"], "Z": s["Z"], "dW": s["dW"], "dX": s["dX"]}
    if "db" in s:
        B.conv_bwd_bias(d, s["dY"], s["db"])
        r["db"] = s["db"]
    return r


def _pool(x, k):
    """Means over the k x k tiles, a ragged tile over the elements that it has."""
    H, W = x.shape[2:]
    x = torch.nn.functional.pad(x, (0, -W % k, 0, -H % k))
    n = torch.nn.functional.pad(torch.ones(1, 1, H, W, dtype=x.dtype, device=x.device), (0, -W % k, 0, -H % k))
    tiles = [t.unflatten(3, (-1, k)).unflatten(2, (-1, k)).sum(dim=(3, 5)) for t in (x, n)]
    return tiles[0] / tiles[1]


def _inflate(z, k, H, W):
    return z.repeat_interleave(k, 2).repeat_interleave(k, 3)[:, :, :H, :W]


def exact(case, seed):
    t = {n: v.double() for n, v in _inputs(case, seed).items()}
    N, C, H, W, k = (case[n] for n in ("N", "C", "H", "W", "k"))
    if case["op"] == "compress":
        return {"Z": _pool(t["X"], k)}
    if case["op"] == "norm":
        def per(v):
            return v.view(1, C, 1, 1)
        scale = t["gamma"] * t["invstd"]
        shift = t["beta"] - t["mean"] * scale
        xn = (t["Y"] * per(scale) + per(shift)).relu()
        zin = _pool(t["Y"], k)
        xhat = (_inflate(zin, k, H, W) - per(t["mean"])) * per(t["invstd"])
        dbeta, dgamma, m = t["dY"].sum(dim=(0, 2, 3)), (t["dY"] * xhat).sum(dim=(0, 2, 3)), N * H * W
        dx = per(scale) * (t["dY"] - per(dbeta) / m - xhat * per(dgamma) / m)
        return {"X": xn, "Z": _pool(xn, k), "Zin": zin, "dgamma": dgamma, "dbeta": dbeta, "dX": dx}
    K, R, st, pad = case["K"], case["R"], case["stride"], case["R"] // 2
    P, Q = _out(case, H), _out(case, W)

    def padded(x):
        return torch.nn.functional.pad(x, (pad, pad, pad, pad))

    def tap(x, r, s):  # the pixels that tap (r, s) meets, as [channel][image, row, column]
        v = x[:, :, r:r + (P - 1) * st + 1:st, s:s + (Q - 1) * st + 1:st]
        return v.permute(1, 0, 2, 3).reshape(x.shape[1], -1)

    taps = [(r, s) for r in range(R) for s in range(R)]
    z = _pool(t["X"], k)
    dym = t["dY"].permute(1, 0, 2, 3).reshape(K, -1)
    xh = padded(_inflate(z, k, H, W))
    dw = torch.empty(K, C, R, R, dtype=torch.float64, device=DEV)
    for r, s in taps:
        dw[:, :, r, s] = dym @ tap(xh, r, s).t()
    if case["op"] == "dw":
        return {"dW": dw}
    xp = padded(t["X"])
    y = torch.zeros(K, N * P * Q, dtype=torch.float64, device=DEV)
    dxp = torch.zeros_like(xp)
    for r, s in taps:
        y += t["W"][:, :, r, s] @ tap(xp, r, s)
        part = (t["W"][:, :, r, s].t() @ dym).view(C, N, P, Q).permute(1, 0, 2, 3)
        dxp[:, :, r:r + (P - 1) * st + 1:st, s:s + (Q - 1) * st + 1:st] += part
    y = y.view(K, N, P, Q).permute(1, 0, 2, 3)
    if case["bias"]:
        y = y + t["b"].view(1, K, 1, 1)
    out = {"Y": y, "Z": z, "dW": dw, "dX": dxp[:, :, pad:pad + H, pad:pad + W]}
    if case["bias"]:
        out["db"] = t["dY"].sum(dim=(0, 2, 3))
    return out
