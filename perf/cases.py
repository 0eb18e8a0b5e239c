"""Timed cases of the 1-bit FQT layers, with reference results in 64 bits.

A case is one pass through the public entry points: a layer backward (fqt_layer_backward), a
binary forward (fqt_binary_forward) or a training pass of one binary layer module (forward and
autograd backward).  Shapes are those of the VGG-16 and ResNet-18 layers, the GEMM sweep and the
small linear layer the benchmark runs; draw() gives more of the same ranges, ragged ones among
them.  Inputs follow the repository's synthetic recipes: X, W ~ N(0, 1), dY with uneven group
ranges (per-sample or per-channel lognormal scale, Student-t).
"""
import math

import numpy as np
import torch
import torch.nn.functional as F

from paper_2408_14267_amd import fqt, train
from paper_2408_14267_amd.workloads import LayerShape

DEV = "cuda"
BERNOULLI, OFF = 0, 2


def _conv(name, op, N, C, D, H, W, k, s, p, dtype, bits, recipe, agp=BERNOULLI):
    return dict(name=name, op=op, kind="conv2d", N=N, C=C, D=D, H=H, W=W, k=k, s=s, p=p,
                dtype=dtype, bits=bits, recipe=recipe, agp=agp)


def _linear(name, op, N, C, D, dtype, bits, recipe, agp=BERNOULLI):
    return dict(name=name, op=op, kind="linear", N=N, C=C, D=D, H=1, W=1, k=1, s=1, p=0,
                dtype=dtype, bits=bits, recipe=recipe, agp=agp)


def listed():
    return [
        # The smallest layer of the suite: launches and latency are all it costs.
        _linear("bwd_linear_32x256x128", "backward", 32, 256, 128, "f32", 2, "sample_lognormal"),
        # The benchmark layer: VGG-16 at 32 px, 3x3 256 -> 256 on 8x8 maps, batch 128.
        _conv("bwd_conv_256_8x8", "backward", 128, 256, 256, 8, 8, 3, 1, 1, "f32", 4,
              "sample_lognormal"),
        # A down-sampling layer: the first 3x3/2 convolution of ResNet-18 at 224 px.
        _conv("bwd_conv_64_128_56x56_s2", "backward", 64, 64, 128, 56, 56, 3, 2, 1, "f32", 4,
              "student_t"),
        # The largest layer: VGG-16 at 224 px, conv2, bf16 activations and gradients.
        _conv("bwd_conv_64_224x224_bf16", "backward", 64, 64, 64, 224, 224, 3, 1, 1, "bf16", 2,
              "channel_lognormal"),
        # A deep, contraction-heavy layer: VGG-16 at 224 px, conv9.
        _conv("bwd_conv_512_28x28_bf16", "backward", 64, 512, 512, 28, 28, 3, 1, 1, "bf16", 2,
              "channel_lognormal"),
        # Odd maps: the last stage of ResNet-18 at 224 px has 7x7 pixels.
        _conv("bwd_conv_512_7x7", "backward", 64, 512, 512, 7, 7, 3, 1, 1, "f32", 4, "student_t"),
        # The largest fully connected layer: VGG-16 at 224 px, fc6.
        _linear("bwd_linear_25088_4096_bf16", "backward", 64, 25088, 4096, "bf16", 2,
                "channel_lognormal"),
        # A point of the binary GEMM sweep: 1-bit codes of every group (no pruning).
        _linear("bwd_linear_4608x4096x4096_b1", "backward", 4608, 4096, 4096, "f32", 1,
                "sample_lognormal", OFF),
        # Forward of the benchmark layer.
        _conv("fwd_conv_256_8x8", "forward", 128, 256, 256, 8, 8, 3, 1, 1, "f32", 4, "student_t"),
        # Forward of a large layer: VGG-16 at 224 px, conv4.
        _conv("fwd_conv_128_112x112_bf16", "forward", 64, 128, 128, 112, 112, 3, 1, 1, "bf16", 2,
              "student_t"),
        # Forward of fc6.
        _linear("fwd_linear_25088_4096_bf16", "forward", 64, 25088, 4096, "bf16", 2, "student_t"),
        # Training pass of one layer module: ResNet-18 at 224 px, first stage.
        _conv("train_conv_64_56x56", "train", 64, 64, 64, 56, 56, 3, 1, 1, "f32", 4, "student_t"),
    ]


# Bounds of a drawn case: elements of X and of dY, of W, and multiply-accumulates of a product.
MAX_MAP, MAX_W, MAX_MACS = 60_000_000, 60_000_000, 60_000_000_000


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        op = rng.choice(["backward"] * 4 + ["forward"] * 2 + ["train"] * 2)
        dtype = "f32" if op == "train" else rng.choice(["f32", "bf16"])
        bits = rng.choice([1, 2, 2, 3, 4, 4, 8])
        agp = OFF if rng.random() < 0.15 else BERNOULLI
        recipe = rng.choice(["sample_lognormal", "channel_lognormal", "student_t"])
        if rng.random() < 0.3:
            c = _linear(None, op, logint(16, 4608), logint(64, 25088), logint(10, 8192), dtype,
                        bits, recipe, agp)
        else:
            k = rng.choice([1, 3, 3, 3, 3, 5, 7])
            s = 2 if rng.random() < 0.25 else 1
            H = rng.choice([4, 7, 8, 14, 16, 28, 32, 56, 112, logint(4, 224)])
            W = H if rng.random() < 0.8 else max(4, H + rng.randint(-3, 3))
            C = rng.choice([3, 16, 64, 128, 256, 512, logint(3, 512)])
            D = rng.choice([16, 64, 128, 256, 512, logint(8, 512)])
            c = _conv(None, op, logint(1, 256), C, D, H, W, k, s, k // 2, dtype, bits, recipe, agp)
        del c["name"]
        L = _shape(c)
        R = L.N * L.Ho * L.Wo
        K = L.C * L.kh * L.kw
        if (L.N * L.C * L.H * L.W <= MAX_MAP and R * L.D <= MAX_MAP and L.D * K <= MAX_W and
                R * L.D * K <= MAX_MACS and R * K <= 4 * MAX_MACS // 64):
            return c


def _shape(c):
    return LayerShape("layer", c["kind"], c["N"], c["C"], c["D"], c["H"], c["W"], c["k"], c["k"],
                      c["s"], c["s"], c["p"], c["p"])


def _inputs(c, seed):
    """X, W, dY and Gamma of the case on the device, made from the seed alone."""
    L = _shape(c)
    g = torch.Generator(device=DEV).manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=g, device=DEV)

    x, w, dy = normal(*L.x_shape), normal(*L.w_shape), normal(*L.dy_shape)
    ones = (1,) * (dy.dim() - 2)
    if c["recipe"] == "sample_lognormal":
        dy *= torch.exp(2.0 * normal(L.N)).view(L.N, 1, *ones)
    elif c["recipe"] == "channel_lognormal":
        dy *= torch.exp(1.5 * normal(L.D)).view(1, L.D, *ones)
    else:                                   # Student-t with 3 degrees of freedom
        chi = normal(*L.dy_shape).square_()
        for _ in range(2):
            chi += normal(*L.dy_shape).square_()
        dy /= chi.div_(3.0).sqrt_()
    gamma = 0.5 + torch.rand(L.D, generator=g, device=DEV)
    if c["op"] != "backward":
        gamma /= math.sqrt(w[0].numel())
    if c["dtype"] == "bf16":
        x, dy = x.bfloat16(), dy.bfloat16()
    return L, x, w, dy, gamma


def prepare(case, seed):
    L, x, w, dy, gamma = _inputs(case, seed)
    if case["op"] == "train":
        if case["kind"] == "linear":
            mod = train.BinaryLinear(L.C, L.D, bits=case["bits"], agp_mode=case["agp"], layer_id=1,
                                     seed=seed)
        else:
            mod = train.BinaryConv2d(L.C, L.D, L.kh, L.sh, L.ph, bits=case["bits"],
                                     agp_mode=case["agp"], layer_id=1, seed=seed)
        mod = mod.to(DEV)
        with torch.no_grad():
            mod.weight.copy_(w)
            mod.gamma.copy_(gamma)
        return dict(op="train", mod=mod, x=x.requires_grad_(True), dy=dy)
    dt = fqt.dtype_code(case["dtype"])
    desc = fqt.layer_desc(L, dy_dtype=dt, x_dtype=dt, dx_dtype=dt)
    if case["op"] == "forward":
        return dict(op="forward", desc=desc, x=x, w=w, gamma=gamma, y=torch.empty_like(dy),
                    ws=fqt.workspace(desc, None, fqt.FQT_WS_FORWARD))
    cfg = fqt.quant_cfg(case["bits"], case["agp"], seed, 0, 1)
    return dict(op="backward", desc=desc, cfg=cfg, x=x, w=w, dy=dy, dx=torch.empty_like(x),
                dw=torch.empty_like(w), ws=fqt.workspace(desc, cfg))


def run(state):
    s = state
    if s["op"] == "backward":
        fqt.fqt_layer_backward(s["desc"], s["cfg"], s["x"], s["w"], s["dy"], s["dx"], s["dw"],
                               s["ws"])
        return {"dx": s["dx"], "dw": s["dw"]}
    if s["op"] == "forward":
        fqt.fqt_binary_forward(s["desc"], s["x"], s["w"], s["gamma"], s["y"], None, s["ws"])
        return {"y": s["y"]}
    y = s["mod"](s["x"])
    dx, dw, dgamma = torch.autograd.grad(y, (s["x"], s["mod"].weight, s["mod"].gamma), s["dy"])
    return {"y": y, "dx": dx, "dw": dw, "dgamma": dgamma}


def work(case):
    L = _shape(case)
    e = 2 if case["dtype"] == "bf16" else 4
    x, w, y = L.N * L.C * L.H * L.W, L.D * L.C * L.kh * L.kw, L.N * L.D * L.Ho * L.Wo
    product = 2.0 * L.binary_macs()
    # Pruning keeps about 1/b of the groups of each product.
    kept = 1.0 if case["agp"] == OFF else 1.0 / case["bits"]
    fwd_bytes, bwd_bytes = e * (x + y) + 4 * (w + L.D), e * (2 * x + y) + 8 * w
    if case["op"] == "forward":
        return {"bytes": fwd_bytes, "flops": product}
    if case["op"] == "backward":
        return {"bytes": bwd_bytes, "flops": 2 * kept * product}
    return {"bytes": fwd_bytes + bwd_bytes + 8 * L.D, "flops": (1 + 2 * kept) * product}


def tolerance(case):
    # The products are exact integers; what rounds is the rescale S * I + Z' * c of each output.
    # In float32 its two terms cancel where a group's range is far from zero: up to 1.3e-5 of dW
    # against 64 bits, below 1e-6 elsewhere; a bfloat16 output rounds by 1.7e-3.
    if case["dtype"] == "bf16":
        return {"rel": 7e-3, "max": 2e-2}
    return {"rel": 5e-5, "max": 2e-3}


# ----------------------------------------------------------------------------- 64-bit reference

M32 = 0xFFFFFFFF


def _mulhilo(m, a):
    """High and low 32 bits of m * a for a constant m and a tensor a of 32-bit values (int64)."""
    lo = (a & 0xFFFF) * m
    hi = (a >> 16) * m + (lo >> 16)
    return hi >> 16, ((hi & 0xFFFF) << 16) | (lo & 0xFFFF)


def _philox(blk, stream, seed):
    """Philox4x32-10 words of the blocks `blk` (int64 tensor, below 2^32) for layer 1, step 0."""
    c = [blk, torch.full_like(blk, stream << 30), torch.ones_like(blk), torch.zeros_like(blk)]
    k0, k1 = seed & M32, (seed >> 32) & M32
    for _ in range(10):
        h0, l0 = _mulhilo(0xD2511F53, c[0])
        h1, l1 = _mulhilo(0xCD9E8D57, c[2])
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c


def _select(lo, hi, bits, agp, stream, seed):
    """Kept mask, float64 scale and offset, float32 zero point and B / R of one group set."""
    B, G = (1 << bits) - 1, lo.numel()
    z = (lo.float().cpu().numpy() + np.float32(0)).astype(np.float32)
    r = (hi.float().cpu().numpy() - z).astype(np.float32)
    with np.errstate(divide="ignore"):
        inv = np.where(r > 0, np.float32(B) / r, np.float32(0)).astype(np.float32)
    keep, p = np.ones(G, bool), np.ones(G)
    if agp != OFF:
        rmax = float(r.max())
        w = np.floor(np.ldexp(r.astype(np.float64) / (rmax if rmax > 0 else 1.0), 40)).astype(np.int64)
        sat, W = np.zeros(G, bool), int(w.sum())
        while True:                          # groups whose probability would pass 1 are capped
            new = ~sat & (w > 0) & ((G - bits * int(sat.sum())) * w >= bits * W)
            if not new.any():
                break
            sat |= new
            W -= int(w[new].sum())
        A = G - bits * int(sat.sum())
        words = torch.stack(_philox(torch.arange((G + 3) // 4), stream, seed), 1).reshape(-1)[:G]
        u = words.tolist()
        for i in range(G):
            if sat[i]:
                continue
            aw = A * int(w[i]) if A > 0 else 0
            p[i] = aw / (bits * W) if W > 0 else 0.0
            keep[i] = W > 0 and u[i] * bits * W < aw << 32
    with np.errstate(divide="ignore", invalid="ignore"):
        S = np.where(keep, r.astype(np.float64) / (B * p), 0.0)
        Z = np.where(keep, z.astype(np.float64) / p, 0.0)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).to(DEV) for a in (keep, S, Z, z, inv)]
    return dict(zip(("keep", "S", "Z", "z", "inv"), dev))


def _codes(v, u24):
    q = torch.floor(v)
    return (q + (u24 < (v - q) * 16777216.0)).double()


def _sign(t):
    return torch.where(t > 0, 1.0, -1.0).double()


def _backward64(L, x, w, g, bits, agp, seed):
    """dX and dW in float64 from the float32 stochastic-rounding codes of g [N][D][P]."""
    N, D, P, K = L.N, L.D, L.Ho * L.Wo, L.C * L.kh * L.kw
    g = g.reshape(N, D, P)
    s = _select(g.amin((1, 2)), g.amax((1, 2)), bits, agp, 1, seed)
    c = _select(g.amin((0, 2)), g.amax((0, 2)), bits, agp, 2, seed)
    sw = _sign(w).reshape(D, K)
    dx = torch.zeros(N, L.C, L.H, L.W, dtype=torch.float64, device=DEV)
    I = torch.zeros(D, K, dtype=torch.float64, device=DEV)
    T = torch.zeros(K, dtype=torch.float64, device=DEV)
    B = float((1 << bits) - 1)
    step = max(1, int(4e7 // (P * max(K, D))))
    for n0 in range(0, N, step):
        n1 = min(N, n0 + step)
        n = n1 - n0
        gv = g[n0:n1].float() + 0.0
        e0, e1 = n0 * D * P, n1 * D * P
        b0 = e0 // 4
        u = torch.stack(_philox(torch.arange(b0, (e1 + 3) // 4, device=DEV), 0, seed), 1)
        u = (u.reshape(-1)[e0 - 4 * b0:e1 - 4 * b0] >> 8).float().view(n, D, P)

        def rounded(p, dims):
            z, inv, keep = (p[k][dims] for k in ("z", "inv", "keep"))
            return _codes(((gv - z) * inv).clamp(0.0, B), u) * keep

        qs = rounded({k: s[k][n0:n1] for k in s}, (slice(None), None, None))
        qc = rounded(c, (None, slice(None), None))
        xs = F.pad(_sign(x[n0:n1]).reshape(n, L.C, L.H, L.W), (L.pw, L.pw, L.ph, L.ph), value=-1.0)
        cols = F.unfold(xs, (L.kh, L.kw), stride=L.stride).permute(1, 0, 2).reshape(K, n * P)
        I += qc.permute(1, 0, 2).reshape(D, n * P) @ cols.t()
        T += cols.sum(1)
        rows = sw.t() @ (s["S"][n0:n1, None, None] * qs + s["Z"][n0:n1, None, None]).permute(
            1, 0, 2).reshape(D, n * P)
        rows = rows.view(K, n, P).permute(1, 0, 2).contiguous()
        dx[n0:n1] = F.fold(rows, (L.H, L.W), (L.kh, L.kw), padding=L.pad, stride=L.stride)
    dw = c["S"][:, None] * I + c["Z"][:, None] * T
    return dx.reshape(L.x_shape), dw.reshape(L.w_shape)


def _forward64(L, x, w):
    """The integer product of the binary forward in float64, [N][D][P]."""
    N, D, P, K = L.N, L.D, L.Ho * L.Wo, L.C * L.kh * L.kw
    sw, out = _sign(w).reshape(D, K), torch.empty(N, D, P, dtype=torch.float64, device=DEV)
    step = max(1, int(4e7 // (P * max(K, D))))
    for n0 in range(0, N, step):
        n1 = min(N, n0 + step)
        xs = _sign(x[n0:n1]).reshape(n1 - n0, L.C, L.H, L.W)
        xs = F.pad(xs, (L.pw, L.pw, L.ph, L.ph), value=-1.0)
        cols = F.unfold(xs, (L.kh, L.kw), stride=L.stride).permute(1, 0, 2).reshape(K, -1)
        out[n0:n1] = (sw @ cols).view(D, n1 - n0, P).permute(1, 0, 2)
    return out


def exact(case, seed):
    L, x, w, dy, gamma = _inputs(case, seed)
    if case["op"] == "backward":
        dx, dw = _backward64(L, x, w, dy, case["bits"], case["agp"], seed)
        return {"dx": dx, "dw": dw}
    I = _forward64(L, x, w)
    y = (I * gamma.double()[:, None]).reshape(dy.shape)
    if case["op"] == "forward":
        return {"y": y}
    g = dy * gamma.view(1, -1, *(1,) * (dy.dim() - 2))
    dx, dw = _backward64(L, x, w, g, case["bits"], case["agp"], seed)
    dgamma = (dy.reshape(I.shape).double() * I).sum((0, 2))
    return {"y": y, "dx": dx * (x.abs() <= 1), "dw": dw, "dgamma": dgamma}
