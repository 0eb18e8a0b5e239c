"""The layer backward (its own code kernels and operand formats) against the same layer through
the separate entries: quantize, the sign packers and the products launch, bit for bit."""
import sys

import pytest

from paper_2408_14267_amd.workloads import LayerShape

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _conv(N, C, D, H, W, k, s, p):
    return LayerShape("c", "conv2d", N, C, D, H, W, k, k, s, s, p, p)


# (layer, bits, agp, dtype, spread of the group ranges)
CASES = [
    # Lines of 256 rows: whole samples, tiles that meet several samples (100, 12 and 4 pixels a
    # sample), ragged channels and rows, every code width; nearly all groups pruned (spread 6).
    (_conv(64, 8, 130, 32, 32, 3, 1, 1), 4, 0, "f32", 1.5),
    (_conv(250, 5, 170, 10, 10, 3, 1, 1), 2, 0, "bf16", 1.5),
    (_conv(701, 3, 520, 3, 4, 3, 1, 1), 8, 0, "f32", 1.0),
    (_conv(1001, 4, 1020, 2, 2, 3, 1, 1), 3, 0, "bf16", 1.5),
    (_conv(70, 6, 65, 40, 36, 3, 1, 1), 1, 2, "f32", 1.0),
    (_conv(64, 8, 128, 64, 64, 3, 2, 1), 1, 0, "bf16", 1.5),
    (_conv(96, 8, 128, 28, 28, 3, 1, 1), 6, 0, "f32", 6.0),
    (_conv(66, 9, 70, 34, 34, 1, 1, 0), 2, 1, "f32", 2.0),
    # The tap form of dW (3 x 3, at least 768 words): both code formats, rows whose length is and
    # is not a multiple of 32, a ragged last word, one to three channel and slot blocks.
    (_conv(65, 40, 70, 30, 26, 3, 1, 1), 2, 0, "bf16", 1.5),
    (_conv(13, 33, 40, 66, 62, 3, 1, 1), 8, 2, "f32", 1.0),
    (_conv(2, 29, 20, 224, 224, 3, 1, 1), 2, 2, "f32", 1.0),
    (_conv(13, 70, 200, 64, 64, 3, 1, 1), 1, 2, "bf16", 1.0),
    (_conv(13, 65, 150, 64, 64, 3, 1, 1), 3, 2, "f32", 1.0),
    (_conv(800, 27, 80, 1, 64, 3, 1, 1), 5, 0, "f32", 1.0),
    (_conv(2, 23, 20, 224, 224, 3, 1, 1), 2, 2, "f32", 1.0),     # (too few channels for it)
    # Linear layers of few rows (dW bound by its stores), dX from W itself where W has the channels
    # and dW a launch of its own, else from packed signs: one, two and four row tiles, ragged D and
    # C, b = 8, the many-group selection.
    (LayerShape("fc", "linear", 20, 2050, 1030), 3, 0, "f32", 1.5),
    (LayerShape("fc", "linear", 64, 4096, 2600), 2, 0, "bf16", 1.5),
    (LayerShape("fc", "linear", 128, 1026, 2050), 8, 0, "f32", 1.0),
    (LayerShape("fc", "linear", 65, 6000, 1000), 1, 2, "f32", 1.0),
    (LayerShape("fc", "linear", 64, 2051, 2100), 4, 0, "f32", 1.5),
    (LayerShape("fc", "linear", 33, 3000, 1500), 4, 1, "bf16", 3.0),
    (LayerShape("fc", "linear", 20, 8198, 1030), 3, 0, "f32", 1.5),
    (LayerShape("fc", "linear", 128, 8194, 1100), 8, 0, "f32", 1.0),
    (LayerShape("fc", "linear", 65, 9000, 600), 1, 2, "bf16", 1.0),
    (LayerShape("fc", "linear", 33, 5000, 1500), 4, 1, "bf16", 3.0),
    # Few rows and so many outputs that the register tiles would take them: dX from W itself reads
    # byte codes also for b <= 2.
    (LayerShape("fc", "linear", 128, 65472, 18), 2, 0, "f32", 1.5),
    (LayerShape("fc", "linear", 128, 65536, 18), 2, 0, "f32", 1.5),
    (LayerShape("fc", "linear", 100, 65536, 70), 1, 2, "bf16", 1.0),
    (LayerShape("fc", "linear", 64, 131072, 16), 2, 0, "f32", 1.5),
    # Large linear layers: dX with the channels along the lanes and nibble operands, dW from
    # nibble codes (b <= 2) over ragged words, W packed by row passes.
    (LayerShape("fc", "linear", 4100, 4100, 1100), 1, 2, "f32", 1.0),
    (LayerShape("fc", "linear", 2050, 8196, 2050), 2, 0, "bf16", 1.5),
    (LayerShape("fc", "linear", 2600, 6500, 1026), 4, 0, "f32", 1.5),
    (LayerShape("fc", "linear", 530, 2048, 2052), 2, 0, "f32", 1.5),
    (LayerShape("fc", "linear", 513, 2050, 2051), 1, 2, "f32", 1.0),
    # Register-tile dX of convolutions: 25 taps, D above 2048, stride 2, one channel tile.
    (_conv(50, 40, 16, 60, 60, 5, 1, 2), 2, 2, "f32", 1.0),
    (_conv(300, 40, 2112, 16, 16, 3, 1, 1), 2, 0, "f32", 1.0),   # (just too few kept samples)
    (_conv(330, 40, 2112, 16, 16, 3, 1, 1), 2, 0, "f32", 1.0),
    (_conv(90, 40, 20, 75, 75, 3, 2, 1), 1, 2, "bf16", 1.0),
    (_conv(90, 20, 70, 57, 57, 3, 1, 1), 8, 0, "f32", 1.0),
    # Many dW blocks of pruned slots: after the dX blocks in the in-block reduction of up to 64 words
    # and of more, before them where dX has more tiles and with split partials; a set where every
    # channel may be kept.
    (_conv(40, 512, 300, 7, 7, 3, 1, 1), 8, 0, "f32", 1.5),
    (_conv(100, 256, 600, 7, 7, 3, 1, 1), 8, 0, "f32", 1.5),
    (_conv(100, 512, 300, 7, 7, 3, 1, 1), 8, 0, "f32", 1.5),
    (_conv(40, 64, 300, 28, 28, 3, 1, 1), 8, 0, "bf16", 1.5),
    (_conv(40, 512, 300, 7, 7, 3, 1, 1), 4, 2, "f32", 1.0),
    (LayerShape("fc", "linear", 4800, 2050, 900), 3, 0, "f32", 1.5),     # after register tiles
    # Register tiles of a linear layer with few live waves, and the split form just below the line.
    (LayerShape("fc", "linear", 2050, 4100, 130), 8, 0, "bf16", 1.0),
    (LayerShape("fc", "linear", 1540, 4100, 130), 6, 0, "f32", 1.0),
]


@pytest.mark.parametrize("layer,bits,agp,dtype,spread", CASES)
def test_layer_matches_the_entries(layer, bits, agp, dtype, spread):
    from paper_2408_14267_amd import fqt
    print(f"[gpu layer codes] {layer} b={bits} agp={agp} {dtype}", flush=True)
    sys.stdout.flush()
    g = torch.Generator(device="cuda").manual_seed(8)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda")

    ones = (1,) * (len(layer.dy_shape) - 2)
    dy = normal(*layer.dy_shape) * torch.exp(spread * normal(layer.N)).view(layer.N, 1, *ones)
    dy = (dy * torch.exp(spread * normal(layer.D)).view(1, layer.D, *ones)).to(td)
    x, w = normal(*layer.x_shape).to(td), normal(*layer.w_shape)
    dt = fqt.dtype_code(dtype)
    desc = fqt.layer_desc(layer, dt, dt, fqt.FQT_F32, dt)
    cfg = fqt.quant_cfg(bits, agp, 17, 3, 2)
    q = fqt.QGrad(desc, cfg)
    fqt.fqt_agp_scq_quantize(desc, cfg, dy, q, fqt.workspace(desc, cfg, fqt.FQT_WS_QUANTIZE))
    K, R = layer.C * layer.kh * layer.kw, layer.N * layer.Ho * layer.Wo
    xs = torch.empty((R + 63) // 64 * K, dtype=torch.int64, device="cuda")
    wsb = torch.empty(K * 64 * ((layer.D + 63) // 64), dtype=torch.int8, device="cuda")
    wsum = torch.empty(K, dtype=torch.int32, device="cuda")
    fqt.fqt_pack_input_signs(desc, x, xs)
    fqt.fqt_pack_weight_signs(desc, w, wsb, wsum)
    dx, dw = torch.empty_like(x), torch.empty_like(w)
    fqt.fqt_binary_products(desc, cfg, q, xs, wsb, wsum, dx, dw,
                            fqt.workspace(desc, cfg, fqt.FQT_WS_GEMM_DW))
    ws = torch.full((fqt.fqt_workspace_size(desc, cfg),), 0xAB, dtype=torch.uint8, device="cuda")
    fqt.fqt_workspace_init(ws)
    dx2, dw2 = torch.full_like(x, 7.0), torch.full_like(w, 7.0)
    for _ in range(2):
        fqt.fqt_layer_backward(desc, cfg, x, w, dy, dx2, dw2, ws)
        torch.cuda.synchronize()
        assert torch.equal(dx2, dx), "dX"
        assert torch.equal(dw2, dw), "dW"
    assert torch.count_nonzero(dw).item() > 0


@pytest.mark.parametrize("N,D,H,W,dtype", [
    (31, 261, 16, 16, "bf16"),     # a last block whose waves lie past the last channel
    (3, 1, 32, 33, "f32"), (2, 6, 20, 13, "f32"), (1, 1024, 16, 17, "f32"), (1024, 5, 16, 16, "bf16"),
    (2, 65, 112, 112, "f32"),      # planes in segments, a ragged last batch
    (700, 130, 16, 18, "f32"),     # several channels per wave
])
def test_line_statistics(N, D, H, W, dtype):
    """Without AGP the offsets are the groups' minima and the scales their ranges over B, exactly."""
    from paper_2408_14267_amd import fqt
    layer = LayerShape("c", "conv2d", N, 1, D, H, W)
    print(f"[gpu layer codes] statistics {layer} {dtype}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(9)
    dy = torch.randn(layer.dy_shape, generator=g, device="cuda") + 0.5
    if dtype == "bf16":
        dy = dy.to(torch.bfloat16)
    desc, cfg = fqt.layer_desc(layer, fqt.dtype_code(dtype)), fqt.quant_cfg(2, fqt.FQT_AGP_OFF)
    q, ws = fqt.QGrad(desc, cfg), fqt.workspace(desc, cfg, fqt.FQT_WS_QUANTIZE)
    y = dy.float()
    for _ in range(2):                                  # (the merged keys are left zero)
        fqt.fqt_agp_scq_quantize(desc, cfg, dy, q, ws)
        torch.cuda.synchronize()
        for dims, offset, scale in (((1, 2, 3), q.psq_offset, q.psq_scale), ((0, 2, 3), q.pcq_offset, q.pcq_scale)):
            lo, hi = y.amin(dims), y.amax(dims)
            assert torch.equal(offset, lo) and torch.equal(scale, ((hi - lo).double() / 3).float())


# Register tiles of dX: two groups of taps, strides and paddings that differ by direction, one and two
# channel tiles, D past the f16 line sums, b = 8's bias, a ragged last tile.
TILES = [
    (LayerShape("c", "conv2d", 20, 40, 33, 48, 48, 7, 7, 1, 1, 3, 3), 2, 2),
    (LayerShape("c", "conv2d", 80, 9, 70, 61, 45, 5, 3, 2, 3, 2, 0), 3, 0),
    (LayerShape("c", "conv2d", 60, 9, 70, 45, 61, 8, 8, 3, 2, 0, 4), 8, 2),
    (LayerShape("c", "conv2d", 110, 70, 20, 40, 52, 3, 3, 2, 2, 1, 1), 8, 0),
    (LayerShape("c", "conv2d", 48, 200, 2100, 16, 16, 2, 2, 1, 1, 1, 1), 1, 2),
    (LayerShape("c", "conv2d", 96, 40, 65, 30, 30, 1, 1, 2, 2, 0, 0), 4, 2),
]


@pytest.mark.parametrize("layer,bits,agp", TILES)
def test_register_tiles_against_fold(layer, bits, agp):
    """dX of the entry and of the layer, bit for bit, against the float64 product of the byte codes and
    the signs, folded, and rescaled in float32 as the method states it."""
    from paper_2408_14267_amd import fqt
    print(f"[gpu layer codes] tiles {layer} b={bits} agp={agp}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(12)
    x, w, dy = (torch.randn(s, generator=g, device="cuda") for s in (layer.x_shape, layer.w_shape, layer.dy_shape))
    desc, cfg = fqt.layer_desc(layer), fqt.quant_cfg(bits, agp, 17, 3, 2)
    q = fqt.QGrad(desc, cfg)
    fqt.fqt_agp_scq_quantize(desc, cfg, dy, q, fqt.workspace(desc, cfg, fqt.FQT_WS_QUANTIZE))
    C, D, P, K = layer.C, layer.D, layer.Ho * layer.Wo, layer.C * layer.kh * layer.kw
    Wd = (D + 63) // 64
    wsb = torch.empty(K * 64 * Wd, dtype=torch.int8, device="cuda")
    wsum = torch.empty(K, dtype=torch.int32, device="cuda")
    fqt.fqt_pack_weight_signs(desc, w, wsb, wsum)
    kept = q.psq_kept[:int(q.psq_count)].long()
    signs = torch.where(w.view(D, K) > 0, 1.0, -1.0).double().t().contiguous()
    fold = lambda cols: torch.nn.functional.fold(cols, (layer.H, layer.W), (layer.kh, layer.kw),
                                                 padding=layer.pad, stride=layer.stride)
    c = fold(signs.sum(1).view(1, K, 1).expand(1, K, P).contiguous()).float()
    codes = q.psq_codes.view(2 * Wd, layer.N * P, 32)
    want = torch.zeros_like(x)
    for j, n in enumerate(kept.tolist()):
        rows = codes[:, j * P:(j + 1) * P].permute(0, 2, 1).reshape(64 * Wd, P)[:D].double()
        i = fold((signs @ rows).view(1, K, P)).float()          # (integers below 2^24)
        want[n] = (q.psq_scale[n] * i + q.psq_offset[n] * c)[0]
    dx, dx2, dw = torch.full_like(x, 7.0), torch.full_like(x, 7.0), torch.empty_like(w)
    fqt.fqt_binary_gemm_dx(desc, cfg, q, wsb, wsum, dx)
    fqt.fqt_layer_backward(desc, cfg, x, w, dy, dx2, dw, fqt.workspace(desc, cfg))
    torch.cuda.synchronize()
    assert len(kept) > 0
    assert torch.equal(dx, want), "dX of the entry"
    assert torch.equal(dx2, want), "dX of the layer"


@pytest.mark.parametrize("stride,pad", [(2, 1), (3, 1), (1, 1), (2, 2)])
@pytest.mark.parametrize("bits", [2, 4])
def test_padded_one_tap_on_one_pixel_maps(stride, pad, bits):
    """A padded 1 x 1 convolution on 1 x 1 maps, large enough for register tiles: output pixel p meets
    the input pixel where p * stride = pad, and where no p does dX is 0 (its zero-point term too)."""
    from paper_2408_14267_amd import fqt
    layer = _conv(1024, 16400, 12, 1, 1, 1, stride, pad)
    print(f"[gpu layer codes] {layer} b={bits}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(6)
    x, w = (torch.randn(s, generator=g, device="cuda") for s in (layer.x_shape, layer.w_shape))
    dy = torch.randn(layer.dy_shape, generator=g, device="cuda") + 3.0
    desc, cfg = fqt.layer_desc(layer), fqt.quant_cfg(bits, 0, 17, 3, 2)
    q = fqt.QGrad(desc, cfg)
    fqt.fqt_agp_scq_quantize(desc, cfg, dy, q, fqt.workspace(desc, cfg, fqt.FQT_WS_QUANTIZE))
    wsb = torch.empty(layer.C * 64, dtype=torch.int8, device="cuda")
    wsum = torch.empty(layer.C, dtype=torch.int32, device="cuda")
    fqt.fqt_pack_weight_signs(desc, w, wsb, wsum)
    # The rescale of exact integers from the byte codes of the pixel that the tap meets.
    want = torch.zeros(layer.N, layer.C, device="cuda")
    kept = q.psq_kept[:int(q.psq_count)].long()
    if pad % stride == 0:
        P = layer.Ho * layer.Wo
        rows = torch.arange(len(kept), device="cuda") * P + pad // stride * (layer.Wo + 1)
        codes = q.psq_codes.view(2, layer.N * P, 32)[0, rows, :layer.D].float()
        signs = torch.where(w.view(layer.D, layer.C) > 0, 1.0, -1.0)
        want[kept] = q.psq_scale[kept, None] * (codes @ signs) + q.psq_offset[kept, None] * signs.sum(0)
    dx, dx2, dw = torch.full_like(x, 7.0), torch.full_like(x, 7.0), torch.empty_like(w)
    fqt.fqt_binary_gemm_dx(desc, cfg, q, wsb, wsum, dx)
    fqt.fqt_layer_backward(desc, cfg, x, w, dy, dx2, dw, fqt.workspace(desc, cfg))
    torch.cuda.synchronize()
    assert len(kept) > 0
    assert torch.equal(dx.view_as(want), want), "dX of the entry"
    assert torch.equal(dx2.view_as(want), want), "dX of the layer"


@pytest.mark.parametrize("layer,bits,agp", [
    (_conv(13, 40, 70, 64, 64, 3, 1, 1), 2, 0),                  # dW by taps
    (LayerShape("fc", "linear", 64, 4096, 1030), 4, 0),          # few rows, dX from W itself
    (LayerShape("fc", "linear", 20, 4100, 3080), 4, 0),          # the forward too
    (LayerShape("fc", "linear", 2050, 8196, 1030), 1, 2),        # W by row passes, nibble codes
])
def test_captured_calls_replay(layer, bits, agp):
    """Backward and forward captured in one HIP graph and replayed with eager work between the
    replays equal the eager calls bit for bit."""
    from paper_2408_14267_amd import fqt
    print(f"[layer codes] replay {layer} b={bits}", file=sys.stderr, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda shape: torch.randn(shape, device="cuda", generator=gen)
    x, w, dy, gamma = rnd(layer.x_shape), rnd(layer.w_shape), rnd(layer.dy_shape), rnd((layer.D,))
    desc, cfg = fqt.layer_desc(layer), fqt.quant_cfg(bits, agp, 3, 0, 1)
    ws, wf = fqt.workspace(desc, cfg), fqt.workspace(desc, None, fqt.FQT_WS_FORWARD)

    def calls(dx, dw, y, stream=None):
        fqt.fqt_layer_backward(desc, cfg, x, w, dy, dx, dw, ws, stream)
        fqt.fqt_binary_forward(desc, x, w, gamma, y, None, wf, stream)

    want = torch.empty_like(x), torch.empty_like(w), torch.empty_like(dy)
    got = torch.empty_like(x), torch.empty_like(w), torch.empty_like(dy)
    calls(*want)
    torch.cuda.synchronize()
    side, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side), torch.cuda.graph(g, stream=side):
        calls(*got, side)
    torch.cuda.synchronize()
    other = torch.empty_like(x), torch.empty_like(w), torch.empty_like(dy)
    for r in range(3):
        for t in got:
            t.fill_(7.0)
        g.replay()
        torch.cuda.synchronize()
        for name, a, b in zip(("dx", "dw", "y"), got, want):
            assert torch.equal(a.view(torch.int32), b.view(torch.int32)), f"replay {r} {name}"
        calls(*other)                                             # eager work between
        torch.cuda.synchronize()
