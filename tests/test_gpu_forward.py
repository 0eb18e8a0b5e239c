"""Every form of the binary forward against a plain torch product of the signs: the integer
product bit for bit, Y within the one rounding of gamma * I."""
import sys

import pytest

from paper_2408_14267_amd.workloads import LayerShape

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _conv(N, C, D, H, W, k, s, p):
    return LayerShape("c", "conv2d", N, C, D, H, W, k, k, s, s, p, p)


def _linear(N, C, D):
    return LayerShape("fc", "linear", N, C, D)


# (layer, X / Y dtype, W dtype, element offset of X, W, Y and I in their buffers)
CASES = [
    # Wave tiles of 64 x 64, contraction whole: odd maps (element stores), maps of 4-pixel
    # pieces, one pixel per sample, ragged channels.
    (_conv(64, 70, 100, 57, 57, 3, 1, 1), "f32", "f32", 0),
    (_conv(64, 33, 70, 56, 56, 3, 1, 1), "bf16", "f32", 0),
    (_conv(40, 64, 128, 60, 56, 3, 1, 1), "f32", "bf16", 1),
    (_linear(4100, 200, 2050), "f32", "f32", 0),
    # The contraction of a 64 x 64 tile over four waves: 7x7, 12-pixel, 16-pixel and 28-pixel maps.
    (_conv(64, 130, 700, 7, 7, 3, 1, 1), "f32", "f32", 0),
    (_conv(200, 128, 1024, 3, 4, 3, 1, 1), "bf16", "f32", 0),
    (_conv(160, 128, 900, 4, 4, 3, 1, 1), "f32", "f32", 0),
    (_conv(90, 65, 1000, 7, 4, 3, 1, 1), "f32", "f32", 1),
    (_linear(1500, 1100, 1600), "bf16", "f32", 0),
    # 32 x 32 tiles: few and many steps, 5x5 and 2-stride taps, large padding, small maps.
    (_conv(3, 5, 9, 6, 7, 1, 1, 0), "f32", "f32", 0),
    (_conv(5, 200, 40, 9, 11, 5, 2, 2), "f32", "f32", 0),
    (_conv(4, 3, 33, 13, 13, 7, 2, 5), "bf16", "bf16", 0),
    (_conv(130, 64, 64, 2, 2, 3, 1, 1), "f32", "f32", 0),
    (_conv(130, 64, 64, 1, 1, 3, 1, 1), "f32", "f32", 0),
    (_linear(129, 65, 31), "f32", "f32", 0),
    # Linear layers of few rows, W packed: last chunks of the contraction, odd and misaligned
    # rows of W.
    (_linear(1, 1, 1), "f32", "f32", 0),
    (_linear(16, 127, 17), "f32", "f32", 1),
    (_linear(17, 129, 100), "bf16", "f32", 0),
    (_linear(33, 640, 1000), "bf16", "f32", 0),
    (_linear(64, 4224, 300), "f32", "f32", 0),
    (_linear(128, 1026, 515), "f32", "bf16", 0),
    (_linear(20, 1027, 64), "f32", "bf16", 0),
    (_linear(9, 4994, 40), "f32", "bf16", 1),
    # The same with W large enough to be read as it is (and just not): every tile count, ragged
    # rows and outputs, the last blocks and chunks.
    (_linear(1, 2048, 3072), "f32", "f32", 0),
    (_linear(16, 2047, 3072), "f32", "f32", 0),
    (_linear(16, 2050, 3071), "bf16", "f32", 0),
    (_linear(16, 2049, 3073), "f32", "f32", 1),
    (_linear(17, 4097, 3100), "bf16", "f32", 0),
    (_linear(32, 2176, 4100), "f32", "bf16", 0),
    (_linear(33, 4994, 3090), "f32", "bf16", 0),
    (_linear(64, 2050, 3089), "bf16", "bf16", 1),
    (_linear(65, 2051, 3075), "f32", "bf16", 0),
    (_linear(128, 2057, 5003), "f32", "f32", 0),
    (_linear(129, 2057, 3075), "f32", "f32", 0),
]


def _buffer(t, offset):
    b = torch.empty(t.numel() + offset, dtype=t.dtype, device=t.device)
    v = b[offset:].view(t.shape)
    v.copy_(t)
    return v


def _reference(layer, x, w):
    N, D, P, K = layer.N, layer.D, layer.Ho * layer.Wo, layer.C * layer.kh * layer.kw
    sw = torch.where(w > 0, 1.0, -1.0).double().reshape(D, K)
    out = torch.empty(N, D, P, dtype=torch.float64, device=x.device)
    for n0 in range(0, N, 32):
        xs = torch.where(x[n0:n0 + 32] > 0, 1.0, -1.0).double()
        xs = xs.reshape(-1, layer.C, layer.H, layer.W)
        xs = torch.nn.functional.pad(xs, (layer.pw, layer.pw, layer.ph, layer.ph), value=-1.0)
        cols = torch.nn.functional.unfold(xs, (layer.kh, layer.kw), stride=layer.stride)
        n = cols.shape[0]
        cols = cols.permute(1, 0, 2).reshape(K, n * P)
        out[n0:n0 + 32] = (sw @ cols).view(D, n, P).permute(1, 0, 2)
    return out.reshape(layer.dy_shape)


@pytest.mark.parametrize("layer,dtype,wdtype,offset", CASES)
def test_forward_forms(layer, dtype, wdtype, offset):
    from paper_2408_14267_amd import fqt
    print(f"[gpu forward] {layer} {dtype} {wdtype} offset {offset}", flush=True)
    sys.stdout.flush()
    g = torch.Generator(device="cuda").manual_seed(3)
    td = {"f32": torch.float32, "bf16": torch.bfloat16}
    x = torch.randn(layer.x_shape, generator=g, device="cuda").to(td[dtype])
    w = torch.randn(layer.w_shape, generator=g, device="cuda").to(td[wdtype])
    x.view(-1)[:2] = 0.0                                  # sign(0) = -1
    w.view(-1)[:1] = float("nan")                         # sign(NaN) = -1
    gamma = torch.randn(layer.D, generator=g, device="cuda")
    ref = _reference(layer, x, w)
    dt = fqt.dtype_code(dtype)
    desc = fqt.layer_desc(layer, dt, dt, fqt.dtype_code(wdtype), dt)
    x, w = _buffer(x, offset), _buffer(w, offset)
    y = _buffer(torch.full(layer.dy_shape, 7.0, dtype=td[dtype], device="cuda"), offset)
    i = _buffer(torch.full(layer.dy_shape, 7, dtype=torch.int32, device="cuda"), offset)
    ws = torch.full((fqt.fqt_workspace_size(desc, None, fqt.FQT_WS_FORWARD),), 0x77,
                    dtype=torch.uint8, device="cuda")
    shape = (1, -1) + (1,) * (ref.dim() - 2)
    want = gamma.double().view(shape) * ref
    rel = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -24     # one rounding to the output type
    for out in (i, None):
        fqt.fqt_binary_forward(desc, x, w, gamma, y, out, ws)
        torch.cuda.synchronize()
        assert torch.equal(i.double(), ref), "integer product"
        assert ((y.double() - want).abs() <= rel * want.abs()).all(), "Y"
        y.fill_(7.0)


def test_forward_packed_rows_past_two_gib():
    """67 million pixels: the packed X exceeds 2 GiB and its rows take 64-bit addresses."""
    from paper_2408_14267_amd import fqt
    layer = _conv(1, 1, 2, 8200, 8200, 1, 2, 0)
    print(f"[gpu forward] {layer}", flush=True)
    x = torch.randn(layer.x_shape, device="cuda")
    w = torch.tensor([1.0, -1.0], device="cuda").view(layer.w_shape)
    gamma = torch.tensor([0.5, 2.0], device="cuda")
    desc = fqt.layer_desc(layer)
    y = torch.empty(layer.dy_shape, device="cuda")
    fqt.fqt_binary_forward(desc, x, w, gamma, y, None, fqt.workspace(desc, None, fqt.FQT_WS_FORWARD))
    torch.cuda.synchronize()
    s = torch.where(x[0, 0, ::2, ::2] > 0, 1.0, -1.0)
    assert torch.equal(y[0, 0], 0.5 * s) and torch.equal(y[0, 1], -2.0 * s)
