"""fqt_train_backward against the same steps taken one by one: dY = dH * gamma through
fqt_layer_backward (dX and dW bit for bit, dX masked where |X| > 1), dgamma against float64."""
import sys

import pytest

from paper_2408_14267_amd.workloads import LayerShape

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _conv(N, C, D, H, W, k, s, p):
    return LayerShape("c", "conv2d", N, C, D, H, W, k, k, s, s, p, p)


CASES = [
    (_conv(9, 16, 70, 8, 8, 3, 1, 1), 4, 0),          # 64-pixel tiles, merged keys
    (_conv(5, 7, 70, 9, 9, 3, 1, 1), 3, 0),           # odd maps: element by element
    (_conv(3, 20, 66, 36, 36, 3, 1, 1), 2, 0),        # per-plane statistics, a ragged last batch
    (_conv(40, 3, 10, 40, 40, 3, 2, 1), 8, 2),        # planes of a strided layer, AGP off
    (_conv(2, 70, 9, 362, 362, 3, 1, 1), 2, 0),       # register-tile dX: 16-byte and element stores
    (_conv(1, 1, 4, 1024, 513, 3, 1, 1), 2, 0),       # one channel tile per wave in dX
    (LayerShape("fc", "linear", 37, 300, 132), 4, 0),     # channel quads
    (LayerShape("fc", "linear", 70, 64, 77), 1, 0),       # odd rows
    (LayerShape("fc", "linear", 1500, 96, 1300), 2, 0),   # more than 1024 groups
    (_conv(64, 8, 300, 14, 14, 3, 1, 1), 4, 0),       # several row tiles per block, whole quads
    (_conv(64, 8, 300, 15, 15, 3, 1, 1), 4, 0),       # and element by element
    (LayerShape("fc", "linear", 33, 5000, 1030), 4, 0),   # few rows, dX from W itself
    (LayerShape("fc", "linear", 2050, 4100, 300), 2, 0),  # register-tile dX along the channels
]


@pytest.mark.parametrize("layer,bits,agp", CASES)
def test_train_backward_matches_the_steps(layer, bits, agp):
    from paper_2408_14267_amd import fqt
    print(f"[gpu train fused] {layer} b={bits}", flush=True)
    sys.stdout.flush()
    g = torch.Generator(device="cuda").manual_seed(4)
    x = torch.randn(layer.x_shape, generator=g, device="cuda")
    w = torch.randn(layer.w_shape, generator=g, device="cuda")
    gamma = torch.randn(layer.D, generator=g, device="cuda")
    dh = torch.randn(layer.dy_shape, generator=g, device="cuda")
    x.view(-1)[:1] = 1.0
    K = layer.C * layer.kh * layer.kw
    i = torch.randint(-K, K + 1, layer.dy_shape, generator=g, device="cuda", dtype=torch.int32)
    shape = (1, -1) + (1,) * (dh.dim() - 2)
    desc, cfg = fqt.layer_desc(layer), fqt.quant_cfg(bits, agp, 5, 3, 2)
    dx, dw = torch.empty_like(x), torch.empty_like(w)
    fqt.fqt_layer_backward(desc, cfg, x, w, (dh * gamma.view(shape)).contiguous(), dx, dw,
                           fqt.workspace(desc, cfg))
    dx = dx * (x.abs() <= 1)
    terms = dh.double() * i.double()
    dims = (0,) + tuple(range(2, dh.dim()))
    want, size = terms.sum(dims), terms.abs().sum(dims)
    ws = fqt.train_workspace(desc, cfg)
    for _ in range(2):                          # a reused workspace gives the same result
        dx2, dw2 = torch.full_like(x, 7.0), torch.full_like(w, 7.0)
        dgamma = torch.full_like(gamma, 7.0)
        fqt.fqt_train_backward(desc, cfg, x, w, gamma, i, dh, dx2, dw2, dgamma, ws)
        torch.cuda.synchronize()
        assert torch.equal(dx2, dx), "dX"
        assert torch.equal(dw2, dw), "dW"
        # A lane adds up to 64 products in float32, then 6 levels of lanes: below 128 roundings of 2^-24.
        assert ((dgamma.double() - want).abs() <= 128 * 2.0 ** -24 * size).all(), "dgamma"


def test_module_gradients_of_any_layout_and_create_graph():
    """An expanded and a misaligned gradient give what a contiguous copy gives; with
    create_graph, dgamma stays differentiable in the gradient (d dgamma / d dH = I)."""
    from paper_2408_14267_amd import train
    print("[gpu train fused] module layouts", flush=True)
    torch.manual_seed(1)
    mod = train.BinaryConv2d(8, 12, 3, 1, 1, bits=2, layer_id=3, seed=9).cuda()
    x = torch.randn(4, 8, 6, 6, device="cuda", requires_grad=True)
    args = (x, mod.weight, mod.gamma)

    def grads(dy, **kw):
        mod.step = 0
        y = mod(x)
        return y, torch.autograd.grad(y, args, dy, **kw)

    base = torch.randn(4 * 12 * 36 + 1, device="cuda")
    shifted = base[1:].view(4, 12, 6, 6)
    expanded = torch.randn(1, 12, 1, 1, device="cuda").expand(4, 12, 6, 6)
    for dy in (shifted, expanded, shifted.to(memory_format=torch.channels_last)):
        for a, b in zip(grads(dy)[1], grads(dy.contiguous().clone())[1]):
            assert torch.equal(a, b)
    dy = shifted.clone().requires_grad_(True)
    y, (dx, dw, dgamma) = grads(dy, create_graph=True)
    plain = grads(dy.detach())[1]
    assert torch.equal(dx, plain[0]) and torch.equal(dw, plain[1])
    assert torch.allclose(dgamma.detach(), plain[2], rtol=1e-5, atol=1e-4)
    second, = torch.autograd.grad(dgamma.sum(), dy)
    assert torch.equal(second, torch.round(y.detach() / mod.gamma.detach().view(1, -1, 1, 1)))


def test_current_stream_with_and_without_the_raw_handle(monkeypatch):
    from paper_2408_14267_amd import fqt
    side = torch.cuda.Stream()
    for stream in (torch.cuda.default_stream(), side):
        with torch.cuda.stream(stream):
            assert fqt.current_stream() == stream.cuda_stream
            with monkeypatch.context() as m:
                m.setattr(fqt, "_raw_stream", None)
                assert fqt.current_stream() == stream.cuda_stream


def test_module_bits_and_agp_change_between_steps():
    """Workspace sizes follow the code width and the pruning mode: a module whose settings change takes
    a workspace of the new size (and the old one again when they change back)."""
    from paper_2408_14267_amd import fqt, train
    print("[gpu train fused] module settings change", flush=True)
    torch.manual_seed(2)
    mod = train.BinaryConv2d(64, 64, 3, 1, 1, bits=1, agp_mode=fqt.FQT_AGP_OFF).cuda()
    x = torch.randn(64, 64, 32, 32, device="cuda", requires_grad=True)
    dy = torch.randn(64, 64, 32, 32, device="cuda")

    def grads(m):
        m.step = 5
        return torch.autograd.grad(m(x), (x, m.weight, m.gamma), dy)

    for bits, agp in ((1, 2), (8, 2), (8, 0), (1, 2)):
        mod.bits, mod.agp_mode = bits, agp
        fresh = train.BinaryConv2d(64, 64, 3, 1, 1, bits=bits, agp_mode=agp).cuda()
        fresh.load_state_dict(mod.state_dict())
        for a, b in zip(grads(mod), grads(fresh)):
            assert torch.equal(a, b), (bits, agp)


def test_module_workspaces_are_one_per_stream():
    """Two streams may run one module at a time each: they take workspaces of their own.  A capture
    takes one that is there, whatever stream it came from."""
    from paper_2408_14267_amd import fqt, train
    print("[gpu train fused] module workspaces", flush=True)
    mod = train.BinaryLinear(40, 24, bits=2).cuda()
    desc, cfg = mod.desc((16, 40)), fqt.quant_cfg(2)
    side = torch.cuda.Stream()
    first = mod.ws_forward(desc), mod.ws_backward(desc, cfg)
    with torch.cuda.stream(side):
        other = mod.ws_forward(desc), mod.ws_backward(desc, cfg)
        again = mod.ws_forward(desc), mod.ws_backward(desc, cfg)
    assert all(a.data_ptr() != b.data_ptr() for a, b in zip(first, other))
    assert all(a is b for a, b in zip(other, again))
    assert all(a is b for a, b in zip(first, (mod.ws_forward(desc), mod.ws_backward(desc, cfg))))
    x = torch.randn(16, 40, device="cuda", requires_grad=True)
    dy = torch.randn(16, 24, device="cuda")
    step = lambda: torch.autograd.grad(mod(x), (x, mod.weight, mod.gamma), dy)
    mod.step = 0
    want = [t.clone() for t in step()]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    mod.step = 0
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        got = step()
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            assert torch.equal(a, b)
        step()                                  # eager work between the replays
        torch.cuda.synchronize()
    assert len(mod._ws) == 2 and all(len(v) == 2 for v in mod._ws.values())
