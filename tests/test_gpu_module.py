"""GPU tests of the autograd / nn.Module front end: what autograd returns for Y, dX, dW is what the
oracle computes for the same tensors, flows and seeds."""
import numpy as np
import pytest
import torch

from test_gpu_parity import check_product, dev, host, mx, oracle_layer  # noqa: F401  (mx: the fixture)

pytestmark = pytest.mark.gpu


def _padded(a, rows):
    out = np.zeros((rows, a.shape[1]), a.dtype)
    out[: a.shape[0]] = a
    return out


def _run_module(lin, X3, dY3):
    x = dev(X3).requires_grad_(True)
    y = lin(x)
    (y * dev(dY3)).sum().backward()                     # dL/dY = dY exactly
    return y.detach(), x.grad, lin.weight.grad


@pytest.mark.parametrize("flow", ["tetrajet", "microscaling"])
def test_module_forward_backward_matches_oracle(mx, orc, flow):
    """x[2, 100, 96] (200 tokens: padded to 224 with zero rows), 96 -> 160, with bias: Y, dX, dW from
    autograd against the oracle's products of the oracle's codes, for both flows of Sec. 3.3."""
    import mx_workloads as wl
    N, D, C, Np = 200, 96, 160, 224
    X, W, dY = wl.linear_layer(N, D, C, seed=2, outliers=2)
    lin = mx.MxLinear(D, C, bias=True, flow=flow, seed=3, layer_id=5)
    with torch.no_grad():
        lin.weight.copy_(dev(W))
        lin.bias.copy_(dev(np.linspace(-1, 1, C, dtype=np.float32)))
    y, dx, dw = _run_module(lin, X.reshape(2, 100, D), dY.reshape(2, 100, C))
    assert y.shape == (2, 100, C) and dx.shape == (2, 100, D) and dw.shape == (C, D)
    seed = ((3 << 16) | 5) << 32                        # first call of the module with seed 3 and layer id 5
    Xp, dYp = _padded(X, Np), _padded(dY, Np)
    if flow == "tetrajet":
        xt, wt, dy = oracle_layer(orc, Xp, W, dYp, seed=seed)
    else:                                               # Eqs. 6-7: deterministic, from the full-precision tensors
        xt = orc.quantize_transposed(Xp, round_t=0, tensor_id_t=6, pre_quant=0, round_row=0, tensor_id_row=1, seed=seed)
        wt = orc.quantize_transposed(W, round_t=0, tensor_id_t=4, pre_quant=0, round_row=0, tensor_id_row=2, seed=seed)
        dy = orc.quantize_transposed(dYp, round_t=0, tensor_id_t=5, pre_quant=0, round_row=0, tensor_id_row=3, seed=seed)
    bias = np.linspace(-1, 1, C, dtype=np.float32)
    y_nobias = torch.zeros((Np, C), device="cuda")
    y_nobias[:N] = y.reshape(N, C) - dev(bias)
    # subtracting the bias again costs one FP32 rounding of |y|: allow for it next to the product's 1e-5
    ref = orc.gemm_f64(xt[2], xt[3], wt[2], wt[3])
    absref = np.abs(orc.dequantize(xt[2], xt[3])) @ np.abs(orc.dequantize(wt[2], wt[3])).T
    err = np.abs(host(y_nobias).astype(np.float64) - ref)
    assert np.all(err <= 1e-5 * absref + 2.0 ** -22 * (np.abs(ref) + 1.0)), err.max()
    dxp = torch.zeros((Np, D), device="cuda")
    dxp[:N] = dx.reshape(N, D)
    ref_dx = orc.gemm_f64(dy[2], dy[3], wt[0], wt[1])
    assert np.all(ref_dx[N:] == 0.0)                    # zero gradient rows quantize to zero
    check_product(orc, dxp, dy[2], dy[3], wt[0], wt[1], "dX " + flow)
    check_product(orc, dw, dy[0], dy[1], xt[0], xt[1], "dW " + flow)
    want_db = dY.astype(np.float64).sum(0)
    assert np.allclose(host(lin.bias.grad), want_db, rtol=1e-5, atol=1e-5 * np.abs(dY).sum(0).max())
    # a second call draws new rounding streams (seed advances with the call count)
    y2, dx2, _ = _run_module(lin, X.reshape(2, 100, D), dY.reshape(2, 100, C))
    assert torch.equal(y2, y)                           # the forward quantizers are deterministic
    if flow == "tetrajet":
        assert not torch.equal(dx2, dx)
    else:
        assert torch.equal(dx2, dx)


def test_module_qema_and_bf16(mx, orc):
    """bf16 activations and weights, weight through Q-EMA: two training-mode forwards advance the
    moving average exactly as the oracle does, and Y is the product with the Q-EMA codes."""
    import mx_workloads as wl
    N, D, C = 256, 128, 96
    X, _, _ = wl.linear_layer(N, D, C, seed=6, dtype="bf16")
    lin = mx.MxLinear(D, C, bias=False, dtype=torch.bfloat16, qema=True, beta=0.99, seed=1)
    ema = None
    for t, W in enumerate(wl.weight_walk(C, D, seed=6, steps=1, sigma=5e-3)):
        W = wl.round_to_bf16(W)
        if ema is None:
            ema = np.zeros_like(W)
        wc, wsc = orc.ema_weight_quant(W, ema, beta=0.99, update_ema=2 if t == 0 else 1)
        with torch.no_grad():
            lin.weight.copy_(dev(W, "bf16"))
        y = lin(dev(X, "bf16"))
        assert np.array_equal(host(lin.w_ema), ema), t
    assert y.dtype == torch.bfloat16
    xq = orc.quantize(X)
    ref = orc.gemm_f64(xq[0], xq[1], wc, wsc)
    absref = np.abs(orc.dequantize(xq[0], xq[1])) @ np.abs(orc.dequantize(wc, wsc)).T
    err = np.abs(host(y.detach().float()).astype(np.float64) - ref)
    assert np.all(err <= 1e-5 * absref + 2.0 ** -8 * np.abs(ref))      # bf16 output rounding
    # evaluation mode leaves the moving average alone
    lin.eval()
    before = lin.w_ema.clone()
    lin(dev(X, "bf16"))
    assert torch.equal(before, lin.w_ema)


def test_module_trains_a_small_mlp(mx):
    """Two MXFP4 layers fit a random teacher: the loss must fall (a property, not a parity check --
    gradients that were wrong in sign, scale or transposition would not descend)."""
    torch.manual_seed(0)
    Din, H, Dout, N = 64, 128, 32, 512
    teacher = torch.randn(Din, Dout, device="cuda") / Din ** 0.5
    x = torch.randn(N, Din, device="cuda")
    target = torch.tanh(x @ teacher)
    net = torch.nn.Sequential(mx.MxLinear(Din, H, seed=1), torch.nn.GELU(), mx.MxLinear(H, Dout, seed=2))
    opt = torch.optim.AdamW(net.parameters(), lr=3e-3, weight_decay=0.0)
    losses = []
    for _ in range(60):
        opt.zero_grad()
        loss = torch.nn.functional.mse_loss(net(x), target)
        loss.backward()
        opt.step()
        losses.append(float(loss.detach()))
    assert losses[-1] < 0.5 * losses[0], (losses[0], losses[-1])


def test_module_device_seed_equals_host_seed_and_replays_in_a_graph(mx):
    """device_seed=True: the same Y, dX, dW as the host-side key, call for call (eagerly); and a whole
    forward + backward recorded into a graph gives, replay after replay, what the eager module gives on
    its next calls (new rounding numbers each time, so the gradients of two replays differ)."""
    import mx_workloads as wl
    N, D, C = 96, 64, 128
    X, W, dY = wl.linear_layer(N, D, C, seed=8)
    lins = [mx.MxLinear(D, C, bias=True, seed=0x9ABC, layer_id=0xDEF0, device_seed=ds) for ds in (False, True)]
    for lin in lins:
        with torch.no_grad():
            lin.weight.copy_(dev(W))
            lin.bias.copy_(dev(np.linspace(-2, 2, C, dtype=np.float32)))

    def eager(lin):
        x = dev(X).requires_grad_(True)
        lin.weight.grad = lin.bias.grad = None
        y = lin(x)
        (y * dev(dY)).sum().backward()
        return y.detach().clone(), x.grad.clone(), lin.weight.grad.clone(), lin.bias.grad.clone()

    for call in range(2):
        a, b = eager(lins[0]), eager(lins[1])
        for u, v, nm in zip(a, b, ("Y", "dX", "dW", "dbias")):
            assert torch.equal(u, v), (call, nm)
    # record call 3 of the device-seed module; replays are then calls 3, 4, 5 of the host-seed module
    lin = lins[1]
    xs = dev(X).requires_grad_(True)
    dys = dev(dY)
    lin.weight.grad = lin.bias.grad = None
    graph = torch.cuda.CUDAGraph()
    before = lin.seed_state.clone()
    with torch.cuda.graph(graph):
        ys = lin(xs)
        (ys * dys).sum().backward()
    lin.seed_state.copy_(before)                       # recording ran nothing: the key still names call 2
    seen = []
    for call in range(3):
        graph.replay()
        torch.cuda.synchronize()
        want = eager(lins[0])
        for u, v, nm in zip((ys, xs.grad, lin.weight.grad, lin.bias.grad), want, ("Y", "dX", "dW", "dbias")):
            assert torch.equal(u, v), (call, nm)
        seen.append(xs.grad.clone())
    assert not torch.equal(seen[0], seen[1]) and not torch.equal(seen[1], seen[2])


def test_layers_of_a_model_round_with_independent_streams(mx):
    """Two layers of the same shape built with default arguments, given the same weight, input and output
    gradient: the deterministic forward agrees bit for bit, the stochastically rounded backward does not
    (each layer's Philox key carries its own layer id, Sec. 3.4's independence)."""
    import mx_workloads as wl
    N, D, C = 96, 64, 128
    X, W, dY = wl.linear_layer(N, D, C, seed=12)
    a, b = mx.MxLinear(D, C, bias=False), mx.MxLinear(D, C, bias=False)
    assert a.layer_id != b.layer_id and a.key_high != b.key_high
    outs = []
    for lin in (a, b):
        with torch.no_grad():
            lin.weight.copy_(dev(W))
        outs.append(_run_module(lin, X, dY))
    assert torch.equal(outs[0][0], outs[1][0])
    assert not torch.equal(outs[0][1], outs[1][1]) and not torch.equal(outs[0][2], outs[1][2])


def test_device_seed_backward_uses_the_key_of_its_own_forward(mx):
    """Two forward calls before the first backward (micro-batches): with the key in device memory each
    backward still rounds with the key of its own forward, as the host-side key does."""
    import mx_workloads as wl
    N, D, C = 64, 64, 96
    X, W, dY = wl.linear_layer(N, D, C, seed=13)
    grads = []
    for ds in (False, True):
        lin = mx.MxLinear(D, C, bias=False, seed=4, layer_id=9, device_seed=ds)
        with torch.no_grad():
            lin.weight.copy_(dev(W))
        x1, x2 = dev(X).requires_grad_(True), dev(X).requires_grad_(True)
        y1, y2 = lin(x1), lin(x2)
        (y1 * dev(dY)).sum().backward()
        (y2 * dev(dY)).sum().backward()
        grads.append((x1.grad.clone(), x2.grad.clone()))
    assert torch.equal(grads[0][0], grads[1][0]) and torch.equal(grads[0][1], grads[1][1])
    assert not torch.equal(grads[0][0], grads[0][1])


@pytest.mark.parametrize("tokens,xt,wt,flow,qema", [
    (1, "bf16", "f32", "tetrajet", False), (33, "f32", "f32", "tetrajet", False), (200, "bf16", "bf16", "microscaling", False),
    (255, "bf16", "f32", "microscaling", True), (300, "bf16", "bf16", "tetrajet", True), (4095, "bf16", "f32", "tetrajet", False),
    (4097, "bf16", "f32", "tetrajet", False), (4225, "f32", "f32", "microscaling", False)])
def test_module_equals_the_calls_on_padded_tensors(mx, tokens, xt, wt, flow, qema):
    """Ragged token counts, mixed source types, column sums and every subset of wanted gradients: bit for bit what the
    separate calls give on explicitly padded tensors (which the parity tests hold against the oracle)."""
    D, C, tdt = 160, 96, {"f32": torch.float32, "bf16": torch.bfloat16}
    g = torch.Generator(device="cuda")
    g.manual_seed(tokens)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    x, dy = rnd(tokens, D).to(tdt[xt]), (rnd(tokens, C) * 1e-3).to(tdt[xt])
    lin = mx.MxLinear(D, C, bias=True, dtype=tdt[wt], flow=flow, qema=qema, seed=7, layer_id=3)
    with torch.no_grad():
        lin.bias.copy_(rnd(C))
    seed, tetra, Np = ((7 << 16) | 3) << 32, flow == "tetrajet", (tokens + 31) // 32 * 32
    pad = lambda t: torch.cat([t, t.new_zeros((Np - tokens, t.shape[1]))])
    rt, pre = (mx.ROUND_SR if tetra else mx.ROUND_RTN), int(tetra)
    xtq, xts, xq, xs = mx.mx_quantize_transposed(pad(x), rt, 6, pre, True, mx.ROUND_RTN, 1, seed=seed)
    w = lin.weight.detach()
    if qema:
        wq, ws = mx.mx_ema_weight_quant(w, torch.zeros(C, D, device="cuda"), lin.beta, 2)
        if tetra:
            wtq, wts, _, _ = mx.mx_quantize_transposed(None, rt, 4, 1, False, row_in=(wq, ws), seed=seed, shape=(C, D))
        else:
            wtq, wts, _, _ = mx.mx_quantize_transposed(w, rt, 4, 0, False, seed=seed)
    else:
        wtq, wts, wq, ws = mx.mx_quantize_transposed(w, rt, 4, pre, True, mx.ROUND_RTN, 2, seed=seed)
    y0 = mx.mx_linear_fwd_bias(xq, xs, wq, ws, lin.bias.detach().float(), out_dtype=x.dtype)[:tokens]
    u8 = lambda *s: torch.empty(s, dtype=torch.uint8, device="cuda")
    out, db0 = (u8(C, Np // 2), u8(C, Np // 32), u8(Np, C // 2), u8(Np, C // 32)), torch.empty(C, device="cuda")
    mx.mx_quantize_transposed_batch([{"src": pad(dy), "out": out, "tensor_id_t": 5, "tensor_id_row": 3, "pre_quant": 0, "seed": seed,
                                      "col_sums": db0}], rt, rt)
    dx0 = mx.mx_linear_bwd_dx(out[2], out[3], wtq, wts, out_dtype=x.dtype)[:tokens]
    dw0 = mx.mx_linear_bwd_dw(out[0], out[1], xtq, xts).to(w.dtype)
    for want in range(1, 8):
        lin.calls, lin._ema_started = 0, False
        xg = x.clone().requires_grad_(bool(want & 1))
        lin.weight.requires_grad_(bool(want & 2))
        lin.bias.requires_grad_(bool(want & 4))
        y = lin(xg)
        asked = [t for t in (xg, lin.weight, lin.bias) if t.requires_grad]
        grads = iter(torch.autograd.grad(y, asked, dy))
        assert torch.equal(y, y0), want
        for t, ref in ((xg, dx0), (lin.weight, dw0), (lin.bias, db0.to(w.dtype))):
            if t.requires_grad:
                assert torch.equal(next(grads), ref), want
    lin.calls, lin._ema_started = 0, False
    with torch.no_grad():
        assert torch.equal(lin(x), y0)
        assert torch.equal(lin(x.reshape(1, tokens, 1, D)).reshape(tokens, C), y0)


def test_step_refuses_what_the_c_interface_refuses(mx):
    """MxLinearStep's buffers are attributes that a program may replace; each call is refused before anything is launched."""
    B = mx.binding

    def refused(code, call, *args):
        with pytest.raises(mx.MxError) as e:
            call(*args)
        assert e.value.code == code, e.value

    z = lambda *s, **kw: torch.zeros(s, device="cuda", **kw)
    X, W, dY = z(64, 64), z(96, 64), z(64, 96)
    step = lambda: mx.MxLinearStep(64, 64, 96, out_dtype=torch.float32)
    shifted = lambda t, by: torch.empty(t.numel() + by, dtype=t.dtype, device="cuda")[by:].view(t.shape)
    for name, by, call, arg in (("y", 1, "forward", (X, W)), ("dx", 1, "backward", (dY,)), ("dw", 1, "backward", (dY,)),
                                ("xtq", 4, "forward", (X, W)), ("wq", 4, "forward", (X, W)), ("dyq", 4, "backward", (dY,))):
        s = step()
        setattr(s, name, shifted(getattr(s, name), by))
        refused(B.MX_ERR_ALIGN, getattr(s, call), *arg, 1)
    s = step()
    s.y = z(64, 96, dtype=torch.float16)
    with pytest.raises(TypeError):
        s.forward(X, W, 1)
    # more rows than the tile quantizer's index takes
    n = 65535 * 128 + 32
    s = mx.MxLinearStep(n, 32, 32)
    refused(B.MX_ERR_SHAPE, s.forward, z(n, 32, dtype=torch.bfloat16), z(32, 32, dtype=torch.bfloat16), 1)
    refused(B.MX_ERR_SHAPE, s.backward, z(n, 32, dtype=torch.bfloat16), 1)


@pytest.mark.parametrize("dt", [torch.float16, torch.float64])
@pytest.mark.parametrize("tokens", [33, 4100])
def test_bias_of_another_floating_type(mx, dt, tokens):
    """The bias enters the product as FP32 and its gradient comes back in its own type."""
    torch.manual_seed(tokens)
    lin, ref = (mx.MxLinear(64, 96, seed=1, layer_id=2) for _ in range(2))
    ref.load_state_dict(lin.state_dict())
    lin.bias = torch.nn.Parameter(torch.randn(96, device="cuda").to(dt))
    ref.bias = torch.nn.Parameter(lin.bias.detach().float())
    x, dy = torch.randn(tokens, 64, device="cuda"), torch.randn(tokens, 96, device="cuda")
    y, y0 = lin(x), ref(x)
    g, g0 = (torch.autograd.grad(v, (m.weight, m.bias), dy) for v, m in ((y, lin), (y0, ref)))
    assert torch.equal(y, y0) and torch.equal(g[0], g0[0]) and g[1].dtype == dt and torch.equal(g[1], g0[1].to(dt))
    with torch.no_grad():
        assert torch.equal(lin(x), y0)


@pytest.mark.parametrize("options", [{}, {"bias": False}, {"device_seed": True}, {"qema": True}])
def test_traced_module_replays_the_pass(mx, options):
    """torch.jit.trace records the pass as one call: outputs and gradients on other inputs are the module's own."""
    torch.manual_seed(5)
    lin, ref = (mx.MxLinear(64, 96, seed=1, layer_id=2, **options) for _ in range(2))
    ref.load_state_dict(lin.state_dict())
    xs = [torch.randn(3, 32, 64, device="cuda") for _ in range(4)]
    lin.eval()
    with torch.no_grad():
        traced = torch.jit.trace(lin, xs[0], check_trace=False)
        want = [ref.eval()(x) for x in xs]
        for x, y in zip(xs, want):
            assert torch.equal(traced(x), y)
    traced = torch.jit.trace(lin, xs[0].clone().requires_grad_(True), check_trace=False)     # one forward call of its own
    key, dy = lin.calls - 1, torch.randn(3, 32, 96, device="cuda")
    for x in xs:
        got, ours = x.clone().requires_grad_(True), x.clone().requires_grad_(True)
        if lin.seed_state is not None:
            ref.seed_state.copy_(lin.seed_state)             # the trace advances the word that it shares with the module
        ref.calls = key                                      # a key from the host is a constant of the trace
        y, y0 = traced(got), ref(ours)
        assert torch.equal(y, y0)
        g = torch.autograd.grad(y, (got, *lin.parameters()), dy)
        for a, b in zip(g, torch.autograd.grad(y0, (ours, *ref.parameters()), dy)):
            assert torch.equal(a, b)


def test_saved_operands_through_hooks(mx):
    """Hooks that move the saved operands away and back change nothing; what does not come back as it was is refused, as MxError
    out of the backward pass."""
    lin = mx.MxLinear(64, 96, seed=1, layer_id=2)
    x, dy = torch.randn(40, 64, device="cuda", requires_grad=True), torch.randn(40, 96, device="cuda")
    want = torch.autograd.grad(lin(x), (x, lin.weight, lin.bias), dy)
    for whole, unpack in ((True, lambda t: t.cuda()), (False, lambda t: t.cuda()[:-256]), (False, lambda t: t), (False, lambda t: t.cuda().float())):
        lin.calls = 0
        with torch.autograd.graph.saved_tensors_hooks(lambda t: t.cpu(), unpack):
            y = lin(x)
        backward = lambda: torch.autograd.grad(y, (x, lin.weight, lin.bias), dy)
        if whole:
            assert all(torch.equal(a, b) for a, b in zip(backward(), want))
        else:
            with pytest.raises(mx.MxError) as e:
                backward()
            assert e.value.code == mx.binding.MX_ERR_SHAPE


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("tokens,D,C,xt,wt", [(1, 32, 32, "f32", "bf16"), (33, 160, 96, "bf16", "f32"), (257, 96, 2080, "bf16", "bf16"),
                                              # one launch: one K step, two, a ragged second one; the last sizes that it
                                              # takes, and one more row of tiles, one more group of columns
                                              (64, 256, 64, "f32", "f32"), (65, 288, 96, "bf16", "f32"), (3, 512, 64, "f32", "bf16"),
                                              (1000, 512, 1024, "bf16", "bf16"), (1025, 512, 1024, "bf16", "f32"), (130, 544, 64, "bf16", "bf16"),
                                              # more chunks than one per lane of the row kernel's grid covers
                                              (8200, 1056, 96, "bf16", "f32"), (2113, 4128, 64, "f32", "f32")])
def test_forward_without_gradients_equals_the_one_with(mx, mode, tokens, D, C, xt, wt):
    """Row quantizers alone (both tensors in one launch, one or four chunks per lane) against the fused ones, which the
    parity tests hold against the oracle; both scale rules, every pair of source types."""
    tdt = {"f32": torch.float32, "bf16": torch.bfloat16}
    torch.manual_seed(tokens)
    x = torch.randn(tokens, D, device="cuda").mul_(torch.randn(tokens, 1, device="cuda").exp_()).to(tdt[xt])
    for bias in (True, False):
        lin = mx.MxLinear(D, C, bias=bias, dtype=tdt[wt], scale_mode=mode, seed=1, layer_id=1)
        if bias:
            with torch.no_grad():
                lin.bias.normal_()
        y = lin(x).detach()
        with torch.no_grad():
            assert torch.equal(lin(x), y)
        wq, ws = mx.mx_quantize(lin.weight.detach(), scale_mode=mode)
        xq, xs = mx.mx_quantize(x, scale_mode=mode)
        args = (xq, xs, wq, ws) + ((lin.bias.detach().float(),) if bias else ())
        assert torch.equal((mx.mx_linear_fwd_bias if bias else mx.mx_linear_fwd)(*args, out_dtype=x.dtype), y)


@pytest.mark.parametrize("flow", ["tetrajet", "microscaling"])
@pytest.mark.parametrize("xt,wt", [("bf16", "f32"), ("f32", "bf16"), ("f32", "f32")])
def test_module_with_the_floor_scale_rule(mx, flow, xt, wt):
    """Eq. 2's scale rule through the native pass, mixed source types in one launch: the separate calls' bits."""
    tdt, tokens, Np, D, C = {"f32": torch.float32, "bf16": torch.bfloat16}, 70, 96, 160, 96
    torch.manual_seed(1)
    x, dy = torch.randn(tokens, D, device="cuda").to(tdt[xt]), (torch.randn(tokens, C, device="cuda") * 1e-3).to(tdt[xt])
    lin = mx.MxLinear(D, C, dtype=tdt[wt], flow=flow, scale_mode=1, seed=7, layer_id=3)
    xg = x.clone().requires_grad_(True)
    y = lin(xg)
    dx, dw, db = torch.autograd.grad(y, (xg, lin.weight, lin.bias), dy)
    seed, tetra = ((7 << 16) | 3) << 32, flow == "tetrajet"
    pad = lambda t: torch.cat([t, t.new_zeros((Np - tokens, t.shape[1]))])
    rt, pre = (mx.ROUND_SR if tetra else mx.ROUND_RTN), int(tetra)
    xtq, xts, xq, xs = mx.mx_quantize_transposed(pad(x), rt, 6, pre, True, mx.ROUND_RTN, 1, scale_mode=1, seed=seed)
    wtq, wts, wq, ws = mx.mx_quantize_transposed(lin.weight.detach(), rt, 4, pre, True, mx.ROUND_RTN, 2, scale_mode=1, seed=seed)
    dtq, dts, dq, ds = mx.mx_quantize_transposed(pad(dy), rt, 5, 0, True, rt, 3, scale_mode=1, seed=seed)
    assert torch.equal(y, mx.mx_linear_fwd_bias(xq, xs, wq, ws, lin.bias.detach().float(), out_dtype=x.dtype)[:tokens])
    assert torch.equal(dx, mx.mx_linear_bwd_dx(dq, ds, wtq, wts, out_dtype=x.dtype)[:tokens])
    assert torch.equal(dw, mx.mx_linear_bwd_dw(dtq, dts, xtq, xts).to(dw.dtype))
    # FP32 sums of `tokens` values in some order, then one rounding to the bias's type
    ref, mag = dy.double().sum(0), dy.double().abs().sum(0)
    assert bool(((db.double() - ref).abs() <= tokens * 2.0 ** -24 * mag + (ref.abs() * 2.0 ** -8 if wt == "bf16" else 0.0)).all())


def _check_backward_pass(mx, n, d, c, dtype):
    g = torch.Generator(device="cuda")
    g.manual_seed(n + d + c)
    x, w, dy = (torch.randn(s, generator=g, device="cuda").to(dtype) for s in ((n, d), (c, d), (n, c)))
    st = mx.MxLinearStep(n, d, c, out_dtype=dtype)
    st.forward(x, w, 7)
    dx, dw = (t.clone() for t in st.backward(dy, 7))
    assert torch.equal(dx, mx.mx_linear_bwd_dx(st.dyq, st.dys, st.wtq, st.wts, out_dtype=dtype))
    assert torch.equal(dw, mx.mx_linear_bwd_dw(st.dytq, st.dyts, st.xtq, st.xts, out_dtype=torch.float32))
    # the module: a workspace each
    lin = mx.MxLinear(d, c, bias=False, dtype=dtype, seed=7 >> 16, layer_id=0)
    with torch.no_grad():
        lin.weight.copy_(w)
    lin.key_high, lin.calls = 0, 7
    xg = x.clone().requires_grad_(True)
    gx, gw = torch.autograd.grad(lin(xg), (xg, lin.weight), dy)
    assert torch.equal(gx, dx)
    if n % 128 == 0 or n < 4096:                        # otherwise the module's dW sums over more rows, in another order
        assert torch.equal(gw, dw.to(dtype))


@pytest.mark.parametrize("n,d,c", [
    # tiles of dW / dX: 64 / 64 (with idle workgroups between the two), K split 64 / 128x64, 64 / 128, 128x64 / 64,
    # 128x64 / 128x64, 128x64 / 128, 64 / 128 with all of K at once, 128x64 / the same, the smallest, 128x64 / K split 64, dX on the main kernel (apart)
    (256, 192, 768), (12608, 192, 576), (4064, 2048, 480), (1024, 768, 3072), (2048, 768, 3072), (4064, 2048, 992), (25216, 1536, 384), (3968, 4096, 352), (32, 32, 32),
    (512, 1024, 4096), (25216, 384, 1536)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_products_of_a_backward_pass_in_one_launch(mx, n, d, c, dtype):
    """The native backward pass gives what the separate calls give for the same operands, bit for bit."""
    _check_backward_pass(mx, n, d, c, dtype)


def _split_both(mx, n, d, c):
    """Workspace bytes of dX and dW, each of which splits K."""
    need = [mx.mx_linear_workspace_bytes(which, n, c, d) for which in (mx.binding.GEMM_BWD_DX, mx.binding.GEMM_BWD_DW)]
    assert min(need) > 0
    return need


@pytest.mark.parametrize("n,d,c", [
    (4096, 64, 4096), (4128, 64, 4128), (4096, 96, 5120)])                  # the second: ragged K
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_backward_pass_that_splits_both_products(mx, n, d, c, dtype):
    """MxLinearStep has one workspace for both, so that they must run one after the other; MxLinear gives each its own."""
    _split_both(mx, n, d, c)
    kernel = mx.binding.host().gemm_kernel_name
    assert kernel(c, d, n, False) == kernel(n, d, c, False) == "64x64"                               # one launch but for the workspace
    _check_backward_pass(mx, n, d, c, dtype)


def test_memory_of_a_backward_pass_that_splits_both_products(mx):
    """On the main kernel they run one after the other: the pass holds one workspace at a time."""
    n, d, c = 8192, 768, 8192
    need = _split_both(mx, n, d, c)
    assert mx.binding.host().gemm_kernel_name(n, d, c, False) == "main" and min(need) > 40 << 20
    lin = mx.MxLinear(d, c, bias=False, dtype=torch.bfloat16, seed=1, layer_id=1)
    x, dy = torch.randn(n, d, device="cuda").bfloat16().requires_grad_(True), torch.randn(n, c, device="cuda").bfloat16()
    y = lin(x)
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    held = torch.cuda.memory_allocated()
    torch.autograd.grad(y, (x, lin.weight), dy)
    torch.cuda.synchronize()
    results, packed = 2 * (n * d + c * d), 2 * n * c * 17 // 32
    assert torch.cuda.max_memory_allocated() - held <= results + packed + max(need) + (4 << 20)


def _kernels_of(graph):
    """Nodes of a recorded graph, through the HIP library that this process has loaded."""
    import ctypes
    hip = ctypes.CDLL(next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line))
    count = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(count)) == 0
    return count.value


@pytest.mark.parametrize("tokens,D,C,nodes", [(197, 256, 96, 1), (197, 288, 96, 2), (1000, 512, 1024, 2), (7168, 512, 64, 1), (33, 384, 3072, 1)])
def test_forward_recorded_into_a_graph(mx, tokens, D, C, nodes):
    """Beyond 256 columns a recorded call runs the separate kernels where they take less device time; every replay gives what the
    eager call gives for the values that the input then holds."""
    torch.manual_seed(D)
    lin = mx.MxLinear(D, C, dtype=torch.bfloat16, seed=1, layer_id=1)
    x = torch.randn(tokens, D, device="cuda").bfloat16()
    with torch.no_grad():
        lin.bias.normal_()
        lin(x)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(graph):
            y = lin(x)
        assert _kernels_of(graph) == nodes
        for _ in range(3):
            x.copy_(torch.randn(tokens, D, device="cuda").mul_(torch.randn(tokens, 1, device="cuda").exp_()))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(y, lin(x))
