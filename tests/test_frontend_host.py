"""Host-side checks of the native front ends (no GPU: each call is refused before anything is launched)."""
import pytest

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def mx():
    import paper_2502_20853_amd as mx
    from paper_2502_20853_amd import build
    if build.is_stale():
        build.build()
    mx.binding.host()
    return mx


def refused(mx, code, call, *args, **kw):
    """The call raises MxError with this code of the C interface."""
    with pytest.raises(mx.MxError) as e:
        call(*args, **kw)
    assert e.value.code == code, e.value
    return str(e.value)


def misaligned(*shape):
    n = 1
    for s in shape:
        n *= s
    return torch.zeros(n + 1)[1:].view(shape)


def test_refusals_carry_the_code_of_the_c_interface(mx):
    B = mx.binding
    lin = mx.MxLinear(64, 96, device="cpu")
    assert "MX_ERR_SHAPE (-2)" in refused(mx, B.MX_ERR_SHAPE, lin, torch.zeros(0, 64))
    step = mx.MxLinearStep(64, 64, 96, device="cpu")
    X, W, dY = torch.zeros(64, 64), torch.zeros(96, 64), torch.zeros(64, 96)
    refused(mx, B.MX_ERR_ALIGN, step.forward, misaligned(64, 64), W, 1)
    refused(mx, B.MX_ERR_ALIGN, step.forward, torch.zeros(64, 66)[:, :64], W, 1)
    refused(mx, B.MX_ERR_SHAPE, step.forward, X[:1].expand(64, 64), W, 1)
    refused(mx, B.MX_ERR_ALIGN, step.backward, misaligned(64, 96), 1)
    p = torch.nn.Parameter(misaligned(32))
    p.grad = torch.zeros(32)
    refused(mx, B.MX_ERR_ALIGN, mx.QRampingAdamW([], [p]).step)
    q = torch.nn.Parameter(torch.zeros(32))
    q.grad = misaligned(32)
    refused(mx, B.MX_ERR_ALIGN, mx.QRampingAdamW([], [q]).step)
    state = [{}]
    for bad in (dict(lr=-1.0), dict(b1=1.0), dict(b2=0.0), dict(eps=-1.0), dict(wd=float("nan"))):
        h = dict(lr=1e-3, b1=0.9, b2=0.999, eps=1e-8, wd=0.0, **{})
        h.update(bad)
        refused(mx, B.MX_ERR_MODE, B.host().ramping_step, [q], state, 0, False, 0, h["lr"], h["b1"], h["b2"], h["eps"], h["wd"])


def test_linear_refuses_sizes_the_kernels_do_not_take(mx):
    """weight is a parameter that a program may replace after the constructor's checks."""
    B = mx.binding
    for c, d in ((40, 64), (96, 48), (96, 0), (0, 64)):
        lin = mx.MxLinear(64, 96, bias=False, device="cpu")
        lin.weight = torch.nn.Parameter(torch.zeros(c, d))
        for grad in (True, False):
            with torch.set_grad_enabled(grad):
                refused(mx, B.MX_ERR_SHAPE, lin, torch.zeros(32, d))
    lin = mx.MxLinear(64, 96, qema=True, device="cpu")
    lin.w_ema = misaligned(96, 64)
    refused(mx, B.MX_ERR_ALIGN, lin, torch.zeros(32, 64))
    for beta in (1.0, -0.1, float("nan")):
        refused(mx, B.MX_ERR_MODE, mx.MxLinear(64, 96, qema=True, beta=beta, device="cpu"), torch.zeros(32, 64))
    with pytest.raises(ValueError):
        mx.MxLinear(64, 96, qema=True, device="cpu").to(torch.bfloat16)(torch.zeros(32, 64))


def test_unknown_scale_modes_are_refused(mx):
    B = mx.binding
    X, W, dY = torch.zeros(64, 64), torch.zeros(96, 64), torch.zeros(64, 96)
    for mode in (-1, 2, 7):
        step = mx.MxLinearStep(64, 64, 96, device="cpu", scale_mode=mode)
        refused(mx, B.MX_ERR_MODE, mx.MxLinear(64, 96, device="cpu", scale_mode=mode), X)
        refused(mx, B.MX_ERR_MODE, step.forward, X, W, 1)
        refused(mx, B.MX_ERR_MODE, step.backward, dY, 1)
        w = torch.nn.Parameter(torch.zeros(4, 64))
        refused(mx, B.MX_ERR_MODE, mx.QRampingAdamW([w], scale_mode=mode).step)          # the first step opens a window


def test_optimizer_refuses_lengths_the_kernels_do_not_take(mx):
    """A parameter group that is added later does not pass the constructor's checks."""
    B = mx.binding
    for shape, quantized in (((10,), False), ((0,), False), ((2, 48), True), ((1, 40), True), ((64,), True), ((0, 32), True)):
        opt = mx.QRampingAdamW([], [torch.nn.Parameter(torch.zeros(32))])
        p = torch.nn.Parameter(torch.zeros(shape))
        opt.add_param_group({"params": [p], "quantized": quantized})
        p.grad = torch.zeros(shape)
        if len(shape) == 2 or not quantized:
            refused(mx, B.MX_ERR_SHAPE, opt.step)
        else:
            with pytest.raises(ValueError):                                  # no rows and columns to make a state for
                opt.step()


def test_seeds_of_any_integer_type(mx):
    """What ctypes takes as a 64-bit word: any integer, modulo 2^64."""
    np = pytest.importorskip("numpy")
    for seed, word in ((3, 3), (True, 1), (-1, 2 ** 64 - 1), (2 ** 64 + 5, 5), (np.int64(7), 7), (np.uint64(2 ** 63), 2 ** 63), (np.int32(-2), 2 ** 64 - 2)):
        assert mx.binding.seed_args(seed) == (word, None)
    for seed in (1.5, "1", None):
        with pytest.raises(TypeError):
            mx.binding.seed_args(seed)
    t = torch.zeros(1, dtype=torch.int64)
    assert mx.binding.seed_args(t)[1] is t


def test_a_refused_call_does_not_start_the_moving_average(mx):
    lin = mx.MxLinear(64, 96, qema=True, device="cpu")
    for x in (torch.zeros(32, 32), torch.zeros(32, 64, dtype=torch.float16), torch.zeros(0, 64)):
        with pytest.raises(Exception):
            lin(x)
    assert not lin._ema_started                              # the next call starts it from the weight


def test_qema_is_looked_at_on_every_call(mx):
    lin = mx.MxLinear(64, 96, qema=True, device="cpu")
    lin.w_ema = misaligned(96, 64)
    refused(mx, mx.binding.MX_ERR_ALIGN, lin, torch.zeros(32, 64))
    lin.qema = False
    with pytest.raises(RuntimeError, match="runs on the GPU"):               # switched off: the buffer plays no part
        lin(torch.zeros(32, 64))
    lin = mx.MxLinear(64, 96, device="cpu")
    lin.qema = True
    with pytest.raises(ValueError):                                          # switched on without one
        lin(torch.zeros(32, 64))


@pytest.mark.parametrize("which", ["x", "weight", "bias"])
@pytest.mark.parametrize("frozen", [True, False])
def test_forward_mode_tangents_are_refused(mx, which, frozen):
    """A dual tensor does not require grad: with frozen weights, or under no_grad, nothing but this check sees it."""
    import torch.autograd.forward_ad as fwd
    lin, x = mx.MxLinear(64, 96, device="cpu").requires_grad_(not frozen), torch.zeros(32, 64)
    w, b = lin.weight.detach(), lin.bias.detach()
    with fwd.dual_level():
        dual = lambda t: fwd.make_dual(t, torch.ones_like(t))
        if which == "x":
            x = dual(x)
        elif which == "weight":
            del lin.weight
            lin.weight = dual(w)
        else:
            del lin.bias
            lin.bias = dual(b)
        for grad in (True, False):
            with torch.set_grad_enabled(grad), pytest.raises(NotImplementedError):
                lin(x)
        with fwd._set_fwd_grad_enabled(False), pytest.raises(RuntimeError, match="runs on the GPU"):     # tangents switched off
            lin(x)


def test_one_launch_where_it_is_not_slower(mx):
    """A second K step costs device time: a call that is recorded into a graph takes it only where the separate kernels take longer."""
    fits = mx.binding.host().linear_fits_one_launch
    for captured in (False, True):
        assert fits(197, 768, 192, True, captured) and fits(1, 1024, 256, False, captured) and fits(16384, 64, 256, False, captured)
        assert not fits(197, 768, 544, True, captured) and not fits(16385, 64, 256, False, captured)
    for m, n, k in ((1, 1024, 288), (512, 384, 384), (1576, 384, 384), (2000, 512, 512), (7168, 64, 480)):
        assert fits(m, n, k, False, False) and not fits(m, n, k, False, True)
    assert fits(7168, 64, 512, False, True) and fits(16384, 64, 288, False, True)            # an X of 3.5 M elements
    assert fits(64, 3072, 512, True, True) and not fits(64, 3072, 512, False, True) and not fits(64, 3040, 512, True, True)


def test_kernel_of_the_fused_gelu_stage(mx):
    """128 x 128 tiles beyond one round of the main kernel's tiles up to K = 896; where one round holds them all, up to K = 640 and
    in rounds filled to less than 70 %."""
    kernel = lambda m, n, k: mx.binding.host().gemm_kernel_name(m, n, k, True)
    for k in (768, 896):
        assert kernel(12608, 1024, k) == kernel(8192, 2048, k) == kernel(4096, 4096, k) == "main"
        assert kernel(11520, 1024, k) == "main" and kernel(11264, 1024, k) == "128x128"          # 180 and 176 of 256
        assert kernel(16640, 1024, k) == kernel(32768, 1024, k) == kernel(25216, 3072, k) == "128x128"
    for k in (512, 640):
        assert kernel(12608, 1024, k) == kernel(8192, 2048, k) == kernel(25216, 3072, k) == "128x128"
    assert kernel(25216, 3072, 1024) == kernel(25216, 3072, 4096) == "main" and kernel(16640, 1024, 2048) == "128x128"
    assert kernel(1024, 4096, 896) == "64x64"


def test_tail_of_a_tile_quantizer_launch(mx):
    """The tiles beyond a multiple of 256 (one per compute unit) are issued as halves where they are up to 128, or 64 of FP32 with
    nothing stochastic; with more of them up to a quarter of a round, unless six waves share a SIMD and all run at once as they are."""
    groups = lambda tiles, src, row_sr, t_sr: mx.binding.host().tile_workgroups(128 * tiles, 128, src, row_sr, t_sr)
    for src, row_sr, t_sr in ((1, False, False), (1, True, False), (0, True, False), (1, False, True), (0, False, False), (0, True, True)):
        tail = lambda tiles: groups(tiles, src, row_sr, t_sr) - tiles
        few = 64 if (src, row_sr, t_sr) == (0, False, False) else 128
        assert tail(1) == 1 and tail(128) == 128 and tail(256) == 0 and tail(257) == 1 and tail(512 + few) == few and tail(512 + few + 1) == 0
        for base in (768, 1024, 1280, 1536, 2304):
            assert tail(base) == 0 and tail(base + 1) == 1 and tail(base + few) == few
        assert tail(768 + few + 1) == 0 and tail(1600) == 64 and tail(2304 + few + 1) == 0
        six = not t_sr and (src == 1 or row_sr)
        assert tail(1280 + few + 1) == (0 if six and few == 128 else few + 1)                     # 1409 to 1536 tiles
        assert tail(1536 - 1) == (0 if six else 255)
        assert tail(2560 + 255) == 255 and tail(1792 + 129) == 0
    assert groups(1024, 2, False, True) == 1024 and groups(1025, 2, False, True) == 1026 and groups(2048 + 200, 2, False, True) == 2448
    assert groups(1280, 1, True, True) == 1280 and groups(1024 + 200, 1, True, True) == 1424 and groups(1280 + 200, 1, True, True) == 1480
    assert groups(200, 2, False, True) == groups(200, 1, True, True) == 400 and groups(513, 0, False, True) == 514
