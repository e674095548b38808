"""Seeded sweeps of shapes and flags (all within the documented limits): quantizers bit for bit against
the oracle, products against the FP64 product, on shapes no other test names."""
import numpy as np
import pytest
import torch

from test_gpu_parity import assert_same_bytes, check_product, dev, host, mixed_matrix, mx, random_packed  # noqa: F401

pytestmark = pytest.mark.gpu


def test_sweep_row_quantizer(mx, orc):
    rng = np.random.default_rng(101)
    for case in range(40):
        rows, cols = int(rng.integers(1, 300)), 32 * int(rng.integers(1, 40))
        pad = 8 * int(rng.integers(0, 4))
        dtype = ("f32", "bf16")[case % 2]
        rnd, mode = int(rng.integers(0, 2)), int(rng.integers(0, 2))
        seed, tid, base = int(rng.integers(0, 2 ** 63)), int(rng.integers(0, 2 ** 32)), 8 * int(rng.integers(0, 2 ** 40))
        x = mixed_matrix(rows, cols + pad, seed=200 + case, dtype=dtype)[:, :cols]      # ld = cols + pad
        want = orc.quantize(np.ascontiguousarray(x), round=rnd, scale_mode=mode, seed=seed, tensor_id=tid, index_base=base)
        src = dev(mixed_matrix(rows, cols + pad, seed=200 + case, dtype=dtype), dtype)[:, :cols]
        got = mx.mx_quantize(src, rnd, mode, seed=seed, tensor_id=tid, index_base=base)
        what = "case %d: %dx%d ld %d %s round %d mode %d" % (case, rows, cols, cols + pad, dtype, rnd, mode)
        assert_same_bytes(got[1], want[1], what + " scales")
        assert_same_bytes(got[0], want[0], what + " codes")


def test_sweep_transposed_quantizer(mx, orc):
    rng = np.random.default_rng(102)
    shapes = [(32 * int(rng.integers(1, 30)), 32 * int(rng.integers(1, 30))) for _ in range(28)]
    shapes += [(4096 + 32 * int(rng.integers(0, 64)), 4096 + 32 * int(rng.integers(0, 40))) for _ in range(3)]   # wide tiles + tail
    shapes += [(32 * int(rng.integers(600, 900)), 32 * int(rng.integers(20, 30))) for _ in range(3)]            # tall and narrow
    for case, (rows, cols) in enumerate(shapes):
        dtype = ("bf16", "f32")[case % 2]
        round_t, round_row, pre = int(rng.integers(0, 2)), int(rng.integers(0, 2)), int(rng.integers(0, 2))
        mode, want_row = int(rng.integers(0, 2)), bool(rng.integers(0, 4) > 0)
        seed, base = int(rng.integers(0, 2 ** 63)), 8 * int(rng.integers(0, 2 ** 36))
        pad = 8 * int(rng.integers(0, 3))
        full = mixed_matrix(rows, cols + pad, seed=300 + case, dtype=dtype)
        kw = dict(round_t=round_t, tensor_id_t=6, pre_quant=pre, want_row=want_row, round_row=round_row, tensor_id_row=1,
                  scale_mode=mode, seed=seed, index_base=base)
        want = orc.quantize_transposed(np.ascontiguousarray(full[:, :cols]), **kw)
        got = mx.mx_quantize_transposed(dev(full, dtype)[:, :cols], **kw)
        what = "case %d: %dx%d ld %d %s t %d row %d pre %d mode %d" % (case, rows, cols, cols + pad, dtype, round_t, round_row, pre, mode)
        for g, w, nm in zip(got, want, ("codes_t", "scales_t", "codes_row", "scales_row")):
            if w is None:
                assert g is None
            else:
                assert_same_bytes(g, w, what + " " + nm)


def test_sweep_products(mx, orc):
    rng = np.random.default_rng(103)
    for case in range(36):
        m, n = int(rng.integers(1, 700)), int(rng.integers(1, 700))
        k = 32 * int(rng.integers(1, 12)) if case % 3 == 0 else 128 * int(rng.integers(1, 24))
        ac, as_ = random_packed(m, k, 400 + case)
        bc, bs = random_packed(n, k, 500 + case)
        out = torch.float32 if case % 4 else torch.bfloat16
        if n % 4 == 0 and case % 2:
            bias = rng.standard_normal(n).astype(np.float32)
            got = mx.mx_linear_fwd_bias(dev(ac), dev(as_), dev(bc), dev(bs), dev(bias), out_dtype=torch.float32)
            ref = orc.gemm_f64(ac, as_, bc, bs) + bias.astype(np.float64)[None, :]
            absref = np.abs(orc.dequantize(ac, as_)) @ np.abs(orc.dequantize(bc, bs)).T + np.abs(bias)[None, :]
            err = np.abs(host(got).astype(np.float64) - ref)
            assert np.all(err <= 1e-5 * absref), ("case %d: %dx%dx%d with bias" % (case, m, n, k), (err / absref).max())
            continue
        got = mx.mx_linear_fwd(dev(ac), dev(as_), dev(bc), dev(bs), out_dtype=out).float()
        check_product(orc, got, ac, as_, bc, bs, "case %d: %dx%dx%d" % (case, m, n, k),
                      tol=1e-5 if out == torch.float32 else 2.0 ** -8)


@pytest.mark.parametrize("m,n,k", [
    # 64 x 64 tiles (up to 256 of them): one row, tile edges, one K step, several, ragged tails of 32, 64 and 96
    (1, 4, 32), (64, 64, 512), (65, 63, 544), (63, 129, 1120), (224, 192, 768), (1024, 1024, 96),
    # one tile more: 128 x 64 tiles, up to 768 of them
    (1025, 1024, 96), (1031, 1030, 288), (4096, 1536, 160),
    # one more: 128 x 128 tiles; K % 128 == 0 below and above 512
    (4097, 1536, 160), (12801, 452, 384), (12672, 578, 416),
    # in steps of 128 up to K = 256, all of K at once above that: ragged K, rows and columns that end inside a wave's tile
    (12801, 452, 256), (12801, 452, 288), (4163, 1570, 352),
    # the main kernel from 128 tiles of 256 x 256 on (ragged edges, shifted last scale block)
    (32765, 250, 640), (32641, 36, 512), (8200, 1028, 1152),
    # short K, a second round of 256 x 256 tiles that is less than a quarter full: 128 x 128 tiles; one more K step
    (8450, 2044, 768), (8450, 2044, 896),
    # K splits of the 64 x 64 and 128 x 64 tiles (uneven, ragged K), and of the main kernel
    (100, 132, 4128), (192, 768, 12608), (1100, 2080, 8224), (516, 764, 41088)])
def test_products_at_the_lines_between_kernels(mx, orc, m, n, k):
    ac, as_ = random_packed(m, k, 600 + m % 97)
    bc, bs = random_packed(n, k, 700 + n % 89)
    got = mx.mx_linear_fwd(dev(ac), dev(as_), dev(bc), dev(bs))
    check_product(orc, got, ac, as_, bc, bs, "%dx%dx%d" % (m, n, k))
    if n % 4 == 0:                                       # bf16 with bias: one rounding of the FP32 sum
        bias = np.linspace(-2, 2, n, dtype=np.float32)
        y = mx.mx_linear_fwd_bias(dev(ac), dev(as_), dev(bc), dev(bs), dev(bias), out_dtype=torch.bfloat16)
        assert torch.equal(y, (got + dev(bias)).bfloat16())


@pytest.mark.parametrize("m,n,k", [
    # 64 x 64 tiles, up to 1024 of them: one row, edges, a column count that ends inside a tile
    (1, 32, 512), (33, 544, 640), (1000, 4096, 512),
    # 128 x 128 tiles: one row of tiles more, edges in rows and columns (scale rows of odd length)
    (1025, 4096, 512), (1632, 2720, 512),
    # one well-filled round of the main kernel's tiles: 128 x 128 up to K = 640, the main kernel beyond; more than one round:
    # 128 x 128 up to K = 896.  Edges in rows and columns
    (4063, 3040, 512), (4063, 3040, 896), (4063, 3040, 1024), (4100, 1120, 2176), (4063, 3040, 768), (5700, 3040, 896)])
def test_fused_gelu_at_the_lines_between_kernels(mx, orc, m, n, k):
    """The pre-activation is what mx_linear_fwd_bias stores, and the codes are round_D of GELU of it: every kernel of the
    fused stage takes the FP32 sum, so dequantized values differ from the oracle's only next to a threshold
    (GELU's error is below 2^-18 of the value; a threshold is met with that probability)."""
    xc, xs = random_packed(m, k, 800 + m % 97)
    wc, ws = random_packed(n, k, 900 + n % 89)
    ws[:] = 127 - 8                                      # pre-activations of order 1 and 10
    xs[:] = 127 + np.arange(m, dtype=np.int64)[:, None] % 4
    bias = np.linspace(-3, 3, n, dtype=np.float32)
    args = (dev(xc), dev(xs), dev(wc), dev(ws), dev(bias))
    for mode in (0, 1):
        y, aq, as_ = mx.mx_linear_fwd_gelu_quant(*args, out_dtype=torch.float32, scale_mode=mode)
        assert torch.equal(y, mx.mx_linear_fwd_bias(*args, out_dtype=torch.float32))
        A = orc.gelu(y.cpu().numpy().astype(np.float64)).astype(np.float32)
        want_c, want_s = orc.quantize(A, scale_mode=mode)
        got, want = orc.dequantize(host(aq), host(as_)), orc.dequantize(want_c, want_s)
        # one group's scale may move with its maximum, one value's code at a threshold: 2^-17 of the values, and a few
        assert np.count_nonzero(got != want) <= 32 * (1 + m * n // 2 ** 17), (m, n, k, mode)
        assert np.count_nonzero(host(as_) != want_s) <= 1 + m * n // 2 ** 22, (m, n, k, mode)


@pytest.mark.parametrize("rows,cols", [(32, 32), (96, 64), (128, 128), (160, 96), (256, 160), (288, 2080), (2112, 8256)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_fused_quantizer_at_the_edges_of_its_tiles(mx, orc, rows, cols, dtype):
    """Macro tiles of 128 rows x 128 or 64 columns (the last shape has 128-column tiles and a tail of halves): both sources and
    packed codes, both roundings, bit for bit."""
    x = mixed_matrix(rows, cols, seed=1000 + rows + cols, dtype=dtype)
    for rnd, pre in ((1, 1), (1, 0), (0, 0), (0, 1)):
        kw = dict(round_t=rnd, tensor_id_t=6, pre_quant=pre, round_row=rnd if pre == 0 else 0, tensor_id_row=1, seed=7)
        got, want = mx.mx_quantize_transposed(dev(x, dtype), **kw), orc.quantize_transposed(x, **kw)
        for g, w, nm in zip(got, want, ("codes_t", "scales_t", "codes_row", "scales_row")):
            assert_same_bytes(g, w, "%s round %d pre %d %s" % (dtype, rnd, pre, nm))
        if pre:
            t = mx.mx_quantize_transposed(None, rnd, 6, 1, False, row_in=(got[2], got[3]), seed=7, shape=(rows, cols))
            assert_same_bytes(t[0], want[0], "codes_t from packed codes")
            assert_same_bytes(t[1], want[1], "scales_t from packed codes")


@pytest.mark.parametrize("rows,cols,rt,pre", [(9248, 4128, 0, 0), (9248, 4128, 0, 1), (14368, 8224, 1, 1), (14368, 8224, 1, 0)])
def test_fused_quantizer_of_large_f32_sources(mx, orc, rows, cols, rt, pre):
    """From 36 Mi elements on (112 Mi with stochastic column groups) macro tiles of 256 rows: the last one 32 rows tall and
    32 columns wide, bit for bit."""
    x = np.tile(mixed_matrix(rows // 4, cols // 4, seed=rows + pre, dtype="f32"), (4, 4))
    kw = dict(round_t=rt, tensor_id_t=6, pre_quant=pre, round_row=rt if pre == 0 else 0, tensor_id_row=1, seed=7)
    got, want = mx.mx_quantize_transposed(dev(x), **kw), orc.quantize_transposed(x, **kw)
    for g, w, nm in zip(got, want, ("codes_t", "scales_t", "codes_row", "scales_row")):
        assert_same_bytes(g, w, nm)


@pytest.mark.parametrize("before", [0, 1, 40, 700, 10 ** 6])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_block_numbers_across_a_counter_word(mx, orc, dtype, before):
    """Philox block numbers reach 2^32 `before` blocks into the tensor (0: they start there, 10^6: they stay below)."""
    rows, cols, base = 160, 224, (1 << 35) - 8 * before
    x = mixed_matrix(rows, cols, seed=900, dtype=dtype)
    src, key = dev(x, dtype), dict(seed=(5 << 40) + 9, index_base=base)
    got, want = mx.mx_quantize(src, 1, 0, tensor_id=3, **key), orc.quantize(x, round=1, scale_mode=0, tensor_id=3, **key)
    for g, w, nm in zip(got, want, ("codes", "scales")):
        assert_same_bytes(g, w, "rows " + nm)
    for pre, round_row in ((0, 1), (1, 0), (1, 1)):
        kw = dict(round_t=1, tensor_id_t=5, pre_quant=pre, want_row=True, round_row=round_row, tensor_id_row=3, **key)
        for g, w, nm in zip(mx.mx_quantize_transposed(src, **kw), orc.quantize_transposed(x, **kw), ("codes_t", "scales_t", "codes_row", "scales_row")):
            assert_same_bytes(g, w, "pre %d row %d %s" % (pre, round_row, nm))
    kw = dict(round_t=1, tensor_id_t=6, pre_quant=1, want_row=False, **key)
    got = mx.mx_quantize_transposed(None, 1, 6, 1, False, row_in=mx.mx_quantize(src), shape=(rows, cols), **key)
    for g, w, nm in zip(got[:2], orc.quantize_transposed(x, **kw)[:2], ("codes_t", "scales_t")):
        assert_same_bytes(g, w, "from packed codes " + nm)


@pytest.mark.parametrize("rows", [40960, 40992, 82112, 102432])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_transposed_at_the_lines_between_tile_widths(mx, orc, dtype, rows):
    """192 columns: 640, 642, 1284 and 1602 tiles of 128 columns, the last 128, 0, 4 and 66 as halves."""
    x = mixed_matrix(rows, 192, seed=901, dtype=dtype)
    src = dev(x, dtype)
    for pre, round_row in ((1, 0), (0, 1)):
        kw = dict(round_t=1, tensor_id_t=6, pre_quant=pre, want_row=True, round_row=round_row, tensor_id_row=1, seed=77)
        for g, w, nm in zip(mx.mx_quantize_transposed(src, **kw), orc.quantize_transposed(x, **kw), ("codes_t", "scales_t", "codes_row", "scales_row")):
            assert_same_bytes(g, w, "%d rows pre %d row %d %s" % (rows, pre, round_row, nm))


@pytest.mark.parametrize("rows", [57472, 90112, 90240, 98336])
def test_deterministic_transposed_at_the_lines_between_tile_widths(mx, orc, rows):
    """192 bf16 columns, both outputs deterministic: 898, 1408, 1410 and 1538 tiles; the last 0, 128, 0 and 2 are issued as halves."""
    x = mixed_matrix(rows, 192, seed=902, dtype="bf16")
    kw = dict(round_t=0, tensor_id_t=6, pre_quant=0, want_row=True, round_row=0, tensor_id_row=1, seed=77)
    for g, w, nm in zip(mx.mx_quantize_transposed(dev(x, "bf16"), **kw), orc.quantize_transposed(x, **kw), ("codes_t", "scales_t", "codes_row", "scales_row")):
        assert_same_bytes(g, w, "%d rows %s" % (rows, nm))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("m,n,k", [(200, 132, 96), (3100, 2056, 96), (6300, 1064, 160), (6400, 1064, 352), (3200, 2080, 512)])
def test_products_into_padded_and_shifted_rows(mx, dtype, m, n, k):
    """Rows of whole 64-byte sectors and others, below and above 24 MB: the values do not depend on where they are stored, and nothing
    outside of the matrix is written.  The last size also through the fused GELU stage."""
    (ac, as_), (bc, bs) = random_packed(m, k, 31), random_packed(n, k, 32)
    bs[:] = 127 - 8
    a, s, b, t = dev(ac), dev(as_), dev(bc), dev(bs)
    bias = torch.linspace(-2, 2, n, device="cuda")
    want = mx.mx_linear_fwd_bias(a, s, b, t, bias, out_dtype=dtype)
    es = want.element_size()
    for pad, shift in ((0, 0), (16, 0), (16, 16), (64 - n * es % 64, 0), (64 - n * es % 64, 16), (80, 48)):
        pitch = n + pad // es
        flat = torch.full((m * pitch + 64,), 7.0, dtype=dtype, device="cuda")
        out = flat[shift // es: shift // es + m * pitch].view(m, pitch)[:, :n]
        rest = torch.ones_like(flat, dtype=torch.bool)
        rest[shift // es: shift // es + m * pitch].view(m, pitch)[:, :n] = False
        for fused in (False, True) if k >= 512 and n % 32 == 0 else (False,):
            out.zero_()
            if fused:
                mx.mx_linear_fwd_gelu_quant(a, s, b, t, bias, out=out)
            else:
                mx.mx_linear_fwd_bias(a, s, b, t, bias, out=out)
            assert torch.equal(out, want), (pad, shift, fused)
            assert bool((flat[rest] == 7.0).all()), (pad, shift, fused)
