"""The element codec over its whole domain, through the public quantizers and bit for bit against the oracle: every bf16
value under every scale that a group with it can have, every code times every pair of row and column scales, and FP32
thresholds with their neighbours at every scale.  These are what the FP4 conversion instructions of gfx950 stand on."""
import numpy as np
import pytest
import torch

from test_gpu_parity import assert_same_bytes, dev, mx  # noqa: F401

pytestmark = pytest.mark.gpu

NAMES = ("codes_t", "scales_t", "codes_row", "scales_row")


def bf16(patterns):
    return (np.asarray(patterns, np.uint32) << 16).view(np.float32)


def f32(patterns):
    return np.asarray(patterns, np.uint32).view(np.float32)


def largest_of_each_scale(orc, mode):
    """{scale byte: largest bf16 magnitude (as a pattern) of a group with that byte}"""
    last = {}
    for p in range(1, 0x7F80):
        last[orc.shared_exponent(bf16([p])[0], mode) + 127] = p
    return last


def groups_of(values, maximum):
    """Rows of 32: the group's maximum, then 31 of the values (padded with zeros)."""
    n = -(-values.size // 31)
    out = np.zeros((n, 32), np.float32)
    out[:, 0] = maximum
    flat = np.zeros(n * 31, np.float32)
    flat[: values.size] = values
    out[:, 1:] = flat.reshape(n, 31)
    return out


def whole(groups):
    """A multiple of 32 groups (the last one repeated)."""
    return np.concatenate([groups] + [groups[-1:]] * (-groups.shape[0] % 32))


def check_rows_and_columns(mx, orc, x, dtype, mode, pre):
    for rnd in (0, 1):
        got, want = mx.mx_quantize(dev(x, dtype), rnd, mode, seed=5, tensor_id=3), orc.quantize(x, round=rnd, scale_mode=mode, seed=5, tensor_id=3)
        assert_same_bytes(got[1], want[1], "row scales, round %d mode %d" % (rnd, mode))
        assert_same_bytes(got[0], want[0], "row codes, round %d mode %d" % (rnd, mode))
        xt = np.ascontiguousarray(x.T)                     # the groups as 32x1 column groups
        kw = dict(round_t=rnd, tensor_id_t=6, pre_quant=pre, round_row=0 if pre else rnd, tensor_id_row=1, scale_mode=mode, seed=5)
        for g, w, nm in zip(mx.mx_quantize_transposed(dev(xt, dtype), **kw), orc.quantize_transposed(xt, **kw), NAMES):
            assert_same_bytes(g, w, "%s, round %d mode %d" % (nm, rnd, mode))


@pytest.mark.parametrize("mode", [0, 1])
def test_every_bf16_value_under_every_scale(mx, orc, mode):
    both = lambda p: np.concatenate([p, p | 0x8000])
    parts = [groups_of(bf16(both(np.arange(0, last + 1, dtype=np.uint32))), bf16([last])[0])
             for _, last in sorted(largest_of_each_scale(orc, mode).items())]
    check_rows_and_columns(mx, orc, whole(np.concatenate(parts)), "bf16", mode, 0)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("pre", [0, 1])
def test_f32_thresholds_and_neighbours_at_every_scale(mx, orc, mode, pre):
    rng = np.random.default_rng(mode)
    points = np.array([0, 0.25, 0.5, 0.75, 1, 1.25, 1.5, 1.75, 2, 2.5, 3, 3.5, 4, 5, 6, 7, 7.5], np.float64)
    parts = []
    for byte, last in sorted(largest_of_each_scale(orc, mode).items()):
        if pre and byte > 251:                             # |x| < 2^126 with double quantization
            continue
        top = int(last) << 16
        with np.errstate(over="ignore"):                   # what overflows is above the group's maximum
            p = (points * 2.0 ** (byte - 127)).astype(np.float32).view(np.uint32).astype(np.int64)
        p = np.concatenate([p + d for d in range(-3, 4)] + [np.arange(8), rng.integers(0, top + 1, 64), top - rng.integers(0, min(top, 1 << 24) + 1, 64)])
        p = p[(p >= 0) & (p <= top)]
        parts.append(groups_of(f32(np.concatenate([p, p | 0x80000000])), f32([top])[0]))
    x = whole(np.concatenate(parts))
    if pre:                                                # column groups across the scales as well: small ones under large ones
        x = np.concatenate([x, x[rng.permutation(x.shape[0])]])
    check_rows_and_columns(mx, orc, x, "f32", mode, pre)


@pytest.mark.parametrize("mode", [0, 1])
def test_every_code_at_every_pair_of_scales(mx, orc, mode):
    """Blocks of 32 rows x 32 columns of packed row results: row 0 holds 6 at one scale, the others every code at 31 scales,
    or all at that of row 0."""
    B = np.arange(0, 252)
    blocks = [(big, np.full(31, big)) for big in B] + [(big, B[i : i + 31]) for big in B for i in range(0, B.size, 31)]
    blocks += [blocks[-1]] * (-len(blocks) % 4)
    rows, cols = 32, 32 * len(blocks)
    codes = np.zeros((rows, cols), np.uint8)
    scales = np.zeros((rows, len(blocks)), np.uint8)
    for k, (big, small) in enumerate(blocks):
        codes[0, 32 * k : 32 * k + 32] = 7
        scales[0, k] = big
        codes[1:, 32 * k : 32 * k + 32] = np.arange(32) % 16
        scales[1 : 1 + small.size, k] = small
    packed = np.ascontiguousarray(codes[:, ::2] | codes[:, 1::2] << 4)
    for rnd in (0, 1):
        for seed in (1, 2):
            got = mx.mx_quantize_transposed(None, rnd, 6, 1, False, row_in=(dev(packed), dev(scales)), scale_mode=mode, seed=seed, shape=(rows, cols))
            want = orc.quantize_transposed(np.zeros((rows, cols), np.float32), round_t=rnd, tensor_id_t=6, pre_quant=1, want_row=False,
                                           row_in=(packed, scales), scale_mode=mode, seed=seed)
            assert_same_bytes(got[1], want[1], "scales, round %d" % rnd)
            assert_same_bytes(got[0], want[0], "codes, round %d" % rnd)
