"""FP32 filter banks on the matrix cores, at the edges of their tiles and
channel blocks.  Integer values small enough that every sum is exact in FP32
(|x|, |f|, |g| <= 4: at most 64 * 25 * 16 < 2^24 per output, and 16 per pixel
of a filter gradient), so every result equals the FP64 oracle's exactly."""
import numpy as np
import pytest
import torch

import oracle
from paper_2504_01266_amd import workloads as wl

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def ints(seed, *shape):
    return wl.rng(seed, *shape).integers(-4, 5, shape).astype(np.float32)


# (n, C_in, C_out): one to four output blocks per work-group, several groups,
# padded channels on either side, more source channels than one staging step
CHANNELS = [(2, 16, 64), (1, 64, 16), (1, 3, 16), (1, 8, 8), (1, 12, 24), (1, 33, 17), (1, 16, 48), (1, 20, 130)]
# widths and heights around the 64-column strips, the 8-row tiles and the
# 16-byte chunks; the narrowest the kernels take
SIZES = [(1, 4), (2, 5), (7, 63), (8, 64), (9, 65), (17, 131), (70, 33)]


@pytest.mark.parametrize("k", [1, 3, 5])
@pytest.mark.parametrize("nio", CHANNELS)
@pytest.mark.parametrize("hw", SIZES)
def test_forward_and_gradients_exact(gpu_lib, nio, hw, k):
    n, ci, co = nio
    x, f, g = ints(1, n, ci, *hw), ints(2, co, ci, k, k), ints(3, n, co, *hw)
    print(nio, hw, k, flush=True)
    for border in ("clamp", "zero"):
        y = gpu_lib.forward(dev(x), dev(f), mode="bank", border=border)
        ref = oracle.forward(x.astype(np.float64), f.astype(np.float64), "bank", border=border)
        assert np.array_equal(y.double().cpu().numpy(), ref), border
    gi, gf = gpu_lib.backward(dev(x), dev(f), dev(g), mode="bank")
    assert np.array_equal(gi.double().cpu().numpy(),
                          oracle.grad_input(g.astype(np.float64), f.astype(np.float64), x.shape, "bank"))
    assert np.array_equal(gf.double().cpu().numpy(),
                          oracle.grad_filter(x.astype(np.float64), g.astype(np.float64), f.shape, "bank"))


@pytest.mark.parametrize("k", [3, 5])
def test_views_with_odd_strides(gpu_lib, k):
    """Unaligned rows, channel and image strides of a larger buffer, on every
    operand; nothing outside the output views is written."""
    r = wl.rng(7, k)
    big = lambda c: dev(r.integers(-4, 5, (3, c + 2, 41, 83)).astype(np.float32))  # noqa: E731
    xb, gb, yb, ib = big(16), big(32), big(32), big(16)
    cut = lambda t, c: t[::2, 1:1 + c, 2:39, 3:78]  # noqa: E731
    x, g, y, gi = cut(xb, 16), cut(gb, 32), cut(yb, 32), cut(ib, 16)
    f = dev(ints(8, 32, 16, k, k))
    host = lambda t: t.double().cpu().numpy()  # noqa: E731
    y_keep, i_keep = yb.clone(), ib.clone()
    gpu_lib.forward(x, f, mode="bank", outs=[y])
    assert np.array_equal(host(y), oracle.forward(host(x), host(f), "bank"))
    _, gf = gpu_lib.backward(x, f, g, mode="bank", grad_input=gi)
    assert np.array_equal(host(gi), oracle.grad_input(host(g), host(f), tuple(x.shape), "bank"))
    assert np.array_equal(host(gf), oracle.grad_filter(host(x), host(g), tuple(f.shape), "bank"))
    cut(y_keep, 32).copy_(y)
    cut(i_keep, 16).copy_(gi)
    assert torch.equal(yb, y_keep) and torch.equal(ib, i_keep)


@pytest.mark.parametrize("nio", [(1, 16, 64), (1, 40, 16)])
def test_bands_equal_the_whole_bitwise(gpu_lib, nio):
    n, ci, co = nio
    k, h, w = 3, 45, 100
    x = dev(wl.rng(9, ci).standard_normal((n, ci, h, w), dtype=np.float32))
    f = dev(wl.rng(10, ci).standard_normal((co, ci, k, k), dtype=np.float32))
    whole = gpu_lib.forward(x, f, mode="bank")
    parts = []
    for y0, y1 in [(0, 1), (1, 14), (14, 40), (40, 45)]:
        lo, hi = max(0, y0 - 1), min(h, y1 + 1)
        parts.append(gpu_lib.forward(x[:, :, lo:hi], f, mode="bank", rows=(y0 - lo, y1 - lo)))
    assert torch.equal(torch.cat(parts, dim=2), whole)


def test_gradients_repeat_bitwise(gpu_lib):
    x = dev(wl.rng(11, 1).standard_normal((2, 16, 90, 150), dtype=np.float32))
    f = dev(wl.rng(11, 2).standard_normal((64, 16, 3, 3), dtype=np.float32))
    g = dev(wl.rng(11, 3).standard_normal((2, 64, 90, 150), dtype=np.float32))
    a = gpu_lib.backward(x, f, g, mode="bank")
    b = gpu_lib.backward(x, f, g, mode="bank")
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


@pytest.mark.parametrize("case", [(32, 64, 256, 70, 4, 1), (32, 64, 256, 66, 5, 3), (512, 16, 16, 258, 4, 3)])
def test_weight_gradient_over_several_row_segments(gpu_lib, case):
    """Units with more rows than a wave adds up before its sums go to memory
    (with one and with four row splits), so the partials are added to."""
    n, ci, co, h, w, k = case
    x, g = ints(12, n, ci, h, w), ints(13, n, co, h, w)
    f = ints(14, co, ci, k, k)
    print(case, flush=True)
    _, gf = gpu_lib.backward(dev(x), dev(f), dev(g), mode="bank", need_input=False)
    assert np.array_equal(gf.double().cpu().numpy(),
                          oracle.grad_filter(x.astype(np.float64), g.astype(np.float64), f.shape, "bank"))


def test_autotuning_a_bank_with_one_tiling_records_nothing(gpu_lib, tmp_path):
    """The FP32 banks on the matrix cores have no tiling variants: autotuning
    one reports variant 1 and leaves the table alone (its key is shared with
    VALU banks of few channels)."""
    x, f = ints(15, 1, 16, 40, 70), ints(16, 64, 16, 3, 3)
    gpu_lib.tune_clear()
    try:
        assert gpu_lib.autotune_forward(dev(x), dev(f), mode="bank") == 1
        gpu_lib.tune_save(str(tmp_path / "tune.json"))
        assert "[0, 2, 3, 2," not in (tmp_path / "tune.json").read_text()
    finally:
        gpu_lib.tune_clear()
