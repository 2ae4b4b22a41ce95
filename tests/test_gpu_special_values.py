"""Infinities, NaN and subnormal values through the FP32 banks on the matrix
cores, which pad channels to fours and sixteens, and the 8-bit 3 x 3 filter
with its dot products.  Padded channels must not reach a result: an output is
infinite or NaN where its own terms say so.  (A weight gradient's padded pixels
do reach it: zero times what the image's last columns hold.)"""
import numpy as np
import pytest
import torch

import oracle
from paper_2504_01266_amd import workloads as wl
from test_bank_routes import valu_workspace

pytestmark = pytest.mark.gpu

CASES = [(2, 16, 64, 9, 70), (1, 19, 37, 17, 64), (1, 64, 16, 11, 131)]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    return t.double().cpu().numpy()


def nonzero_ints(r, *shape):
    return (r.integers(1, 5, shape) * r.choice([-1, 1], shape)).astype(np.float32)


def weight_gradient(x, g, k):
    """F-bar in 64 bits, every product taken as it is."""
    n, _, h, w = x.shape
    q = (k - 1) // 2
    out = np.empty((g.shape[1], x.shape[1], k, k))
    for u in range(k):
        rows = np.clip(np.arange(h) + u - q, 0, h - 1)
        for v in range(k):
            cols = np.clip(np.arange(w) + v - q, 0, w - 1)
            s = x[:, :, rows][..., cols]
            for o in range(g.shape[1]):
                out[o, :, u, v] = (g[:, o, None] * s).sum(axis=(0, 2, 3))
    return out


def same(got, want):
    np.testing.assert_array_equal(got, want)  # (NaN equals NaN here)


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("k", [1, 3, 5])
@pytest.mark.filterwarnings("ignore:invalid value")
def test_infinities_and_nan_in_fp32_banks(gpu_lib, case, k):
    n, ci, co, h, w = case
    r = wl.rng(91, *case, k)
    x, g, f = nonzero_ints(r, n, ci, h, w), nonzero_ints(r, n, co, h, w), nonzero_ints(r, co, ci, k, k)
    # (the last channels and corners of the image among them)
    for i, v in enumerate((np.inf, -np.inf, np.nan)):
        x[i % n, (ci - 1, 0, ci // 2)[i], (0, h - 1, h // 2)[i], (0, 40, 17)[i]] = v
        g[i % n, (co - 1, 0, co // 2)[i], (h - 1, 0, h // 2)[i], (w - 1, 0, 33)[i]] = v
    x64, g64, f64 = (a.astype(np.float64) for a in (x, g, f))
    print(case, k, flush=True)
    for border in ("clamp", "zero"):
        same(host(gpu_lib.forward(dev(x), dev(f), mode="bank", border=border)),
             oracle.forward(x64, f64, "bank", border=border))
    gi, _ = gpu_lib.backward(dev(x), dev(f), dev(g), mode="bank", need_filter=False)
    same(host(gi), oracle.grad_input(g64, f64, x.shape, "bank"))
    # infinite weights meet no padded channel either
    f[co - 1, ci - 1, 0, 0], f[0, 0, k - 1, k - 1] = np.inf, -np.inf
    x = nonzero_ints(r, n, ci, h, w)
    same(host(gpu_lib.forward(dev(x), dev(f), mode="bank")),
         oracle.forward(x.astype(np.float64), f.astype(np.float64), "bank"))


WEIGHT_CASES = [(2, 16, 64, 90, 90, 1), (1, 24, 37, 170, 128, 1), (2, 16, 64, 9, 70, 3), (1, 24, 37, 17, 64, 3),
                (1, 64, 60, 11, 131, 3), (2, 16, 64, 9, 70, 5), (9, 30, 32, 17, 64, 5), (1, 64, 60, 11, 131, 5)]


@pytest.mark.parametrize("case", WEIGHT_CASES)
@pytest.mark.filterwarnings("ignore:invalid value")
def test_infinities_and_nan_in_fp32_weight_gradients(gpu_lib, case):
    n, ci, co, h, w, k = case
    r = wl.rng(93, *case)
    x, g = nonzero_ints(r, n, ci, h, w), nonzero_ints(r, n, co, h, w)
    for i, v in enumerate((np.inf, -np.inf, np.nan)):
        x[i % n, (ci - 1, 0, ci // 2)[i], (0, h - 1, h // 2)[i], (0, 40, 17)[i]] = v
        g[i % n, (co - 1, 0, co // 2)[i], (h - 1, 0, h // 2)[i], (w - 1, 0, 33)[i]] = v
    f = dev(np.zeros((co, ci, k, k), np.float32))
    print(case, flush=True)
    assert gpu_lib.backward_workspace(dev(x), f, "bank") != valu_workspace(n, ci, co, h, w, k)
    _, gf = gpu_lib.backward(dev(x), f, dev(g), mode="bank", need_input=False)
    same(host(gf), weight_gradient(x.astype(np.float64), g.astype(np.float64), k))


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("k", [1, 3, 5])
def test_subnormal_values_in_fp32_banks(gpu_lib, case, k):
    """Whole multiples of the smallest subnormal: every sum is one too, exact."""
    n, ci, co, h, w = case
    r = wl.rng(92, *case, k)
    tiny = np.float32(2.0 ** -149)
    x, g, f = nonzero_ints(r, n, ci, h, w), nonzero_ints(r, n, co, h, w), nonzero_ints(r, co, ci, k, k)
    print(case, k, flush=True)
    same(host(gpu_lib.forward(dev(x * tiny), dev(f), mode="bank")),
         oracle.forward(x.astype(np.float64), f.astype(np.float64), "bank") * 2.0 ** -149)
    gi, _ = gpu_lib.backward(dev(x), dev(f), dev(g * tiny), mode="bank", need_filter=False)
    same(host(gi), oracle.grad_input(g.astype(np.float64), f.astype(np.float64), x.shape, "bank") * 2.0 ** -149)
    _, gf = gpu_lib.backward(dev(x * tiny), dev(f), dev(g), mode="bank", need_input=False)
    same(host(gf), weight_gradient(x.astype(np.float64), g.astype(np.float64), k) * 2.0 ** -149)


TAPS = [[np.inf] + [0.0] * 8, [0.0] * 8 + [-np.inf], [np.nan] + [1.0] * 8, [np.inf, -np.inf] + [0.5] * 7,
        [1e38] * 9, [-1e-42] * 9, [2.0 ** -130] * 9, [127.0, -128.0] + [0.0] * 7, [np.nan] * 9]


@pytest.mark.parametrize("taps", range(len(TAPS)))
@pytest.mark.parametrize("channels", [1, 3, 4])
def test_special_taps_of_the_8_bit_filter(gpu_lib, taps, channels):
    """Factors 1 to 4 and 5 take different kernels: the bytes of a uniform
    image agree (inside it, and at its corner with zero borders)."""
    f = dev(np.array(TAPS[taps], np.float32).reshape(3, 3))
    for value in (0, 7):
        x = torch.full((1, 5, 40, channels), value, dtype=torch.uint8, device="cuda").permute(0, 3, 1, 2)
        clamp = [gpu_lib.upsample_forward(x, f, s, out_dtype=torch.uint8) for s in range(1, 6)]
        zero = [gpu_lib.upsample_forward(x, f, s, out_dtype=torch.uint8, border="zero") for s in range(1, 6)]
        for s in range(1, 5):
            assert torch.equal(clamp[s - 1], clamp[4][:, :, :5 * s, :40 * s])
            assert torch.equal(zero[s - 1][:, :, 0, 0], zero[4][:, :, 0, 0])
            assert torch.equal(zero[s - 1][:, :, 2 * s, 2 * s], zero[4][:, :, 12, 12])
