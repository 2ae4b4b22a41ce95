"""The reduction of the weight gradient's partial sums on either side of the
number of partials that one launch takes.  Integer operands: exact."""
import numpy as np
import pytest
import torch

import oracle
from paper_2504_01266_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("planes", [1, 255, 257, 7281, 7282, 7290])  # 9 taps x 7281 = 65529 values
def test_shared_filter_over_many_planes(gpu_lib, planes):
    r = wl.rng(83, planes)
    x, g = (r.integers(-4, 5, (1, planes, 3, 5)).astype(np.float32) for _ in range(2))
    f = np.zeros((3, 3), np.float32)
    print(planes, flush=True)
    _, gf = gpu_lib.backward(*(torch.from_numpy(a).cuda() for a in (x, f, g)), need_input=False)
    np.testing.assert_array_equal(gf.cpu().numpy(), oracle.grad_filter(x, g, (1, 1, 3, 3), "shared")[0, 0])


@pytest.mark.parametrize("channels", [255, 256, 257])  # 9 taps x 256 = 2304 outputs, one partial set each
def test_depthwise_filters_by_the_number_of_outputs(gpu_lib, channels):
    r = wl.rng(84, channels)
    x, g = (r.integers(-4, 5, (2, channels, 6, 7)).astype(np.float32) for _ in range(2))
    f = np.zeros((channels, 1, 3, 3), np.float32)
    print(channels, flush=True)
    _, gf = gpu_lib.backward(*(torch.from_numpy(a).cuda() for a in (x, f, g)), mode="depthwise", need_input=False)
    np.testing.assert_array_equal(gf.cpu().numpy(), oracle.grad_filter(x, g, f.shape, "depthwise"))


@pytest.mark.parametrize("planes", [4095, 4096, 4097])  # partial sets of one output
def test_one_tap_over_many_planes(gpu_lib, planes):
    r = wl.rng(85, planes)
    x, g = (r.integers(-4, 5, (1, planes, 2, 3)).astype(np.float32) for _ in range(2))
    print(planes, flush=True)
    _, gf = gpu_lib.backward(*(torch.from_numpy(a).cuda() for a in (x, np.zeros((1, 1), np.float32), g)),
                             need_input=False)
    np.testing.assert_array_equal(gf.cpu().numpy(), oracle.grad_filter(x, g, (1, 1, 1, 1), "shared")[0, 0])
