"""Calls at the largest grid of one launch, on a machine without a GPU (the
pointers are not memory): a call that the limit allows fails at the launch,
one beyond it is refused before."""
import ctypes

import pytest
import torch

from paper_2504_01266_amd import binding as B

pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="the launch would run")
LIMIT = 2 ** 32 // 256 - 1  # work-groups
PLANES = LIMIT // 9         # 64 rows x 513 columns: 9 tiles of 64 x 64, 10 of 32 x 128


def planes(n, h, w):
    return B.F2dTensor(1 << 20, B.F32, 1, 1, n, h, w, n * h * w, h * w, w)


@pytest.mark.parametrize("border", ["clamp", "zero"])
def test_default_tiling_stays_within_one_launch(border):
    f = B.F2dFilter(1 << 20, B.F32, 1, 1, 9)
    for n, want in ((PLANES, B.EHIP), (PLANES + 1, B.EUNSUPPORTED)):
        x = planes(n, 64, 513)
        got = B.load().filter2d_forward(ctypes.byref(x), ctypes.byref(f), ctypes.byref(B.make_opts(border=border)),
                                        ctypes.byref(planes(n, 64, 513)), 1, None)
        assert got == want, B.last_error()


def test_default_tiling_of_the_adjoint_stays_within_one_launch():
    f = B.F2dFilter(1 << 20, B.F32, 1, 1, 9)
    x = planes(PLANES, 56, 505)  # with its frame 64 x 513
    need = B.load().filter2d_backward_workspace(ctypes.byref(x), ctypes.byref(f), ctypes.byref(B.make_opts()))
    got = B.load().filter2d_backward(ctypes.byref(x), ctypes.byref(f), ctypes.byref(planes(PLANES, 56, 505)), 1,
                                     ctypes.byref(B.make_opts()), ctypes.byref(planes(PLANES, 56, 505)), None,
                                     ctypes.c_void_p(1 << 20), need, None)
    assert got == B.EHIP, B.last_error()
