"""Which FP32 banks' weight gradients take the matrix cores, seen in the
workspace that the library asks for (host only): small layers keep the VALU
plan, frame plus one partial per tile run and channel pair."""
import ctypes

import pytest

from paper_2504_01266_amd import binding as B


def up(b):
    return (max(b, 1) + 255) // 256 * 256


def valu_workspace(n, c, o, h, w, k):
    r = (k - 1) // 2
    frame = up(n * c * (2 * r * (w + 2 * r) + 2 * r * h) * 4) if n * c * r else 0
    tiles = ((h + 63) // 64) * ((w + 63) // 64)
    run = min(max(tiles * n * c * o // 8192, 1), 16)
    return frame + up(n * c * o * ((tiles + run - 1) // run) * k * k * 4)


@pytest.mark.parametrize("n,c,o,h,w,k,valu", [
    (1, 16, 16, 112, 112, 5, True), (8, 16, 16, 56, 56, 5, True), (1, 16, 64, 56, 56, 5, True),
    (1, 48, 16, 112, 112, 5, True), (1, 16, 16, 224, 224, 5, True), (1, 64, 64, 14, 14, 5, False),
    (1, 16, 64, 112, 112, 5, False), (8, 16, 16, 112, 112, 5, False), (4, 16, 64, 256, 256, 5, False),
    (8, 16, 16, 56, 56, 3, True), (1, 16, 32, 160, 160, 3, True), (2, 16, 16, 100, 70, 3, True),
    (1, 16, 16, 28, 28, 3, False),
    (1, 16, 16, 128, 128, 3, False), (32, 16, 16, 56, 56, 3, False), (16, 16, 64, 1024, 1024, 3, False),
    (4, 3, 16, 41, 55, 1, True), (8, 16, 64, 512, 512, 1, False)])
def test_small_layers_keep_the_valu_plan(n, c, o, h, w, k, valu):
    x = B.F2dTensor(4096, B.F32, 1, n, c, h, w, c * h * w, h * w, w)
    f = B.F2dFilter(4096, B.F32, o, c, k)
    need = B.load().filter2d_backward_workspace(ctypes.byref(x), ctypes.byref(f), ctypes.byref(B.make_opts("bank")))
    assert (need == valu_workspace(n, c, o, h, w, k)) == valu
