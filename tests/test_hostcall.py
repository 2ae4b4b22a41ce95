"""The native marshalling module on calls that never reach a kernel (CPU
tensors, refused by the library or before it): the errors are those of the
ctypes descriptors, and refused calls return the library's status."""
import pytest
import torch

from paper_2504_01266_amd import binding as B


@pytest.fixture(scope="module")
def native():
    B.load()
    return B._native


IMG, TAPS = torch.zeros(1, 3, 8, 9), torch.zeros(3, 3)


def fwd(native, image=IMG, filt=TAPS, mode=0, epilogue=0, rows=None, outs=None, variant=0, out_dtype=None, border=0):
    return native.forward(image, filt, mode, epilogue, rows, outs, variant, out_dtype, border, 0)


@pytest.mark.parametrize("kw", [{"image": torch.zeros(5)}, {"image": torch.zeros(1, 1, 2, 3, 4)},
                                {"filt": torch.zeros(3)}, {"filt": torch.zeros(3, 5)},
                                {"filt": torch.zeros(1, 1, 3, 5)}, {"filt": torch.zeros(3, 6)[:, ::2]},
                                {"rows": (1, 2, 3)}, {"outs": [torch.zeros(4)]}])
def test_what_descriptors_cannot_express_is_a_value_error(native, kw):
    with pytest.raises(ValueError):
        fwd(native, **kw)


@pytest.mark.parametrize("kw", [{"image": IMG.double()}, {"filt": TAPS.half()}, {"out_dtype": torch.float64}])
def test_unknown_element_types_are_key_errors(native, kw):
    with pytest.raises(KeyError):
        fwd(native, **kw)


@pytest.mark.parametrize("kw", [{"image": None}, {"filt": 3}, {"out_dtype": "u8"}, {"rows": 5}, {"outs": [None]}])
def test_other_objects_are_type_errors(native, kw):
    with pytest.raises(TypeError):
        fwd(native, **kw)


def test_depthwise_without_channels(native):
    with pytest.raises(ZeroDivisionError):
        fwd(native, image=torch.zeros(1, 0, 4, 4), filt=torch.zeros(2, 1, 3, 3), mode=1)


def test_refused_calls_return_the_status_and_outputs(native):
    status, outs = fwd(native, filt=torch.zeros(2, 2))
    assert status == B.EINVAL and "k=2" in B.last_error() and outs[0].shape == IMG.shape
    status, _ = fwd(native, rows=(2, 20))
    assert status == B.EINVAL and "rows" in B.last_error()
    given = [torch.zeros(1, 3, 8, 8)]
    status, outs = fwd(native, outs=given)
    assert status == B.EINVAL and outs is given
    status, outs = native.upsample(IMG, TAPS, 2, None, None, 0, 0)
    assert status == B.EUNSUPPORTED and outs.shape == (1, 3, 16, 18)
    status, _ = native.separable(IMG, torch.zeros(17), torch.zeros(17), None, None, None, 0)
    assert status == B.EUNSUPPORTED
    with pytest.raises(ValueError):
        native.separable(IMG, torch.zeros(3), torch.zeros(5), None, None, None, 0)
    status, gi, gf = native.backward(IMG, torch.zeros(2, 2), [IMG], 0, True, True, None, None, None, 0)
    assert status == B.EINVAL and gi.shape == IMG.shape and gf.shape == (2, 2)
    status, gi, gf = native.backward(IMG.byte(), TAPS, [IMG], 0, True, False, None, None, None, 0)
    assert status != B.OK and gf is None
    with pytest.raises(ValueError):
        native.backward(IMG, TAPS, [IMG], 0, False, True, None, None, torch.zeros(8), 0)
