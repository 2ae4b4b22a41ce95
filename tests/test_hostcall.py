"""The native marshalling module on calls that never reach a kernel (CPU
tensors, refused by the library or before it): the errors are those of the
ctypes descriptors, and refused calls return the library's status."""
import ctypes
import weakref

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


# ---- what the module hands to the library, seen by functions in its place --

P = ctypes.POINTER
ENTRY = {
    "filter2d_forward": (ctypes.c_int32, P(B.F2dTensor), P(B.F2dFilter), P(B.F2dOpts), P(B.F2dTensor),
                         ctypes.c_int32, ctypes.c_void_p),
    "filter2d_upsample_forward": (ctypes.c_int32, P(B.F2dTensor), P(B.F2dFilter), ctypes.c_int32, P(B.F2dOpts),
                                  P(B.F2dTensor), ctypes.c_void_p),
    "filter2d_forward_separable": (ctypes.c_int32, P(B.F2dTensor), ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int32,
                                   P(B.F2dOpts), P(B.F2dTensor), ctypes.c_void_p),
    "filter2d_backward_workspace": (ctypes.c_size_t, P(B.F2dTensor), P(B.F2dFilter), P(B.F2dOpts)),
    "filter2d_backward": (ctypes.c_int32, P(B.F2dTensor), P(B.F2dFilter), P(B.F2dTensor), ctypes.c_int32,
                          P(B.F2dOpts), P(B.F2dTensor), ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t,
                          ctypes.c_void_p),
}


@pytest.fixture
def hooked(native):
    """Replaces C entry points by Python functions for one test."""
    lib, kept = B.load(), []

    def connect(**hooks):
        def address(name):
            if name not in hooks:
                return ctypes.cast(getattr(lib, name), ctypes.c_void_p).value
            kept.append(ctypes.CFUNCTYPE(*ENTRY[name])(hooks[name]))
            return ctypes.cast(kept[-1], ctypes.c_void_p).value
        native.connect(*[address(n) for n in ENTRY])

    yield connect
    connect()


def test_outputs_without_a_length_are_refused(native):
    for make in (lambda: (torch.empty_like(IMG) for _ in range(1)), lambda: map(torch.empty_like, [IMG])):
        with pytest.raises(TypeError):
            fwd(native, outs=make())


def test_outputs_made_by_a_sequence_live_until_the_call(native, hooked):
    class Fresh:  # sized and iterable, keeping nothing
        refs = []

        def __len__(self):
            return 2

        def __iter__(self):
            for _ in range(2):
                t = torch.empty(1, 3, 8, 9)
                self.refs.append(weakref.ref(t))
                yield t

    alive = []
    hooked(filter2d_forward=lambda *a: alive.append([r() is not None for r in Fresh.refs]) or B.OK)
    status, outs = fwd(native, filt=torch.zeros(6, 1, 3, 3), mode=1, outs=Fresh())
    assert status == B.OK and alive == [[True, True]] and isinstance(outs, Fresh)


def test_argument_errors_come_before_the_device(native, monkeypatch):
    def no_device(*_):
        raise RuntimeError("no device")

    monkeypatch.setattr(B, "_raw_stream", no_device)
    monkeypatch.setattr(B, "_current_device", lambda: 0)
    row, u8 = torch.zeros(5), IMG.byte()
    for call in (lambda: B.forward(row, TAPS), lambda: B.upsample_forward(row.byte(), TAPS, 2),
                 lambda: B.forward_separable(IMG, torch.zeros(3), torch.zeros(5)),
                 lambda: B.backward(row, TAPS, row)):
        with pytest.raises(ValueError):
            call()
    for call in (lambda: B.forward(IMG, TAPS), lambda: B.upsample_forward(u8, TAPS, 2),
                 lambda: B.forward_separable(IMG, torch.zeros(3), torch.zeros(3)),
                 lambda: B.backward(IMG, TAPS, IMG)):
        with pytest.raises(RuntimeError, match="no device"):
            call()


def test_factors_and_rows_that_are_no_whole_numbers(native, hooked):
    seen = []
    hooked(filter2d_upsample_forward=lambda x, f, s, *_: seen.append(s) or B.OK,
           filter2d_forward_separable=lambda x, a, b, k, o, *_: seen.append((o[0].row_begin, o[0].row_end)) or B.OK)
    u8, taps = IMG.byte(), torch.zeros(3)
    for scale in (2.5, 2.0, None):
        with pytest.raises(TypeError):
            B.upsample_forward(u8, TAPS, scale)
    for rows in ((None, None), (None, 4), (0, None), (0.0, 4.0)):
        with pytest.raises(TypeError):
            B.forward_separable(IMG, taps, taps, rows=rows)
    assert seen == []
    native.upsample(u8, TAPS, 2.5, torch.zeros(1, 3, 16, 18).byte(), None, 0, 0)  # a given output: int(scale)
    native.separable(IMG, taps, taps, 2, 4, None, 0)
    assert seen == [2, (2, 4)]
