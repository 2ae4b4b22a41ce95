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


def fields(s):
    return {n: getattr(s, n) for n, _ in s._fields_}


def nhwc(dtype, c=3):
    return torch.zeros(2, 6, 7, c, dtype=dtype).permute(0, 3, 1, 2)


U8, I32, F32, BF16 = torch.uint8, torch.int32, torch.float32, torch.bfloat16
# image, filter, keywords of B.forward, expected element type and interleaving of new outputs
FORWARD = [
    (torch.zeros(6, 7), torch.zeros(3, 3), {}, F32, False),
    (torch.zeros(3, 6, 7), torch.zeros(3, 3), {"rows": (1, 4)}, F32, False),
    (torch.zeros(2, 3, 8, 9)[:, :, 1:7, 1:8], torch.zeros(6, 1, 5, 5), {"mode": "depthwise"}, F32, False),
    (torch.zeros(2, 3, 6, 1), torch.zeros(4, 3, 3, 3), {"mode": "bank", "border": "zero", "variant": 2}, F32, False),
    (torch.zeros(2, 3, 6, 7), torch.zeros(4, 3, 1, 1), {"mode": "bank"}, F32, False),
    (torch.zeros(2, 3, 6, 7, dtype=BF16), torch.zeros(4, 3, 3, 3, dtype=BF16), {"mode": "bank"}, F32, False),
    (torch.zeros(2, 3, 6, 7, dtype=BF16), torch.zeros(4, 3, 3, 3, dtype=BF16), {"mode": "bank", "out_dtype": BF16},
     BF16, False),
    (torch.zeros(2, 3, 6, 7, dtype=U8), torch.zeros(6, 1, 3, 3, dtype=I32),
     {"mode": "depthwise", "epilogue": B.EPI_SUMSQ_PAIRS}, I32, False),
    (torch.zeros(2, 3, 6, 7, dtype=U8), torch.zeros(3, 3), {}, F32, False),
    (nhwc(U8), torch.zeros(3, 3, dtype=I32), {}, I32, True),
    (nhwc(U8, 4), torch.zeros(3, 3), {"out_dtype": U8, "rows": (2, 6)}, U8, True),
    (nhwc(U8), torch.zeros(1, 3, 1, 1), {"mode": "bank", "out_dtype": U8}, U8, False),
]


@pytest.mark.parametrize("case", range(len(FORWARD)))
def test_forward_describes_its_tensors_as_the_ctypes_binding(native, hooked, case):
    image, filt, kw, dtype, inter = FORWARD[case]
    seen = []

    def record(x, f, o, ys, n, stream):
        seen.append((fields(x[0]), fields(f[0]), fields(o[0]), [fields(ys[j]) for j in range(n)], stream))
        return B.OK

    hooked(filter2d_forward=record)
    mode, border = B._MODES[kw.get("mode", "shared")], B._BORDERS[kw.get("border", "clamp")]
    args = (image, filt, mode, kw.get("epilogue", 0), kw.get("rows"))
    tail = (kw.get("variant", 0), kw.get("out_dtype"), border, 77)
    status, outs = native.forward(*args, None, *tail)
    image4, (fd, filt4) = B._as4(image), B.filter_desc(filt)
    r0, r1 = kw.get("rows") or (0, image4.size(2))
    want = [fields(B.tensor_desc(image4)), fields(fd),
            fields(B.make_opts(mode, kw.get("epilogue", 0), (r0, r1), kw.get("variant", 0), border))]
    assert status == B.OK and list(seen[0][:3]) == want and seen[0][4] == 77
    assert seen[0][3] == [fields(B.tensor_desc(o)) for o in outs]
    channels = filt4.size(0) if mode == B.BANK else image4.size(1)
    assert len(outs) == B.out_count(mode, filt4.shape, image4.size(1), kw.get("epilogue", 0))
    for o in outs:
        assert o.dtype == dtype and o.shape == (image4.size(0), channels, r1 - r0, image4.size(3))
        assert B.interleaved(o) == inter and (inter or o.is_contiguous())
    # given outputs: the same descriptors, in 3-D where the image has one plane group
    given = [torch.zeros(o.shape, dtype=o.dtype) for o in outs]
    status, back = native.forward(*args, [g[0] if g.size(0) == 1 else g for g in given], *tail)
    assert status == B.OK and seen[1][3] == [fields(B.tensor_desc(g)) for g in given]
    assert [b.data_ptr() for b in back] == [g.data_ptr() for g in given]


def test_the_other_calls_describe_their_tensors_as_the_ctypes_binding(native, hooked):
    seen = {}

    def up(x, f, s, o, y, stream):
        seen["up"] = (fields(x[0]), fields(f[0]), s, fields(o[0]), fields(y[0]), stream)
        return B.OK

    def sep(x, a, b, k, o, y, stream):
        seen["sep"] = (fields(x[0]), a, b, k, fields(o[0]), fields(y[0]), stream)
        return B.OK

    def work(x, f, o):
        seen["work"] = (fields(x[0]), fields(f[0]), fields(o[0]))
        return 1000

    def back(x, f, gs, n, o, gi, gf, ws, ws_bytes, stream):
        seen["back"] = (fields(x[0]), fields(f[0]), [fields(gs[j]) for j in range(n)], fields(o[0]),
                        fields(gi[0]) if gi else None, gf, bool(ws), ws_bytes, stream)
        return B.OK

    hooked(filter2d_upsample_forward=up, filter2d_forward_separable=sep, filter2d_backward_workspace=work,
           filter2d_backward=back)
    image, taps = nhwc(U8), torch.zeros(3, 3)
    _, y = native.upsample(image, taps, 3, None, U8, B.BORDER_ZERO, 5)
    assert y.shape == (2, 3, 18, 21) and y.dtype == U8 and B.interleaved(y)
    assert seen["up"] == (fields(B.tensor_desc(image)), fields(B.filter_desc(taps)[0]), 3,
                          fields(B.make_opts("shared", 0, None, 0, "zero")), fields(B.tensor_desc(y)), 5)
    x, a, b = torch.zeros(3, 6, 7), torch.zeros(5), torch.zeros(5)
    _, y = native.separable(x, a, b, 1, 5, None, 6)
    assert y.shape == (1, 3, 4, 7) and y.dtype == F32
    assert seen["sep"] == (fields(B.tensor_desc(x[None])), a.data_ptr(), b.data_ptr(), 5,
                           fields(B.make_opts("shared", 0, (1, 5))), fields(B.tensor_desc(y)), 6)
    for x, f, gs, mode, ws in [
            (torch.zeros(6, 7), taps, [torch.zeros(6, 7)], "shared", None),
            (torch.zeros(2, 3, 6, 7), torch.zeros(6, 1, 3, 3), [torch.zeros(2, 3, 6, 7)] * 2, "depthwise",
             torch.zeros(2000, dtype=U8)),
            (torch.zeros(2, 3, 6, 7, dtype=BF16), torch.zeros(4, 3, 5, 5, dtype=BF16), [torch.zeros(2, 4, 6, 7)], "bank",
             torch.zeros(10, dtype=U8))]:
        _, gi, gf = native.backward(x, f, gs, B._MODES[mode], True, True, ws, None, None, 8)
        described = (fields(B.tensor_desc(B._as4(x))), fields(B.filter_desc(f)[0]))
        opts = fields(B.make_opts(mode))
        assert seen["work"] == (*described, opts)
        assert gi.shape == B._as4(x).shape and gi.dtype == F32 and gf.shape == f.shape and gf.dtype == F32
        assert seen["back"] == (*described, [fields(B.tensor_desc(B._as4(g))) for g in gs], opts,
                                fields(B.tensor_desc(gi)), gf.data_ptr(), True, 1000, 8)
        _, gi, gf = native.backward(x, f, gs, B._MODES[mode], False, False, ws, None, None, 8)
        assert gi is None and gf is None and seen["back"][4:6] == (None, None)
