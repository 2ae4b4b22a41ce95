// Native argument marshalling for the Python binding: describes torch tensors
// as f2d_tensor / f2d_filter, allocates the outputs the caller did not give
// and calls the C ABI.  Built as the extension module _hostcall.
//
// Marshalling in Python (ctypes structures, views, shape and stride look-ups)
// took 11 of the 14.5 us of a 5x5 filter's call on 1 x 3 x 64 x 64; here it takes
// 1.6 of 5, of which a new output is 1.0 and the current stream 0.35.
//
// Errors are those of the ctypes binding: ValueError for tensors the
// descriptors cannot express, KeyError for element types the library does not
// know, and the library's status, returned to the caller.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/Dtype.h>
#include <torch/csrc/DynamicTypes.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/object_ptr.h>

#include <ATen/ATen.h>

#include <vector>

#include "filter2d.h"

namespace {

decltype(&filter2d_forward) g_forward = nullptr;
decltype(&filter2d_upsample_forward) g_upsample = nullptr;
decltype(&filter2d_forward_separable) g_separable = nullptr;
decltype(&filter2d_backward_workspace) g_workspace = nullptr;
decltype(&filter2d_backward) g_backward = nullptr;

const at::Tensor& tensor_of(PyObject* o, const char* what) {
  TORCH_CHECK_TYPE(THPVariable_Check(o), what, " must be a tensor");
  return THPVariable_Unpack(o);
}

// 2-D and 3-D tensors stand for [1][1][h][w] and [1][c][h][w].
at::Tensor as4(const at::Tensor& t) {
  if (t.dim() == 2) return t.view({1, 1, t.size(0), t.size(1)});
  if (t.dim() == 3) return t.unsqueeze(0);
  return t;
}

bool dtype_code(const at::Tensor& t, int32_t* code) {
  switch (t.scalar_type()) {
    case at::kByte: *code = F2D_U8; return true;
    case at::kInt: *code = F2D_I32; return true;
    case at::kFloat: *code = F2D_F32; return true;
    case at::kBFloat16: *code = F2D_BF16; return true;
    default: {
      PyObject* d = reinterpret_cast<PyObject*>(torch::getTHPDtype(t.scalar_type()));
      PyErr_SetObject(PyExc_KeyError, d);
      return false;
    }
  }
}

// The tensor descriptor; false with a Python error set where there is none.
bool describe(const at::Tensor& t, f2d_tensor* d) {
  if (t.dim() != 4) {
    PyErr_SetString(PyExc_ValueError, "expected a 4-D [n][c][h][w] tensor");
    return false;
  }
  d->stride_w = static_cast<int32_t>(t.size(3) > 1 ? t.stride(3) : 1);
  if (!dtype_code(t, &d->dtype)) return false;
  d->data = t.data_ptr();
  d->n = t.size(0);
  d->c = t.size(1);
  d->h = t.size(2);
  d->w = t.size(3);
  d->stride_n = t.stride(0);
  d->stride_c = t.stride(1);
  d->stride_h = t.stride(2);
  return true;
}

bool describe_filter(const at::Tensor& f, f2d_filter* d) {
  const bool two = f.dim() == 2;
  if (!two && f.dim() != 4) {
    PyErr_SetString(PyExc_ValueError, "expected a [f_out][f_in][k][k] filter");
    return false;
  }
  const int64_t kh = f.size(two ? 0 : 2), kw = f.size(two ? 1 : 3);
  if (kh != kw) {
    PyErr_SetString(PyExc_ValueError, "expected a [f_out][f_in][k][k] filter");
    return false;
  }
  if (!f.is_contiguous()) {
    PyErr_SetString(PyExc_ValueError, "the filter must be contiguous");
    return false;
  }
  if (!dtype_code(f, &d->dtype)) return false;
  d->data = f.data_ptr();
  d->f_out = two ? 1 : static_cast<int32_t>(f.size(0));
  d->f_in = two ? 1 : static_cast<int32_t>(f.size(1));
  d->k = static_cast<int32_t>(kh);
  return true;
}

// An [n][c][h][w] view of interleaved [n][h][w][c] storage.
bool interleaved(const at::Tensor& t) {
  return t.dim() == 4 && t.size(1) > 1 && t.stride(1) == 1 && t.stride(3) == t.size(1);
}

at::Tensor new_out(const at::Tensor& image, const at::Tensor& filt, int64_t c, int64_t h, int64_t w,
                   PyObject* out_dtype, bool il) {
  at::ScalarType dt = at::kFloat;
  if (out_dtype != Py_None) {
    TORCH_CHECK_TYPE(THPDtype_Check(out_dtype), "out_dtype must be a torch.dtype");
    dt = reinterpret_cast<THPDtype*>(out_dtype)->scalar_type;
  } else if (image.scalar_type() == at::kByte && filt.scalar_type() == at::kInt) {
    dt = at::kInt;
  }
  const auto opt = at::TensorOptions().dtype(dt).device(image.device());
  if (il) return at::empty({image.size(0), h, w, c}, opt).permute({0, 3, 1, 2});
  return at::empty({image.size(0), c, h, w}, opt);
}

// The stream's address, or a function that returns it: the device is asked only
// when the arguments are in order.
bool stream_of(PyObject* o, void** out) {
  THPObjectPtr made;
  if (!PyLong_Check(o)) {
    made = PyObject_CallObject(o, nullptr);
    if (!made) return false;
    o = made.get();
  }
  *out = PyLong_AsVoidPtr(o);
  return !PyErr_Occurred();
}

PyObject* py_connect(PyObject*, PyObject* args) {
  PyObject* a[5];
  if (!PyArg_ParseTuple(args, "OOOOO", &a[0], &a[1], &a[2], &a[3], &a[4])) return nullptr;
  g_forward = reinterpret_cast<decltype(g_forward)>(PyLong_AsVoidPtr(a[0]));
  g_upsample = reinterpret_cast<decltype(g_upsample)>(PyLong_AsVoidPtr(a[1]));
  g_separable = reinterpret_cast<decltype(g_separable)>(PyLong_AsVoidPtr(a[2]));
  g_workspace = reinterpret_cast<decltype(g_workspace)>(PyLong_AsVoidPtr(a[3]));
  g_backward = reinterpret_cast<decltype(g_backward)>(PyLong_AsVoidPtr(a[4]));
  if (PyErr_Occurred()) return nullptr;
  Py_RETURN_NONE;
}

// forward(image, filt, mode, epilogue, rows | None, outs | None, variant,
//         out_dtype | None, border, stream) -> (status, [outputs])
PyObject* py_forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  TORCH_CHECK_TYPE(n == 10, "forward takes 10 arguments");
  const at::Tensor image = as4(tensor_of(a[0], "image"));
  const at::Tensor& filt = tensor_of(a[1], "filt");
  f2d_filter fd;
  if (!describe_filter(filt, &fd)) return nullptr;
  f2d_opts opts;
  opts.channels = static_cast<int32_t>(PyLong_AsLong(a[2]));
  opts.epilogue = static_cast<int32_t>(PyLong_AsLong(a[3]));
  opts.variant = static_cast<int32_t>(PyLong_AsLong(a[6]));
  opts.border = static_cast<int32_t>(PyLong_AsLong(a[8]));
  if (PyErr_Occurred()) return nullptr;
  f2d_tensor x;
  if (!describe(image, &x)) return nullptr;
  opts.row_begin = 0;
  opts.row_end = x.h;
  if (a[4] != Py_None) {
    PyObject* r = PySequence_Fast(a[4], "rows must be a pair");
    if (!r) return nullptr;
    if (PySequence_Fast_GET_SIZE(r) != 2) {
      Py_DECREF(r);
      PyErr_SetString(PyExc_ValueError, "rows must be a pair");
      return nullptr;
    }
    opts.row_begin = PyLong_AsLongLong(PySequence_Fast_GET_ITEM(r, 0));
    opts.row_end = PyLong_AsLongLong(PySequence_Fast_GET_ITEM(r, 1));
    Py_DECREF(r);
    if (PyErr_Occurred()) return nullptr;
  }
  THPObjectPtr list, seq;  // seq holds given outputs (and what makes them) until the call is enqueued
  std::vector<f2d_tensor> descs;
  if (a[5] == Py_None) {
    int64_t count = 1;
    if (opts.channels == F2D_CH_DEPTHWISE) {
      if (x.c == 0) {
        PyErr_SetString(PyExc_ZeroDivisionError, "an image without channels");
        return nullptr;
      }
      count = fd.f_out / x.c + (opts.epilogue == F2D_EPI_SUMSQ_PAIRS ? 1 : 0);
    }
    const bool bank = opts.channels == F2D_CH_BANK;
    list = PyList_New(count);
    if (!list) return nullptr;
    descs.resize(count);
    for (int64_t j = 0; j < count; ++j) {
      at::Tensor o = new_out(image, filt, bank ? fd.f_out : x.c, opts.row_end - opts.row_begin, x.w, a[7],
                             !bank && interleaved(image));
      if (!describe(o, &descs[j])) return nullptr;
      PyObject* w = THPVariable_Wrap(std::move(o));
      if (!w) return nullptr;
      PyList_SET_ITEM(list.get(), j, w);
    }
  } else {
    if (PyObject_Size(a[5]) < 0) return nullptr;  // TypeError: iterators without a length are refused
    seq = PySequence_Fast(a[5], "outs must be a sequence of tensors");
    if (!seq) return nullptr;
    const Py_ssize_t count = PySequence_Fast_GET_SIZE(seq.get());
    descs.resize(count);
    for (Py_ssize_t j = 0; j < count; ++j)
      if (!describe(as4(tensor_of(PySequence_Fast_GET_ITEM(seq.get(), j), "outs")), &descs[j])) return nullptr;
    Py_INCREF(a[5]);
    list = a[5];
  }
  void* stream;
  if (!stream_of(a[9], &stream)) return nullptr;
  f2d_status st;
  {
    pybind11::gil_scoped_release nogil;
    st = g_forward(&x, &fd, &opts, descs.data(), static_cast<int32_t>(descs.size()), stream);
  }
  return Py_BuildValue("(iN)", static_cast<int>(st), list.release());
  END_HANDLE_TH_ERRORS
}

// upsample(image, filt, scale, out | None, out_dtype | None, border, stream) -> (status, out)
PyObject* py_upsample(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  TORCH_CHECK_TYPE(n == 7, "upsample takes 7 arguments");
  const at::Tensor image = as4(tensor_of(a[0], "image"));
  const at::Tensor& filt = tensor_of(a[1], "filt");
  f2d_filter fd;
  if (!describe_filter(filt, &fd)) return nullptr;
  // a new output takes whole factors only, a given one what int() takes
  THPObjectPtr factor(a[3] == Py_None ? PyNumber_Index(a[2]) : PyNumber_Long(a[2]));
  if (!factor) return nullptr;
  const int64_t scale = PyLong_AsLongLong(factor.get());
  f2d_opts opts{};
  opts.channels = F2D_CH_SHARED;
  opts.border = static_cast<int32_t>(PyLong_AsLong(a[5]));
  if (PyErr_Occurred()) return nullptr;
  f2d_tensor x, y;
  if (!describe(image, &x)) return nullptr;
  THPObjectPtr out;
  if (a[3] == Py_None) {
    at::Tensor o = new_out(image, filt, x.c, x.h * scale, x.w * scale, a[4], interleaved(image));
    if (!describe(o, &y)) return nullptr;
    out = THPVariable_Wrap(std::move(o));
    if (!out) return nullptr;
  } else {
    if (!describe(as4(tensor_of(a[3], "out")), &y)) return nullptr;
    Py_INCREF(a[3]);
    out = a[3];
  }
  void* stream;
  if (!stream_of(a[6], &stream)) return nullptr;
  f2d_status st;
  {
    pybind11::gil_scoped_release nogil;
    st = g_upsample(&x, &fd, static_cast<int32_t>(scale), &opts, &y, stream);
  }
  return Py_BuildValue("(iN)", static_cast<int>(st), out.release());
  END_HANDLE_TH_ERRORS
}

// separable(image, a, b, first row | None, end row, out | None, stream) -> (status, out)
PyObject* py_separable(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  TORCH_CHECK_TYPE(n == 7, "separable takes 7 arguments");
  const at::Tensor image = as4(tensor_of(a[0], "image"));
  const at::Tensor& fa = tensor_of(a[1], "a");
  const at::Tensor& fb = tensor_of(a[2], "b");
  if (fa.dim() != 1 || fb.dim() != 1 || fa.numel() != fb.numel()) {
    PyErr_SetString(PyExc_ValueError, "a and b must be 1-D with the same length k");
    return nullptr;
  }
  if (fa.scalar_type() != at::kFloat || fb.scalar_type() != at::kFloat || !fa.is_contiguous() ||
      !fb.is_contiguous()) {
    PyErr_SetString(PyExc_ValueError, "a and b must be contiguous float32");
    return nullptr;
  }
  f2d_tensor x, y;
  if (!describe(image, &x)) return nullptr;
  f2d_opts opts{};
  opts.channels = F2D_CH_SHARED;
  opts.row_begin = 0;
  opts.row_end = x.h;
  if (a[3] != Py_None) {
    opts.row_begin = PyLong_AsLongLong(a[3]);
    opts.row_end = PyLong_AsLongLong(a[4]);
  }
  if (PyErr_Occurred()) return nullptr;
  THPObjectPtr out;
  if (a[5] == Py_None) {
    at::Tensor o = at::empty({x.n, x.c, opts.row_end - opts.row_begin, x.w},
                             at::TensorOptions().dtype(at::kFloat).device(image.device()));
    if (!describe(o, &y)) return nullptr;
    out = THPVariable_Wrap(std::move(o));
    if (!out) return nullptr;
  } else {
    if (!describe(as4(tensor_of(a[5], "out")), &y)) return nullptr;
    Py_INCREF(a[5]);
    out = a[5];
  }
  void* stream;
  if (!stream_of(a[6], &stream)) return nullptr;
  f2d_status st;
  {
    const float* pa = static_cast<const float*>(fa.data_ptr());
    const float* pb = static_cast<const float*>(fb.data_ptr());
    const int32_t k = static_cast<int32_t>(fa.numel());
    pybind11::gil_scoped_release nogil;
    st = g_separable(&x, pa, pb, k, &opts, &y, stream);
  }
  return Py_BuildValue("(iN)", static_cast<int>(st), out.release());
  END_HANDLE_TH_ERRORS
}

// backward(image, filt, grad_outs, mode, need_input, need_filter, workspace |
//          None, grad_input | None, grad_filter | None, stream)
//   -> (status, grad_input | None, grad_filter | None)
PyObject* py_backward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  TORCH_CHECK_TYPE(n == 10, "backward takes 10 arguments");
  const at::Tensor& given = tensor_of(a[0], "image");
  const at::Tensor image = as4(given);
  const at::Tensor& filt = tensor_of(a[1], "filt");
  f2d_filter fd;
  if (!describe_filter(filt, &fd)) return nullptr;
  f2d_tensor x;
  if (!describe(image, &x)) return nullptr;
  THPObjectPtr seq(PySequence_Fast(a[2], "grad_outs must be a sequence of tensors"));
  if (!seq) return nullptr;
  std::vector<f2d_tensor> gs(PySequence_Fast_GET_SIZE(seq.get()));
  for (size_t j = 0; j < gs.size(); ++j)
    if (!describe(as4(tensor_of(PySequence_Fast_GET_ITEM(seq.get(), j), "grad_outs")), &gs[j])) return nullptr;
  f2d_opts opts{};
  opts.channels = static_cast<int32_t>(PyLong_AsLong(a[3]));
  const bool need_x = PyObject_IsTrue(a[4]) == 1, need_f = PyObject_IsTrue(a[5]) == 1;
  if (PyErr_Occurred()) return nullptr;
  const auto f32 = at::TensorOptions().dtype(at::kFloat).device(image.device());
  THPObjectPtr gi, gf;
  f2d_tensor gid;
  float* gfp = nullptr;
  at::Tensor made_gf;
  if (need_x) {
    if (a[7] != Py_None) {
      if (!describe(tensor_of(a[7], "grad_input"), &gid)) return nullptr;
      Py_INCREF(a[7]);
      gi = a[7];
    } else {
      at::Tensor t = at::empty(image.sizes(), f32);
      if (!describe(t, &gid)) return nullptr;
      gi = THPVariable_Wrap(std::move(t));
      if (!gi) return nullptr;
    }
  }
  if (need_f) {
    if (a[8] != Py_None) {
      const at::Tensor& t = tensor_of(a[8], "grad_filter");
      if (t.numel() != filt.numel() || t.scalar_type() != at::kFloat || !t.is_contiguous()) {
        PyErr_SetString(PyExc_ValueError,
                        "grad_filter must be a contiguous float32 tensor with the filter's size");
        return nullptr;
      }
      made_gf = t;
    } else if (filt.dim() == 2) {
      made_gf = at::empty({1, 1, filt.size(0), filt.size(1)}, f32);
    } else {
      made_gf = at::empty(filt.sizes(), f32);
    }
    gfp = static_cast<float*>(made_gf.data_ptr());
  }
  const size_t bytes = g_workspace(&x, &fd, &opts);
  at::Tensor ws;
  if (a[6] != Py_None) ws = tensor_of(a[6], "workspace");
  if (!ws.defined() || static_cast<size_t>(ws.numel()) < bytes)
    ws = at::empty({static_cast<int64_t>(bytes > 1 ? bytes : 1)},
                   at::TensorOptions().dtype(at::kByte).device(image.device()));
  void* stream;
  if (!stream_of(a[9], &stream)) return nullptr;
  f2d_status st;
  {
    void* wp = ws.data_ptr();
    pybind11::gil_scoped_release nogil;
    st = g_backward(&x, &fd, gs.data(), static_cast<int32_t>(gs.size()), &opts, need_x ? &gid : nullptr, gfp, wp,
                    bytes, stream);
  }
  if (!need_x) {
    Py_INCREF(Py_None);
    gi = Py_None;
  }
  if (need_f) {
    if (filt.dim() == 2) {
      gf = THPVariable_Wrap(made_gf.view(filt.sizes()));
    } else if (a[8] != Py_None) {
      Py_INCREF(a[8]);
      gf = a[8];
    } else {
      gf = THPVariable_Wrap(std::move(made_gf));
    }
    if (!gf) return nullptr;
  } else {
    Py_INCREF(Py_None);
    gf = Py_None;
  }
  return Py_BuildValue("(iNN)", static_cast<int>(st), gi.release(), gf.release());
  END_HANDLE_TH_ERRORS
}

#define F2D_FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL
PyMethodDef g_methods[] = {
    {"connect", py_connect, METH_VARARGS, "Addresses of the C entry points."},
    {"forward", F2D_FAST(py_forward), nullptr},
    {"upsample", F2D_FAST(py_upsample), nullptr},
    {"separable", F2D_FAST(py_separable), nullptr},
    {"backward", F2D_FAST(py_backward), nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_hostcall", nullptr, -1, g_methods, nullptr, nullptr, nullptr,
                        nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__hostcall() { return PyModule_Create(&g_module); }
