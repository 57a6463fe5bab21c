// The Python binding's short path: one C call that takes torch tensors,
// checks them, allocates the result, asks for torch's current stream and
// calls the library's C ABI.
//
// Written in Python (with ctypes) these steps take 7 us of the 10.4 us that a
// call on a small image takes, more than its kernel: a 256 x 256 filter call
// went from 10.4 us to 4.1 us in a bare loop (4.6 to 4.9 us over three images in
// turn), of which the launch itself is 3.2 us.
//
// Only the plain case is handled here: exact torch.Tensor arguments of the
// right type and shape on the GPU, no stream argument, no Python mode that
// wants to see the calls. Anything else returns NotImplemented and the
// caller's Python code checks it, reports it or runs it. A nonzero pf_status
// is returned as an int. Nothing is kept between calls but the addresses of
// the library's functions.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "pf.h"

namespace {

decltype(&pf_filter2d_f32) f_filter2d;
decltype(&pf_filter_sep_f32) f_sep;
decltype(&pf_filter_chain_f32) f_chain;
decltype(&pf_filter2d_f32_border) f_border;
decltype(&pf_filter2d_u8) f_u8;
decltype(&pf_sum_workspace) f_sum_ws;
decltype(&pf_sum_f32) f_sum;
decltype(&pf_sum_f32_noalloc) f_sum_noalloc;
decltype(&pf_hist_workspace) f_hist_ws;
decltype(&pf_hist256_u8) f_hist;
decltype(&pf_server_submit) f_submit;
decltype(&pf_server_result) f_result;

PyObject *not_handled() {
    Py_INCREF(Py_NotImplemented);
    return Py_NotImplemented;
}

// Other Python threads run while the call allocates and enqueues.
struct NoGil {
    PyThreadState *s = PyEval_SaveThread();
    ~NoGil() { PyEval_RestoreThread(s); }
};

// The tensor behind `o` if it is a plain GPU tensor of the type and a number
// of dimensions in lo..hi.
const at::Tensor *plain(PyObject *o, at::ScalarType type, int64_t lo, int64_t hi) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.scalar_type() != type || t.layout() != at::kStrided) return nullptr;
    if (t.dim() < lo || t.dim() > hi || !t.is_contiguous()) return nullptr;
    return &t;
}

// Whether t's elements, in memory it owns, reach `bytes` on the GPU.
bool room(const at::Tensor &t, int64_t bytes) {
    if (!t.defined() || !t.is_cuda()) return false;
    const int64_t size = t.element_size();
    return t.numel() * size >= bytes && (int64_t)t.storage().nbytes() - t.storage_offset() * size >= bytes;
}

// `out`: none given, or a plain tensor with as many elements as x.
bool out_for(PyObject *out, const at::Tensor &x, int64_t lo, int64_t hi) {
    if (out == Py_None) return true;
    const at::Tensor *t = plain(out, x.scalar_type(), lo, hi);
    return t && room(*t, x.numel() * x.element_size());
}

bool small_int(PyObject *o, int32_t *v) {
    if (!PyLong_CheckExact(o)) return false;
    int over = 0;
    const long x = PyLong_AsLongAndOverflow(o, &over);
    if (over || x < INT32_MIN || x > INT32_MAX) return false;
    *v = (int32_t)x;
    return true;
}

void *stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

// Sizes of an h x w image that the C ABI takes as int32.
bool image_sizes(const at::Tensor &x, int32_t *h, int32_t *w) {
    const int64_t a = x.size(-2), b = x.size(-1);
    if (a > INT32_MAX || b > INT32_MAX) return false;
    *h = (int32_t)a;
    *w = (int32_t)b;
    return true;
}

// Runs call(y) for the result y (`out` if given, else like(x)) and returns
// y, or the status.
template <class Like, class Call>
PyObject *run(PyObject *out, Like &&like, Call &&call) {
    pf_status st;
    if (out != Py_None) {
        {
            NoGil g;
            st = call(THPVariable_Unpack(out));
        }
        if (st != PF_OK) return PyLong_FromLong(st);
        Py_INCREF(out);
        return out;
    }
    at::Tensor y;
    {
        NoGil g;
        y = like();
        st = call(y);
    }
    return st == PF_OK ? THPVariable_Wrap(std::move(y)) : PyLong_FromLong(st);
}

// Every entry: argument count, no function mode, and no C++ exception past
// this point (the caller's Python path then meets and reports the cause).
template <class F>
PyObject *entry(Py_ssize_t n, Py_ssize_t want, F &&f) {
    if (n != want || at::impl::torch_function_mode_enabled()) return not_handled();
    try {
        return f();
    } catch (const std::exception &) {
        PyErr_Clear();
        return not_handled();
    }
}

bool square_filter(const at::Tensor *f) { return f && f->size(0) == f->size(1) && f->size(0) % 2 == 1 && f->size(0) < 1024; }

// filter2d(x, f, exact, out)
PyObject *filter2d(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry(n, 4, [&]() -> PyObject * {
        const at::Tensor *x = plain(a[0], at::kFloat, 2, 2), *f = plain(a[1], at::kFloat, 2, 2);
        int32_t h, w;
        if (!x || !square_filter(f) || !image_sizes(*x, &h, &w)) return not_handled();
        if (!out_for(a[3], *x, 2, 2)) return not_handled();
        const int exact = PyObject_IsTrue(a[2]);
        if (exact < 0) return nullptr;
        return run(
            a[3], [&] { return at::empty_like(*x); },
            [&](const at::Tensor &y) {
                return f_filter2d(h, w, (int32_t)(f->size(0) / 2), (const float *)x->data_ptr(),
                                  (const float *)f->data_ptr(), (float *)y.data_ptr(), exact ? PF_FLAG_EXACT : 0, stream());
            });
    });
}

// The calls with a border rule: pf_filter2d_f32_border (passes null) and
// pf_filter_chain_f32.
PyObject *bordered(PyObject *px, PyObject *pf, PyObject *ppasses, PyObject *pborder, PyObject *pexact, PyObject *out) {
    const at::Tensor *x = plain(px, at::kFloat, 2, 2), *f = plain(pf, at::kFloat, 2, 2);
    int32_t h, w, passes = 0, border;
    if (!x || !square_filter(f) || !image_sizes(*x, &h, &w)) return not_handled();
    if ((ppasses && !small_int(ppasses, &passes)) || !small_int(pborder, &border)) return not_handled();
    if (!out_for(out, *x, 2, 2)) return not_handled();
    const int exact = PyObject_IsTrue(pexact);
    if (exact < 0) return nullptr;
    return run(
        out, [&] { return at::empty_like(*x); },
        [&](const at::Tensor &y) {
            const int32_t r = (int32_t)(f->size(0) / 2), flags = exact ? PF_FLAG_EXACT : 0;
            const float *in = (const float *)x->data_ptr(), *taps = (const float *)f->data_ptr();
            float *o = (float *)y.data_ptr();
            return ppasses ? f_chain(h, w, r, passes, border, in, taps, o, flags, stream())
                           : f_border(h, w, r, border, in, taps, o, flags, stream());
        });
}

// filter2d_border(x, f, border, exact, out)
PyObject *filter2d_border(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry(n, 5, [&] { return bordered(a[0], a[1], nullptr, a[2], a[3], a[4]); });
}

// filter_chain(x, f, passes, border, exact, out)
PyObject *filter_chain(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry(n, 6, [&] { return bordered(a[0], a[1], a[2], a[3], a[4], a[5]); });
}

// filter_sep(x, fx, fy, exact, out)
PyObject *filter_sep(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry(n, 5, [&]() -> PyObject * {
        const at::Tensor *x = plain(a[0], at::kFloat, 2, 2), *fx = plain(a[1], at::kFloat, 1, 1),
                         *fy = plain(a[2], at::kFloat, 1, 1);
        int32_t h, w;
        if (!x || !fx || !fy || !image_sizes(*x, &h, &w)) return not_handled();
        const int64_t k = fx->numel();
        if (k != fy->numel() || k % 2 != 1 || k >= 1024) return not_handled();
        if (!out_for(a[4], *x, 2, 2)) return not_handled();
        const int exact = PyObject_IsTrue(a[3]);
        if (exact < 0) return nullptr;
        return run(
            a[4], [&] { return at::empty_like(*x); },
            [&](const at::Tensor &y) {
                return f_sep(h, w, (int32_t)(k / 2), (const float *)x->data_ptr(), (const float *)fx->data_ptr(),
                             (const float *)fy->data_ptr(), (float *)y.data_ptr(), exact ? PF_FLAG_EXACT : 0, stream());
            });
    });
}

// filter2d_u8(x, f, shift, out)
PyObject *filter2d_u8(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry(n, 4, [&]() -> PyObject * {
        const at::Tensor *x = plain(a[0], at::kByte, 2, 3), *f = plain(a[1], at::kChar, 2, 2);
        int32_t h, w, shift;
        if (!x || !square_filter(f) || !image_sizes(*x, &h, &w) || !small_int(a[2], &shift)) return not_handled();
        const int64_t c = x->dim() == 3 ? x->size(0) : 1;
        if (c > INT32_MAX || !out_for(a[3], *x, 2, 3)) return not_handled();
        return run(
            a[3], [&] { return at::empty_like(*x); },
            [&](const at::Tensor &y) {
                return f_u8((int32_t)c, h, w, (int32_t)(f->size(0) / 2), shift, (const uint8_t *)x->data_ptr(),
                            (const int8_t *)f->data_ptr(), (uint8_t *)y.data_ptr(), 0, stream());
            });
    });
}

// A float64 workspace of `bytes`, or the caller's.
at::Tensor workspace_for(PyObject *given, size_t bytes, const at::Tensor &x) {
    if (given != Py_None) return THPVariable_Unpack(given);
    return at::empty({std::max<int64_t>((int64_t)(bytes + 7) / 8, 1)}, x.options().dtype(at::kDouble));
}

// A reduction's result (`bytes` of it) or, for bytes < 0, its workspace: none
// given, or a tensor of any type with that room.
bool buffer(PyObject *o, int64_t bytes) {
    if (o == Py_None) return true;
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.defined() && room(t, bytes >= 0 ? bytes : t.numel() * (int64_t)t.element_size());
}

// sum_f32(x, out, workspace)
PyObject *sum_f32(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry(n, 3, [&]() -> PyObject * {
        const at::Tensor *x = plain(a[0], at::kFloat, 0, 64);
        if (!x || !buffer(a[1], 2 * sizeof(double)) || !buffer(a[2], -1)) return not_handled();
        size_t need = 0;
        if (f_sum_ws(x->numel(), &need) != PF_OK) return not_handled();
        return run(
            a[1], [&] { return at::empty({2}, x->options().dtype(at::kDouble)); },
            [&](const at::Tensor &y) {
                const at::Tensor ws = workspace_for(a[2], need, *x);
                return f_sum(x->numel(), (const float *)x->data_ptr(), (double *)y.data_ptr(), ws.data_ptr(),
                             (size_t)ws.numel() * ws.element_size(), stream());
            });
    });
}

// sum_f32_noalloc(x, out)
PyObject *sum_f32_noalloc(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry(n, 2, [&]() -> PyObject * {
        const at::Tensor *x = plain(a[0], at::kFloat, 0, 64);
        if (!x || !buffer(a[1], 2 * sizeof(double))) return not_handled();
        return run(
            a[1], [&] { return at::empty({2}, x->options().dtype(at::kDouble)); },
            [&](const at::Tensor &y) {
                return f_sum_noalloc(x->numel(), (const float *)x->data_ptr(), (double *)y.data_ptr(), stream());
            });
    });
}

// hist256_u8(x, out, workspace)
PyObject *hist256_u8(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry(n, 3, [&]() -> PyObject * {
        const at::Tensor *x = plain(a[0], at::kByte, 0, 64);
        if (!x || !buffer(a[1], 256 * sizeof(int64_t)) || !buffer(a[2], -1)) return not_handled();
        size_t need = 0;
        if (f_hist_ws(x->numel(), &need) != PF_OK) return not_handled();
        // One sub-histogram per CU and 32 KiB of data (see pf_hist256_u8).
        need = std::max(need, (size_t)1024 * (size_t)std::min<int64_t>(x->numel() / 32768 + 1, 256));
        return run(
            a[1], [&] { return at::empty({256}, x->options().dtype(at::kLong)); },
            [&](const at::Tensor &y) {
                const at::Tensor ws = workspace_for(a[2], need, *x);
                return f_hist(x->numel(), (const uint8_t *)x->data_ptr(), (int64_t *)y.data_ptr(), ws.data_ptr(),
                              (size_t)ws.numel() * ws.element_size(), stream());
            });
    });
}

// server_submit(handle, x, r, kind, filt, arrival_ns): the ticket (tickets
// start at 1), or minus the status. filt: a C-contiguous float32 buffer.
PyObject *server_submit(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry(n, 6, [&]() -> PyObject * {
        const at::Tensor *x = plain(a[1], at::kFloat, 2, 2);
        int32_t h, w, r, kind;
        if (!x || !image_sizes(*x, &h, &w) || !small_int(a[2], &r) || !small_int(a[3], &kind)) return not_handled();
        if (!PyLong_CheckExact(a[0]) || !PyLong_CheckExact(a[5])) return not_handled();
        void *srv = PyLong_AsVoidPtr(a[0]);
        const int64_t arrival = PyLong_AsLongLong(a[5]);
        if (PyErr_Occurred()) {
            PyErr_Clear();
            return not_handled();
        }
        Py_buffer b;
        if (PyObject_GetBuffer(a[4], &b, PyBUF_FORMAT | PyBUF_C_CONTIGUOUS) != 0) {
            PyErr_Clear();
            return not_handled();
        }
        PyObject *res = nullptr;
        // Too few weights for the kind and radius: the Python code says so.
        const int64_t k = 2 * (int64_t)r + 1, weights = kind == PF_KIND_2D ? k * k : 2 * k;
        if (b.itemsize == 4 && b.format && b.format[0] == 'f' && !b.format[1] &&
            (r < 0 || r > PF_R_MAX || b.len >= 4 * weights)) {
            int64_t ticket = 0;
            pf_status st;
            {
                NoGil g;
                st = f_submit((pf_server *)srv, h, w, r, kind, (const float *)x->data_ptr(), 0, (const float *)b.buf,
                              stream(), arrival, &ticket);
            }
            res = PyLong_FromLongLong(st == PF_OK ? ticket : -(int64_t)st);
        } else {
            res = not_handled();
        }
        PyBuffer_Release(&b);
        return res;
    });
}

// server_result(handle, ticket, h, w, out): the status. The library copies on
// the null stream: under another current stream the caller's Python code orders
// the copy against it.
PyObject *server_result(PyObject *, PyObject *const *a, Py_ssize_t n) {
    return entry(n, 5, [&]() -> PyObject * {
        const at::Tensor *out = plain(a[4], at::kFloat, 2, 2);
        int32_t h, w;
        if (!out || stream() || !small_int(a[2], &h) || !small_int(a[3], &w)) return not_handled();
        if (!room(*out, 4 * (int64_t)h * w)) return not_handled();
        if (!PyLong_CheckExact(a[0]) || !PyLong_CheckExact(a[1])) return not_handled();
        void *srv = PyLong_AsVoidPtr(a[0]);
        const int64_t ticket = PyLong_AsLongLong(a[1]);
        if (PyErr_Occurred()) {
            PyErr_Clear();
            return not_handled();
        }
        pf_status st;
        {
            NoGil g;
            st = f_result((pf_server *)srv, ticket, h, w, (float *)out->data_ptr(), 0);
        }
        return PyLong_FromLong(st);
    });
}

// bind(addresses): the C ABI's functions, in the order below, from the
// library that the Python binding loaded.
PyObject *bind(PyObject *, PyObject *arg) {
    void **to[] = {(void **)&f_filter2d, (void **)&f_sep,  (void **)&f_chain,       (void **)&f_border,  (void **)&f_u8,
                   (void **)&f_sum_ws,   (void **)&f_sum,  (void **)&f_sum_noalloc, (void **)&f_hist_ws, (void **)&f_hist,
                   (void **)&f_submit,   (void **)&f_result};
    constexpr Py_ssize_t count = sizeof to / sizeof *to;
    if (!PyTuple_Check(arg) || PyTuple_GET_SIZE(arg) != count) {
        PyErr_SetString(PyExc_TypeError, "bind takes one tuple of function addresses");
        return nullptr;
    }
    for (Py_ssize_t i = 0; i < count; ++i) {
        void *p = PyLong_AsVoidPtr(PyTuple_GET_ITEM(arg, i));
        if (!p) return PyErr_Occurred() ? nullptr : (PyErr_SetString(PyExc_ValueError, "null address"), nullptr);
        *to[i] = p;
    }
    Py_RETURN_NONE;
}

#define PF_ENTRY(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {PF_ENTRY(filter2d),    PF_ENTRY(filter2d_border), PF_ENTRY(filter_chain), PF_ENTRY(filter_sep),
                         PF_ENTRY(filter2d_u8), PF_ENTRY(sum_f32),         PF_ENTRY(hist256_u8),   PF_ENTRY(sum_f32_noalloc),
                         PF_ENTRY(server_submit), PF_ENTRY(server_result),
                         {"bind", bind, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) { return PyModule_Create(&module); }
