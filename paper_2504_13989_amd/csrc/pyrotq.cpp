// Python side of the C ABI: argument marshalling for torch tensors, in native code.
//
// A call on a few rows is bounded by the host: the kernel of a 16 x 4096 launch takes 3 us, and the HIP runtime
// about as long to launch it.  Marshalling the same call in Python (shape and stride queries, two output
// tensors, the current stream as an object, ten ctypes conversions) took 9 us on top; here it is a few hundred ns
// for the checks and about half a microsecond for each output tensor, which come straight from the caching
// allocator without a trip through the operator dispatcher.
// The interpreter lock is released around every call into the library, as ctypes does.
#include <Python.h>

#include <ATen/hip/EmptyTensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>
#include <vector>

#include "../../include/rotq.h"

namespace {

PyObject* g_error = nullptr;          // binding.RotqError(code, where)

// A Python error has been set.
struct Raised {};

[[noreturn]] void raise(PyObject* type, const char* text) {
    PyErr_SetString(type, text);
    throw Raised{};
}

void check(int code, const char* where) {
    if (code == RQ_OK) return;
    PyObject* e = g_error ? PyObject_CallFunction(g_error, "is", code, where) : nullptr;
    if (e) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    } else if (!PyErr_Occurred()) {
        PyErr_Format(PyExc_RuntimeError, "%s: %s (%d)", where, rq_strerror(code), code);
    }
    throw Raised{};
}

const at::Tensor& tensor(PyObject* o) {
    if (!THPVariable_Check(o)) raise(PyExc_TypeError, "expected a torch tensor");
    return THPVariable_Unpack(o);
}

long integer(PyObject* o) {
    long v;
    if (PyLong_Check(o)) {
        v = PyLong_AsLong(o);
    } else {
        PyObject* i = PyNumber_Long(o);
        if (!i) throw Raised{};
        v = PyLong_AsLong(i);
        Py_DECREF(i);
    }
    if (v == -1 && PyErr_Occurred()) throw Raised{};
    return v;
}

float real(PyObject* o) {
    const double v = PyFloat_AsDouble(o);
    if (v == -1.0 && PyErr_Occurred()) throw Raised{};
    return (float)v;
}

bool truth(PyObject* o) {
    const int v = PyObject_IsTrue(o);
    if (v < 0) throw Raised{};
    return v != 0;
}

const rq_hadamard_t* handle(PyObject* o) {
    void* p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) throw Raised{};
    return static_cast<const rq_hadamard_t*>(p);
}

int order(const rq_hadamard_t* h, const char* where) {
    int n = 0;
    check(rq_hadamard_info(h, &n, nullptr, nullptr, nullptr, nullptr), where);
    return n;
}

void* stream(PyObject* o) {
    if (o == Py_None) return c10::hip::getCurrentHIPStream().stream();
    PyObject* v = PyObject_GetAttrString(o, "cuda_stream");
    if (!v) throw Raised{};
    void* p = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    if (!p && PyErr_Occurred()) throw Raised{};
    return p;
}

int dtype_code(at::ScalarType t) {
    switch (t) {
        case at::kBFloat16: return RQ_BF16;
        case at::kFloat: return RQ_F32;
        case at::kHalf: return RQ_F16;
        default: return -1;
    }
}

// Rows of a tensor whose last dimension is contiguous and whose leading dimensions collapse to one row index
// with a single stride.
struct Rows {
    const void* X;
    int dtype;
    int64_t rows, ld;
    int d;
    c10::Device device;
};

Rows rows_of(PyObject* o) {
    const at::Tensor& x = tensor(o);
    if (!x.is_cuda()) raise(PyExc_ValueError, "x must be a device tensor");
    const int64_t nd = x.dim();
    if (nd < 1) raise(PyExc_IndexError, "x must have at least one dimension");
    if (x.stride(nd - 1) != 1) raise(PyExc_ValueError, "last dimension must be contiguous");
    const int code = dtype_code(x.scalar_type());
    if (code < 0) raise(PyExc_TypeError, "unsupported input dtype");
    const int64_t d = x.size(nd - 1);
    if (d > INT32_MAX) raise(PyExc_ValueError, "rows are too wide");
    Rows r{x.const_data_ptr(), code, 0, d, (int)d, x.device()};
    if (x.is_contiguous()) {
        r.rows = d > 0 ? x.numel() / d : 0;
    } else {
        if (nd != 2) raise(PyExc_ValueError, "non-contiguous input must be 2-D");
        r.rows = x.size(0);
        if (r.rows > 1) r.ld = x.stride(0);
    }
    return r;
}

// An output tensor: the caller's, or a new one.  `ref` is a new reference.
struct Out {
    PyObject* ref = nullptr;
    void* data = nullptr;
    Out() = default;
    Out(const Out&) = delete;
    Out& operator=(const Out&) = delete;
    ~Out() { Py_XDECREF(ref); }
    PyObject* take() {
        PyObject* r = ref;
        ref = nullptr;
        return r;
    }
    void given(PyObject* o) {
        data = tensor(o).data_ptr();
        Py_INCREF(o);
        ref = o;
    }
    void adopt(at::Tensor&& y) {
        data = y.data_ptr();
        ref = THPVariable_Wrap(std::move(y));
        if (!ref) throw Raised{};
    }
    void make(PyObject* o, at::IntArrayRef size, at::ScalarType t, c10::Device device) {
        if (o != Py_None) return given(o);
        adopt(at::Tensor(at::detail::empty_cuda(size, t, device, std::nullopt)));
    }
};

// The results of a quantizing call: codes [rows, row_bytes], then one or two float tensors of `size`.  Each has a storage
// of its own: torch does not save tensors of different types that share one, and a result that is resized must not
// grow into another.  (One allocation for all of them would save the host 0.5 us a call.)
void make_results(c10::Device device, int64_t rows, int64_t row_bytes, at::IntArrayRef size, std::initializer_list<PyObject*> given,
                  std::initializer_list<Out*> outs) {
    PyObject* const* g = given.begin();
    Out* const* o = outs.begin();
    o[0]->make(g[0], {rows, row_bytes}, at::kByte, device);
    for (size_t i = 1; i < outs.size(); ++i) o[i]->make(g[i], size, at::kFloat, device);
}

template <typename F>
int unlocked(F f) {
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return rc;
}

PyObject* tuple2(Out& a, Out& b) {
    PyObject* t = PyTuple_New(2);
    if (!t) throw Raised{};
    PyTuple_SET_ITEM(t, 0, a.take());
    PyTuple_SET_ITEM(t, 1, b.take());
    return t;
}
PyObject* tuple3(Out& a, Out& b, Out& c) {
    PyObject* t = PyTuple_New(3);
    if (!t) throw Raised{};
    PyTuple_SET_ITEM(t, 0, a.take());
    PyTuple_SET_ITEM(t, 1, b.take());
    PyTuple_SET_ITEM(t, 2, c.take());
    return t;
}

// Function bodies: called with at least `Arity` arguments, may throw Raised or a torch / C++ exception.
using Body = PyObject* (*)(PyObject* const*);

template <Body body, int Arity>
PyObject* entry(PyObject*, PyObject* const* a, Py_ssize_t n) {
    if (n != Arity) {
        PyErr_Format(PyExc_TypeError, "expected %d arguments, got %zd", Arity, n);
        return nullptr;
    }
    try {
        return body(a);
    } catch (const Raised&) {
    } catch (const c10::OutOfMemoryError& e) {
        // torch.OutOfMemoryError, as its own operators raise it
        PyObject* m = PyImport_ImportModule("torch");
        PyObject* t = m ? PyObject_GetAttrString(m, "OutOfMemoryError") : nullptr;
        if (!t) PyErr_Clear();
        PyErr_SetString(t ? t : PyExc_RuntimeError, e.what_without_backtrace());
        Py_XDECREF(t);
        Py_XDECREF(m);
    } catch (const c10::Error& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what_without_backtrace());
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}

int width(PyObject* o, const char* where) {
    const long bits = integer(o);
    if (bits != 3 && bits != 4) check(RQ_ERR_ARG, where);
    return (int)bits;
}

// (handle, x, bits, clip, codes, scales, stream)
PyObject* rotate_quantize(PyObject* const* a) {
    const char* where = "rq_rotate_quantize";
    const rq_hadamard_t* h = handle(a[0]);
    const Rows x = rows_of(a[1]);
    const int bits = width(a[2], where), n = order(h, where);
    const float clip = real(a[3]);
    void* s = stream(a[6]);
    Out codes, scales;
    make_results(x.device, x.rows, (int64_t)n * bits / 8, {x.rows}, {a[4], a[5]}, {&codes, &scales});
    check(unlocked([&] {
        return rq_rotate_quantize(h, x.X, x.dtype, x.rows, x.d, x.ld, bits, clip, codes.data,
                                  static_cast<float*>(scales.data), s);
    }), where);
    return tuple2(codes, scales);
}

// (handle, x, bits, clip, codes, scales, mins, stream)
PyObject* rotate_quantize_asym(PyObject* const* a) {
    const char* where = "rq_rotate_quantize_asym";
    const rq_hadamard_t* h = handle(a[0]);
    const Rows x = rows_of(a[1]);
    const int bits = width(a[2], where), n = order(h, where);
    const float clip = real(a[3]);
    void* s = stream(a[7]);
    const int64_t groups = n >= RQ_GROUP ? n / RQ_GROUP : 1;
    Out codes, scales, mins;
    make_results(x.device, x.rows, (int64_t)n * bits / 8, {x.rows, groups}, {a[4], a[5], a[6]}, {&codes, &scales, &mins});
    check(unlocked([&] {
        return rq_rotate_quantize_asym(h, x.X, x.dtype, x.rows, x.d, x.ld, bits, clip, codes.data,
                                       static_cast<float*>(scales.data), static_cast<float*>(mins.data), s);
    }), where);
    return tuple3(codes, scales, mins);
}

// (x, bits, clip, codes, scales, stream)
PyObject* quantize(PyObject* const* a) {
    const char* where = "rq_quantize";
    const Rows x = rows_of(a[0]);
    const int bits = width(a[1], where);
    const float clip = real(a[2]);
    void* s = stream(a[5]);
    Out codes, scales;
    make_results(x.device, x.rows, (int64_t)x.d * bits / 8, {x.rows}, {a[3], a[4]}, {&codes, &scales});
    check(unlocked([&] {
        return rq_quantize(x.X, x.dtype, x.rows, x.d, x.ld, bits, clip, codes.data, static_cast<float*>(scales.data), s);
    }), where);
    return tuple2(codes, scales);
}

// (x, bits, clip, codes, scales, mins, stream)
PyObject* quantize_asym(PyObject* const* a) {
    const char* where = "rq_quantize_asym";
    const Rows x = rows_of(a[0]);
    const int bits = width(a[1], where);
    const float clip = real(a[2]);
    void* s = stream(a[6]);
    const int64_t groups = x.d >= RQ_GROUP ? x.d / RQ_GROUP : 1;
    Out codes, scales, mins;
    make_results(x.device, x.rows, (int64_t)x.d * bits / 8, {x.rows, groups}, {a[3], a[4], a[5]}, {&codes, &scales, &mins});
    check(unlocked([&] {
        return rq_quantize_asym(x.X, x.dtype, x.rows, x.d, x.ld, bits, clip, codes.data,
                                static_cast<float*>(scales.data), static_cast<float*>(mins.data), s);
    }), where);
    return tuple3(codes, scales, mins);
}

// The floating-point result of rotate / dequantize_rotate: out (or None), d_out (or None), out_dtype (or None).
struct FloatOut {
    Out y;
    int code;
    int64_t d_out, ld;
    FloatOut(PyObject* out, PyObject* d_out_o, PyObject* dtype_o, int n, int64_t rows, c10::Device device) {
        d_out = d_out_o == Py_None ? n : integer(d_out_o);
        if (d_out > INT32_MAX) d_out = INT32_MAX;      // refused by the library
        at::ScalarType t = at::kFloat;
        if (out == Py_None && dtype_o != Py_None) {
            if (!THPDtype_Check(dtype_o)) raise(PyExc_TypeError, "out_dtype must be a torch dtype");
            t = reinterpret_cast<THPDtype*>(dtype_o)->scalar_type;
        } else if (out != Py_None) {
            t = tensor(out).scalar_type();
        }
        code = dtype_code(t);
        if (code < 0) raise(PyExc_ValueError, "output dtype must be float32, bfloat16 or float16");
        y.make(out, {rows, d_out}, t, device);
        ld = d_out;
        if (out != Py_None) {
            const int64_t st = tensor(out).stride(0);
            ld = rows > 1 || st > d_out ? st : d_out;
        }
    }
};

// (handle, x, transpose, d_out, out_dtype, out, stream)
PyObject* rotate(PyObject* const* a) {
    const char* where = "rq_rotate";
    const rq_hadamard_t* h = handle(a[0]);
    const Rows x = rows_of(a[1]);
    const int transpose = truth(a[2]);
    void* s = stream(a[6]);
    FloatOut o(a[5], a[3], a[4], order(h, where), x.rows, x.device);
    check(unlocked([&] {
        return rq_rotate(h, x.X, x.dtype, x.rows, x.d, x.ld, transpose, o.y.data, o.code, (int)o.d_out, o.ld, s);
    }), where);
    return o.y.take();
}

// (handle, codes, scales, bits, mins, transpose, d_out, out_dtype, out, stream)
PyObject* dequantize_rotate(PyObject* const* a) {
    const char* where = "rq_dequantize_rotate";
    const rq_hadamard_t* h = handle(a[0]);
    const at::Tensor& codes = tensor(a[1]);
    const float* scales = static_cast<const float*>(tensor(a[2]).const_data_ptr());
    const int bits = (int)integer(a[3]);
    const float* mins = a[4] == Py_None ? nullptr : static_cast<const float*>(tensor(a[4]).const_data_ptr());
    const int transpose = truth(a[5]);
    const int64_t rows = codes.size(0);
    void* s = stream(a[9]);
    FloatOut o(a[8], a[6], a[7], order(h, where), rows, codes.device());
    check(unlocked([&] {
        return rq_dequantize_rotate(h, codes.const_data_ptr(), scales, mins, rows, bits, transpose, o.y.data, o.code,
                                    (int)o.d_out, o.ld, s);
    }), where);
    return o.y.take();
}

// (handle, codes, scales, bits, mins, out, stream)
PyObject* dequantize(PyObject* const* a) {
    const bool asym = a[4] != Py_None;
    const char* where = asym ? "rq_dequantize_asym" : "rq_dequantize";
    const rq_hadamard_t* h = handle(a[0]);
    const at::Tensor& codes = tensor(a[1]);
    const float* scales = static_cast<const float*>(tensor(a[2]).const_data_ptr());
    const int bits = (int)integer(a[3]);
    const float* mins = asym ? static_cast<const float*>(tensor(a[4]).const_data_ptr()) : nullptr;
    const int64_t rows = codes.size(0);
    void* s = stream(a[6]);
    Out y;
    y.make(a[5], {rows, (int64_t)order(h, where)}, at::kFloat, codes.device());
    check(unlocked([&] {
        float* Y = static_cast<float*>(y.data);
        return asym ? rq_dequantize_asym(h, codes.const_data_ptr(), scales, mins, rows, bits, Y, s)
                    : rq_dequantize(h, codes.const_data_ptr(), scales, rows, bits, Y, s);
    }), where);
    return y.take();
}

// A sequence of clip ratios as floats (a float32 array is copied whole).
std::vector<float> clip_list(PyObject* o) {
    Py_buffer b;
    if (PyObject_CheckBuffer(o) && PyObject_GetBuffer(o, &b, PyBUF_ND | PyBUF_FORMAT) == 0) {
        if (b.ndim == 1 && b.itemsize == 4 && b.format && std::strcmp(b.format, "f") == 0) {
            const float* p = static_cast<const float*>(b.buf);
            std::vector<float> v(p, p + b.shape[0]);
            PyBuffer_Release(&b);
            return v;
        }
        PyBuffer_Release(&b);
    }
    PyErr_Clear();
    PyObject* f = PySequence_Fast(o, "clips must be a sequence of numbers");
    if (!f) throw Raised{};
    const Py_ssize_t k = PySequence_Fast_GET_SIZE(f);
    std::vector<float> v((size_t)k);
    for (Py_ssize_t i = 0; i < k; ++i) {
        const double c = PyFloat_AsDouble(PySequence_Fast_GET_ITEM(f, i));
        if (c == -1.0 && PyErr_Occurred()) {
            Py_DECREF(f);
            throw Raised{};
        }
        v[(size_t)i] = (float)c;
    }
    Py_DECREF(f);
    return v;
}

// Device scratch of at least `bytes`: the caller's tensor, or a new one.
struct Scratch {
    at::Tensor own;
    void* data;
    size_t bytes;
    Scratch(PyObject* o, size_t need, c10::Device device) {
        if (o != Py_None) {
            const at::Tensor& t = tensor(o);
            data = t.data_ptr();
            bytes = (size_t)t.numel() * t.element_size();
        } else {
            const int64_t words = (int64_t)((need > 8 ? need : 8) + 7) / 8;
            own = at::Tensor(at::detail::empty_cuda({words}, at::kDouble, device, std::nullopt));
            data = own.data_ptr();
            bytes = (size_t)words * 8;
        }
    }
};

// (handle, x, bits, clips, mse, workspace, stream, asym)
PyObject* quant_error(PyObject* const* a) {
    const bool asym = truth(a[7]);
    const char* where = asym ? "rq_quant_error_asym" : "rq_quant_error";
    const rq_hadamard_t* h = handle(a[0]);
    const Rows x = rows_of(a[1]);
    const int bits = (int)integer(a[2]);
    const std::vector<float> clips = clip_list(a[3]);
    const int k = (int)clips.size();
    void* s = stream(a[6]);
    Out mse;
    mse.make(a[4], {k}, at::kFloat, x.device);
    const Scratch ws(a[5], rq_quant_error_workspace(x.rows, k), x.device);
    check(unlocked([&] {
        auto fn = asym ? rq_quant_error_asym : rq_quant_error;
        return fn(h, x.X, x.dtype, x.rows, x.d, x.ld, bits, clips.data(), k, static_cast<float*>(mse.data), ws.data,
                  ws.bytes, s);
    }), where);
    return mse.take();
}

// (handle, x, bits, clips, mse, stream)
PyObject* quant_error_noalloc(PyObject* const* a) {
    const char* where = "rq_quant_error_noalloc";
    const rq_hadamard_t* h = handle(a[0]);
    const Rows x = rows_of(a[1]);
    const int bits = (int)integer(a[2]);
    const std::vector<float> clips = clip_list(a[3]);
    void* s = stream(a[5]);
    Out mse;
    mse.given(a[4]);
    check(unlocked([&] {
        return rq_quant_error_noalloc(h, x.X, x.dtype, x.rows, x.d, x.ld, bits, clips.data(), (int)clips.size(),
                                      static_cast<float*>(mse.data), s);
    }), where);
    return mse.take();
}

// (handle, x, bits, eps, max_evals, workspace, stream, asym)
PyObject* gbs_search(PyObject* const* a) {
    const bool asym = truth(a[7]);
    const char* where = asym ? "rq_gbs_search_asym" : "rq_gbs_search";
    const rq_hadamard_t* h = handle(a[0]);
    const Rows x = rows_of(a[1]);
    const int bits = (int)integer(a[2]);
    const float eps = real(a[3]);
    const long evals = integer(a[4]);
    if (evals < 1 || evals > 256) check(RQ_ERR_ARG, where);
    void* s = stream(a[6]);
    const Scratch ws(a[5], rq_gbs_workspace(x.rows), x.device);
    std::vector<float> tc((size_t)evals), tm((size_t)evals);
    float clip = 0.0f, mse = 0.0f;
    int n = 0;
    check(unlocked([&] {
        auto fn = asym ? rq_gbs_search_asym : rq_gbs_search;
        return fn(h, x.X, x.dtype, x.rows, x.d, x.ld, bits, eps, (int)evals, ws.data, ws.bytes, s, &clip, &mse, tc.data(),
                  tm.data(), &n);
    }), where);
    PyObject* trace = PyList_New(n);
    if (!trace) throw Raised{};
    for (int i = 0; i < n; ++i) {
        PyObject* p = Py_BuildValue("(dd)", (double)tc[(size_t)i], (double)tm[(size_t)i]);
        if (!p) {
            Py_DECREF(trace);
            throw Raised{};
        }
        PyList_SET_ITEM(trace, i, p);
    }
    return Py_BuildValue("(ddN)", (double)clip, (double)mse, trace);
}

// Called once by the binding: the class of the errors raised for the library's error codes.
PyObject* set_error(PyObject*, PyObject* cls) {
    Py_INCREF(cls);
    Py_XSETREF(g_error, cls);
    Py_RETURN_NONE;
}

#define RQ_ENTRY(name, arity) \
    {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&entry<name, arity>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    RQ_ENTRY(rotate_quantize, 7),   RQ_ENTRY(rotate_quantize_asym, 8), RQ_ENTRY(quantize, 6),
    RQ_ENTRY(quantize_asym, 7),     RQ_ENTRY(rotate, 7),               RQ_ENTRY(dequantize_rotate, 10),
    RQ_ENTRY(dequantize, 7),        RQ_ENTRY(quant_error, 8),          RQ_ENTRY(quant_error_noalloc, 6),
    RQ_ENTRY(gbs_search, 8),        {"set_error", set_error, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
#undef RQ_ENTRY

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pyrotq", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pyrotq() { return PyModule_Create(&module); }
