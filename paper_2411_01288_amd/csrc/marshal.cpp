// Argument marshalling of the four calls of a pass (route, index, fwd, bwd) for binding.py: the same checks as its
// _ptr, on the tensors themselves.  A step of a small layer is a few dozen microseconds of kernels and passes 23 tensors; read
// attribute by attribute from Python their checks took longer than the launches (issuing a step of 256 x 64 x 256 in fp32
// 42 -> 25 us, a serving pass of 16 tokens 33 -> 25 us).  Whatever is not a plain dense tensor of the expected kind (a subclass, an
// active function mode, None, a wrong size) goes to _ptr, which decides and words the error.
#include <Python.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/PythonTorchFunctionTLS.h>

#include <initializer_list>

#include "../../include/hexa_moe.h"

namespace {

typedef decltype(&hexa_moe_route) route_fn;
typedef decltype(&hexa_moe_index) index_fn;
typedef decltype(&hexa_moe_fwd) fwd_fn;
typedef decltype(&hexa_moe_bwd) bwd_fn;

// the library's functions (the library that binding.py has loaded), and objects of binding.py
struct {
    route_fn route;
    index_fn index;
    fwd_fn fwd;
    bwd_fn bwd;
    PyObject* shape_type;
    PyObject* ptr;          // binding._ptr
    PyObject* dtype[4];     // torch.float32, bfloat16, float16 (by hexa_dtype), int32
} g;
constexpr int kInt32 = 3;
constexpr at::ScalarType kScalar[4] = {at::kFloat, at::kBFloat16, at::kHalf, at::kInt};

struct Failed {};           // a Python error is set

PyObject* checked(PyObject* o) {
    if (!o) throw Failed{};
    return o;
}
struct Ref {                // owns a reference
    PyObject* o;
    explicit Ref(PyObject* p) : o(checked(p)) {}
    Ref(const Ref&) = delete;
    ~Ref() { Py_DECREF(o); }
};

bool plain_tensor(PyObject* t) { return THPVariable_CheckExact(t) && !at::impl::torch_function_mode_enabled(); }

void* address(PyObject* number) {
    if (number == Py_None) return nullptr;
    void* p = PyLong_AsVoidPtr(number);
    if (!p && PyErr_Occurred()) throw Failed{};
    return p;
}

// device pointer of a dense tensor of these sizes, NULL for None
void* ptr(PyObject* t, std::initializer_list<int64_t> dims, int dtype, const char* name) {
    if (plain_tensor(t)) {
        const at::Tensor& x = THPVariable_Unpack(t);
        if (x.is_cuda() && x.is_contiguous() && x.scalar_type() == kScalar[dtype] && x.sizes().equals(dims)) return x.data_ptr();
    }
    const Ref d(PyTuple_New((Py_ssize_t)dims.size()));
    Py_ssize_t i = 0;
    for (const int64_t n : dims) PyTuple_SET_ITEM(d.o, i++, checked(PyLong_FromLongLong(n)));
    const Ref r(PyObject_CallFunction(g.ptr, "OOOs", t, d.o, g.dtype[dtype], name));
    return address(r.o);
}
// any tensor: where it lies, and its elements
void* buffer(PyObject* t, size_t& elements) {
    if (plain_tensor(t)) {
        const at::Tensor& x = THPVariable_Unpack(t);
        elements = (size_t)x.numel();
        return x.data_ptr();
    }
    const Ref p(PyObject_CallMethod(t, "data_ptr", nullptr)), n(PyObject_CallMethod(t, "numel", nullptr));
    elements = PyLong_AsSize_t(n.o);
    if (PyErr_Occurred()) throw Failed{};
    return address(p.o);
}

hexa_moe_shape shape_of(PyObject* o) {
    const int is = PyObject_IsInstance(o, g.shape_type);
    if (is < 0) throw Failed{};
    Py_buffer view;
    if (!is || PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "shape: need a Shape (see make_shape)");
        throw Failed{};
    }
    hexa_moe_shape s{};
    if ((size_t)view.len == sizeof(s)) s = *static_cast<const hexa_moe_shape*>(view.buf);
    PyBuffer_Release(&view);
    return s;
}
int dtype_of(const hexa_moe_shape& s) {
    if (s.dtype < 0 || s.dtype >= kInt32) {      // (as the table of dtypes in binding.py answers)
        PyErr_Format(PyExc_KeyError, "%d", (int)s.dtype);
        throw Failed{};
    }
    return s.dtype;
}
void* item(PyObject* map, const char* key, std::initializer_list<int64_t> dims, int dtype) {
    const Ref k(PyUnicode_InternFromString(key));
    const Ref t(PyObject_GetItem(map, k.o));
    return ptr(t.o, dims, dtype, key);
}
hexa_moe_idx idx_of(const hexa_moe_shape& s, PyObject* map) {
    const int64_t A = (int64_t)s.T * s.k, E = s.E;
    hexa_moe_idx i{};
    i.counts = (int32_t*)item(map, "counts", {E}, kInt32);
    i.offsets = (int32_t*)item(map, "offsets", {E + 1}, kInt32);
    i.perm = (int32_t*)item(map, "perm", {A}, kInt32);
    i.inv = (int32_t*)item(map, "inv", {A}, kInt32);
    return i;
}

// An entry point: argument count, exceptions, and the launches without the interpreter's lock.
template <int N, typename F>
PyObject* call(PyObject* const* args, Py_ssize_t n, F marshal) {
    HANDLE_TH_ERRORS
    if (n != N) {
        PyErr_Format(PyExc_TypeError, "%d arguments expected, %zd given", N, n);
        return nullptr;
    }
    try {
        const auto launch = marshal(args);
        int status;
        Py_BEGIN_ALLOW_THREADS
        status = (int)launch();
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(status);
    } catch (const Failed&) {
        return nullptr;
    }
    END_HANDLE_TH_ERRORS
}

// (shape, logits, gate_mode, topk_idx, gate, stream)
PyObject* route(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return call<6>(args, n, [](PyObject* const* a) {
        const hexa_moe_shape s = shape_of(a[0]);
        const auto* logits = (const float*)ptr(a[1], {s.T, s.E}, HEXA_F32, "logits");
        const long mode = PyLong_AsLong(a[2]);
        if (mode == -1 && PyErr_Occurred()) throw Failed{};
        auto* topk = (int32_t*)ptr(a[3], {s.T, s.k}, kInt32, "topk_idx");
        auto* gate = (float*)ptr(a[4], {s.T, s.k}, HEXA_F32, "gate");
        void* st = address(a[5]);
        return [=] { return g.route(&s, logits, (int32_t)mode, topk, gate, st); };
    });
}

// (shape, topk_idx, idx, scratch, stream)
PyObject* index(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return call<5>(args, n, [](PyObject* const* a) {
        const hexa_moe_shape s = shape_of(a[0]);
        const auto* topk = (const int32_t*)ptr(a[1], {s.T, s.k}, kInt32, "topk_idx");
        const hexa_moe_idx idx = idx_of(s, a[2]);
        size_t bytes = 0;
        void* scratch = buffer(a[3], bytes);
        void* st = address(a[4]);
        return [=] { return g.index(&s, topk, idx, scratch, bytes, st); };
    });
}

// (shape, x, topk_idx, gate, W1, b1, W2, b2, idx, workspace, y, stream)
PyObject* fwd(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return call<12>(args, n, [](PyObject* const* a) {
        const hexa_moe_shape s = shape_of(a[0]);
        const int64_t T = s.T, d = s.d_model, f = s.d_ff, E = s.E, k = s.k;
        const int dt = dtype_of(s);
        const void* x = ptr(a[1], {T, d}, dt, "x");
        const auto* topk = (const int32_t*)ptr(a[2], {T, k}, kInt32, "topk_idx");
        const auto* gate = (const float*)ptr(a[3], {T, k}, HEXA_F32, "gate");
        const void *W1 = ptr(a[4], {E, d, f}, dt, "W1"), *b1 = ptr(a[5], {E, f}, dt, "b1");
        const void *W2 = ptr(a[6], {E, f, d}, dt, "W2"), *b2 = ptr(a[7], {E, d}, dt, "b2");
        const hexa_moe_idx idx = idx_of(s, a[8]);
        void* y = ptr(a[10], {T, d}, dt, "y");
        size_t bytes = 0;
        void* ws = buffer(a[9], bytes);
        void* st = address(a[11]);
        return [=] { return g.fwd(&s, x, topk, gate, W1, b1, W2, b2, idx, y, ws, bytes, st); };
    });
}

// (shape, dY, x, topk_idx, gate, W1, W2, idx, workspace, out, stream)
PyObject* bwd(PyObject*, PyObject* const* args, Py_ssize_t n) {
    return call<11>(args, n, [](PyObject* const* a) {
        const hexa_moe_shape s = shape_of(a[0]);
        const int64_t T = s.T, d = s.d_model, f = s.d_ff, E = s.E, k = s.k;
        const int dt = dtype_of(s);
        const void *dY = ptr(a[1], {T, d}, dt, "dY"), *x = ptr(a[2], {T, d}, dt, "x");
        const auto* topk = (const int32_t*)ptr(a[3], {T, k}, kInt32, "topk_idx");
        const auto* gate = (const float*)ptr(a[4], {T, k}, HEXA_F32, "gate");
        const void *W1 = ptr(a[5], {E, d, f}, dt, "W1"), *W2 = ptr(a[6], {E, f, d}, dt, "W2");
        const hexa_moe_idx idx = idx_of(s, a[7]);
        size_t bytes = 0;
        void* ws = buffer(a[8], bytes);
        void* dx = item(a[9], "dx", {T, d}, dt);
        auto* dW1 = (float*)item(a[9], "dW1", {E, d, f}, HEXA_F32);
        auto* db1 = (float*)item(a[9], "db1", {E, f}, HEXA_F32);
        auto* dW2 = (float*)item(a[9], "dW2", {E, f, d}, HEXA_F32);
        auto* db2 = (float*)item(a[9], "db2", {E, d}, HEXA_F32);
        const Ref dg(PyObject_CallMethod(a[9], "get", "s", "dgate"));
        auto* dgate = (float*)ptr(dg.o, {T, k}, HEXA_F32, "dgate");
        void* st = address(a[10]);
        return [=] { return g.bwd(&s, dY, x, topk, gate, W1, W2, idx, ws, bytes, dx, dW1, db1, dW2, db2, dgate, st); };
    });
}

// ((addresses of hexa_moe_route, _index, _fwd, _bwd), Shape, _ptr, (float32, bfloat16, float16, int32))
PyObject* bind(PyObject*, PyObject* args) {
    unsigned long long r, i, f, b;
    PyObject *shape_type, *py_ptr, *d[4];
    if (!PyArg_ParseTuple(args, "(KKKK)OO(OOOO)", &r, &i, &f, &b, &shape_type, &py_ptr, &d[0], &d[1], &d[2], &d[3])) return nullptr;
    g.route = (route_fn)r; g.index = (index_fn)i; g.fwd = (fwd_fn)f; g.bwd = (bwd_fn)b;
    Py_INCREF(shape_type); g.shape_type = shape_type;
    Py_INCREF(py_ptr); g.ptr = py_ptr;
    for (int q = 0; q < 4; ++q) { Py_INCREF(d[q]); g.dtype[q] = d[q]; }
    Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    {"route", (PyCFunction)(void (*)(void))route, METH_FASTCALL, nullptr},
    {"index", (PyCFunction)(void (*)(void))index, METH_FASTCALL, nullptr},
    {"fwd", (PyCFunction)(void (*)(void))fwd, METH_FASTCALL, nullptr},
    {"bwd", (PyCFunction)(void (*)(void))bwd, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// torch: the version this was built for (it reads tensors as laid out there; the binding compares)
PyMODINIT_FUNC PyInit__marshal() {
    PyObject* m = PyModule_Create(&kModule);
    if (m && PyModule_AddStringConstant(m, "torch", BUILT_FOR_TORCH) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
