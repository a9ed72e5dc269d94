// The marshalling of hbl.py's calls on small problems, natively: a forward call of a few tokens is two launches of 2 to 3 us, and
// its checks, allocations and argument conversion took 7 us in Python.  Every function takes the call's arguments as they
// come, and either makes the call and returns its result, returns the library's status (an int) if it is not 0, or returns None
// without having done anything where an argument is not the ordinary one (another type, layout, device or size than a plain
// contiguous device tensor that fits): the Python code then takes the call and raises what it raises.
// (16 x 256 -> 256, fp32, outputs and workspace allocated by the call, calls in a row: 11.9 -> 8.0 us with two launches, 5.3 with one.)
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/Functions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "hbitlinear.h"

namespace {

// Entry points of the loaded library (bind()).
struct Library {
    decltype(&hbl_hbitlinear_forward) forward[2];   // with the transform, plain
    decltype(&hbl_ln_bitlinear_forward) ln_forward;
    decltype(&hbl_bitlinear_forward_small) small;
    decltype(&hbl_workspace_bytes) workspace_bytes;
    decltype(&hbl_fwht) fwht;
    decltype(&hbl_kv_quant_absmax) kv_quant;
    decltype(&hbl_kv_dequant) kv_dequant;
    decltype(&hbl_kv_packed_bytes) kv_packed_bytes;
} lib;

PyObject* decline() { Py_RETURN_NONE; }

// A plain contiguous device tensor with memory of its own: nothing that a mode, a transform or a subclass stands behind.
bool ordinary(const at::Tensor& t) {
    using K = c10::DispatchKey;
    static const c10::DispatchKeySet other({K::Python, K::PythonTLSSnapshot, K::Functionalize, K::FuncTorchBatched,
                                            K::FuncTorchGradWrapper, K::Batched, K::Conjugate, K::Negative, K::ZeroTensor});
    return t.defined() && t.is_cuda() && t.layout() == c10::kStrided && t.has_storage() && !t.key_set().has_any(other) && t.is_contiguous();
}
// The tensor behind a Python object, or nullptr if it is not an ordinary one.  (torch.Tensor and Parameter, no other subclass.)
const at::Tensor* tensor(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return ordinary(t) ? &t : nullptr;
}
// Integers and floats as they are written; others (numpy scalars, bools as sizes) take the Python path.
bool get_int(PyObject* o, int64_t& v) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0 && v > -(int64_t{1} << 31) && v < (int64_t{1} << 31);
}
bool get_float(PyObject* o, float& v) {
    if (!PyFloat_CheckExact(o)) return false;
    v = (float)PyFloat_AS_DOUBLE(o);
    return true;
}
int x_dtype(const at::Tensor& t) {
    return t.scalar_type() == at::kBFloat16 ? HBL_BF16 : (t.scalar_type() == at::kFloat ? HBL_F32 : -1);
}
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// Other threads run during the allocations and the library's call, as they do during torch.empty and a call through ctypes.  An
// exception (an allocation that fails) passes the destructor, which takes the lock back, on its way to END_HANDLE_TH_ERRORS.
template <typename Call>
int without_gil(Call call) {
    struct Released {
        PyThreadState* const state = PyEval_SaveThread();
        ~Released() { PyEval_RestoreThread(state); }
    } released;
    return call();
}
constexpr int kDeclined = 1;   // beside the library's statuses, which are not positive

PyObject* result(int rc, PyObject* given, const at::Tensor& t) {
    if (rc == kDeclined) return decline();
    if (rc != HBL_OK) return PyLong_FromLong(rc);
    if (given != nullptr && given != Py_None) {
        Py_INCREF(given);
        return given;
    }
    return THPVariable_Wrap(t);
}

// Memory that a call reads (a lazily cloned tensor is read where it is) or writes (its own copy is made here, which may fail).
const void* input(const at::Tensor& t) { return t.const_data_ptr(); }
const float* floats(const at::Tensor& t) { return t.const_data_ptr<float>(); }

// What the projection calls share: x [T, K], packed weights, scales, y (allocated if it is not given).
struct Projection {
    const at::Tensor *x, *packed, *scales;
    at::Tensor y, workspace;
    int64_t T, K, N, bits;
    int dtype;
    float eps;
    // y and the workspace that were not given; without the interpreter's lock
    bool allocate(bool with_workspace) {
        if (!y.defined()) y = at::empty({T, N}, x->options().dtype(at::kBFloat16));
        if (with_workspace && !workspace.defined())
            workspace = at::empty({(int64_t)lib.workspace_bytes(T, K, N, (int)bits)}, x->options().dtype(at::kByte));
        return ordinary(y) && (!with_workspace || ordinary(workspace));
    }
};
bool get_projection(PyObject* x, PyObject* packed, PyObject* n, PyObject* scales, PyObject* bits, PyObject* eps, PyObject* y,
                    Projection& p) {
    p.x = tensor(x);
    p.packed = tensor(packed);
    p.scales = tensor(scales);
    if (!p.x || !p.packed || !p.scales || p.x->dim() != 2 || !get_int(n, p.N) || !get_int(bits, p.bits) || !get_float(eps, p.eps))
        return false;
    p.T = p.x->size(0);
    p.K = p.x->size(1);
    p.dtype = x_dtype(*p.x);
    if (p.dtype < 0 || p.N <= 0 || p.K <= 0 || p.K > (1 << 24) || p.packed->scalar_type() != at::kByte ||
        p.packed->numel() < p.N * p.K / 4 + 4 * p.N || p.scales->scalar_type() != at::kFloat || p.scales->numel() < 1)
        return false;
    if (y != Py_None) {
        const at::Tensor* t = tensor(y);
        if (!t || t->scalar_type() != at::kBFloat16 || t->dim() != 2 || t->size(0) != p.T || t->size(1) != p.N) return false;
        p.y = *t;
    }
    return true;
}
bool get_workspace(PyObject* o, Projection& p) {
    if (o == Py_None) return true;
    const at::Tensor* t = tensor(o);
    if (!t || t->scalar_type() != at::kByte) return false;
    p.workspace = *t;
    return true;
}

// forward(plain, x, packed, N, scales, bits, eps, y, workspace)
PyObject* forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Projection p;
    int64_t plain;
    if (n != 9 || !get_int(a[0], plain) || !get_projection(a[1], a[2], a[3], a[4], a[5], a[6], a[7], p) || !get_workspace(a[8], p))
        return decline();
    void* s = stream();
    const int rc = without_gil([&] {
        if (!p.allocate(true)) return kDeclined;
        return lib.forward[plain != 0](input(*p.x), p.dtype, p.T, p.K, input(*p.packed), p.N, floats(*p.scales), p.scales->numel(),
                                       (int)p.bits, p.eps, p.y.data_ptr(), p.workspace.data_ptr(), p.workspace.numel(), s);
    });
    return result(rc, a[7], p.y);
    END_HANDLE_TH_ERRORS
}

// ln_forward(x, gain, ln_eps, hadamard, packed, N, scales, bits, eps, y, workspace)
PyObject* ln_forward(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Projection p;
    float ln_eps;
    if (n != 11 || !PyBool_Check(a[3]) || !get_float(a[2], ln_eps)) return decline();
    const at::Tensor* gain = tensor(a[1]);
    if (!gain || gain->scalar_type() != at::kFloat || !get_projection(a[0], a[4], a[5], a[6], a[7], a[8], a[9], p) ||
        gain->numel() != p.K || !get_workspace(a[10], p))
        return decline();
    void* s = stream();
    const int hadamard = a[3] == Py_True;
    const int rc = without_gil([&] {
        if (!p.allocate(true)) return kDeclined;
        return lib.ln_forward(input(*p.x), p.dtype, p.T, p.K, floats(*gain), ln_eps, hadamard, input(*p.packed), p.N, floats(*p.scales),
                              p.scales->numel(), (int)p.bits, p.eps, p.y.data_ptr(), p.workspace.data_ptr(), p.workspace.numel(), s);
    });
    return result(rc, a[9], p.y);
    END_HANDLE_TH_ERRORS
}

// small(x, packed, N, scales, y, bits, hadamard, eps)
PyObject* small(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    Projection p;
    if (n != 8 || !PyBool_Check(a[6]) || a[4] == Py_None || !get_projection(a[0], a[1], a[2], a[3], a[5], a[7], a[4], p)) return decline();
    void* s = stream();
    const int hadamard = a[6] == Py_True;
    const int rc = without_gil([&] {
        return lib.small(input(*p.x), p.dtype, p.T, p.K, input(*p.packed), p.N, floats(*p.scales), p.scales->numel(), (int)p.bits, p.eps,
                         hadamard, p.y.data_ptr(), s);
    });
    return result(rc, a[4], p.y);
    END_HANDLE_TH_ERRORS
}

// fwht(x, bf16 out): allocates the output
PyObject* fwht(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 2 || !PyBool_Check(a[1])) return decline();
    const at::Tensor* x = tensor(a[0]);
    if (!x || x->dim() != 2 || x_dtype(*x) < 0) return decline();
    const bool bf16 = a[1] == Py_True;
    at::Tensor out;
    void* s = stream();
    const int rc = without_gil([&] {
        out = at::empty({x->size(0), x->size(1)}, x->options().dtype(bf16 ? at::kBFloat16 : at::kFloat));
        if (!ordinary(out)) return kDeclined;
        return lib.fwht(input(*x), x_dtype(*x), x->size(0), x->size(1), out.data_ptr(), bf16 ? HBL_BF16 : HBL_F32, s);
    });
    return result(rc, nullptr, out);
    END_HANDLE_TH_ERRORS
}

// kv_quant(x, bits, eps): allocates (packed, scales)
PyObject* kv_quant(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    int64_t bits;
    float eps;
    if (n != 3 || !get_int(a[1], bits) || !get_float(a[2], eps)) return decline();
    const at::Tensor* x = tensor(a[0]);
    if (!x || x->dim() != 2 || x_dtype(*x) < 0) return decline();
    const int64_t rows = x->size(0), d = x->size(1);
    if (lib.kv_packed_bytes(rows, d, (int)bits) == 0) return decline();   // (no rows, or a shape that is refused)
    at::Tensor packed, scales;
    void* s = stream();
    const int rc = without_gil([&] {
        packed = at::empty({rows, d * bits / 8}, x->options().dtype(at::kByte));
        scales = at::empty({rows}, x->options().dtype(at::kFloat));
        if (!ordinary(packed) || !ordinary(scales)) return kDeclined;
        return lib.kv_quant(input(*x), x_dtype(*x), rows, d, (int)bits, eps, packed.data_ptr(), scales.data_ptr<float>(), s);
    });
    PyObject* first = result(rc, nullptr, packed);
    if (rc != HBL_OK || !first) return first;
    PyObject* second = THPVariable_Wrap(scales);
    PyObject* both = second ? PyTuple_Pack(2, first, second) : nullptr;
    Py_DECREF(first);
    Py_XDECREF(second);
    return both;
    END_HANDLE_TH_ERRORS
}

// kv_dequant(packed, scales, d, bits, bf16 out): allocates the output
PyObject* kv_dequant(PyObject*, PyObject* const* a, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    int64_t d, bits;
    if (n != 5 || !get_int(a[2], d) || !get_int(a[3], bits) || !PyBool_Check(a[4])) return decline();
    const at::Tensor *packed = tensor(a[0]), *scales = tensor(a[1]);
    if (!packed || !scales || scales->dim() != 1 || scales->scalar_type() != at::kFloat) return decline();
    const int64_t rows = scales->size(0);
    const size_t need = lib.kv_packed_bytes(rows, d, (int)bits);
    if (need == 0 || packed->scalar_type() != at::kByte || (size_t)packed->numel() < need) return decline();
    const bool bf16 = a[4] == Py_True;
    at::Tensor out;
    void* s = stream();
    const int rc = without_gil([&] {
        out = at::empty({rows, d}, packed->options().dtype(bf16 ? at::kBFloat16 : at::kFloat));
        if (!ordinary(out)) return kDeclined;
        return lib.kv_dequant(input(*packed), floats(*scales), rows, d, (int)bits, out.data_ptr(), bf16 ? HBL_BF16 : HBL_F32, s);
    });
    return result(rc, nullptr, out);
    END_HANDLE_TH_ERRORS
}

// bind(addresses of the library's functions, in the order of `Library`)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    void* f[9];
    if (n != 9) {
        PyErr_SetString(PyExc_TypeError, "nine addresses");
        return nullptr;
    }
    for (int i = 0; i < 9; ++i) {
        f[i] = PyLong_AsVoidPtr(a[i]);
        if (f[i] == nullptr) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address");
            return nullptr;
        }
    }
    lib = Library{{reinterpret_cast<decltype(&hbl_hbitlinear_forward)>(f[0]), reinterpret_cast<decltype(&hbl_hbitlinear_forward)>(f[1])},
                  reinterpret_cast<decltype(&hbl_ln_bitlinear_forward)>(f[2]), reinterpret_cast<decltype(&hbl_bitlinear_forward_small)>(f[3]),
                  reinterpret_cast<decltype(&hbl_workspace_bytes)>(f[4]), reinterpret_cast<decltype(&hbl_fwht)>(f[5]),
                  reinterpret_cast<decltype(&hbl_kv_quant_absmax)>(f[6]), reinterpret_cast<decltype(&hbl_kv_dequant)>(f[7]),
                  reinterpret_cast<decltype(&hbl_kv_packed_bytes)>(f[8])};
    Py_RETURN_NONE;
}

#define HBL_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {HBL_METHOD(bind), HBL_METHOD(forward), HBL_METHOD(ln_forward), HBL_METHOD(small), HBL_METHOD(fwht),
                         HBL_METHOD(kv_quant), HBL_METHOD(kv_dequant), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host_call() {
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", HBL_BUILT_FOR) < 0) {   // torch's version
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
