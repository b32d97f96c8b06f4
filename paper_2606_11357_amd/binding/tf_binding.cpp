// The matmul calls of tilefuse.py in native code: argument checks, the output,
// the workspace and the current stream, then the C ABI call, in one entry from
// Python.  A decode GEMV runs 5 to 7 us on the GPU; the same steps through
// Python and ctypes took about 10 us a call on the host, so a loop of them
// waited for Python.  Measured on MI355X, us a call in a loop: W8 K = N = 4096,
// one row 10.2 -> 5.5, W4 16 x 2048 x 2048 10.2 -> 5.4, W4 K = 4096, N = 14336,
// one row 10.2 -> 6.7 (each now the GPU's time); 4.6 us of host work a call, most
// of it the launch.
//
// Only calls in the common form are taken here (plain contiguous tensors of
// the documented types and shapes, Python integers); anything else returns
// NotImplemented, and the general path in tilefuse.py runs it or raises.  The
// library's functions are handed over as addresses (bind), so that whichever
// build of the library the binding loaded is the one that is called.
#include <ATen/ops/empty.h>
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

using MatmulFn = int (*)(const uint16_t*, const void*, uint16_t*, int64_t, int64_t, int64_t, int, void*, size_t, void*);
using BytesFn = int64_t (*)(int, int64_t, int64_t, int64_t, int);

constexpr int kFns = 8;                  // (bits 4, 8) x (gemm, gemv) x (fp16, bf16)
MatmulFn g_fn[kFns];
BytesFn g_bytes;
PyObject* g_stream;                      // device index -> current stream's handle
PyObject* g_workspaces;                  // device index -> cached workspace
PyObject* g_workspace;                   // (device, bytes) -> workspace, grown if need be

// bind((address of each matmul function), address of tf_workspace_bytes,
//      current stream function, workspace dict, default_workspace)
PyObject* bind(PyObject*, PyObject* args) {
    PyObject *fns, *stream, *dict, *ws;
    unsigned long long bytes;
    if (!PyArg_ParseTuple(args, "O!KOO!O", &PyTuple_Type, &fns, &bytes, &stream, &PyDict_Type, &dict, &ws))
        return nullptr;
    if (PyTuple_GET_SIZE(fns) != kFns) {
        PyErr_SetString(PyExc_ValueError, "bind needs eight functions");
        return nullptr;
    }
    for (int i = 0; i < kFns; ++i) {
        const unsigned long long a = PyLong_AsUnsignedLongLong(PyTuple_GET_ITEM(fns, i));
        if (PyErr_Occurred()) return nullptr;
        g_fn[i] = reinterpret_cast<MatmulFn>(a);
    }
    g_bytes = reinterpret_cast<BytesFn>(bytes);
    Py_XSETREF(g_stream, Py_NewRef(stream));
    Py_XSETREF(g_workspaces, Py_NewRef(dict));
    Py_XSETREF(g_workspace, Py_NewRef(ws));
    Py_RETURN_NONE;
}

PyObject* not_here() { return Py_NewRef(Py_NotImplemented); }

// A reference held until the end of the scope.
struct Held {
    PyObject* o = nullptr;
    ~Held() { Py_XDECREF(o); }
};

// A plain tensor (no subclass) on the GPU, contiguous.
const at::Tensor* plain(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return t.is_cuda() && t.layout() == at::kStrided && t.is_contiguous() ? &t : nullptr;
}

PyObject* matmul_common(PyObject* const* a, Py_ssize_t n) {
    if (n != 9 || !g_bytes) return not_here();
    for (const int i : {0, 4, 5, 6})
        if (!PyLong_CheckExact(a[i])) return not_here();
    int over = 0;
    const long bits = PyLong_AsLong(a[0]);
    const bool gemv = a[1] == Py_True;
    const int64_t K = PyLong_AsLongLongAndOverflow(a[4], &over);
    if (over) return not_here();
    const int64_t N = PyLong_AsLongLongAndOverflow(a[5], &over);
    if (over) return not_here();
    const int64_t group = PyLong_AsLongLongAndOverflow(a[6], &over);
    if (over || group != (int)group) return not_here();
    const at::Tensor *A = plain(a[2]), *packed = plain(a[3]);
    if (!A || !packed || A->dim() != 2 || A->size(1) != K || A->size(0) < 1 || N < 1) return not_here();
    const bool bf = A->scalar_type() == at::kBFloat16;
    if (!bf && A->scalar_type() != at::kHalf) return not_here();
    const int64_t M = A->size(0);
    const int dev = A->get_device();
    PyObject *out_o = a[7], *ws_o = a[8];
    // the workspace: False none, None the device's cached one, or the caller's
    Held held;                       // the cached workspace, over the call
    void* ws = nullptr;
    size_t ws_bytes = 0;
    if (ws_o == Py_None) {
        const int64_t need = g_bytes((int)bits, M, K, N, (int)group);
        if (need < 0) return not_here();
        if (need > 0) {
            const Held key{PyLong_FromLong(dev)};
            if (!key.o) return nullptr;
            held.o = Py_XNewRef(PyDict_GetItemWithError(g_workspaces, key.o));
            if (!held.o && PyErr_Occurred()) return nullptr;
            const at::Tensor* t = held.o ? plain(held.o) : nullptr;
            if (!t || t->numel() < need) {
                const Held device{PyObject_GetAttrString(a[2], "device")};
                if (!device.o) return nullptr;
                Py_XSETREF(held.o, PyObject_CallFunction(g_workspace, "OL", device.o, (long long)need));
                if (!held.o) return nullptr;
                t = plain(held.o);
                if (!t) return not_here();
            }
            ws = t->data_ptr();
            ws_bytes = t->nbytes();
        }
    } else if (ws_o != Py_False) {
        const at::Tensor* t = plain(ws_o);
        if (!t) return not_here();
        ws = t->data_ptr();
        ws_bytes = t->nbytes();
    }
    at::Tensor made;
    const at::Tensor* out;
    if (out_o == Py_None) {
        made = at::empty({M, N}, A->options().requires_grad(false));
        out = &made;
    } else {
        out = plain(out_o);
        if (!out || out->scalar_type() != A->scalar_type() || out->dim() != 2 || out->size(0) != M ||
            out->size(1) != N)
            return not_here();
    }
    const Held index{PyLong_FromLong(dev)};
    const Held handle{index.o ? PyObject_CallOneArg(g_stream, index.o) : nullptr};
    if (!handle.o) return nullptr;
    void* stream = PyLong_AsVoidPtr(handle.o);
    const MatmulFn fn = g_fn[(bits == 8 ? 4 : 0) + (gemv ? 2 : 0) + (bf ? 1 : 0)];
    const uint16_t* x = static_cast<const uint16_t*>(A->data_ptr());
    const void* pk = packed->data_ptr();
    uint16_t* y = static_cast<uint16_t*>(out->data_ptr());
    int rc;
    Py_BEGIN_ALLOW_THREADS;
    rc = fn(x, pk, y, M, K, N, (int)group, ws, ws_bytes, stream);
    Py_END_ALLOW_THREADS;
    if (rc != 0) return PyLong_FromLong(rc);
    return out_o == Py_None ? THPVariable_Wrap(std::move(made)) : Py_NewRef(out_o);
}

// matmul(bits, gemv, A, packed, K, N, group, out, workspace): the output, the
// library's status if it is not 0, or NotImplemented.
PyObject* matmul(PyObject*, PyObject* const* a, Py_ssize_t n) {
    // No exception leaves a C entry.  Any access to a tensor may throw (a nested
    // tensor with rows of different lengths has no size(1); memory may be short),
    // and none follows the launch but the wrapping of the output: the general path
    // meets the same condition and raises it as torch does.
    try {
        return matmul_common(a, n);
    } catch (...) {
        return PyErr_Occurred() ? nullptr : not_here();
    }
}

PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, "Hand over the library's functions."},
    {"matmul", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(matmul)), METH_FASTCALL,
     "One matmul call of the library, or NotImplemented."},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tf_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__tf_binding() { return PyModule_Create(&module); }
