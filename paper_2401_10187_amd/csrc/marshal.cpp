// The binding's per-call work in native code: looks at the tensors of a Kron-Matmul, makes the result and crosses the C-ABI.
// Only what it can take as it is: plain CUDA tensors that are contiguous, of one type and on the current device.  For
// everything else, mistakes included, call() returns NotImplemented and binding.py goes the long way, which also
// says what is wrong.
//
// Python objects cost about 0.05 to 0.1 us for each attribute that is asked for, and ctypes about as much for each argument that
// it converts: back to back, 10 x (52x50, 65x20) as a plain call 7.9 -> 5.8 us (what the GPU needs), 16 x 8x8^3 prepared 4.3 -> 3.6.
#include <Python.h>
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/core/DeviceGuard.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <stdint.h>

namespace {

typedef int (*PlainFn)(int, int, const int*, const int*, const void*, const void* const*, void*, int, void*);
typedef int (*WorkspaceFn)(int, int, const int*, const int*, const void*, const void* const*, void*, int, void*, size_t, void*);

constexpr int MAX_FACTORS = 64;
PlainFn g_plain[2];              // factors as they are, factors given transposed
WorkspaceFn g_workspace[2];
PyObject* g_raw_stream;          // device index -> handle of torch's current stream
PyObject* g_fail;                // (status, transposed, with workspace): raises

// The interpreter is left to other threads meanwhile, and taken back however the block ends.
struct WithoutGil {
    PyThreadState* state = PyEval_SaveThread();
    ~WithoutGil() { PyEval_RestoreThread(state); }
};

// Handle of torch's current stream on a device; false with a Python error set.
bool current_stream(PyObject* index, void** stream)
{
    PyObject* r = PyObject_CallOneArg(g_raw_stream, index);
    if (!r) return false;
    *stream = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    return !PyErr_Occurred();
}

PyObject* fail(int status, bool transposed, bool with_ws)
{
    PyObject* r = PyObject_CallFunction(g_fail, "iii", status, (int)transposed, (int)with_ws);
    Py_XDECREF(r);
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, "a Kron-Matmul failed");
    return nullptr;
}

// A plain strided CUDA tensor with memory of its own (no wrapper of functorch, no conjugate or negative view).
bool plain(PyObject* o, const at::Tensor*& t)
{
    if (!THPVariable_CheckExact(o)) return false;
    t = &THPVariable_Unpack(o);
    const c10::TensorImpl* i = t->unsafeGetTensorImpl();
    return t->defined() && t->is_cuda() && t->layout() == at::kStrided && i->has_storage() && !i->is_python_dispatch() &&
           !i->key_set().has_any(c10::DispatchKeySet({c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                                      c10::DispatchKey::Functionalize, c10::DispatchKey::Conjugate, c10::DispatchKey::Negative,
                                                      c10::DispatchKey::ZeroTensor, c10::DispatchKey::Python}));
}

PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    if (nargs != 5) {
        PyErr_SetString(PyExc_TypeError, "call(X, Fs, Y, workspace, transposed)");
        return nullptr;
    }
    PyObject *const fs = args[1], *const yo = args[2], *const wo = args[3];
    const bool transposed = args[4] == Py_True;
    if ((args[4] != Py_True && args[4] != Py_False) || !(PyList_CheckExact(fs) || PyTuple_CheckExact(fs)) || !g_fail) Py_RETURN_NOTIMPLEMENTED;
    if (at::impl::torch_function_mode_enabled() || c10::impl::TorchDispatchModeTLS::any_modes_set()) Py_RETURN_NOTIMPLEMENTED;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(fs);
    PyObject* const* items = PySequence_Fast_ITEMS(fs);
    if (n < 1 || n > MAX_FACTORS) Py_RETURN_NOTIMPLEMENTED;
    HANDLE_TH_ERRORS
    {
        const at::Tensor *x, *f, *w = nullptr;
        if (!plain(args[0], x) || x->dim() != 2 || !x->is_contiguous()) Py_RETURN_NOTIMPLEMENTED;
        const at::ScalarType type = x->scalar_type();
        const c10::Device device = x->device();
        if ((type != at::kFloat && type != at::kDouble) || c10::impl::VirtualGuardImpl(c10::DeviceType::CUDA).getDevice() != device) Py_RETURN_NOTIMPLEMENTED;
        int P[MAX_FACTORS], Q[MAX_FACTORS];
        const void* ptr[MAX_FACTORS];
        const int64_t most = (int64_t)1 << 30;
        int64_t kin = 1, kout = 1;
        for (Py_ssize_t i = 0; i < n; ++i) {
            if (!plain(items[i], f) || f->scalar_type() != type || f->device() != device || f->dim() != 2 || !f->is_contiguous()) Py_RETURN_NOTIMPLEMENTED;
            const int64_t p = f->size(transposed ? 1 : 0), q = f->size(transposed ? 0 : 1);
            if (p < 1 || q < 1 || p > most || q > most || kin > most / p || kout > most / q) Py_RETURN_NOTIMPLEMENTED;
            kin *= p;
            kout *= q;
            P[i] = (int)p;
            Q[i] = (int)q;
            ptr[i] = f->const_data_ptr();
        }
        const int64_t M = x->size(0);
        if (M < 1 || M > most || x->size(1) != kin) Py_RETURN_NOTIMPLEMENTED;
        const void* ws = nullptr;
        if (wo != Py_None) {
            if (!plain(wo, w) || w->device() != device || !w->is_contiguous()) Py_RETURN_NOTIMPLEMENTED;
            ws = w->data_ptr();
        }
        at::Tensor made;
        const at::Tensor* y = &made;
        if (yo == Py_None) made = x->new_empty({M, kout});
        else if (!plain(yo, y) || y->scalar_type() != type || y->device() != device || !y->is_contiguous() || y->dim() != 2 || y->size(0) != M || y->size(1) != kout)
            Py_RETURN_NOTIMPLEMENTED;
        void* const out = y->data_ptr();
        const void* const in = x->const_data_ptr();
        const size_t ws_bytes = w ? w->nbytes() : 0;
        PyObject* index = PyLong_FromLong(device.index());
        void* stream = nullptr;
        const bool ok = index && current_stream(index, &stream);
        Py_XDECREF(index);
        if (!ok) return nullptr;
        int status;
        {
            WithoutGil other_threads;
            const int code = type == at::kFloat ? 0 : 1;
            status = w ? g_workspace[transposed]((int)M, (int)n, P, Q, in, ptr, out, code, const_cast<void*>(ws), ws_bytes, stream)
                       : g_plain[transposed]((int)M, (int)n, P, Q, in, ptr, out, code, stream);
        }
        if (status != 0) return fail(status, transposed, w != nullptr);
        if (yo != Py_None) {
            Py_INCREF(yo);
            return yo;
        }
        return THPVariable_Wrap(std::move(made));
    }
    END_HANDLE_TH_ERRORS
}

// A call whose arguments are all known: bind(M, n, P, Q, X, F, Y, dtype, workspace, workspace bytes, with workspace, transposed,
// device index) with the addresses of what binding.py has checked and keeps alive.
struct Bound {
    PyObject_HEAD
    vectorcallfunc vectorcall;
    int M, n, code, with_ws, transposed;
    const int *P, *Q;
    const void *X, *ws;
    const void* const* F;
    void* Y;
    size_t ws_bytes;
    PyObject* index;
};

// status 0, or raises; bound(stream or None)
PyObject* bound_call(PyObject* self, PyObject* const* args, size_t nargsf, PyObject* kwnames)
{
    Bound* b = reinterpret_cast<Bound*>(self);
    if (PyVectorcall_NARGS(nargsf) != 1 || kwnames) {
        PyErr_SetString(PyExc_TypeError, "bound(stream)");
        return nullptr;
    }
    void* stream = nullptr;
    if (args[0] == Py_None) {
        if (!current_stream(b->index, &stream)) return nullptr;
    } else {
        stream = PyLong_AsVoidPtr(args[0]);
        if (PyErr_Occurred()) return nullptr;
    }
    int status;
    try {                                                // (HANDLE_TH_ERRORS also sets torch's warnings up, 0.05 us)
        WithoutGil other_threads;
        status = b->with_ws ? g_workspace[b->transposed](b->M, b->n, b->P, b->Q, b->X, b->F, b->Y, b->code, const_cast<void*>(b->ws), b->ws_bytes, stream)
                            : g_plain[b->transposed](b->M, b->n, b->P, b->Q, b->X, b->F, b->Y, b->code, stream);
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
    if (status != 0) return fail(status, b->transposed, b->with_ws);
    Py_RETURN_NONE;
}

void bound_dealloc(PyObject* self)
{
    Py_XDECREF(reinterpret_cast<Bound*>(self)->index);
    Py_TYPE(self)->tp_free(self);
}

PyTypeObject BoundType = {PyVarObject_HEAD_INIT(nullptr, 0)};

PyObject* bind(PyObject*, PyObject* args)
{
    unsigned long long P, Q, X, F, Y, ws, bytes;
    int M, n, code, with_ws, transposed, index;
    if (!PyArg_ParseTuple(args, "iiKKKKKiKKppi", &M, &n, &P, &Q, &X, &F, &Y, &code, &ws, &bytes, &with_ws, &transposed, &index)) return nullptr;
    Bound* b = PyObject_New(Bound, &BoundType);
    if (!b) return nullptr;
    b->vectorcall = bound_call;
    b->M = M;
    b->n = n;
    b->code = code;
    b->with_ws = with_ws;
    b->transposed = transposed;
    b->P = reinterpret_cast<const int*>(P);
    b->Q = reinterpret_cast<const int*>(Q);
    b->X = reinterpret_cast<const void*>(X);
    b->F = reinterpret_cast<const void* const*>(F);
    b->Y = reinterpret_cast<void*>(Y);
    b->ws = reinterpret_cast<const void*>(ws);
    b->ws_bytes = (size_t)bytes;
    b->index = PyLong_FromLong(index);
    if (!b->index) {
        Py_DECREF(b);
        return nullptr;
    }
    return reinterpret_cast<PyObject*>(b);
}

// start(addresses of kronmatmul, _transposed, _ws, _transposed_ws; current raw stream of a device; what raises on failure)
PyObject* start(PyObject*, PyObject* args)
{
    unsigned long long a, b, c, d;
    PyObject *stream, *raise;
    if (!PyArg_ParseTuple(args, "KKKKOO", &a, &b, &c, &d, &stream, &raise)) return nullptr;
    g_plain[0] = reinterpret_cast<PlainFn>(a);
    g_plain[1] = reinterpret_cast<PlainFn>(b);
    g_workspace[0] = reinterpret_cast<WorkspaceFn>(c);
    g_workspace[1] = reinterpret_cast<WorkspaceFn>(d);
    Py_INCREF(stream);
    Py_INCREF(raise);
    Py_XSETREF(g_raw_stream, stream);
    Py_XSETREF(g_fail, raise);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL, "call(X, Fs, Y, workspace, transposed) -> Y, or NotImplemented"},
    {"bind", bind, METH_VARARGS, "a call with all its arguments"},
    {"start", start, METH_VARARGS, "the library's entry points and what torch is asked for"},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void)
{
    BoundType.tp_name = "paper_2401_10187_amd._marshal.Bound";
    BoundType.tp_basicsize = sizeof(Bound);
    BoundType.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL;
    BoundType.tp_vectorcall_offset = offsetof(Bound, vectorcall);
    BoundType.tp_call = PyVectorcall_Call;
    BoundType.tp_dealloc = bound_dealloc;
    if (PyType_Ready(&BoundType) < 0) return nullptr;
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "built_for", KM_BUILT_FOR) < 0) Py_CLEAR(m);      // the torch whose headers these are
    return m;
}
