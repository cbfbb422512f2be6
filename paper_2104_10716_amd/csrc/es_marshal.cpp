// es_marshal.cpp -- native argument marshalling for the hot entry points: torch tensors in, one C-ABI call out.
//
// A Python program calls es_spmm once per layer; on a graph of a few thousand
// rows the kernel takes about 4 us, and reading fifteen tensor attributes,
// finding the current stream and converting twenty ctypes arguments in Python
// took another 8 (13 us per call in all; 4 with this module).  Nothing is
// computed here.  Every function returns the C entry point's status, or None when
// an argument is not the plain case (wrong type, shape, device or stride, or a
// tensor without memory of its own: sparse, fake, a wrapper): the caller then goes
// through the checks written in Python, which name the fault.
// No exception leaves a function, and the C call runs without the interpreter lock,
// as a ctypes call does: a launch that waits for room in a queue stops no other thread.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "es_spmm.h"

namespace {

decltype(&es_spmm_ws) g_spmm_ws = nullptr;
decltype(&es_spmm_backward) g_backward = nullptr;
decltype(&es_spmm_backward_ws) g_backward_ws = nullptr;
decltype(&es_spmm_backward_workspace_bytes) g_backward_bytes = nullptr;
decltype(&es_spmm_backward_pull) g_pull = nullptr;

// Strided, with a storage that holds its elements, and not a Python-dispatched
// wrapper.  A fake tensor calls itself a device tensor and answers with a null
// address, which as `vals` would mean an unweighted graph.
bool has_memory(const at::Tensor& t)
{
    return t.defined() && t.layout() == at::kStrided && !t.unsafeGetTensorImpl()->is_python_dispatch() &&
           t.has_storage() && (t.data_ptr() || t.numel() == 0);
}

bool as_tensor(PyObject* o, at::ScalarType type, const at::Tensor** out)
{
    if (!THPVariable_Check(o)) return false;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.scalar_type() != type || !has_memory(t)) return false;
    *out = &t;
    return true;
}

// A reference that is dropped at the end of the scope.
struct Owned {
    PyObject* p;
    ~Owned() { Py_XDECREF(p); }
};

// An int, or what converts to one without loss (a NumPy integer); false, with no
// error left behind, for anything else.
bool as_long(PyObject* o, long long* out)
{
    Owned index{PyNumber_Index(o)};
    int overflow = 0;
    if (index.p) *out = PyLong_AsLongLongAndOverflow(index.p, &overflow);
    if (index.p && !overflow) return true;
    PyErr_Clear();
    return false;
}

// One of `names`, or an integer: its code.
bool as_code(PyObject* o, const char* const* names, int n, int32_t* out)
{
    if (PyUnicode_Check(o)) {
        for (int i = 0; i < n; ++i)
            if (PyUnicode_CompareWithASCIIString(o, names[i]) == 0) { *out = i; return true; }
        return false;
    }
    long long v;
    if (!as_long(o, &v) || v < INT32_MIN || v > INT32_MAX) return false;
    *out = (int32_t)v;
    return true;
}

// The low 64 bits of an integer.
bool as_seed(PyObject* o, uint64_t* out)
{
    Owned index{PyNumber_Index(o)};
    if (index.p) *out = PyLong_AsUnsignedLongLongMask(index.p);
    if (index.p && !PyErr_Occurred()) return true;
    PyErr_Clear();
    return false;
}

const char* const kModes[] = {"full", "bucket", "fastrand"};
const char* const kNorms[] = {"none", "mean", "rsqrt", "rescale", "inv_degree"};

// None: torch's current stream; an int: the address; else a stream object of torch.
bool as_stream(PyObject* o, void** out)
{
    if (o == Py_None) {
        *out = c10::hip::getCurrentHIPStream().stream();
        return true;
    }
    Owned address{PyLong_Check(o) ? (Py_INCREF(o), o) : PyObject_GetAttrString(o, "cuda_stream")};
    if (address.p && PyLong_Check(address.p)) {
        *out = PyLong_AsVoidPtr(address.p);
        if (*out || !PyErr_Occurred()) return true;
    }
    PyErr_Clear();
    return false;
}

// `call` (noexcept: every address is read before) without the interpreter lock
template <class Call>
PyObject* unlocked(Call&& call)
{
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// What every product has in common: X (gathered) and Y (written), [N x F] with
// unit column stride, and the sampler's arguments.
struct Product {
    const float* x;
    float* y;
    int64_t N;
    int32_t F, ldx, ldy, W, mode, norm;
    uint64_t seed;
    void* stream;

    // the scalars first: what they may run (an object's __index__) comes before any address is read
    bool scalars(PyObject* w, PyObject* m, PyObject* sd, PyObject* nm, PyObject* f, PyObject* st)
    {
        F = -1;
        return as_code(w, nullptr, 0, &W) && as_code(m, kModes, 3, &mode) && as_seed(sd, &seed) &&
               as_code(nm, kNorms, 5, &norm) && (f == Py_None || (as_code(f, nullptr, 0, &F) && F >= 0)) &&
               as_stream(st, &stream);
    }

    bool matrices(int64_t n, PyObject* xt, PyObject* yt)
    {
        N = n;
        const at::Tensor *X, *Y;
        if (!as_tensor(xt, at::kFloat, &X) || !as_tensor(yt, at::kFloat, &Y)) return false;
        if (X->dim() != 2 || Y->dim() != 2 || X->stride(1) != 1 || Y->stride(1) != 1) return false;
        if (X->size(0) != N || Y->size(0) != N) return false;
        if (F < 0) {
            if (X->size(1) > INT32_MAX) return false;
            F = (int32_t)X->size(1);
        }
        if (F > X->size(1) || F > Y->size(1)) return false;
        const int64_t lx = N > 1 ? X->stride(0) : std::max<int64_t>(X->size(1), 1);
        const int64_t ly = N > 1 ? Y->stride(0) : std::max<int64_t>(Y->size(1), 1);
        if (lx > INT32_MAX || ly > INT32_MAX || lx < 0 || ly < 0) return false;
        x = static_cast<const float*>(X->data_ptr());
        y = static_cast<float*>(Y->data_ptr());
        ldx = (int32_t)lx; ldy = (int32_t)ly;
        return true;
    }
};

struct Csr {
    const int32_t *rowptr, *colidx;
    const float* vals;
    int64_t N, nnz, stored;                            // nnz: the caller's hint, or stored

    bool parse(PyObject* rp, PyObject* ci, PyObject* va, PyObject* nz)
    {
        int32_t hint = 0;
        if (nz != Py_None && !as_code(nz, nullptr, 0, &hint)) return false;
        const at::Tensor *r, *c, *v;
        if (!as_tensor(rp, at::kInt, &r) || !as_tensor(ci, at::kInt, &c)) return false;
        N = r->numel() - 1;
        nnz = stored = c->numel();
        vals = nullptr;
        if (va != Py_None) {
            if (!as_tensor(va, at::kFloat, &v) || v->numel() != nnz) return false;
            vals = static_cast<const float*>(v->data_ptr());
        }
        rowptr = static_cast<const int32_t*>(r->data_ptr());
        colidx = static_cast<const int32_t*>(c->data_ptr());
        if (nz != Py_None) nnz = hint;
        return true;
    }
};

// bind(es_spmm_ws, es_spmm_backward, es_spmm_backward_pull, es_spmm_backward_ws,
// es_spmm_backward_workspace_bytes): addresses of the C entry points
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (n != 5) { PyErr_SetString(PyExc_TypeError, "bind takes five addresses"); return nullptr; }
    void* p[5];
    for (int i = 0; i < 5; ++i) {
        p[i] = PyLong_AsVoidPtr(a[i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null entry point");
            return nullptr;
        }
    }
    g_spmm_ws = reinterpret_cast<decltype(g_spmm_ws)>(p[0]);
    g_backward = reinterpret_cast<decltype(g_backward)>(p[1]);
    g_pull = reinterpret_cast<decltype(g_pull)>(p[2]);
    g_backward_ws = reinterpret_cast<decltype(g_backward_ws)>(p[3]);
    g_backward_bytes = reinterpret_cast<decltype(g_backward_bytes)>(p[4]);
    Py_RETURN_NONE;
}

// spmm(rowptr, colidx, vals, X, Y, W, mode, seed, norm, workspace, F, stream, nnz)
PyObject* spmm(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Csr g;
    Product p;
    if (n != 13 || !g_spmm_ws || !p.scalars(a[5], a[6], a[7], a[8], a[10], a[11]) ||
        !g.parse(a[0], a[1], a[2], a[12]) || !p.matrices(g.N, a[3], a[4]))
        Py_RETURN_NONE;
    void* ws = nullptr;
    size_t ws_bytes = 0;
    if (a[9] != Py_None) {
        if (!THPVariable_Check(a[9])) Py_RETURN_NONE;
        const at::Tensor& t = THPVariable_Unpack(a[9]);
        if (!t.is_cuda() || !has_memory(t) || !t.is_contiguous()) Py_RETURN_NONE;
        ws = t.data_ptr();
        ws_bytes = t.nbytes();
    }
    return unlocked([&] {
        return g_spmm_ws(g.rowptr, g.colidx, g.vals, p.x, p.y, g.N, g.nnz, p.F, p.ldx, p.ldy, p.W, p.mode, p.seed,
                         p.norm, nullptr, ws, ws_bytes, p.stream);
    });
}

// `bytes` from torch's allocator, in the pool of the stream that will use them: given
// back as soon as the work on them is queued, they are handed out again in that stream's order only.
struct Scratch {
    void* p = nullptr;
    Scratch(size_t bytes, hipStream_t stream) noexcept
    {
        if (!bytes || !lendable(stream)) return;
        // The allocator may ask the runtime for memory.  In another thread's capture of a graph (of global
        // mode) that is an error which ends the capture, unless this thread's mode is relaxed.
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) { (void)hipGetLastError(); return; }
        try {
            p = c10::hip::HIPCachingAllocator::raw_alloc_with_stream(bytes, stream);
        } catch (...) {
            p = nullptr;                               // no room: the caller's form without a workspace
        }
        (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
    // Not to a stream that is being captured (torch may not know of the capture, and a graph would
    // outlive the memory), nor to one of another device: the allocator serves the current one.
    static bool lendable(hipStream_t stream) noexcept
    {
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        hipDevice_t device = -1;
        int current = -1;
        if (hipStreamIsCapturing(stream, &capture) == hipSuccess && hipStreamGetDevice(stream, &device) == hipSuccess &&
            hipGetDevice(&current) == hipSuccess)
            return capture == hipStreamCaptureStatusNone && device == current;
        (void)hipGetLastError();                       // the launches report their own errors
        return false;
    }
    ~Scratch()
    {
        if (p) c10::hip::HIPCachingAllocator::raw_delete(p);
    }
};

// backward(rowptr, colidx, vals, dY, dX, W, mode, seed, norm, F, stream, nnz)
PyObject* backward(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    Csr g;
    Product p;
    if (n != 12 || !g_backward || !p.scalars(a[5], a[6], a[7], a[8], a[9], a[10]) ||
        !g.parse(a[0], a[1], a[2], a[11]) || !p.matrices(g.N, a[3], a[4]))
        Py_RETURN_NONE;
    return unlocked([&] {
        // sized by the entries there are: nnz may be a hint (a negative one is refused, by the form without a workspace)
        const size_t bytes = g.nnz < 0 ? 0 : g_backward_bytes(g.N, g.stored, p.F, p.W, p.mode);
        if (bytes) {
            const Scratch ws(bytes, static_cast<hipStream_t>(p.stream));
            if (ws.p)
                return g_backward_ws(g.rowptr, g.colidx, g.vals, p.x, p.y, g.N, g.stored, p.F, p.ldx, p.ldy, p.W,
                                     p.mode, p.seed, p.norm, ws.p, bytes, p.stream);
        }
        return g_backward(g.rowptr, g.colidx, g.vals, p.x, p.y, g.N, g.nnz, p.F, p.ldx, p.ldy, p.W, p.mode, p.seed,
                          p.norm, p.stream);
    });
}

// pull(rowptr, t, dY, dX, W, mode, seed, norm, F, stream); t: the dict of es_spmm_transpose_graph
PyObject* pull(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    static const char* const names[] = {"t_ptr", "t_row", "t_idx", "t_slot", "t_vals", "t_pinv", "t_rows"};
    const at::Tensor *rp, *t[7];
    Product p;
    if (n != 10 || !g_pull || !p.scalars(a[4], a[5], a[6], a[7], a[8], a[9]) || !as_tensor(a[0], at::kInt, &rp) ||
        !PyDict_Check(a[1]))
        Py_RETURN_NONE;
    for (int i = 0; i < 7; ++i) {
        PyObject* o = PyDict_GetItemString(a[1], names[i]);
        if (!o || !as_tensor(o, i == 4 ? at::kFloat : at::kInt, &t[i])) Py_RETURN_NONE;
    }
    const int64_t N = rp->numel() - 1;
    if (!p.matrices(N, a[2], a[3])) Py_RETURN_NONE;
    int32_t* q[7];
    for (int i = 0; i < 7; ++i) q[i] = i == 4 ? nullptr : static_cast<int32_t*>(t[i]->data_ptr());
    const float* t_vals = static_cast<const float*>(t[4]->data_ptr());
    const int32_t* rowptr = static_cast<const int32_t*>(rp->data_ptr());
    const int64_t nnz = t[1]->numel();
    return unlocked([&] {
        return g_pull(rowptr, q[0], q[1], q[2], q[3], t_vals, q[5], q[6], p.x, p.y, N, nnz, p.F, p.ldx, p.ldy, p.W,
                      p.mode, p.seed, p.norm, p.stream);
    });
}

// readable(tensor): whether has_memory holds
PyObject* readable(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (n != 1 || !THPVariable_Check(a[0])) Py_RETURN_FALSE;
    return PyBool_FromLong(has_memory(THPVariable_Unpack(a[0])));
}

// `f`, with anything its tensors throw turned into None
template <PyObject* (*f)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* a, Py_ssize_t n)
{
    try {
        return f(self, a, n);
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

#define ES_METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(guarded<f>)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {ES_METHOD(bind), ES_METHOD(spmm), ES_METHOD(backward), ES_METHOD(pull), ES_METHOD(readable),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_es_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__es_marshal() { return PyModule_Create(&module); }
