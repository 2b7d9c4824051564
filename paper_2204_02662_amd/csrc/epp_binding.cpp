// CPython entry points of the calls that a training loop makes on every layer of every pass: argument
// checks on the tensors' C++ objects, current stream, call of the C ABI (include/epp.h).
//
// On a small graph such a call is all host work: a kernel of 4 us, and 7.5 us to check five arguments,
// look up the stream and marshal the call from Python through ctypes.  Here the same steps take 1.5 us beside the
// launch itself.  Messages and exceptions are those of the module that imports this one (__init__.py).
//
// What PyTorch's C++ throws (a tensor of unknown shape, as tracing makes them, asked for its sizes) leaves
// every entry point as the Python exception it stands for: past a C function it would end the process.

#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <c10/core/impl/VirtualGuardImpl.h>
#include <c10/hip/HIPCachingAllocator.h>

#include <atomic>

#include "epp.h"

namespace {

PyObject* g_error = nullptr;       // EppError(code, message)
PyObject* g_raw_stream = nullptr;  // torch._C._cuda_getCurrentRawStream(device index)
PyObject *s_handle, *s_cached_n, *s_n;

// Positional and keyword arguments of a call, in the order of `names`.
bool take_args(const char* fn, PyObject* const* args, Py_ssize_t n, PyObject* kw, const char* const* names, int count,
               PyObject** out) {
    for (int i = 0; i < count; ++i) out[i] = i < n ? args[i] : nullptr;
    if (n > count) {
        PyErr_Format(PyExc_TypeError, "%s() takes %d arguments (%zd given)", fn, count, n);
        return false;
    }
    const Py_ssize_t n_kw = kw ? PyTuple_GET_SIZE(kw) : 0;
    for (Py_ssize_t j = 0; j < n_kw; ++j) {
        PyObject* key = PyTuple_GET_ITEM(kw, j);
        int i = 0;
        while (i < count && PyUnicode_CompareWithASCIIString(key, names[i]) != 0) ++i;
        if (i == count || out[i]) {
            PyErr_Format(PyExc_TypeError, "%s() got an unexpected or repeated argument '%U'", fn, key);
            return false;
        }
        out[i] = args[n + j];
    }
    for (int i = 0; i < count; ++i) {
        if (!out[i]) {
            PyErr_Format(PyExc_TypeError, "%s() misses the argument '%s'", fn, names[i]);
            return false;
        }
    }
    return true;
}

// Library handle of a path or of all paths.
void* handle_of(PyObject* o) {
    PyObject* h = PyObject_GetAttr(o, s_handle);
    if (!h) return nullptr;
    void* p = h == Py_None ? nullptr : PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    if (!p && !PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "the handle has been released");
    return p;
}

// Vertices of its graph (cached by the object), -1 on an error.
int64_t vertices_of(PyObject* o) {
    PyObject* n = PyObject_GetAttr(o, s_cached_n);
    if (n && n == Py_None) {
        Py_DECREF(n);
        n = PyObject_GetAttr(o, s_n);
    }
    if (!n) return -1;
    const int64_t v = PyLong_AsLongLong(n);
    Py_DECREF(n);
    return v;
}

const at::Tensor* bad_tensor(const at::Tensor& t, const char* dtype) {
    const std::string got = std::string(c10::toString(t.scalar_type())), on = t.device().str();
    PyErr_Format(PyExc_ValueError, "expected a contiguous CUDA tensor of %s, got %s on %s", dtype, got.c_str(), on.c_str());
    return nullptr;
}

const at::Tensor* float_tensor(PyObject* o) {
    if (!THPVariable_Check(o)) {
        PyErr_Format(PyExc_TypeError, "expected a tensor, got %s", Py_TYPE(o)->tp_name);
        return nullptr;
    }
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.scalar_type() != at::kFloat || !t.is_contiguous()) return bad_tensor(t, "torch.float32");
    return &t;
}

const at::Tensor* matrix(PyObject* o, const char* what) {
    const at::Tensor* t = float_tensor(o);
    if (t && t->dim() != 2) {
        PyErr_Format(PyExc_ValueError, "%s must be a matrix", what);
        return nullptr;
    }
    return t;
}

// The current stream of the current device; false on an error.
bool current_stream(void** stream) {
    static const c10::impl::DeviceGuardImplInterface* const guard = c10::impl::getDeviceGuardImpl(c10::DeviceType::CUDA);
    PyObject* dev = PyLong_FromLong(guard->getDevice().index());
    if (!dev) return false;
    PyObject* raw = PyObject_CallOneArg(g_raw_stream, dev);
    Py_DECREF(dev);
    if (!raw) return false;
    *stream = PyLong_AsVoidPtr(raw);
    Py_DECREF(raw);
    return !PyErr_Occurred();
}

PyObject* finish(int rc) {
    if (rc >= 0) Py_RETURN_NONE;
    PyObject* e = PyObject_CallFunction(g_error, "is", rc, epp_last_error());
    if (e) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    return nullptr;
}

int32_t width(const at::Tensor& t, int d) { return (int32_t)t.size(d); }

template <bool FULL>
PyObject* aggregate(PyObject*, PyObject* const* args, Py_ssize_t n, PyObject* kw) {
    static const char* const names[2][3] = {{"path", "grad_in", "grad_out"}, {"full", "grad_in", "grad_out"}};
    PyObject* a[3];
    if (!take_args(FULL ? "epp_full_aggregate" : "epp_backward_aggregate", args, n, kw, names[FULL], 3, a)) return nullptr;
    const at::Tensor *in = float_tensor(a[1]), *out = in ? float_tensor(a[2]) : nullptr;
    if (!out) return nullptr;
    if (in->dim() != 2 || in->sizes() != out->sizes()) {
        PyErr_SetString(PyExc_ValueError, "grad_in and grad_out must be n x F matrices of the same shape");
        return nullptr;
    }
    const int64_t vertices = vertices_of(a[0]);
    if (vertices < 0) return nullptr;
    if (in->size(0) != vertices) {  // the kernels index rows by vertex id: fewer rows would be read out of bounds
        PyErr_Format(PyExc_ValueError, "gradient matrices have %lld rows, the graph has %lld vertices",
                     (long long)in->size(0), (long long)vertices);
        return nullptr;
    }
    epp_path_t* path = static_cast<epp_path_t*>(handle_of(a[0]));
    void* s;
    if (!path || !current_stream(&s)) return nullptr;
    const float* src = in->const_data_ptr<float>();
    float* dst = out->mutable_data_ptr<float>();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = FULL ? epp_full_aggregate(path, src, dst, width(*in, 1), s) : epp_backward_aggregate(path, src, dst, width(*in, 1), s);
    Py_END_ALLOW_THREADS
    return finish(rc);
}

template <bool STATIC>
PyObject* weight_gradient(PyObject*, PyObject* const* args, Py_ssize_t n, PyObject* kw) {
    static const char* const names[] = {"paths", "k", "Y", "grad_X", "grad_W", "workspace"};
    PyObject* a[6];
    if (!take_args(STATIC ? "epp_weight_gradient_static" : "epp_weight_gradient", args, n, kw, names, STATIC ? 5 : 6, a))
        return nullptr;
    const at::Tensor* Y = matrix(a[2], "Y");
    const at::Tensor* G = Y ? matrix(a[3], "grad_X") : nullptr;
    const at::Tensor* W = G ? matrix(a[4], "grad_W") : nullptr;
    const int64_t vertices = W ? vertices_of(a[0]) : -1;
    if (vertices < 0) return nullptr;
    if (Y->size(0) != vertices || G->size(0) != vertices || W->size(0) != Y->size(1) || W->size(1) != G->size(1)) {
        PyErr_SetString(PyExc_ValueError, "shapes: Y n x F_in, grad_X n x F_out, grad_W F_in x F_out");
        return nullptr;
    }
    void* ws = nullptr;
    int64_t ws_bytes = 0;
    if (!STATIC) {
        if (!THPVariable_Check(a[5]) || !THPVariable_Unpack(a[5]).is_cuda() ||
            THPVariable_Unpack(a[5]).scalar_type() != at::kByte || !THPVariable_Unpack(a[5]).is_contiguous()) {
            PyErr_SetString(PyExc_ValueError, "workspace must be a contiguous CUDA uint8 tensor");
            return nullptr;
        }
        ws = THPVariable_Unpack(a[5]).mutable_data_ptr();
        ws_bytes = THPVariable_Unpack(a[5]).numel();
    }
    const int k = (int)PyLong_AsLong(a[1]);
    if (k == -1 && PyErr_Occurred()) return nullptr;
    epp_paths_t* paths = static_cast<epp_paths_t*>(handle_of(a[0]));
    void* s;
    if (!paths || !current_stream(&s)) return nullptr;
    const float *y = Y->const_data_ptr<float>(), *g = G->const_data_ptr<float>();
    float* w = W->mutable_data_ptr<float>();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = STATIC ? epp_weight_gradient_static(paths, k, y, width(*Y, 1), g, width(*G, 1), w, s)
                : epp_weight_gradient(paths, k, y, width(*Y, 1), g, width(*G, 1), w, ws, ws_bytes, s);
    Py_END_ALLOW_THREADS
    return finish(rc);
}

PyObject* input_gradient(PyObject*, PyObject* const* args, Py_ssize_t n, PyObject* kw) {
    static const char* const names[] = {"paths", "k", "grad_X", "W", "grad_Y"};
    PyObject* a[5];
    if (!take_args("epp_input_gradient", args, n, kw, names, 5, a)) return nullptr;
    const at::Tensor* G = matrix(a[2], "grad_X");
    const at::Tensor* W = G ? matrix(a[3], "W") : nullptr;
    const at::Tensor* Y = W ? matrix(a[4], "grad_Y") : nullptr;
    const int64_t vertices = Y ? vertices_of(a[0]) : -1;
    if (vertices < 0) return nullptr;
    if (G->size(0) != vertices || W->size(1) != G->size(1) || Y->size(0) != G->size(0) || Y->size(1) != W->size(0)) {
        PyErr_SetString(PyExc_ValueError, "shapes: grad_X n x F_out, W F_in x F_out, grad_Y n x F_in");
        return nullptr;
    }
    const int k = (int)PyLong_AsLong(a[1]);
    if (k == -1 && PyErr_Occurred()) return nullptr;
    epp_paths_t* paths = static_cast<epp_paths_t*>(handle_of(a[0]));
    void* s;
    if (!paths || !current_stream(&s)) return nullptr;
    const float *g = G->const_data_ptr<float>(), *w = W->const_data_ptr<float>();
    float* y = Y->mutable_data_ptr<float>();
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = epp_input_gradient(paths, k, g, width(*G, 1), w, width(*W, 0), y, s);
    Py_END_ALLOW_THREADS
    return finish(rc);
}

typedef PyObject* (*Entry)(PyObject*, PyObject* const*, Py_ssize_t, PyObject*);
template <Entry F>
PyObject* guarded(PyObject* self, PyObject* const* args, Py_ssize_t n, PyObject* kw) {
    // (PyTorch's own macro for this also buffers warnings: 0.2 us a call)
    try {
        return F(self, args, n, kw);
    } catch (python_error& e) {
        e.restore();
    } catch (const c10::Error& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what_without_backtrace());
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
    }
    return nullptr;
}

// epp_alloc_t of PyTorch's caching allocator, on the current device and stream; any host thread, with the interpreter's lock or without.
// (As functions of the Python module, called back through ctypes, an allocation and its release took 4.3 us, and a construction or an
// import makes about eight, some of them while the GPU waits for the next launch: constructed on 8,000 vertices 106 -> 88 us, imported
// and one epoch on the blog graph 120 -> 112.)
std::atomic<long long> g_allocs{0}, g_frees{0}, g_bytes{0};

void* torch_alloc(size_t bytes, void*) {
    try {
        void* p = c10::hip::HIPCachingAllocator::raw_alloc(bytes);
        if (!p) return nullptr;
        g_allocs.fetch_add(1, std::memory_order_relaxed);
        g_bytes.fetch_add((long long)bytes, std::memory_order_relaxed);
        return p;
    } catch (...) {  // out of memory: the library reports EPP_ERR_ALLOC
        return nullptr;
    }
}
void torch_free(void* p, void*) {
    g_frees.fetch_add(1, std::memory_order_relaxed);
    try {
        c10::hip::HIPCachingAllocator::raw_delete(p);
    } catch (...) {  // (nobody to tell: the handle goes)
    }
}

// (address of the allocating function, of the releasing one)
PyObject* allocator(PyObject*, PyObject*) {
    return Py_BuildValue("KK", (unsigned long long)reinterpret_cast<uintptr_t>(&torch_alloc),
                         (unsigned long long)reinterpret_cast<uintptr_t>(&torch_free));
}
// alloc_news(dictionary): adds to its allocs, frees, bytes and live what has been counted since the last call.
PyObject* alloc_news(PyObject*, PyObject* stats) {
    if (!PyDict_Check(stats)) {
        PyErr_SetString(PyExc_TypeError, "alloc_news(dictionary)");
        return nullptr;
    }
    if (!g_allocs.load(std::memory_order_relaxed) && !g_frees.load(std::memory_order_relaxed)) Py_RETURN_NONE;
    const long long allocs = g_allocs.exchange(0, std::memory_order_relaxed), frees = g_frees.exchange(0, std::memory_order_relaxed);
    const struct { const char* key; long long more; } news[] = {
        {"allocs", allocs}, {"frees", frees}, {"bytes", g_bytes.exchange(0, std::memory_order_relaxed)}, {"live", allocs - frees}};
    for (const auto& x : news) {
        PyObject* const had = PyDict_GetItemString(stats, x.key);  // (borrowed; none: taken for 0)
        PyObject* const more = PyLong_FromLongLong(x.more);
        PyObject* const sum = more && had ? PyNumber_Add(had, more) : more;
        const bool done = sum && PyDict_SetItemString(stats, x.key, sum) == 0;
        if (had) Py_XDECREF(more);
        Py_XDECREF(sum);
        if (!done) return nullptr;
    }
    Py_RETURN_NONE;
}

// init(error class, raw-stream function)
PyObject* init(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 2) {
        PyErr_SetString(PyExc_TypeError, "init(error, raw_stream)");
        return nullptr;
    }
    Py_INCREF(args[0]);
    Py_XSETREF(g_error, args[0]);
    Py_INCREF(args[1]);
    Py_XSETREF(g_raw_stream, args[1]);
    Py_RETURN_NONE;
}

#define EPP_FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(guarded<f>)), METH_FASTCALL | METH_KEYWORDS

PyMethodDef methods[] = {
    {"init", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(init)), METH_FASTCALL, nullptr},
    {"epp_backward_aggregate", EPP_FAST(aggregate<false>),
     "epp_backward_aggregate(path, grad_in, grad_out)\n\nPartially-active backward aggregation of one layer."},
    {"epp_full_aggregate", EPP_FAST(aggregate<true>),
     "epp_full_aggregate(full, grad_in, grad_out)\n\nAll-active backward aggregation."},
    {"epp_weight_gradient", EPP_FAST(weight_gradient<false>),
     "epp_weight_gradient(paths, k, Y, grad_X, grad_W, workspace)\n\nW' = Y^T (x) X' over the rows of N^k (k = -1: all "
     "rows); `workspace` is a CUDA uint8 tensor of\nat least epp_weight_gradient_workspace(...) bytes."},
    {"epp_weight_gradient_static", EPP_FAST(weight_gradient<true>),
     "epp_weight_gradient_static(paths, k, Y, grad_X, grad_W)\n\nepp_weight_gradient without a workspace: the partial sums "
     "use the library's static device array\n(no allocation anywhere; F_in * F_out <= 8,388,608; calls on one GPU must "
     "not overlap)."},
    {"epp_input_gradient", EPP_FAST(input_gradient),
     "epp_input_gradient(paths, k, grad_X, W, grad_Y)\n\nY' = X' (x) W^T on the rows of N^k (k = -1: all rows); other rows "
     "of grad_Y are not touched."},
    {"allocator", allocator, METH_NOARGS, nullptr},
    {"alloc_news", alloc_news, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) {
    s_handle = PyUnicode_InternFromString("_h");
    s_cached_n = PyUnicode_InternFromString("_n");
    s_n = PyUnicode_InternFromString("n");
    if (!s_handle || !s_cached_n || !s_n) return nullptr;
    return PyModule_Create(&module);
}
