// The per-call path of attn_fwd and gemm_lrelu in native code: check the tensors, read their pointers and
// torch's current stream, call the library.  Done in Python the same steps take 6 us a call, more than
// the kernels of small problems (1 x 2 x 128 x 64 attention: 4.7 us), so back-to-back calls ran at the
// interpreter's pace.
//
// Only plain calls are served here: anything a check does not recognise (another device, layout, type,
// shape) returns kNotPlain and the caller takes the Python path, which names what is wrong.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <limits.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPGraphsC10Utils.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

namespace {

constexpr long kNotPlain = 1;  // library codes are 0 or negative

typedef int (*AttnFn)(const void*, const void*, const void*, void*, float*, int, int, int, int, int, float, int, void*);
typedef void* (*ScratchFn)(void*, long long);
typedef int (*GemmFn)(const void*, const void*, void*, int, int, int, float, int, void*, ScratchFn, void*);
typedef int (*CapturingFn)(void*);
AttnFn g_attn = nullptr;
GemmFn g_gemm = nullptr;
CapturingFn g_capturing = nullptr;

// Scratch memory of one call, from torch's caching allocator: it belongs to the stream the call runs on, so it
// may go back as soon as the kernels are enqueued (the next owner on that stream comes after them).  That holds
// where a handle is one queue and outlives its work: torch's current stream, but not a handle that only the
// caller knows, nor the per-thread stream, one handle for a queue of every thread.  No memory either
// while the stream is captured, on a device that is not the current one, or when there is none left; the
// call then does without.
class Workspace {
  public:
    Workspace(void* stream, int device) : stream_(stream), device_(device) {}
    // What the library calls if it has a use for the memory (without the interpreter's lock: torch takes it where its allocator needs it).
    static void* take(void* self, long long bytes) { return ((Workspace*)self)->take(bytes); }
    ~Workspace() {
        try {
            if (p_) c10::hip::HIPCachingAllocator::raw_delete(p_);
        } catch (const std::exception&) {
        }
    }
    Workspace(const Workspace&) = delete;
    Workspace& operator=(const Workspace&) = delete;

  private:
    void* take(long long bytes) {
        try {
            if (stream_ != (void*)c10::hip::getCurrentHIPStream(device_).stream() || stream_ == (void*)hipStreamPerThread ||
                c10::hip::current_device() != device_ || g_capturing(stream_))
                return nullptr;
            // A recording in another thread (in the default mode) forbids this thread the allocator's calls to the
            // device, and one such call would end it; they have nothing to do with it.
            const c10::hip::HIPStreamCaptureModeGuard beside(hipStreamCaptureModeRelaxed);
            p_ = c10::hip::HIPCachingAllocator::raw_alloc_with_stream((size_t)bytes, (hipStream_t)stream_);
        } catch (const std::exception&) {
        }
        return p_;
    }

    void* stream_;
    int device_;
    void* p_ = nullptr;
};

const at::Tensor* plain_tensor(PyObject* o, int dim) {
    if (!THPVariable_Check(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || t.layout() != at::kStrided || !t.is_cuda() || t.dim() != dim || !t.is_contiguous()) return nullptr;
    for (int i = 0; i < dim; ++i)
        if (t.size(i) > INT_MAX) return nullptr;
    return &t;
}

int dtype_code(const at::Tensor& t) {  // the library's codes, the same for both entry points
    return t.scalar_type() == at::kHalf ? 0 : t.scalar_type() == at::kBFloat16 ? 1 : -1;
}

// `given`: None for torch's current stream of t's device, or an integer hipStream_t.
bool stream_of(PyObject* given, const at::Tensor& t, void** stream) {
    if (given == Py_None) {
        *stream = (void*)c10::hip::getCurrentHIPStream(t.device().index()).stream();
        return true;
    }
    if (!PyLong_CheckExact(given)) return false;
    *stream = PyLong_AsVoidPtr(given);
    return !PyErr_Occurred();
}

PyObject* not_plain() {
    PyErr_Clear();
    return PyLong_FromLong(kNotPlain);
}

// No exception of torch's may leave an entry point of C: a tensor without storage (inside torch.func.vmap, say)
// throws where its sizes, its data pointer or its stream are asked for.  The Python path then raises its own.
template <PyObject* (*F)(PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
    try {
        return F(args, nargs);
    } catch (const std::exception&) {
        return not_plain();
    }
}

// attn_fwd(q, k, v, out, lse, causal, scale, stream)
PyObject* attn_fwd(PyObject* const* args, Py_ssize_t nargs) {
    if (nargs != 8 || !g_attn) return not_plain();
    const at::Tensor *q = plain_tensor(args[0], 4), *k = plain_tensor(args[1], 4), *v = plain_tensor(args[2], 4),
                     *out = plain_tensor(args[3], 4), *lse = plain_tensor(args[4], 3);
    if (!q || !k || !v || !out || !lse) return not_plain();
    const int dt = dtype_code(*q);
    if (dt < 0 || k->scalar_type() != q->scalar_type() || v->scalar_type() != q->scalar_type() ||
        out->scalar_type() != q->scalar_type() || lse->scalar_type() != at::kFloat || k->sizes() != q->sizes() ||
        v->sizes() != q->sizes() || out->sizes() != q->sizes() || lse->sizes() != q->sizes().slice(0, 3))
        return not_plain();
    const int causal = PyObject_IsTrue(args[5]);
    const double scale = PyFloat_AsDouble(args[6]);
    void* stream;
    if (causal < 0 || (scale == -1.0 && PyErr_Occurred()) || !stream_of(args[7], *q, &stream)) return not_plain();
    void *const pq = q->data_ptr(), *const pk = k->data_ptr(), *const pv = v->data_ptr(), *const po = out->data_ptr(),
               *const pl = lse->data_ptr();
    const int B = (int)q->size(0), H = (int)q->size(1), N = (int)q->size(2), d = (int)q->size(3);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_attn(pq, pk, pv, po, (float*)pl, B, H, N, d, causal, (float)scale, dt, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// gemm_lrelu(a, b, c, slope, stream)
PyObject* gemm_lrelu(PyObject* const* args, Py_ssize_t nargs) {
    if (nargs != 5 || !g_gemm) return not_plain();
    const at::Tensor *a = plain_tensor(args[0], 2), *b = plain_tensor(args[1], 2), *c = plain_tensor(args[2], 2);
    if (!a || !b || !c) return not_plain();
    const int dt = dtype_code(*a);
    if (dt < 0 || b->scalar_type() != a->scalar_type() || c->scalar_type() != a->scalar_type() || b->size(0) != a->size(1) ||
        c->size(0) != a->size(0) || c->size(1) != b->size(1))
        return not_plain();
    const double slope = PyFloat_AsDouble(args[3]);
    void* stream;
    if ((slope == -1.0 && PyErr_Occurred()) || !stream_of(args[4], *a, &stream)) return not_plain();
    void *const pa = a->data_ptr(), *const pb = b->data_ptr(), *const pc = c->data_ptr();
    const int M = (int)a->size(0), N = (int)b->size(1), K = (int)a->size(1);
    Workspace ws(stream, a->device().index());
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_gemm(pa, pb, pc, M, N, K, (float)slope, dt, stream, &Workspace::take, &ws);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// bind(addresses of the library's attn_fwd, gemm_lrelu_with and gemm_lrelu_capturing)
PyObject* bind(PyObject*, PyObject* args) {
    unsigned long long attn = 0, gemm = 0, capturing = 0;
    if (!PyArg_ParseTuple(args, "KKK", &attn, &gemm, &capturing)) return nullptr;
    g_attn = (AttnFn)attn;
    g_capturing = (CapturingFn)capturing;
    g_gemm = (GemmFn)gemm;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"attn_fwd", (PyCFunction)(void (*)(void))guarded<attn_fwd>, METH_FASTCALL, "0, a library error, or NOT_PLAIN"},
                         {"gemm_lrelu", (PyCFunction)(void (*)(void))guarded<gemm_lrelu>, METH_FASTCALL, "0, a library error, or NOT_PLAIN"},
                         {"bind", bind, METH_VARARGS, "addresses of the library's entry points"},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() {
    PyObject* m = PyModule_Create(&module);
    if (m && PyModule_AddIntConstant(m, "NOT_PLAIN", kNotPlain) < 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
