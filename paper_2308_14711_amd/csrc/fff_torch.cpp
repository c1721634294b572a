// The binding's ordinary call, in native code: torch tensors in, one call of the C ABI out.
//
// A forward call on a small batch is a launch or two of 4-10 us; marshalling fifteen arguments and
// checking nine tensors in Python cost another 6.5 us of host time on top of the 3.4 us the
// library and the runtime need, which made every such call host-bound (10.7 us a call whatever the
// kernels took).  Here the same checks are a few loads per tensor.
//
// Each function returns the library's status, or -1 when the call is not an ordinary one (an
// argument of another type, a wrong shape, a CPU tensor, ...): nothing has been enqueued then, and
// binding.py takes the call through its own checks, which name what is wrong.
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPStream.h>

#include "../../include/fff.h"

namespace {

// The arguments of one call.  `ok` falls to false with the first thing that is not as expected.
struct Call {
    PyObject* const* args;
    bool ok = true;
    at::ScalarType dtype = at::ScalarType::Float;

    const at::Tensor* tensor(int i) {
        if (args[i] == Py_None) return nullptr;
        if (!THPVariable_Check(args[i])) {
            ok = false;
            return nullptr;
        }
        return &THPVariable_Unpack(args[i]);
    }
    // Address of a dense device tensor of exactly these sizes (NULL for None).
    void* dense(int i, at::ScalarType want, std::initializer_list<int64_t> sizes) {
        const at::Tensor* t = tensor(i);
        if (!t) return nullptr;
        ok = ok && t->scalar_type() == want && t->sizes() == at::IntArrayRef(sizes.begin(), sizes.size()) &&
             t->is_cuda() && t->is_contiguous();
        return ok ? t->data_ptr() : nullptr;
    }
    // The same for a tensor that must be there.
    void* need(int i, std::initializer_list<int64_t> sizes) {
        void* p = dense(i, dtype, sizes);
        ok = ok && args[i] != Py_None;
        return p;
    }
    int integer(int i, int low, int high) {
        const long v = PyLong_Check(args[i]) ? PyLong_AsLong(args[i]) : (long)low - 1;
        if (v < low || v > high) {
            if (PyErr_Occurred()) PyErr_Clear();
            ok = false;
            return low;
        }
        return (int)v;
    }
    void* stream(int i) {
        if (!ok) return nullptr;
        if (args[i] == Py_None) return c10::hip::getCurrentHIPStream().stream();
        PyObject* h = PyLong_Check(args[i]) ? Py_NewRef(args[i]) : PyObject_GetAttrString(args[i], "cuda_stream");
        void* s = h ? PyLong_AsVoidPtr(h) : nullptr;
        Py_XDECREF(h);
        if (PyErr_Occurred()) {
            PyErr_Clear();
            ok = false;
        }
        return s;
    }
    // x: a matrix of tokens; sets the dtype of the call
    void* tokens(int i, int64_t* T, int64_t* D) {
        const at::Tensor* t = tensor(i);
        if (!t || t->dim() != 2 || (t->scalar_type() != at::ScalarType::Float && t->scalar_type() != at::ScalarType::BFloat16)) {
            ok = false;
            return nullptr;
        }
        dtype = t->scalar_type();
        *T = t->size(0);
        *D = t->size(1);
        return need(i, {*T, *D});
    }
    int64_t columns(int i) {
        const at::Tensor* t = tensor(i);
        if (!t || t->dim() != 2) {
            ok = false;
            return 0;
        }
        return t->size(1);
    }
    int code() const { return dtype == at::ScalarType::BFloat16 ? FFF_BF16 : FFF_F32; }
};

template <class F> PyObject* answer(const Call& c, F call) {
    int rc = -1;
    if (c.ok) {
        Py_BEGIN_ALLOW_THREADS
        rc = call();
        Py_END_ALLOW_THREADS
    }
    return PyLong_FromLong(rc);
}

constexpr int kMaxWidth = 1 << 20;   // sizes beyond the library's own limits are left to its checks

// x, node_w, node_b, leaf_w1, leaf_b1, leaf_w2, leaf_b2, depth, leaf_width, act, out, ...
struct Layer {
    int64_t T = 0, D = 0, O = 0;
    int depth, width, act;
    void *x, *node_w = nullptr, *node_b = nullptr, *w1, *b1, *w2, *b2, *out;
};

// x at argument 0, the leaves at `leaf`, depth / width at `depth`; act and out where given.
Layer layer(Call& c, int leaf, int depth, int width, int act, int out) {
    Layer a;
    a.x = c.tokens(0, &a.T, &a.D);
    a.depth = c.integer(depth, 0, FFF_MAX_DEPTH);
    a.width = c.integer(width, 1, kMaxWidth);
    a.act = c.integer(act, 0, 1);
    a.O = c.columns(out);
    const int64_t n = (int64_t)1 << a.depth;
    a.w1 = c.need(leaf, {n, a.width, a.D});
    a.b1 = c.need(leaf + 1, {n, a.width});
    a.w2 = c.need(leaf + 2, {n, a.width, a.O});
    a.b2 = c.need(leaf + 3, {n, a.O});
    a.out = c.need(out, {a.T, a.O});
    return a;
}

// Scratch of one call from torch's allocator, in the order of the call's stream: handed back once the call has enqueued its work.
// Null where there is none to be had (nothing may throw past the released interpreter lock).
struct Scratch {
    void* p = nullptr;
    Scratch(size_t bytes, hipStream_t s) {
        // an allocator with nothing left asks the device, which must not spoil what another thread captures just now
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        (void)hipThreadExchangeStreamCaptureMode(&mode);
        try {
            p = c10::hip::HIPCachingAllocator::raw_alloc_with_stream(bytes, s);
        } catch (const std::exception&) {
        }
        (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
    ~Scratch() {
        if (p) c10::hip::HIPCachingAllocator::raw_delete(p);
    }
    Scratch(const Scratch&) = delete;
};

// Whether the call is being captured (it is left to binding.py then, which finds out who captures).
bool captured(void* s) {
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing((hipStream_t)s, &capture) == hipSuccess && capture == hipStreamCaptureStatusNone) return false;
    (void)hipGetLastError();
    return true;
}

// x, node_w, node_b, leaf_w1, leaf_b1, leaf_w2, leaf_b2, depth, leaf_width, act, out, leaf_idx, stream, static_scratch
PyObject* forward_hard(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 14) return PyLong_FromLong(-1);
    Call c{args};
    Layer a = layer(c, 3, 7, 8, 9, 10);
    if (a.depth < 1) c.ok = false;
    a.node_w = c.need(1, {((int64_t)1 << a.depth) - 1, a.D});
    a.node_b = c.need(2, {((int64_t)1 << a.depth) - 1});
    int32_t* idx = (int32_t*)c.dense(11, at::ScalarType::Int, {a.T});
    void* s = c.stream(12);
    const int truth = PyObject_IsTrue(args[13]);
    if (truth < 0) {        // a value without one: the caller's own test of it says why
        PyErr_Clear();
        c.ok = false;
    }
    return answer(c, [&] {
        const auto call = [&](auto entry, auto... more) {
            return entry(a.x, a.node_w, a.node_b, a.w1, a.b1, a.w2, a.b2, a.depth, a.width, a.act, a.out, idx, s, a.T, a.D, a.O, c.code(), more...);
        };
        if (truth == 1) return call(fff_forward_hard_static);
        const size_t bytes = fff_hard_scratch_bytes(a.T, a.D, a.O, a.depth, a.width, c.code());
        if (bytes == 0) return call(fff_forward_hard);
        if (captured(s)) return -1;
        const Scratch scratch(bytes, (hipStream_t)s);
        return call(fff_forward_hard_scratch, scratch.p, bytes);
    });
}

// x, gate_w, gate_b, leaf_w1, leaf_b1, leaf_w2, leaf_b2, log2_experts, leaf_width, act, out, expert_idx, stream
PyObject* moe_top1_forward(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 13) return PyLong_FromLong(-1);
    Call c{args};
    Layer a = layer(c, 3, 7, 8, 9, 10);
    void* gate_w = c.need(1, {(int64_t)1 << a.depth, a.D});
    void* gate_b = c.dense(2, c.dtype, {(int64_t)1 << a.depth});
    int32_t* idx = (int32_t*)c.dense(11, at::ScalarType::Int, {a.T});
    void* s = c.stream(12);
    return answer(c, [&] {
        return fff_moe_top1_forward(a.x, gate_w, gate_b, a.w1, a.b1, a.w2, a.b2, a.depth, a.width, a.act, a.out, idx, s,
                                    a.T, a.D, a.O, c.code());
    });
}

// x, node_w, node_b, leaf_w1, leaf_b1, leaf_w2, leaf_b2, depth, leaf_width, act, out, mix, entropy, stream
PyObject* forward_soft(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 14) return PyLong_FromLong(-1);
    Call c{args};
    Layer a = layer(c, 3, 7, 8, 9, 10);
    if (a.depth < 1) c.ok = false;
    const int64_t nodes = ((int64_t)1 << a.depth) - 1;
    a.node_w = c.need(1, {nodes, a.D});
    a.node_b = c.need(2, {nodes});
    float* mix = (float*)c.dense(11, at::ScalarType::Float, {a.T, nodes + 1});
    const at::Tensor* e = c.tensor(12);   // may be longer than the nodes
    float* entropy = e && e->dim() == 1 && e->size(0) >= nodes
                         ? (float*)c.dense(12, at::ScalarType::Float, {e->size(0)}) : nullptr;
    c.ok = c.ok && (entropy || args[12] == Py_None);
    void* s = c.stream(13);
    return answer(c, [&] {
        return fff_forward_soft(a.x, a.node_w, a.node_b, a.w1, a.b1, a.w2, a.b2, a.depth, a.width, a.act, a.out, mix,
                                entropy, s, a.T, a.D, a.O, c.code());
    });
}

// x, ln_gamma, ln_beta, ln_eps, node_w1, node_b1, node_w2, node_b2, leaf_w1, leaf_b1, leaf_w2, leaf_b2,
// depth, node_size, leaf_width, act, residual, out, leaf_idx, stream
PyObject* forward_block(PyObject*, PyObject* const* args, Py_ssize_t n) {
    if (n != 20) return PyLong_FromLong(-1);
    Call c{args};
    Layer a = layer(c, 8, 12, 14, 15, 17);
    if (a.depth < 1) c.ok = false;
    const int64_t nodes = ((int64_t)1 << a.depth) - 1, size = c.integer(13, 1, kMaxWidth);
    void* gamma = c.dense(1, c.dtype, {a.D});
    void* beta = c.dense(2, c.dtype, {a.D});
    const double eps = PyFloat_Check(args[3]) ? PyFloat_AS_DOUBLE(args[3]) : (c.ok = false, 0.0);
    void* w1 = c.need(4, {nodes, size, a.D});
    void* b1 = c.need(5, {nodes, size});
    void* w2 = c.need(6, {nodes, size});
    void* b2 = c.need(7, {nodes});
    const int residual = args[16] == Py_True ? 1 : args[16] == Py_False ? 0 : (c.ok = false, 0);
    int32_t* idx = (int32_t*)c.dense(18, at::ScalarType::Int, {a.T});
    void* s = c.stream(19);
    return answer(c, [&] {
        const auto call = [&](void* scratch, size_t bytes) {
            return fff_forward_block_scratch(a.x, gamma, beta, (float)eps, w1, b1, w2, b2, a.w1, a.b1, a.w2, a.b2, a.depth, (int)size, a.width,
                                             a.act, residual, a.out, idx, s, a.T, a.D, a.O, c.code(), scratch, bytes);
        };
        const size_t bytes = fff_block_scratch_bytes(a.T, a.D, a.O, a.depth, (int)size, a.width, gamma != nullptr, c.code());
        if (bytes == 0) return call(nullptr, 0);
        if (captured(s)) return -1;
        const Scratch scratch(bytes, (hipStream_t)s);
        return call(scratch.p, bytes);
    });
}

// torch's accessors may throw (a tensor without storage, no device): not an ordinary call either
template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject* self, PyObject* const* args, Py_ssize_t n) {
    try {
        return F(self, args, n);
    } catch (const std::exception&) {
        return PyLong_FromLong(-1);
    }
}

#define FFF_METHOD(f) {#f, (PyCFunction)(void (*)(void))guarded<f>, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FFF_METHOD(forward_hard), FFF_METHOD(moe_top1_forward), FFF_METHOD(forward_soft),
                         FFF_METHOD(forward_block), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fff_torch", "Native calls of binding.py", -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__fff_torch(void) { return PyModule_Create(&module); }
