// The chain calls of the Python package: torch tensors in, mcf.h calls out.  A CPython extension,
// because the marshalling (shapes, strides, the output's allocation, the current stream) is most of
// what a small chain costs its caller: 15.3 us a call through ctypes, of which the kernel of
// 1 x [1024,64].[64,128].[128,64] is 4.2 us and the launch 3.
#include <Python.h>

#include <ATen/ops/empty.h>
#include <c10/core/DeviceGuard.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPGraphsC10Utils.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <stdio.h>
#include <string.h>

#include "mcf_internal.h"

namespace {

PyObject *g_error = nullptr; // binding.McfError(status, text)

PyObject *fail(int status, const char *text) {
    PyObject *e = PyObject_CallFunction(g_error, "is", status, text);
    if (e) {
        PyErr_SetObject(g_error, e);
        Py_DECREF(e);
    }
    return nullptr;
}

PyObject *fail_status(int status) {
    const char *more = mcf_last_error();
    char text[512];
    if (*more) snprintf(text, sizeof(text), "%s (%s)", mcf_status_string(status), more);
    else snprintf(text, sizeof(text), "%s", mcf_status_string(status));
    return fail(status, text);
}

// Strides of a [batch, rows, cols] tensor as the C ABI wants them: an empty tensor has no meaningful
// ones (zeros read as packed), and a dimension of extent <= 1 gets the packed one.
void strides3(const at::Tensor &t, int64_t s[3]) {
    const int64_t n0 = t.size(0), n1 = t.size(1), n2 = t.size(2);
    s[0] = s[1] = s[2] = 0;
    if (n0 == 0 || n1 == 0 || n2 == 0) return;
    s[0] = t.stride(0); s[1] = t.stride(1); s[2] = t.stride(2);
    // a single column: keep a row-contiguous (transposed) view recognisable as such
    if (n2 <= 1) s[2] = s[1] == 1 && n1 > 1 ? n1 : 1;
    if (n1 <= 1) s[1] = s[2] == 1 ? n2 : 1;
    if (n0 <= 1) s[0] = 0;
}

// One element broadcast over a whole tensor: every stride is zero, which the C ABI reads as "packed".
bool one_element(const at::Tensor &t) {
    if (t.layout() != at::kStrided || t.numel() <= 1) return false;
    for (int64_t d = 0; d < t.dim(); ++d)
        if (t.size(d) > 1 && t.stride(d) != 0) return false;
    return true;
}

// The workspace of a call from torch's allocator, for the device of its operands (which need not be the current one) and the
// stream that the call runs on: given back right after the launches, it is only handed out again to later work of that
// stream.  While the stream is captured it has to stay with the graph instead.  torch's own capture allocates from the graph's
// pool, which does that; where someone else captures, memory given back would be used by others between the replays:
// nullptr then (and in any capture nothing here may end it, so that an allocation may go past the allocator's cache).
void *workspace(size_t bytes, hipStream_t stream, c10::Device device) {
    namespace alloc = c10::hip::HIPCachingAllocator;
    c10::DeviceGuard on(device);
    if (!mcf::stream_capturing(stream)) return alloc::raw_alloc_with_stream(bytes, stream);
    c10::hip::HIPStreamCaptureModeGuard allowed(hipStreamCaptureModeRelaxed);
    void *ws = alloc::raw_alloc_with_stream(bytes, stream);
    for (const auto &seg : alloc::snapshot().segments)
        if ((size_t)ws - seg.address < seg.total_size && seg.owner_private_pool_id != c10::MempoolId_t(0, 0)) return ws;
    alloc::raw_delete(ws);
    return nullptr;
}

// Lays a call out and launches it; touches nothing of Python's.
int run(mcf_call &call, void *stream, c10::Device device) {
    mcf::Launch l;
    int st = mcf::prepare(&call, &l);
    if (st != MCF_OK) return st;
    void *ws = nullptr;
    if (l.workspace_bytes > 0) {
        // where there is no workspace to be had, ranges that the library chose are not needed
        try {
            ws = workspace((size_t)l.workspace_bytes, (hipStream_t)stream, device);
        } catch (const c10::OutOfMemoryError &) {
            if (call.n_split != 0) throw;
        }
        if (!ws) {
            if (call.n_split != 0) {
                mcf::set_last_error("ranges of n in a graph that torch does not capture");
                return MCF_EUNSUPPORTED;
            }
            call.n_split = 1;
            st = mcf::prepare(&call, &l);
            if (st != MCF_OK) return st;
        }
    }
    st = mcf::launch(&l, ws, l.workspace_bytes, stream);
    if (ws) c10::hip::HIPCachingAllocator::raw_delete(ws);
    return st;
}

// The interpreter lock is let go while a call allocates and launches, both of which may wait for the device
// (and work that is queued may wait for a Python thread); costs 0.1 us a call.
struct NoGil {
    PyThreadState *state = PyEval_SaveThread();
    NoGil() = default;
    NoGil(const NoGil &) = delete;
    ~NoGil() { PyEval_RestoreThread(state); }
};

bool is_tensor(PyObject *o) { return THPVariable_Check(o); }

// chain(kind, scale, causal_offset, A, B, D, F, out, tiles, stream, n_split) -> out
//   kind: 0 plain, 1 softmax, 2 causal softmax; F: None or the third factor (kind 0 or 1)
//   tiles: 0 or the address of an mcf_tiles; stream: None (torch's current one) or a hipStream_t as an integer
//   n_split: ranges of n, 0 for the library's choice (mcf_call)
PyObject *chain(PyObject *, PyObject *const *arg, Py_ssize_t n) {
    if (n != 11) return PyErr_Format(PyExc_TypeError, "chain takes 11 arguments");
    const long kind = PyLong_AsLong(arg[0]);
    double scale = 0.0;
    if (PyFloat_CheckExact(arg[1])) {
        scale = PyFloat_AS_DOUBLE(arg[1]);
    } else if (PyObject *f = PyNumber_Float(arg[1])) { // what float() takes
        scale = PyFloat_AsDouble(f);
        Py_DECREF(f);
    }
    const long long causal_offset = PyLong_AsLongLong(arg[2]);
    const mcf_tiles *tiles = (const mcf_tiles *)PyLong_AsVoidPtr(arg[8]);
    void *stream = arg[9] == Py_None ? nullptr : PyLong_AsVoidPtr(arg[9]);
    const long n_split = PyLong_AsLong(arg[10]);
    if (PyErr_Occurred()) return nullptr;
    if (!is_tensor(arg[3]) || !is_tensor(arg[4]) || !is_tensor(arg[5]) || (arg[6] != Py_None && !is_tensor(arg[6])) ||
        (arg[7] != Py_None && !is_tensor(arg[7])))
        return PyErr_Format(PyExc_TypeError, "A, B, D, F and out must be tensors");
    const at::Tensor &A = THPVariable_Unpack(arg[3]), &B = THPVariable_Unpack(arg[4]), &D = THPVariable_Unpack(arg[5]);
    const at::Tensor *F = arg[6] == Py_None ? nullptr : &THPVariable_Unpack(arg[6]);
    if (A.dim() != 3 || B.dim() != 3 || D.dim() != 3) return fail(MCF_EINVAL, "A, B, D, E must be 3-d [batch, rows, cols]");
    const int64_t b = A.size(0), M = A.size(1), K = A.size(2), N = B.size(2), L = D.size(2);
    if (B.size(0) != b || D.size(0) != b || B.size(1) != K || D.size(1) != N) return fail(MCF_EINVAL, "the shapes of A, B and D do not form a chain");
    if (F && (F->dim() != 3 || F->size(0) != b || F->size(1) != L)) return fail(MCF_EINVAL, "F does not continue D");
    const int64_t cols = F ? F->size(2) : L;
    if (one_element(A) || one_element(B) || one_element(D) || (F && one_element(*F)) || (arg[7] != Py_None && one_element(THPVariable_Unpack(arg[7]))))
        return fail(MCF_EUNSUPPORTED, "an operand is one element broadcast over all of its extent");
    const at::ScalarType type = A.scalar_type();
    if (!A.is_cuda() || !B.is_cuda() || !D.is_cuda()) return fail(MCF_EINVAL, "A, B, D, E must be device tensors");
    if (type != at::kHalf && type != at::kBFloat16) return fail(MCF_EUNSUPPORTED, "unsupported dtype of A");
    if (B.scalar_type() != type || D.scalar_type() != type) return fail(MCF_EINVAL, "A, B, D must share one dtype; E has that dtype or float32");
    if (B.device() != A.device() || D.device() != A.device()) return fail(MCF_EINVAL, "A, B, D, E must live on one device");
    if (F && (F->scalar_type() != type || F->device() != A.device())) return fail(MCF_EINVAL, "F must match A in dtype and device");
    const bool make = arg[7] == Py_None;
    at::Tensor made;
    const at::Tensor &E = make ? made : THPVariable_Unpack(arg[7]);
    if (!make) {
        if (E.dim() != 3 || E.size(0) != b || E.size(1) != M || E.size(2) != cols) return fail(MCF_EINVAL, "the output has the wrong shape");
        if (E.scalar_type() != type && E.scalar_type() != at::kFloat) return fail(MCF_EINVAL, "A, B, D must share one dtype; E has that dtype or float32");
        if (!E.is_cuda() || E.device() != A.device()) return fail(MCF_EINVAL, "A, B, D, E must live on one device");
    }
    mcf_call call;
    mcf_problem &p = call.problem;
    p.batch = b; p.M = M; p.K = K; p.N = N; p.L = L;
    p.in_dtype = type == at::kHalf ? MCF_F16 : MCF_BF16;
    p.out_dtype = !make && E.scalar_type() == at::kFloat ? MCF_F32 : p.in_dtype;
    strides3(A, p.a_stride);
    strides3(B, p.b_stride);
    strides3(D, p.d_stride);
    if (make) memset(p.e_stride, 0, sizeof(p.e_stride)); // packed
    else strides3(E, p.e_stride);
    call.P = F ? cols : 0;
    if (F) strides3(*F, call.f_stride);
    else memset(call.f_stride, 0, sizeof(call.f_stride));
    call.softmax = kind != 0; call.causal = kind == 2;
    call.scale = (float)scale; call.causal_offset = causal_offset;
    call.n_split = (int32_t)n_split;
    call.A = A.data_ptr(); call.B = B.data_ptr(); call.D = D.data_ptr(); call.F = F ? F->data_ptr() : nullptr; call.E = make ? nullptr : E.data_ptr();
    call.tiles = tiles;
    if (arg[9] == Py_None) stream = (void *)c10::hip::getCurrentHIPStream().stream();
    int st = MCF_OK;
    {
        const NoGil released;
        if (make) {
            made = at::empty({b, M, cols}, A.options());
            call.E = made.data_ptr();
        }
        if (!F || cols > 0) st = run(call, stream, A.device()); // (no output columns: nothing to do)
    }
    if (st != MCF_OK) return fail_status(st);
    if (make) return THPVariable_Wrap(std::move(made));
    Py_INCREF(arg[7]);
    return arg[7];
}

// C++ exceptions of torch (out of memory, a stream of another device, ...) become Python ones
PyObject *chain_entry(PyObject *self, PyObject *const *arg, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    return chain(self, arg, n);
    END_HANDLE_TH_ERRORS
}

PyObject *set_error(PyObject *, PyObject *type) {
    Py_INCREF(type);
    Py_XDECREF(g_error);
    g_error = type;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"chain", (PyCFunction)(void (*)(void))chain_entry, METH_FASTCALL, "one chain call on torch tensors"},
                         {"set_error", set_error, METH_O, "the exception type to raise"},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_mcf_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit__mcf_torch() { return PyModule_Create(&module); }
