// The plain calls of the Python binding (attn_fwd and gemm_bf16 on torch's current stream, results allocated here) without
// Python's share of the work: checking three tensors, allocating the results and marshalling two dozen arguments takes
// longer there than a small kernel runs.  Host time per call on the machine measured, Python against this: attn_fwd with its
// keys cut 14.0 against 8.1 us, uncut 8.5 / 4.4, gemm_bf16 7.2 / 3.9.
//
// Each function returns None for everything that is not such a call, however slightly (another type, a subclass, a tensor of
// a transform, a wrong shape), and the Python code then does what it always did, errors included; it returns an int for
// an error code of the library.  The library's entry points arrive as addresses from the binding, which has it loaded.
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cmath>

#include "../../include/attn_workspace.h"
#include "../../include/gemm_workspace.h"

namespace {

using At = at::Tensor;
// The library's entry points, with the headers' own types.
struct Entries {
    decltype(&::attn_fwd) attn_fwd;
    decltype(&::attn_fwd_strided) attn_fwd_strided;
    decltype(&::attn_fwd_workspace_bytes) attn_fwd_workspace_bytes;
    decltype(&::attn_fwd_workspace) attn_fwd_workspace;
    decltype(&::gemm_bf16_workspace_bytes) gemm_bf16_workspace_bytes;
    decltype(&::gemm_bf16_tile) gemm_bf16_tile;
    decltype(&::gemm_bf16_workspace) gemm_bf16_workspace;
} entry = {};

// A torch.Tensor or Parameter proper whose memory is its values: bf16 on a GPU, no subclass, no tensor of a transform.
bool plain(PyObject* obj, int64_t dim) {
    if (!THPVariable_CheckExact(obj)) return false;
    const At& t = THPVariable_Unpack(obj);
    constexpr c10::DispatchKeySet kStrange({c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot, c10::DispatchKey::FuncTorchBatched,
                                            c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize, c10::DispatchKey::BatchedNestedTensor,
                                            c10::DispatchKey::NestedTensor, c10::DispatchKey::ZeroTensor, c10::DispatchKey::Negative, c10::DispatchKey::Conjugate});
    return t.defined() && t.is_cuda() && t.layout() == c10::kStrided && t.scalar_type() == at::kBFloat16 && t.dim() == dim &&
           !t.key_set().has_any(kStrange) && t.stride(dim - 1) == 1;
}
bool fits(int64_t v) { return v >= 0 && v < (int64_t(1) << 31); }

// Memory for a call's parts; undefined where there is none left: such a call runs uncut, as it would without it.
At scratch(size_t need, const At& like) {
    try {
        return at::empty({(int64_t)need}, like.options().dtype(at::kByte));
    } catch (const c10::OutOfMemoryError&) {
        return At();
    }
}
void* stream_of(const At& t) { return (void*)c10::hip::getCurrentHIPStream(t.get_device()).stream(); }

PyObject* attn(PyObject*, PyObject* const* args, Py_ssize_t n) {      // q, k, v, causal, scale
    HANDLE_TH_ERRORS
    if (!entry.attn_fwd || n != 5 || !plain(args[0], 4) || !plain(args[1], 4) || !plain(args[2], 4) || !PyBool_Check(args[3]) || at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
    const At &q = THPVariable_Unpack(args[0]), &k = THPVariable_Unpack(args[1]), &v = THPVariable_Unpack(args[2]);
    const int64_t B = q.size(0), Hq = q.size(1), Sq = q.size(2), D = q.size(3), Hkv = k.size(1), Sk = k.size(2);
    if (k.sizes() != v.sizes() || k.size(0) != B || k.size(3) != D || D == 0 || k.device() != q.device() || v.device() != q.device()) Py_RETURN_NONE;
    if (!fits(B) || !fits(Hq) || !fits(Sq) || !fits(D) || !fits(Hkv) || !fits(Sk)) Py_RETURN_NONE;
    double scale;
    if (args[4] == Py_None) scale = std::pow((double)D, -0.5);
    else if (PyFloat_CheckExact(args[4])) scale = PyFloat_AS_DOUBLE(args[4]);
    else Py_RETURN_NONE;
    const int causal = args[3] == Py_True;
    At o, lse;
    int rc;
    {
        pybind11::gil_scoped_release no_gil;
        o = at::empty_like(q);                       // keeps q's layout for dense views
        if (o.stride(3) != 1) rc = INT_MIN;
        else {
            lse = at::empty({B, Hq, Sq}, q.options().dtype(at::kFloat));
            void* const stream = stream_of(q);
            // few query rows or few heads: the keys are cut over workgroups too (the same conditions as in the Python code)
            const size_t need = Sq <= 64 || B * Hq * Sq <= 160 * 128 ? entry.attn_fwd_workspace_bytes(B, Hq, Hkv, Sq, Sk, D) : 0;
            At ws;
            if (need && (Sk + 64) * std::max(k.stride(2), v.stride(2)) < (int64_t(1) << 31)) ws = scratch(need, q);
            const long long qs[3] = {q.stride(0), q.stride(1), q.stride(2)}, ks[3] = {k.stride(0), k.stride(1), k.stride(2)},
                            vs[3] = {v.stride(0), v.stride(1), v.stride(2)}, os[3] = {o.stride(0), o.stride(1), o.stride(2)};
            if (ws.defined())
                rc = entry.attn_fwd_workspace(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), (float*)lse.data_ptr(), B, Hq, Hkv, Sq, Sk, D, qs, ks, vs, os,
                                              causal, (float)scale, ws.data_ptr(), need, (int)(need / (4 * (size_t)B * Hq * Sq * (D + 2))), stream);
            else if (q.is_contiguous() && k.is_contiguous() && v.is_contiguous() && o.is_contiguous())
                rc = entry.attn_fwd(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), (float*)lse.data_ptr(), B, Hq, Hkv, Sq, Sk, D, causal, (float)scale, stream);
            else
                rc = entry.attn_fwd_strided(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), (float*)lse.data_ptr(), B, Hq, Hkv, Sq, Sk, D, qs, ks, vs, os,
                                            causal, (float)scale, stream);
        }
    }
    if (rc == INT_MIN) Py_RETURN_NONE;
    if (rc != 0) return PyLong_FromLong(rc);
    PyObject* const out[2] = {THPVariable_Wrap(std::move(o)), THPVariable_Wrap(std::move(lse))};
    PyObject* const both = PyTuple_Pack(2, out[0], out[1]);
    Py_XDECREF(out[0]);
    Py_XDECREF(out[1]);
    return both;
    END_HANDLE_TH_ERRORS
}

PyObject* gemm(PyObject*, PyObject* const* args, Py_ssize_t n) {      // a, b, b_is_nk
    HANDLE_TH_ERRORS
    if (!entry.attn_fwd || n != 3 || !plain(args[0], 2) || !plain(args[1], 2) || !PyBool_Check(args[2]) || at::impl::torch_function_mode_enabled()) Py_RETURN_NONE;
    const At &a = THPVariable_Unpack(args[0]), &b = THPVariable_Unpack(args[1]);
    const int nk = args[2] == Py_True;
    const int64_t M = a.size(0), K = a.size(1), N = b.size(nk ? 0 : 1);
    if (b.size(nk ? 1 : 0) != K || b.device() != a.device() || !fits(M) || !fits(N) || !fits(K)) Py_RETURN_NONE;
    At c;
    int rc;
    {
        pybind11::gil_scoped_release no_gil;
        c = at::empty({M, N}, a.options());
        void* const stream = stream_of(a);
        // results of few tiles: k is cut over workgroups too, for operands whose rows start at multiples of 16 bytes
        const size_t need = entry.gemm_bf16_workspace_bytes(M, N, K);
        At ws;
        if (need && !((((uintptr_t)a.data_ptr() | (uintptr_t)b.data_ptr() | (uintptr_t)c.data_ptr()) & 15) || ((a.stride(0) | b.stride(0) | c.stride(0)) & 7)))
            ws = scratch(need, a);
        if (ws.defined())
            rc = entry.gemm_bf16_workspace(a.data_ptr(), b.data_ptr(), c.data_ptr(), M, N, K, a.stride(0), b.stride(0), c.stride(0), nk, 0, 0, ws.data_ptr(), need, stream);
        else
            rc = entry.gemm_bf16_tile(a.data_ptr(), b.data_ptr(), c.data_ptr(), M, N, K, a.stride(0), b.stride(0), c.stride(0), nk, 0, stream);
    }
    if (rc != 0) return PyLong_FromLong(rc);
    return THPVariable_Wrap(std::move(c));
    END_HANDLE_TH_ERRORS
}

// The seven entry points' addresses, in the order of Entries.
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
    void* p[7];
    if (n != 7) { PyErr_SetString(PyExc_TypeError, "seven addresses"); return nullptr; }
    for (int i = 0; i < 7; ++i) {
        p[i] = PyLong_AsVoidPtr(args[i]);
        if (!p[i]) { if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "an address is null"); return nullptr; }
    }
    int at = 0;
    auto next = [&](auto& f) { f = reinterpret_cast<std::remove_reference_t<decltype(f)>>(p[at++]); };
    next(entry.attn_fwd), next(entry.attn_fwd_strided), next(entry.attn_fwd_workspace_bytes), next(entry.attn_fwd_workspace);
    next(entry.gemm_bf16_workspace_bytes), next(entry.gemm_bf16_tile), next(entry.gemm_bf16_workspace);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", (PyCFunction)(void*)bind, METH_FASTCALL, nullptr},
    {"attn", (PyCFunction)(void*)attn, METH_FASTCALL, nullptr},
    {"gemm", (PyCFunction)(void*)gemm, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native() {
    PyObject* const m = PyModule_Create(&module);
    // the torch it was compiled for, which the binding compares with the one in use
    if (m && PyModule_AddStringConstant(m, "torch_version", NATIVE_TORCH) != 0) { Py_DECREF(m); return nullptr; }
    return m;
}
