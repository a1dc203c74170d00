// `signature` and `logsignature` as autograd nodes in C++: the glue of autograd.py (allocations, the choice of stretches, the C
// calls) without the interpreter.  What bounds small calls is the host: a pass of 4 to 6 launches took 50 to 80 us forward and
// backward through Python functions, of which the launches are a quarter, and as much again when the autograd engine's thread runs on
// distant cores and has to fetch the interpreter's state as well.
//
// Beside them `interval`, the query of a Path: eight of them and the scans behind them take 74 us, 107 with queries through ctypes.
//
// They return NotImplemented for every call that is not plain: tensors that are not torch's own, on the CPU or of
// another type, arguments of other types, transforms, modes, tracing and forward gradients, shapes that the library refuses, and paths of
// more than kLongest points.  Those run for 30 us and more in their kernels, most of them for longer than the Python functions take on
// the host, and they keep the Python route in use for what it alone can be asked, with counts and out-of-memory answers put in its way.  The Python functions then take
// the call and raise what they raise, so this file refuses nothing by itself.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/DeviceGuard.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>

#include <optional>

#include "sig.h"

namespace {

using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

constexpr int64_t kLongest = 4096;   // points of a path taken here

struct Declined {};   // the Python functions take the call

enum Mode : int64_t { kSignature, kLogExpand, kLogWords };

// The arguments that are not tensors, in the order they are kept between forward and backward.
struct Call {
    int64_t depth, stream, basepoint, inverse, mode;

    std::vector<int64_t> kept() const { return {depth, stream, basepoint, inverse, mode}; }
    static Call from(const std::vector<int64_t> &v) { return {v[0], v[1], v[2], v[3], v[4]}; }
};

sig_dtype type_of(const at::Tensor &t) { return t.scalar_type() == at::kDouble ? SIG_F64 : SIG_F32; }

hipStream_t stream_of(const at::Tensor &t) { return c10::hip::getCurrentHIPStream(t.device().index()).stream(); }

at::Tensor bytes_like(const at::Tensor &t, int64_t bytes) { return at::empty({bytes}, t.options().dtype(at::kByte)); }

const void *or_null(const at::Tensor &t) { return t.defined() ? t.data_ptr() : nullptr; }

// binding.SigError of a status, as an error of the interpreter.
[[noreturn]] void raise_status(sig_status status)
{
    PyGILState_STATE gil = PyGILState_Ensure();
    if (PyObject *binding = PyImport_ImportModule("paper_2001_00706_amd.binding")) {
        if (PyObject *error = PyObject_GetAttrString(binding, "SigError")) {
            if (PyObject *e = PyObject_CallFunction(error, "is", int(status), sig_status_string(status))) {
                PyErr_SetObject(error, e);
                Py_DECREF(e);
            }
            Py_DECREF(error);
        }
        Py_DECREF(binding);
    }
    python_error failed;
    failed.persist();
    PyGILState_Release(gil);
    throw failed;
}

at::Tensor inverted(const at::Tensor &sig, const Call &c, int64_t d)
{
    at::Tensor out = at::empty_like(sig);
    const sig_status status = sig_invert(sig.data_ptr(), sig.numel() / sig.size(-1), int(d), int(c.depth), type_of(sig), out.data_ptr(),
                                         stream_of(sig));
    if (status != SIG_OK) raise_status(status);
    return out;
}

// The signature itself; path and basepoint points contiguous.
at::Tensor plain_signature(const at::Tensor &path, const at::Tensor &value, const Call &c)
{
    const int64_t B = path.size(0), L = path.size(1), d = path.size(2), S = sig_signature_channels(int(d), int(c.depth));
    const int N = int(c.depth), bp = int(c.basepoint);
    const sig_dtype type = type_of(path);
    const int chunks = c.stream ? 1 : sig_forward_chunks_hint(B, L, int(d), N, bp, type);
    at::Tensor out = c.stream ? at::empty({B, bp ? L : L - 1, S}, path.options()) : at::empty({B, S}, path.options());
    sig_status status;
    if (chunks > 1) {   // few long paths: the scan as a reduction over the length
        const int64_t need = sig_forward_chunked_workspace_bytes(B, L, int(d), N, bp, chunks, type);
        if (need < 0) throw Declined{};
        const at::Tensor ws = bytes_like(path, need);
        status = sig_forward_chunked(path.data_ptr(), B, L, int(d), N, bp, or_null(value), chunks, type, out.data_ptr(), ws.data_ptr(), need,
                                     stream_of(path));
    } else {
        status = sig_signature(path.data_ptr(), B, L, int(d), N, int(c.stream), bp, or_null(value), nullptr, 0, type, out.data_ptr(),
                               stream_of(path));
    }
    if (status != SIG_OK) throw Declined{};
    return out;
}

at::Tensor logarithm(const at::Tensor &sig, const at::Tensor &table, const Call &c, int64_t d)
{
    const int64_t S = sig.size(-1), rows = sig.numel() / S;
    sig_status status;
    at::Tensor out;
    if (c.mode == kLogExpand) {
        out = at::empty_like(sig);
        status = sig_log(sig.data_ptr(), rows, int(d), int(c.depth), type_of(sig), out.data_ptr(), stream_of(sig));
    } else {
        std::vector<int64_t> shape = sig.sizes().vec();
        shape.back() = table.numel();
        out = at::empty(shape, sig.options());
        status = sig_log_words(sig.data_ptr(), rows, int(d), int(c.depth), table.const_data_ptr<int64_t>(), table.numel(), type_of(sig),
                               out.data_ptr(), stream_of(sig));
    }
    if (status != SIG_OK) throw Declined{};
    return out;
}

at::Tensor log_gradient(const at::Tensor &sig, at::Tensor grad, const at::Tensor &table, const Call &c, int64_t d)
{
    const int64_t S = sig.size(-1), rows = sig.numel() / S;
    const sig_dtype type = type_of(sig);
    if (c.mode == kLogWords) {
        at::Tensor all = at::empty_like(sig);
        const sig_status status = sig_lyndon_scatter(grad.data_ptr(), rows, int(d), int(c.depth), table.const_data_ptr<int64_t>(),
                                                     table.numel(), type, all.data_ptr(), stream_of(sig));
        if (status != SIG_OK) raise_status(status);
        grad = all;
    }
    at::Tensor out = at::empty_like(sig);
    const int64_t need = sig_log_backward_workspace_bytes(rows, int(d), int(c.depth), type);
    if (need < 0) raise_status(SIG_ERR_UNSUPPORTED);
    const at::Tensor ws = need > 0 ? bytes_like(sig, need) : at::Tensor();
    const sig_status status = sig_log_backward(sig.data_ptr(), grad.data_ptr(), rows, int(d), int(c.depth), type, out.data_ptr(),
                                               need > 0 ? ws.data_ptr() : nullptr, need, stream_of(sig));
    if (status != SIG_OK) raise_status(status);
    return out;
}

// Gradients with respect to the path and the basepoint, from that with respect to the signature.
variable_list signature_gradients(const at::Tensor &path, const at::Tensor &plain, const at::Tensor &value, at::Tensor grad, const Call &c)
{
    const int64_t B = path.size(0), L = path.size(1), d = path.size(2);
    const int N = int(c.depth), bp = int(c.basepoint);
    const sig_dtype type = type_of(path);
    if (c.inverse) grad = inverted(grad, c, d);   // a signed permutation that is its own transpose
    at::Tensor grad_path = at::empty_like(path), grad_value = value.defined() ? at::empty_like(value) : at::Tensor();
    void *grad_value_at = value.defined() ? grad_value.data_ptr() : nullptr;
    int chunks = c.stream ? 1 : sig_backward_chunks_fastest(B, L, int(d), N, bp, type);
    while (chunks > 1) {   // few long paths: the walk back along the path cut into stretches
        try {
            const int64_t need = sig_backward_chunked_workspace_bytes(B, L, int(d), N, bp, chunks, type);
            const at::Tensor ws = bytes_like(path, need);
            const sig_status status = sig_backward_chunked(path.data_ptr(), grad.data_ptr(), B, L, int(d), N, bp, or_null(value), chunks,
                                                           type, grad_path.data_ptr(), grad_value_at, ws.data_ptr(), need, stream_of(path));
            if (status != SIG_OK) raise_status(status);
            return {grad_path, grad_value};
        } catch (const c10::OutOfMemoryError &) {   // every stretch takes memory: with fewer it may do
            const int fewer = sig_backward_chunks_hint(B, L, int(d), N, bp, type);
            chunks = fewer < chunks ? fewer : 1;
        }
    }
    const int64_t need = sig_backward_workspace_bytes(B, L, int(d), N, int(c.stream), bp, type);
    const at::Tensor ws = need > 0 ? bytes_like(path, need) : at::Tensor();
    // `plain` is as the scan left it, unless plain_signature went by stretches
    const bool scanned = c.stream || sig_forward_chunks_hint(B, L, int(d), N, bp, type) <= 1;
    const sig_status status = (scanned ? sig_backward_scanned : sig_backward)(path.data_ptr(), plain.data_ptr(), grad.data_ptr(), B, L, int(d), N,
                                                                              int(c.stream), bp, or_null(value), type, grad_path.data_ptr(),
                                                                              grad_value_at, need > 0 ? ws.data_ptr() : nullptr, need,
                                                                              stream_of(path));
    if (status != SIG_OK) raise_status(status);
    return {grad_path, grad_value};
}

struct Forward {
    at::Tensor path, value, plain, sig, out;   // sig: the signature whose logarithm is taken
};

Forward run_forward(const at::Tensor &path, const at::Tensor &value, const at::Tensor &table, const Call &c)
{
    Forward f;
    f.path = path.contiguous();
    f.value = value.defined() ? value.contiguous() : value;
    f.plain = plain_signature(f.path, f.value, c);
    const int64_t d = path.size(2);
    f.sig = c.inverse ? inverted(f.plain, c, d) : f.plain;
    f.out = c.mode == kSignature ? f.sig : logarithm(f.sig, table, c, d);
    return f;
}

// What a node is handed besides the tensors it is a function of.
struct Extras {
    Call call;
    at::Tensor table;
};

struct SignatureNode : torch::autograd::Function<SignatureNode> {
    static at::Tensor forward(AutogradContext *ctx, const at::Tensor &path, const std::optional<at::Tensor> &value, const Extras &extras)
    {
        const c10::DeviceGuard guard(path.device());
        const Call &c = extras.call;
        const Forward f = run_forward(path, value.value_or(at::Tensor()), extras.table, c);
        const bool own = c.mode != kSignature && c.inverse;   // the logarithm's signature is not the plain one
        ctx->save_for_backward({f.path, f.plain, f.value, own ? f.sig : at::Tensor()});
        ctx->saved_data["call"] = c.kept();
        if (extras.table.defined()) ctx->saved_data["table"] = extras.table;
        return f.out;
    }

    static variable_list backward(AutogradContext *ctx, variable_list grads)
    {
        const variable_list saved = ctx->get_saved_variables();
        const at::Tensor &path = saved[0], &plain = saved[1], &value = saved[2];
        const Call c = Call::from(ctx->saved_data["call"].toIntVector());
        const c10::DeviceGuard guard(path.device());
        at::Tensor grad = grads[0].contiguous();
        if (c.mode != kSignature) {
            const auto table = ctx->saved_data.find("table");
            grad = log_gradient(saved[3].defined() ? saved[3] : plain, grad,
                                table != ctx->saved_data.end() ? table->second.toTensor() : at::Tensor(), c, path.size(2));
        }
        const variable_list found = signature_gradients(path, plain, value, grad, c);
        return {found[0], found[1], at::Tensor()};
    }
};

bool plain_world()
{
    return !c10::impl::dispatch_mode_enabled() && !at::impl::torch_function_mode_enabled() && !torch::jit::tracer::isTracing() &&
           !c10::impl::tls_local_dispatch_key_set().included_.has(c10::DispatchKey::FuncTorchDynamicLayerFrontMode);
}

bool plain_tensor(const at::Tensor &t)
{
    return t.is_cuda() && t.layout() == at::kStrided && !t.is_conj() && !t.is_neg() && !t._fw_grad(0).defined();
}

// (path, depth, stream, basepoint, inverse, mode, table): the result, or NotImplemented.  mode: 0 the signature, 1 every word of the
// logarithm, 2 the words of `table` (the device table of the Lyndon words; None otherwise).
PyObject *transform(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 7 || !THPVariable_CheckExact(args[0]) || !PyLong_CheckExact(args[1]) || !PyBool_Check(args[2]) || !PyBool_Check(args[4]) ||
        !PyLong_CheckExact(args[5]) || !(PyBool_Check(args[3]) || THPVariable_CheckExact(args[3])) || !plain_world())
        Py_RETURN_NOTIMPLEMENTED;
    const at::Tensor &path = THPVariable_Unpack(args[0]);
    int overflow = 0;
    const int64_t depth = PyLong_AsLongLongAndOverflow(args[1], &overflow);
    if (overflow || depth < 1 || depth > SIG_MAX_DEPTH || !plain_tensor(path) || path.dim() != 3 ||
        (path.scalar_type() != at::kFloat && path.scalar_type() != at::kDouble))
        Py_RETURN_NOTIMPLEMENTED;
    const int64_t B = path.size(0), L = path.size(1), d = path.size(2);
    const Call c = {depth, args[2] == Py_True, args[3] != Py_False, args[4] == Py_True, PyLong_AsLongLong(args[5])};
    std::optional<at::Tensor> value;
    if (!PyBool_Check(args[3])) {
        value = THPVariable_Unpack(args[3]);
        if (!plain_tensor(*value) || value->device() != path.device() || value->scalar_type() != path.scalar_type() ||
            value->dim() != 2 || value->size(0) != B || value->size(1) != d)
            Py_RETURN_NOTIMPLEMENTED;
    }
    at::Tensor table;
    if (c.mode == kLogWords) {
        if (!THPVariable_CheckExact(args[6])) Py_RETURN_NOTIMPLEMENTED;
        table = THPVariable_Unpack(args[6]);
    }
    if (B < 1 || d < 1 || d > 0x7fffffff || L < (c.basepoint ? 1 : 2) || L > kLongest) Py_RETURN_NOTIMPLEMENTED;
    const sig_dtype type = type_of(path);
    const int64_t elems = sig_output_elems(B, L, int(d), int(depth), int(c.stream), int(c.basepoint));
    if (elems < 0) Py_RETURN_NOTIMPLEMENTED;
    const bool grad = at::GradMode::is_enabled() && (path.requires_grad() || (value && value->requires_grad()));
    if (grad && (sig_backward_workspace_bytes(B, L, int(d), int(depth), int(c.stream), int(c.basepoint), type) < 0 ||
                 (c.mode != kSignature &&
                  sig_log_backward_workspace_bytes(elems / sig_signature_channels(int(d), int(depth)), int(d), int(depth), type) < 0)))
        Py_RETURN_NOTIMPLEMENTED;   // no gradient for this shape
    at::Tensor out;
    try {
        pybind11::gil_scoped_release no_gil;
        if (grad) {
            out = SignatureNode::apply(path, value, Extras{c, table});
        } else {
            const at::NoGradGuard no_grad;
            const c10::DeviceGuard guard(path.device());
            out = run_forward(path, value.value_or(at::Tensor()), table, c).out;
        }
    } catch (const Declined &) {
        Py_RETURN_NOTIMPLEMENTED;
    }
    return THPVariable_Wrap(std::move(out));
    END_HANDLE_TH_ERRORS
}

// (prefixes, start, end, d, depth): binding.sig_interval without `out`, or NotImplemented.
PyObject *interval(PyObject *, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 5 || !THPVariable_CheckExact(args[0]) || !plain_world()) Py_RETURN_NOTIMPLEMENTED;
    int64_t v[4];   // start, end, d, depth
    for (int i = 0; i < 4; ++i) {
        int overflow = 0;
        if (!PyLong_CheckExact(args[1 + i])) Py_RETURN_NOTIMPLEMENTED;
        v[i] = PyLong_AsLongLongAndOverflow(args[1 + i], &overflow);
        if (overflow) Py_RETURN_NOTIMPLEMENTED;
    }
    const at::Tensor &prefixes = THPVariable_Unpack(args[0]);
    if (!plain_tensor(prefixes) || prefixes.dim() != 3 || !prefixes.is_contiguous() || v[2] < 1 || v[2] > 0x7fffffff || v[3] < 1 ||
        v[3] > SIG_MAX_DEPTH || (prefixes.scalar_type() != at::kFloat && prefixes.scalar_type() != at::kDouble))
        Py_RETURN_NOTIMPLEMENTED;
    const int64_t B = prefixes.size(0), rows = prefixes.size(1), S = sig_signature_channels(int(v[2]), int(v[3]));
    if (B < 1 || prefixes.size(2) != S || v[0] < 1 || v[0] >= v[1] || v[1] > rows) Py_RETURN_NOTIMPLEMENTED;
    at::Tensor out;
    sig_status status;
    {
        pybind11::gil_scoped_release no_gil;
        const at::NoGradGuard no_grad;
        const c10::DeviceGuard guard(prefixes.device());
        out = at::empty({B, S}, prefixes.options());
        const char *at = static_cast<const char *>(prefixes.data_ptr());
        const int64_t row = S * prefixes.element_size();
        status = sig_interval(at + (v[0] - 1) * row, rows * S, at + (v[1] - 1) * row, rows * S, B, int(v[2]), int(v[3]), type_of(prefixes), out.data_ptr(), S,
                              stream_of(prefixes));
    }
    if (status != SIG_OK) Py_RETURN_NOTIMPLEMENTED;   // the Python function raises what it raises
    return THPVariable_Wrap(std::move(out));
    END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {{"transform", reinterpret_cast<PyCFunction>(transform), METH_FASTCALL, nullptr},
                         {"interval", reinterpret_cast<PyCFunction>(interval), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_sig_torch", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__sig_torch()
{
    PyObject *m = PyModule_Create(&module);
    if (m != nullptr && PyModule_AddStringConstant(m, "built_with", SIG_TORCH_VERSION) < 0) Py_CLEAR(m);
    return m;
}
