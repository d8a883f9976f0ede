// The linear layer's autograd node in native code: what nn.QuartetLinearFunction.apply runs.  Argument checks, output and context
// allocation, the two C ABI calls (quartet_linear_fwd_block, quartet_linear_bwd_block) and the graph edge; no arithmetic.
//
// Why native: a step of a small layer is bound by the host.  As a Python autograd function the step of a 288 x 320 x 352 layer
// took 163-170 us of host time for 17 us of GPU work: seven output tensors, two crossings into Python, and a backward pass
// that has to take the interpreter lock on the engine's own thread.  Here the forward context is one allocation and the
// backward pass never enters Python.
#include <Python.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include <ATen/ATen.h>
#include <c10/core/DeviceGuard.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/function.h>
#include <torch/csrc/autograd/functions/utils.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/autograd/saved_variable.h>
#include <torch/csrc/autograd/VariableTypeUtils.h>
#include <torch/csrc/jit/frontend/tracer.h>

#include "../../include/quartet.h"

namespace {

using torch::autograd::Node;
using torch::autograd::variable_list;

PyObject* g_error = nullptr;   // binding.QuartetError

[[noreturn]] void raise_python(PyObject* type, const std::string& text) {
    pybind11::gil_scoped_acquire gil;
    PyErr_SetString(type, text.c_str());
    python_error e;
    e.persist();
    throw e;
}

void check(int rc) {
    if (rc == QUARTET_OK) return;
    std::string text = rc == QUARTET_EINVAL ? "QUARTET_EINVAL" : rc == QUARTET_ENOTSUP ? "QUARTET_ENOTSUP" : "QUARTET_EHIP";
    if (rc == QUARTET_EHIP) text += " (hipError_t " + std::to_string(quartet_last_hip_error()) + ")";
    raise_python(g_error, text);
}

// The forward context {X_q, M_x, W_q, M_w} as byte ranges of one buffer.
struct Context {
    size_t x_codes, x_scales, x_mask, w_codes, w_scales, w_mask, total;
    Context(int64_t tokens, int64_t in, int64_t out) {
        size_t at = 0;
        auto take = [&](size_t bytes) { const size_t here = at; at += (bytes + 255) & ~(size_t)255; return here; };
        x_codes = take((size_t)(tokens * in) / 2);
        x_scales = take(quartet_scale_bytes(tokens, in));
        x_mask = take((size_t)(tokens * in) / 8);
        w_codes = take((size_t)(out * in) / 2);
        w_scales = take(quartet_scale_bytes(out, in));
        w_mask = take((size_t)(out * in) / 8);
        total = at < 256 ? 256 : at;
    }
};

uint8_t* bytes_of(const at::Tensor& t) { return static_cast<uint8_t*>(t.data_ptr()); }
void* stream_of(const at::Tensor& t) { return c10::hip::getCurrentHIPStream(t.device().index()).stream(); }

// Sizes of one call.
struct Shape {
    std::vector<int64_t> x_sizes;
    int64_t tokens, in, out;
    int hadamard_block;
};

Shape check_arguments(const at::Tensor& x, const at::Tensor& weight, int64_t hadamard_block) {
    if (x.scalar_type() != at::kBFloat16 || weight.scalar_type() != at::kBFloat16)
        raise_python(PyExc_TypeError, "QuartetLinearFunction takes bf16 activations and weights");
    if (!x.is_cuda() || !weight.is_cuda()) raise_python(PyExc_RuntimeError, "QuartetLinearFunction runs on the GPU only");
    if (weight.dim() != 2) raise_python(PyExc_ValueError, "weight must be a matrix [out_features, in_features]");
    const int64_t out = weight.size(0), in = weight.size(1);
    if (x.dim() < 1 || x.size(-1) != in)
        raise_python(PyExc_RuntimeError, "the last dimension of the activations must be in_features = " + std::to_string(in));
    if (hadamard_block != 32 && hadamard_block != 64 && hadamard_block != 128 && hadamard_block != 256)
        raise_python(PyExc_ValueError, "hadamard_block must be 32, 64, 128 or 256");
    const int64_t tokens = in ? x.numel() / in : 0;
    if (tokens % hadamard_block || in % hadamard_block || out % hadamard_block)
        raise_python(PyExc_ValueError, "tokens, in_features and out_features must be multiples of " + std::to_string(hadamard_block));
    return {x.sizes().vec(), tokens, in, out, (int)hadamard_block};
}

// {y, forward context}
std::pair<at::Tensor, at::Tensor> forward(const at::Tensor& x, const at::Tensor& weight, const Shape& s) {
    at::AutoDispatchBelowADInplaceOrView below_autograd;
    c10::DeviceGuard device(x.device());
    const at::Tensor x2 = x.contiguous(), w2 = weight.contiguous();
    std::vector<int64_t> y_sizes = s.x_sizes;
    y_sizes.back() = s.out;
    at::Tensor y = at::empty(y_sizes, x.options());
    const Context c(s.tokens, s.in, s.out);
    at::Tensor ctx = at::empty({(int64_t)c.total}, x.options().dtype(at::kByte));
    uint8_t* b = bytes_of(ctx);
    check(quartet_linear_fwd_block(x2.data_ptr(), w2.data_ptr(), s.tokens, s.in, s.out, s.hadamard_block, y.data_ptr(), QUARTET_DTYPE_BF16,
                                   b + c.x_codes, b + c.x_scales, reinterpret_cast<uint32_t*>(b + c.x_mask), b + c.w_codes,
                                   b + c.w_scales, reinterpret_cast<uint32_t*>(b + c.w_mask), stream_of(x)));
    return {y, ctx};
}

// {dx, dw}; an undefined dy stands for zeros
std::pair<at::Tensor, at::Tensor> backward(const at::Tensor& ctx, const at::Tensor& grad, const Shape& s, uint64_t seed, int rounding) {
    at::NoGradGuard no_grad;
    c10::DeviceGuard device(ctx.device());
    const auto bf16 = ctx.options().dtype(at::kBFloat16);
    const at::Tensor dy = grad.defined() ? grad.reshape({s.tokens, s.out}).to(at::kBFloat16).contiguous() : at::zeros({s.tokens, s.out}, bf16);
    at::Tensor dx = at::empty(s.x_sizes, bf16), dw = at::empty({s.out, s.in}, bf16);
    const size_t nbytes = quartet_linear_workspace_bytes_block(s.tokens, s.in, s.out, s.hadamard_block);
    // from the caching allocator, so calls on several streams or threads never share it
    const at::Tensor ws = at::empty({(int64_t)(nbytes < 256 ? 256 : nbytes)}, ctx.options());
    const Context c(s.tokens, s.in, s.out);
    const uint8_t* b = bytes_of(ctx);
    check(quartet_linear_bwd_block(dy.data_ptr(), s.tokens, s.in, s.out, s.hadamard_block, b + c.x_codes, b + c.x_scales,
                                   reinterpret_cast<const uint32_t*>(b + c.x_mask), b + c.w_codes, b + c.w_scales,
                                   reinterpret_cast<const uint32_t*>(b + c.w_mask), seed, rounding, dx.data_ptr(), dw.data_ptr(),
                                   QUARTET_DTYPE_BF16, ws.data_ptr(), nbytes, stream_of(ctx)));
    return {dx, dw};
}

struct QuartetLinearBackward : public Node {
    torch::autograd::SavedVariable context;
    Shape shape;
    int rounding;
    uint64_t seed;

    std::string name() const override { return "QuartetLinearFunctionBackward"; }
    // the saved context is read and released under the node's lock: threads may run backward passes over a shared graph
    void release_variables() override {
        std::lock_guard<std::mutex> lock(mutex_);
        context.reset_data();
    }

    variable_list apply(variable_list&& grads) override {
        at::Tensor ctx;
        {
            std::lock_guard<std::mutex> lock(mutex_);
            ctx = context.unpack(shared_from_this());
        }
        auto [dx, dw] = backward(ctx, grads[0], shape, seed, rounding);
        return {dx, dw};
    }
};

at::Tensor linear(const at::Tensor& x, const at::Tensor& weight, uint64_t seed, int rounding, int64_t hadamard_block) {
    const Shape shape = check_arguments(x, weight, hadamard_block);
    const bool track = torch::autograd::compute_requires_grad(x, weight);
    auto [y, ctx] = forward(x, weight, shape);
    if (track) {
        auto node = std::shared_ptr<QuartetLinearBackward>(new QuartetLinearBackward(), torch::autograd::deleteNode);
        node->set_next_edges(torch::autograd::collect_next_edges(x, weight));
        node->context = torch::autograd::SavedVariable(ctx, false);
        node->shape = shape;
        node->rounding = rounding; node->seed = seed;
        torch::autograd::set_history(y, node);
    }
    return y;
}

// Calls that the node above does not serve: they take the Python autograd function, which knows what to do with them (or refuses
// them by name).  A tensor with a forward-mode tangent: the result would come back without one, which reads as a zero derivative.
// torch.jit.trace: all it would see of the node is the allocation of its result.  functorch's transforms (vmap, grad, functionalize,
// ...): a tensor without a level would slip through them.
bool needs_python_function(const at::Tensor& x, const at::Tensor& weight) {
    return torch::jit::tracer::isTracing() || c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode) ||
           torch::autograd::isFwGradDefined(x) || torch::autograd::isFwGradDefined(weight);
}

const at::Tensor& tensor_of(PyObject* o) { return THPVariable_Unpack(o); }

PyObject* wrap_pair(std::pair<at::Tensor, at::Tensor> p) {
    PyObject *a = THPVariable_Wrap(std::move(p.first)), *b = THPVariable_Wrap(std::move(p.second));
    PyObject* t = a && b ? PyTuple_Pack(2, a, b) : nullptr;
    Py_XDECREF(a);
    Py_XDECREF(b);
    return t;
}

// linear(x, weight, seed, rounding, hadamard_block): y, or None for a call of needs_python_function
PyObject* py_linear(PyObject*, PyObject* const* args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 5 || !THPVariable_Check(args[0]) || !THPVariable_Check(args[1])) {
        PyErr_SetString(PyExc_TypeError, "linear(x, weight, seed, rounding, hadamard_block): two tensors and three integers");
        return nullptr;
    }
    const uint64_t seed = PyLong_AsUnsignedLongLongMask(args[2]);
    const long rounding = PyLong_AsLong(args[3]), block = PyLong_AsLong(args[4]);
    if (PyErr_Occurred()) return nullptr;
    const at::Tensor x = tensor_of(args[0]), w = tensor_of(args[1]);
    if (needs_python_function(x, w)) Py_RETURN_NONE;
    at::Tensor y;
    {
        pybind11::gil_scoped_release no_gil;
        y = linear(x, w, seed, (int)rounding, block);
    }
    return THPVariable_Wrap(std::move(y));
    END_HANDLE_TH_ERRORS
}

// The two halves for the Python autograd function.
// forward(x, weight, hadamard_block): (y, context)
PyObject* py_forward(PyObject*, PyObject* const* args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 3 || !THPVariable_Check(args[0]) || !THPVariable_Check(args[1])) {
        PyErr_SetString(PyExc_TypeError, "forward(x, weight, hadamard_block): two tensors and an integer");
        return nullptr;
    }
    const long block = PyLong_AsLong(args[2]);
    if (PyErr_Occurred()) return nullptr;
    const at::Tensor x = tensor_of(args[0]), w = tensor_of(args[1]);
    std::pair<at::Tensor, at::Tensor> result;
    {
        pybind11::gil_scoped_release no_gil;
        result = forward(x, w, check_arguments(x, w, block));
    }
    return wrap_pair(std::move(result));
    END_HANDLE_TH_ERRORS
}

// backward(context, dy, x_sizes, out_features, seed, rounding, hadamard_block): (dx, dw)
PyObject* py_backward(PyObject*, PyObject* const* args, Py_ssize_t n) {
    HANDLE_TH_ERRORS
    if (n != 7 || !THPVariable_Check(args[0]) || !THPVariable_Check(args[1])) {
        PyErr_SetString(PyExc_TypeError, "backward(context, dy, x_sizes, out_features, seed, rounding, hadamard_block)");
        return nullptr;
    }
    Shape s;
    for (Py_ssize_t i = 0, dims = PyObject_Length(args[2]); i < dims; ++i) {
        PyObject* size = PySequence_GetItem(args[2], i);
        s.x_sizes.push_back(size ? PyLong_AsLongLong(size) : 0);
        Py_XDECREF(size);
    }
    s.out = PyLong_AsLongLong(args[3]);
    const uint64_t seed = PyLong_AsUnsignedLongLongMask(args[4]);
    const long rounding = PyLong_AsLong(args[5]);
    s.hadamard_block = (int)PyLong_AsLong(args[6]);
    if (PyErr_Occurred()) return nullptr;
    s.tokens = 1;
    for (size_t i = 0; i + 1 < s.x_sizes.size(); ++i) s.tokens *= s.x_sizes[i];
    s.in = s.x_sizes.empty() ? 0 : s.x_sizes.back();
    const at::Tensor ctx = tensor_of(args[0]), dy = tensor_of(args[1]);
    std::pair<at::Tensor, at::Tensor> result;
    {
        pybind11::gil_scoped_release no_gil;
        result = backward(ctx, dy, s, seed, (int)rounding);
    }
    return wrap_pair(std::move(result));
    END_HANDLE_TH_ERRORS
}

PyObject* py_set_error(PyObject*, PyObject* type) {
    Py_INCREF(type);
    Py_XDECREF(g_error);
    g_error = type;
    Py_RETURN_NONE;
}

// The binding's calls without ctypes (binding.py): an entry point's arguments in its order, the stream last.  Pointers are None,
// addresses or contiguous tensors on the GPU, as for the binding; whatever else comes (another type, a tensor subclass, a tensor
// on the host) makes the call return NotImplemented before anything has run, and the binding's own conversion takes it or says what
// is wrong with it.  Integers wrap to their C type and the interpreter lock is released, as with ctypes.  Why: a step of a 256 x 512 x 512
// layer is 15 us of GPU work behind 19 us of host work, half of it the conversion of 36 arguments.
template <bool LAST, typename T>
bool argument(PyObject* o, T& out) {
    if constexpr (std::is_pointer_v<T>) {
        if (PyLong_Check(o)) {
            out = reinterpret_cast<T>(static_cast<uintptr_t>(PyLong_AsUnsignedLongLongMask(o)));
            return true;
        }
        if constexpr (LAST) {
            if (o != Py_None) return false;
            out = c10::hip::getCurrentHIPStream().stream();
            return true;
        }
        if (o == Py_None) {
            out = nullptr;
            return true;
        }
        if (!THPVariable_CheckExact(o)) return false;
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.is_cuda() || !t.is_contiguous()) return false;
        out = static_cast<T>(t.data_ptr());
        return true;
    } else if constexpr (std::is_floating_point_v<T>) {
        if (!PyFloat_CheckExact(o)) return false;
        out = static_cast<T>(PyFloat_AS_DOUBLE(o));
        return true;
    } else {
        if (!PyLong_Check(o)) return false;
        out = static_cast<T>(PyLong_AsUnsignedLongLongMask(o));
        return true;
    }
}

template <auto F>
struct EntryPoint;
template <typename... A, int (*F)(A...)>
struct EntryPoint<F> {
    static PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t n) { return run(args, n, std::index_sequence_for<A...>{}); }
    template <size_t... I>
    static PyObject* run(PyObject* const* args, Py_ssize_t n, std::index_sequence<I...>) {
        std::tuple<std::remove_const_t<A>...> v;
        bool all = n == (Py_ssize_t)sizeof...(A);
        try {
            all = all && (argument<I + 1 == sizeof...(A)>(args[I], std::get<I>(v)) && ...);
        } catch (const std::exception&) {      // a tensor without storage: the binding's own call says so
            all = false;
        }
        if (!all) Py_RETURN_NOTIMPLEMENTED;
        int rc;
        Py_BEGIN_ALLOW_THREADS
        rc = F(std::get<I>(v)...);
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(rc);
    }
};
#define ENTRY_POINT(NAME) \
    {#NAME, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(EntryPoint<&NAME>::call)), METH_FASTCALL, nullptr}

PyMethodDef methods[] = {
    ENTRY_POINT(quartet_linear_fwd),
    ENTRY_POINT(quartet_linear_bwd),
    ENTRY_POINT(quartet_linear_fwd_block),
    ENTRY_POINT(quartet_linear_bwd_block),
    ENTRY_POINT(quartet_quant_fwd),
    ENTRY_POINT(quartet_quant_bwd_sr),
    ENTRY_POINT(quartet_mxfp4_gemm),
    ENTRY_POINT(quartet_mxfp4_gemm_grad),
    {"linear", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(py_linear)), METH_FASTCALL, nullptr},
    {"forward", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(py_forward)), METH_FASTCALL, nullptr},
    {"backward", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(py_backward)), METH_FASTCALL, nullptr},
    {"set_error", py_set_error, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_nn_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__nn_native(void) { return PyModule_Create(&module_def); }
