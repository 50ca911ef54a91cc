// Host path of the hot entry points in native code: the argument checks and the call of the C entry points behind
// binding.py, and the autograd node behind autograd.BCQLinear.  Nothing is computed here.
//
// Why: a call through ctypes is ~9 us of interpreter work around ~5 us of launches, more than most small kernels take,
// and a Python autograd node costs the engine's thread a trip through the interpreter in every backward pass.
// Measured on the host side alone: one binding call 10.6 -> 4.4 us, forward and backward of the module 135 -> 64 us.
//
// Every function returns None when the call is not the plain case (another type, shape, layout, device, a missing
// pointer) or when the C entry point refuses it; the Python code behind it then repeats the call its own way and raises
// what it always raised.
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/jit/frontend/tracer.h>
#include <torch/extension.h>

#include "../../include/bcq.h"
#include "bcq_node.h"

namespace {

using at::Tensor;
using OptTensor = std::optional<Tensor>;

void* current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// a dense tensor of this kind on the current device
bool plain(const Tensor& t, at::ScalarType type, at::IntArrayRef shape) {
    return t.defined() && t.is_cuda() && t.scalar_type() == type && t.sizes() == shape && t.is_contiguous() &&
           !t.key_set().has(c10::DispatchKey::Python) && t.get_device() == c10::hip::current_device();
}
int act_code(const Tensor& t) {
    if (t.scalar_type() == at::kFloat) return BCQ_F32;
    return t.scalar_type() == at::kBFloat16 ? BCQ_BF16 : -1;
}
bool plain_workspace(const OptTensor& w) {
    return !w || (w->is_cuda() && w->is_contiguous() && !w->key_set().has(c10::DispatchKey::Python) &&
                  w->get_device() == c10::hip::current_device());
}
void* ptr(const OptTensor& t) { return t ? t->data_ptr() : nullptr; }
size_t bytes(const OptTensor& t) { return t ? (size_t)t->numel() * t->element_size() : 0; }
const uint32_t* words(const Tensor& t) { return static_cast<const uint32_t*>(t.data_ptr()); }

struct Shape {
    int64_t q = 0, N = 0, K = 0, G = 0;
    bool ok = false;
};
Shape layer_shape(const Tensor& packed, int64_t g) {
    Shape s;
    if (!packed.defined() || packed.dim() != 3 || g < 32) return s;
    s.q = packed.size(0);
    s.N = packed.size(1);
    s.K = packed.size(2) * 32;
    s.G = s.K / g;
    s.ok = plain(packed, at::kInt, {s.q, s.N, s.K / 32});
    return s;
}

// the status of the C call, made without the interpreter lock as ctypes makes it
template <typename F>
bcq_status unlocked(F call) {
    py::gil_scoped_release release;
    return call();
}

py::object fwd_grouped(const Tensor& packed, const Tensor& alpha, const Tensor& x, int64_t g, OptTensor y,
                       const OptTensor& workspace) {
    const Shape s = layer_shape(packed, g);
    if (!s.ok || x.dim() != 2) return py::none();
    const int64_t T = x.size(0);
    const int code = act_code(x);
    if (code < 0 || !plain(x, x.scalar_type(), {T, s.K}) || !plain(alpha, at::kFloat, {s.q, s.N, s.G}) ||
        !plain_workspace(workspace) || (y && !plain(*y, x.scalar_type(), {T, s.N})))
        return py::none();
    if (!y) y = at::empty({T, s.N}, x.options());
    const bcq_status st = unlocked([&] {
        return bcq_linear_fwd_grouped(words(packed), alpha.data_ptr<float>(), x.data_ptr(), code, T, s.N, s.K, g, (int)s.q,
                                      y->data_ptr(), ptr(workspace), bytes(workspace), current_stream());
    });
    return st == BCQ_OK ? py::cast(*y) : py::none();
}

py::object fwd_decode(const Tensor& tiled, const Tensor& alpha, const Tensor& x, int64_t g, OptTensor y,
                      const OptTensor& workspace) {
    if (alpha.dim() < 2 || alpha.dim() > 3 || x.dim() != 2 || g < 32) return py::none();
    const int64_t T = x.size(0), K = x.size(1), q = alpha.size(0), N = alpha.size(1);
    const int code = act_code(x);
    size_t need = 0;
    if (code < 0 || bcq_decode_layout_bytes(N, K, (int)q, &need) != BCQ_OK) return py::none();
    const bool scales = alpha.dim() == 3 ? plain(alpha, at::kFloat, {q, N, K / g}) : (K == g && plain(alpha, at::kFloat, {q, N}));
    if (!scales || !plain(tiled, at::kInt, {(int64_t)(need / 4)}) || !plain(x, x.scalar_type(), {T, K}) ||
        !plain_workspace(workspace) || (y && !plain(*y, x.scalar_type(), {T, N})))
        return py::none();
    if (!y) y = at::empty({T, N}, x.options());
    const bcq_status st = unlocked([&] {
        return bcq_linear_fwd_decode(words(tiled), alpha.data_ptr<float>(), x.data_ptr(), code, T, N, K, g, (int)q,
                                     y->data_ptr(), ptr(workspace), bytes(workspace), current_stream());
    });
    return st == BCQ_OK ? py::cast(*y) : py::none();
}

py::object bwd_input_grouped(const Tensor& packed, const Tensor& alpha, const Tensor& dy, int64_t g,
                             const OptTensor& packed_t, OptTensor dx, const OptTensor& workspace) {
    const Shape s = layer_shape(packed, g);
    if (!s.ok || dy.dim() != 2) return py::none();
    const int64_t T = dy.size(0);
    const int code = act_code(dy);
    if (code < 0 || !plain(dy, dy.scalar_type(), {T, s.N}) || !plain(alpha, at::kFloat, {s.q, s.N, s.G}) ||
        (packed_t && !plain(*packed_t, at::kInt, {s.q, s.K, s.N / 32})) || !plain_workspace(workspace) ||
        (dx && !plain(*dx, dy.scalar_type(), {T, s.K})))
        return py::none();
    if (!dx) dx = at::empty({T, s.K}, dy.options());
    const bcq_status st = unlocked([&] {
        return bcq_linear_bwd_input_grouped(words(packed), static_cast<const uint32_t*>(ptr(packed_t)),
                                            alpha.data_ptr<float>(), dy.data_ptr(), code, T, s.N, s.K, g, (int)s.q,
                                            dx->data_ptr(), ptr(workspace), bytes(workspace), current_stream());
    });
    return st == BCQ_OK ? py::cast(*dx) : py::none();
}

py::object bwd_alpha_grouped(const Tensor& packed, const Tensor& x, const Tensor& dy, int64_t g, int64_t q_train,
                             double grad_scale, OptTensor dalpha, const OptTensor& workspace) {
    const Shape s = layer_shape(packed, g);
    if (!s.ok || x.dim() != 2 || q_train < 1) return py::none();
    const int64_t T = x.size(0);
    const int code = act_code(x);
    if (code < 0 || !plain(x, x.scalar_type(), {T, s.K}) || !plain(dy, x.scalar_type(), {T, s.N}) ||
        !plain_workspace(workspace) || (dalpha && !plain(*dalpha, at::kFloat, {q_train, s.N, s.G})))
        return py::none();
    if (!dalpha) dalpha = at::empty({q_train, s.N, s.G}, x.options().dtype(at::kFloat));
    const bcq_status st = unlocked([&] {
        return bcq_linear_bwd_alpha_grouped(words(packed), x.data_ptr(), dy.data_ptr(), code, T, s.N, s.K, g, (int)s.q,
                                            (int)q_train, (float)grad_scale, dalpha->data_ptr<float>(), ptr(workspace),
                                            bytes(workspace), current_stream());
    });
    return st == BCQ_OK ? py::cast(*dalpha) : py::none();
}

// ---- quantizing and laying out a layer's weights: calls of 5 to 25 us, several per layer
py::object quantize_grouped(const Tensor& W, int64_t q, int64_t g, OptTensor alpha, OptTensor packed, const OptTensor& workspace) {
    if (W.dim() != 2 || q < 1 || q > 8 || g < 32) return py::none();
    const int64_t N = W.size(0), K = W.size(1), G = K / g;
    if (!plain(W, at::kFloat, {N, K}) || (alpha && !plain(*alpha, at::kFloat, {q, N, G})) ||
        (packed && !plain(*packed, at::kInt, {q, N, K / 32})) || !plain_workspace(workspace))
        return py::none();
    if (!alpha) alpha = at::empty({q, N, G}, W.options());
    if (!packed) packed = at::empty({q, N, K / 32}, W.options().dtype(at::kInt));
    const bcq_status st = unlocked([&] {
        return bcq_quantize_grouped(W.data_ptr<float>(), N, K, g, (int)q, alpha->data_ptr<float>(), static_cast<uint32_t*>(packed->data_ptr()),
                                    nullptr, ptr(workspace), bytes(workspace), current_stream());
    });
    return st == BCQ_OK ? py::object(py::make_tuple(*alpha, *packed)) : py::none();
}

py::object pack_transposed(const Tensor& packed, OptTensor packed_t) {
    const Shape s = layer_shape(packed, 32);
    if (!s.ok || s.N % 32 != 0 || (packed_t && !plain(*packed_t, at::kInt, {s.q, s.K, s.N / 32}))) return py::none();
    if (!packed_t) packed_t = at::empty({s.q, s.K, s.N / 32}, packed.options());
    const bcq_status st = unlocked([&] {
        return bcq_pack_transposed(words(packed), s.N, s.K, (int)s.q, static_cast<uint32_t*>(packed_t->data_ptr()), current_stream());
    });
    return st == BCQ_OK ? py::cast(*packed_t) : py::none();
}

py::object pack_decode(const Tensor& packed, OptTensor tiled) {
    const Shape s = layer_shape(packed, 32);
    size_t need = 0;
    if (!s.ok || bcq_decode_layout_bytes(s.N, s.K, (int)s.q, &need) != BCQ_OK || (tiled && !plain(*tiled, at::kInt, {(int64_t)(need / 4)})))
        return py::none();
    if (!tiled) tiled = at::empty({(int64_t)(need / 4)}, packed.options());
    const bcq_status st = unlocked([&] {
        return bcq_pack_decode(words(packed), s.N, s.K, (int)s.q, static_cast<uint32_t*>(tiled->data_ptr()), current_stream());
    });
    return st == BCQ_OK ? py::cast(*tiled) : py::none();
}

// ---- autograd ---------------------------------------------------------------------------------------------------
// The frozen state of a layer, passed to the node beside its two differentiable inputs.
struct Frozen {
    Tensor alpha, packed, twin;  // alpha: scales of the planes that are not trained; alpha, twin may be undefined
    int64_t g, q_train;
    double grad_scale;
};

// Scratch of one call from torch's caching allocator: it belongs to the stream of the call, so passes on several streams
// or threads never share it.
Tensor scratch(int op, int64_t T, const Shape& s, int64_t g, int code, const Tensor& like, bcq_status* st) {
    size_t need = 0;
    *st = bcq_workspace_bytes_grouped(op, T, s.N, s.K, g, (int)s.q, code, &need);
    return *st == BCQ_OK ? at::empty({(int64_t)std::max<size_t>(need, 16)}, like.options().dtype(at::kByte)) : Tensor();
}

// Raised on the engine's thread, like the exception of a Python node
[[noreturn]] void raise_bcq_error(bcq_status st, const char* what) {
    py::gil_scoped_acquire gil;
    py::object error = py::module_::import("paper_2210_03858_amd.binding").attr("BcqError")((int)st, what);
    PyErr_SetObject(reinterpret_cast<PyObject*>(Py_TYPE(error.ptr())), error.ptr());
    python_error raised;
    raised.persist();
    throw std::move(raised);
}

struct Refused {};  // the forward call is not the plain case: the caller takes the Python node

struct BCQLinearNode : public torch::autograd::Function<BCQLinearNode> {
    static Tensor forward(torch::autograd::AutogradContext* ctx, const Tensor& x, const Tensor& alpha_train,
                          const Frozen& f) {
        const Shape s = layer_shape(f.packed, f.g);
        // scales in two plain tensors are joined by the forward's kernels
        const bool parts = f.alpha.defined() && s.ok && f.q_train >= 1 && f.q_train < s.q && !alpha_train.is_neg() && !f.alpha.is_neg() &&
                           plain(alpha_train, at::kFloat, {f.q_train, s.N, s.G}) && plain(f.alpha, at::kFloat, {s.q - f.q_train, s.N, s.G});
        const Tensor alpha = parts ? at::empty({s.q, s.N, s.G}, f.alpha.options())
                                   : (f.alpha.defined() ? at::cat({alpha_train, f.alpha}, 0) : alpha_train).contiguous();
        const Tensor x2 = x.reshape({-1, s.K}).contiguous();
        const int64_t T = x2.size(0);
        const int code = act_code(x2);
        if (!s.ok || code < 0 || !plain(x2, x2.scalar_type(), {T, s.K}) || !plain(alpha, at::kFloat, {s.q, s.N, s.G}))
            throw Refused{};
        bcq_status st = BCQ_OK;
        const Tensor ws = scratch(BCQ_OP_FWD, T, s, f.g, code, x2, &st);
        if (st != BCQ_OK) throw Refused{};
        Tensor y = at::empty({T, s.N}, x2.options());
        if (parts)
            st = bcq_node_forward(words(f.packed), alpha_train.data_ptr<float>(), (int)f.q_train, f.alpha.data_ptr<float>(),
                                  alpha.data_ptr<float>(), x2.data_ptr(), code, T, s.N, s.K, f.g, (int)s.q, y.data_ptr(),
                                  ws.data_ptr(), (size_t)ws.numel(), current_stream());
        else
            st = bcq_linear_fwd_grouped(words(f.packed), alpha.data_ptr<float>(), x2.data_ptr(), code, T, s.N, s.K, f.g,
                                        (int)s.q, y.data_ptr(), ws.data_ptr(), (size_t)ws.numel(), current_stream());
        if (st != BCQ_OK) throw Refused{};
        ctx->save_for_backward({x2, alpha});
        ctx->saved_data["packed"] = f.packed;
        if (f.twin.defined()) ctx->saved_data["twin"] = f.twin;
        ctx->saved_data["g"] = f.g;
        ctx->saved_data["q_train"] = f.q_train;
        ctx->saved_data["grad_scale"] = f.grad_scale;
        ctx->saved_data["x_shape"] = x.sizes().vec();
        std::vector<int64_t> shape = x.sizes().vec();
        shape.back() = s.N;
        return y.reshape(shape);
    }

    static torch::autograd::variable_list backward(torch::autograd::AutogradContext* ctx,
                                                   const torch::autograd::variable_list& grads) {
        const auto saved = ctx->get_saved_variables();
        const Tensor &x2 = saved[0], &alpha = saved[1];
        const Tensor packed = ctx->saved_data["packed"].toTensor();
        const int64_t g = ctx->saved_data["g"].toInt(), q_train = ctx->saved_data["q_train"].toInt();
        const Shape s = layer_shape(packed, g);
        const Tensor dy = grads[0].reshape({-1, s.N}).contiguous();
        const int64_t T = dy.size(0);
        const int code = act_code(dy);
        TORCH_CHECK_VALUE(s.ok && code >= 0 && plain(dy, x2.scalar_type(), {T, s.N}) &&
                              plain(x2, x2.scalar_type(), {T, s.K}) && plain(alpha, at::kFloat, {s.q, s.N, s.G}),
                          "dy must be a contiguous cuda tensor of the activations' dtype");
        const auto twin = ctx->saved_data.find("twin");
        const uint32_t* packed_t = twin == ctx->saved_data.end() ? nullptr : words(twin->second.toTensor());
        const float grad_scale = (float)ctx->saved_data["grad_scale"].toDouble();
        Tensor dx, dalpha;
        const auto workspace = [&](int op) {
            bcq_status st = BCQ_OK;
            const Tensor ws = scratch(op, T, s, g, code, dy, &st);
            if (st != BCQ_OK) raise_bcq_error(st, "bcq_workspace_bytes_grouped");
            return ws;
        };
        if (ctx->needs_input_grad(0)) dx = at::empty({T, s.K}, dy.options());
        if (ctx->needs_input_grad(1)) dalpha = at::empty({q_train, s.N, s.G}, dy.options().dtype(at::kFloat));
        if (dx.defined() && dalpha.defined() && bcq_node_backward_joint(packed_t != nullptr, code, T, s.N, s.K, g, (int)s.q)) {
            const Tensor ws_x = workspace(BCQ_OP_BWD_INPUT), ws_alpha = workspace(BCQ_OP_BWD_ALPHA);
            const bcq_status st = bcq_node_backward(words(packed), alpha.data_ptr<float>(), x2.data_ptr(), dy.data_ptr(), code, T, s.N,
                                                    s.K, g, (int)s.q, (int)q_train, grad_scale, dx.data_ptr(), ws_x.data_ptr(),
                                                    (size_t)ws_x.numel(), dalpha.data_ptr<float>(), ws_alpha.data_ptr(),
                                                    (size_t)ws_alpha.numel(), current_stream());
            if (st != BCQ_OK) raise_bcq_error(st, "bcq_node_backward");
        } else {  // one after the other: each call's scratch is given back before the next takes its own
            if (dx.defined()) {
                const Tensor ws = workspace(BCQ_OP_BWD_INPUT);
                const bcq_status st = bcq_linear_bwd_input_grouped(words(packed), packed_t, alpha.data_ptr<float>(), dy.data_ptr(), code, T,
                                                                   s.N, s.K, g, (int)s.q, dx.data_ptr(), ws.data_ptr(),
                                                                   (size_t)ws.numel(), current_stream());
                if (st != BCQ_OK) raise_bcq_error(st, "bcq_linear_bwd_input_grouped");
            }
            if (dalpha.defined()) {
                const Tensor ws = workspace(BCQ_OP_BWD_ALPHA);
                const bcq_status st = bcq_linear_bwd_alpha_grouped(words(packed), x2.data_ptr(), dy.data_ptr(), code, T, s.N, s.K, g,
                                                                   (int)s.q, (int)q_train, grad_scale, dalpha.data_ptr<float>(),
                                                                   ws.data_ptr(), (size_t)ws.numel(), current_stream());
                if (st != BCQ_OK) raise_bcq_error(st, "bcq_linear_bwd_alpha_grouped");
            }
        }
        if (dx.defined()) dx = dx.reshape(ctx->saved_data["x_shape"].toIntVector());
        return {dx, dalpha, Tensor()};
    }
};

// Tensors and modes that only the Python node handles (or refuses): function transforms, forward-mode gradients, traces,
// dispatch modes, subclasses.
bool transformed(const Tensor& t) {
    return t.key_set().has(c10::DispatchKey::Python) || t.key_set().has(c10::DispatchKey::Functionalize) ||
           t._fw_grad(0).defined();
}

py::object linear(const Tensor& x, const Tensor& alpha_train, const OptTensor& alpha_frozen, const Tensor& packed,
                  const OptTensor& twin, int64_t g, int64_t q_train, double grad_scale) {
    if (c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode) || torch::jit::tracer::isTracing() ||
        c10::impl::TorchDispatchModeTLS::any_modes_set() || transformed(x) || transformed(alpha_train))
        return py::none();
    const Shape s = layer_shape(packed, g);
    if (!s.ok || x.dim() < 1 || x.layout() != at::kStrided || !x.is_cuda() || x.get_device() != c10::hip::current_device() ||
        x.size(-1) != s.K || x.numel() == 0 || act_code(x) < 0 || !alpha_train.is_cuda() ||
        alpha_train.scalar_type() != at::kFloat || (alpha_frozen && alpha_frozen->requires_grad()) ||
        (twin && !plain(*twin, at::kInt, {s.q, s.K, s.N / 32})))
        return py::none();
    const Frozen f{alpha_frozen.value_or(Tensor()), packed, twin.value_or(Tensor()), g, q_train, grad_scale};
    try {
        Tensor y;
        {
            py::gil_scoped_release release;
            y = BCQLinearNode::apply(x, alpha_train, f);
        }
        return py::cast(y);
    } catch (const Refused&) {
        return py::none();
    }
}

// Arguments of other types reach the second form, so that the caller need not catch the TypeError of a failed conversion
// and take one that user code raised inside the call (a saved-tensor hook) for it.
template <typename F>
void define(py::module_& m, const char* name, F f) {
    m.def(name, f);
    m.def(name, [](const py::args&) -> py::object { return py::none(); });
}

}  // namespace

PYBIND11_MODULE(TORCH_EXTENSION_NAME, m) {
    define(m, "fwd_grouped", &fwd_grouped);
    define(m, "fwd_decode", &fwd_decode);
    define(m, "bwd_input_grouped", &bwd_input_grouped);
    define(m, "bwd_alpha_grouped", &bwd_alpha_grouped);
    define(m, "quantize_grouped", &quantize_grouped);
    define(m, "pack_transposed", &pack_transposed);
    define(m, "pack_decode", &pack_decode);
    define(m, "linear", &linear);
}
