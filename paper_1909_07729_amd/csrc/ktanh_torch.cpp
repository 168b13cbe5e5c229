// _ktanh_torch: the host path of ordinary calls.  A CPython module that takes torch tensors, allocates the
// result and enqueues one entry point of libktanh on the current stream, and the differentiable activations
// and LSTM cell as C++ autograd functions over the same entry points.  No arithmetic lives here.
//
// Through Python (argument checks, ctypes, autograd.Function) a call costs the host 8-12 us and a gradient
// step 29 us, two to ten times what the GPU needs for the tensors of a decoding step or of one recurrent
// step; here 4-5 us and 13-20 us.
//
// Every function returns None for anything that is not such a call, and the Python code in binding.py and
// autograd.py then takes it: tensors of another type, device, layout or class, other shapes, a stream given
// by the caller, tracing, dispatch and function modes, functional transforms, forward-mode gradients.  So
// what is refused is refused there, with the messages of old, and nothing is decided here that a mode or a
// transform would have to see.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPFunctions.h>

#include <iterator>

#include "ktanh.h"

namespace {

using at::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

// ------------------------------------------------------------------------------------ entry points
// One uniform form for the element-wise entry points (in, out) and for the gradients (dy, v, dx).
typedef ktanh_status_t (*Unary)(const void *, void *, size_t, const void *lut, ktanh_stream_t);
typedef ktanh_status_t (*Binary)(const void *, const void *, void *, size_t, const void *lut, ktanh_stream_t);

enum Table { NO_TABLE, TABLE32, TABLE64 };
template <class T> struct TableKind { static constexpr Table value = TABLE32; };
template <> struct TableKind<ktanh_lut64_t> { static constexpr Table value = TABLE64; };

template <auto F> struct UnaryOf;
template <class I, class O, class L, ktanh_status_t (*F)(const I *, O *, size_t, const L *, ktanh_stream_t)>
struct UnaryOf<F> {
    static constexpr Table table = TableKind<L>::value;
    static ktanh_status_t call(const void *in, void *out, size_t n, const void *lut, ktanh_stream_t s)
    {
        return F(static_cast<const I *>(in), static_cast<O *>(out), n, static_cast<const L *>(lut), s);
    }
};
template <class I, class O, ktanh_status_t (*F)(const I *, O *, size_t, ktanh_stream_t)>
struct UnaryOf<F> {
    static constexpr Table table = NO_TABLE;
    static ktanh_status_t call(const void *in, void *out, size_t n, const void *, ktanh_stream_t s)
    {
        return F(static_cast<const I *>(in), static_cast<O *>(out), n, s);
    }
};
template <auto F> struct BinaryOf;
template <class E, class L, ktanh_status_t (*F)(const E *, const E *, E *, size_t, const L *, ktanh_stream_t)>
struct BinaryOf<F> {
    static constexpr Table table = TableKind<L>::value;
    static ktanh_status_t call(const void *dy, const void *v, void *dx, size_t n, const void *lut, ktanh_stream_t s)
    {
        return F(static_cast<const E *>(dy), static_cast<const E *>(v), static_cast<E *>(dx), n,
                 static_cast<const L *>(lut), s);
    }
};
template <class E, ktanh_status_t (*F)(const E *, const E *, E *, size_t, ktanh_stream_t)>
struct BinaryOf<F> {
    static constexpr Table table = NO_TABLE;
    static ktanh_status_t call(const void *dy, const void *v, void *dx, size_t n, const void *, ktanh_stream_t s)
    {
        return F(static_cast<const E *>(dy), static_cast<const E *>(v), static_cast<E *>(dx), n, s);
    }
};

constexpr at::ScalarType kBf16 = at::kBFloat16, kF32 = at::kFloat;

struct UnaryEntry {
    const char *name;
    Unary call;
    Table table;
    at::ScalarType in, out;
};
struct BinaryEntry {
    const char *name;
    Binary call;
    Table table;
    at::ScalarType type;
};
#define UNARY(fn, in, out) {#fn, UnaryOf<&fn>::call, UnaryOf<&fn>::table, in, out}
#define BINARY(fn, type) {#fn, BinaryOf<&fn>::call, BinaryOf<&fn>::table, type}

const UnaryEntry kUnary[] = {
    UNARY(ktanh_bf16, kBf16, kBf16), UNARY(ksigmoid, kBf16, kBf16), UNARY(kswish, kBf16, kBf16),
    UNARY(kgelu, kBf16, kBf16), UNARY(ktanh64_bf16, kBf16, kBf16), UNARY(ksigmoid64, kBf16, kBf16),
    UNARY(kswish64, kBf16, kBf16), UNARY(kgelu64, kBf16, kBf16), UNARY(ktanh_f32, kF32, kF32),
    UNARY(ksigmoid_f32, kF32, kF32), UNARY(kswish_f32, kF32, kF32), UNARY(kgelu_f32, kF32, kF32),
    UNARY(ktanh64_f32, kF32, kF32), UNARY(ksigmoid64_f32, kF32, kF32), UNARY(kswish64_f32, kF32, kF32),
    UNARY(kgelu64_f32, kF32, kF32), UNARY(ktanh_f32_to_bf16, kF32, kBf16), UNARY(kpade32_bf16, kBf16, kBf16),
    UNARY(kpade78_bf16, kBf16, kBf16), UNARY(ktaylor2_bf16, kBf16, kBf16), UNARY(ktaylor3_bf16, kBf16, kBf16),
};
const BinaryEntry kBinary[] = {
    BINARY(ktanh_bf16_backward, kBf16), BINARY(ksigmoid_backward, kBf16), BINARY(kswish_backward, kBf16),
    BINARY(kgelu_backward, kBf16), BINARY(kswish64_backward, kBf16), BINARY(kgelu64_backward, kBf16),
    BINARY(ktanh_f32_backward, kF32), BINARY(ksigmoid_f32_backward, kF32), BINARY(kswish_f32_backward, kF32),
    BINARY(kgelu_f32_backward, kF32), BINARY(kswish64_f32_backward, kF32), BINARY(kgelu64_f32_backward, kF32),
};

// ---------------------------------------------------------------------------------------- conditions
// The Python classes that setup() hands over; they live as long as the module, which is never unloaded.
PyObject *g_lut32 = nullptr, *g_lut64 = nullptr, *g_error = nullptr;

// Nothing watches or transforms operations on this thread.
bool ordinary_thread()
{
    const auto included = c10::impl::tls_local_dispatch_key_set().included_;
    return (included.raw_repr() & ~c10::default_included_set.raw_repr()) == 0 &&
           !c10::impl::TorchDispatchModeTLS::any_modes_set() && at::impl::PythonTorchFunctionTLS::stack_len() == 0 &&
           !torch::jit::tracer::isTracing();
}

// A dense tensor on the current GPU with none of the keys of a wrapper, a conjugate or negative view, a
// quantised or sparse layout.
bool ordinary(const Tensor &t, at::ScalarType type)
{
    static const uint64_t known =
        (c10::DispatchKeySet(c10::DispatchKey::CUDA) | c10::DispatchKeySet(c10::DispatchKey::ADInplaceOrView) |
         c10::getAutogradRelatedKeySetFromBackend(c10::BackendComponent::CUDABit) |
         c10::getAutocastRelatedKeySetFromBackend(c10::BackendComponent::CUDABit)).raw_repr();
    return t.is_cuda() && (t.key_set().raw_repr() & ~known) == 0 && t.scalar_type() == type && t.is_contiguous() &&
           t.get_device() == c10::hip::current_device();
}

// The tensor behind a Python object, if it is exactly a torch.Tensor or a Parameter and ordinary().
const Tensor *tensor_of(PyObject *o, at::ScalarType type)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const Tensor &t = THPVariable_Unpack(o);
    return t.defined() && ordinary(t, type) ? &t : nullptr;
}

// A caller's table: None (the default one), or exactly the class that the entry point takes.
class TableArgument {
public:
    TableArgument(PyObject *o, Table kind)
    {
        if (o == Py_None) {
            good_ = true;
            return;
        }
        PyObject *want = kind == TABLE32 ? g_lut32 : kind == TABLE64 ? g_lut64 : nullptr;
        const Py_ssize_t size = kind == TABLE32 ? sizeof(ktanh_lut_t) : sizeof(ktanh_lut64_t);
        if (want == nullptr || reinterpret_cast<PyObject *>(Py_TYPE(o)) != want) return;
        if (PyObject_GetBuffer(o, &view_, PyBUF_SIMPLE) != 0) {
            PyErr_Clear();
            return;
        }
        held_ = true;
        good_ = view_.len == size;
    }
    ~TableArgument()
    {
        if (held_) PyBuffer_Release(&view_);
    }
    TableArgument(const TableArgument &) = delete;
    TableArgument &operator=(const TableArgument &) = delete;
    bool good() const { return good_; }
    const void *pointer() const { return held_ ? view_.buf : nullptr; }

private:
    Py_buffer view_;
    bool held_ = false, good_ = false;
};

ktanh_stream_t current_stream() { return c10::hip::getCurrentHIPStreamMasqueradingAsCUDA().stream(); }

// A status other than KT_OK becomes the KtanhError that the Python front-end raises.
void check_status(ktanh_status_t st, const char *where)
{
    if (st == KT_OK) return;
    pybind11::gil_scoped_acquire gil;
    PyObject *error = PyObject_CallFunction(g_error, "is", (int)st, where);
    if (error != nullptr) {
        PyErr_SetObject(g_error, error);
        Py_DECREF(error);
    }
    python_error carried;
    carried.persist();
    throw carried;
}

// --------------------------------------------------------------------------------- element-wise calls
// name(in, out, lut) -> out, or None
PyObject *unary_call(PyObject *self, PyObject *const *args, Py_ssize_t nargs)
{
    HANDLE_TH_ERRORS
    const UnaryEntry &entry = kUnary[PyLong_AsLong(self)];
    if (nargs != 3 || !ordinary_thread()) Py_RETURN_NONE;
    const Tensor *in = tensor_of(args[0], entry.in);
    if (in == nullptr) Py_RETURN_NONE;
    const Tensor *given = nullptr;
    if (args[1] != Py_None) {
        given = tensor_of(args[1], entry.out);
        if (given == nullptr || given->numel() != in->numel()) Py_RETURN_NONE;
    }
    const TableArgument lut(args[2], entry.table);
    if (!lut.good()) Py_RETURN_NONE;
    Tensor made;
    {
        pybind11::gil_scoped_release no_gil;
        if (given == nullptr)
            made = entry.in == entry.out ? at::empty_like(*in) : at::empty(in->sizes(), in->options().dtype(entry.out));
        const Tensor &out = given == nullptr ? made : *given;
        check_status(entry.call(in->const_data_ptr(), out.mutable_data_ptr(), (size_t)in->numel(), lut.pointer(),
                                current_stream()), entry.name);
    }
    if (given != nullptr) {
        Py_INCREF(args[1]);
        return args[1];
    }
    return THPVariable_Wrap(std::move(made));
    END_HANDLE_TH_ERRORS
}

// name(dy, v, dx, lut) -> dx, or None
PyObject *binary_call(PyObject *self, PyObject *const *args, Py_ssize_t nargs)
{
    HANDLE_TH_ERRORS
    const BinaryEntry &entry = kBinary[PyLong_AsLong(self)];
    if (nargs != 4 || !ordinary_thread()) Py_RETURN_NONE;
    const Tensor *dy = tensor_of(args[0], entry.type), *v = tensor_of(args[1], entry.type);
    if (dy == nullptr || v == nullptr || dy->numel() != v->numel()) Py_RETURN_NONE;
    const Tensor *given = nullptr;
    if (args[2] != Py_None) {
        given = tensor_of(args[2], entry.type);
        if (given == nullptr || given->numel() != dy->numel()) Py_RETURN_NONE;
    }
    const TableArgument lut(args[3], entry.table);
    if (!lut.good()) Py_RETURN_NONE;
    Tensor made;
    {
        pybind11::gil_scoped_release no_gil;
        if (given == nullptr) made = at::empty_like(*dy);
        const Tensor &dx = given == nullptr ? made : *given;
        check_status(entry.call(dy->const_data_ptr(), v->const_data_ptr(), dx.mutable_data_ptr(), (size_t)dy->numel(),
                                lut.pointer(), current_stream()), entry.name);
    }
    if (given != nullptr) {
        Py_INCREF(args[2]);
        return args[2];
    }
    return THPVariable_Wrap(std::move(made));
    END_HANDLE_TH_ERRORS
}

// ---------------------------------------------------------------------------------------- LSTM cell
ktanh_status_t cell_entry(bool wide, const Tensor &gates, const Tensor &c_in, const Tensor &c_out, const Tensor &h_out,
                          size_t T, size_t B, size_t H, const void *lut)
{
    const auto *g = static_cast<const uint16_t *>(gates.const_data_ptr());
    const auto *c = static_cast<const float *>(c_in.const_data_ptr());
    auto *c1 = static_cast<float *>(c_out.mutable_data_ptr());
    auto *h = static_cast<uint16_t *>(h_out.mutable_data_ptr());
    return wide ? klstm_cell64(g, c, c1, h, T, B, H, static_cast<const ktanh_lut64_t *>(lut), current_stream())
                : klstm_cell(g, c, c1, h, T, B, H, static_cast<const ktanh_lut_t *>(lut), current_stream());
}

ktanh_status_t cell_backward_entry(bool wide, const Tensor &gates, const Tensor &c_prev, const Tensor &dh,
                                   const Tensor &dc_next, const Tensor &dgates, const Tensor &dc_prev, const void *lut)
{
    const auto *g = static_cast<const uint16_t *>(gates.const_data_ptr());
    const auto *c = static_cast<const float *>(c_prev.const_data_ptr());
    const auto *d = static_cast<const uint16_t *>(dh.const_data_ptr());
    const auto *dc = static_cast<const float *>(dc_next.const_data_ptr());
    auto *dg = static_cast<uint16_t *>(dgates.mutable_data_ptr());
    auto *dcp = static_cast<float *>(dc_prev.mutable_data_ptr());
    const size_t B = (size_t)c_prev.size(0), H = (size_t)c_prev.size(1);
    return wide ? klstm_cell64_backward(g, c, d, dc, dg, dcp, B, H, static_cast<const ktanh_lut64_t *>(lut), current_stream())
                : klstm_cell_backward(g, c, d, dc, dg, dcp, B, H, static_cast<const ktanh_lut_t *>(lut), current_stream());
}

const char *cell_name(bool wide) { return wide ? "klstm_cell64" : "klstm_cell"; }
const char *cell_backward_name(bool wide) { return wide ? "klstm_cell64_backward" : "klstm_cell_backward"; }

// gates [B, 4H] next to a state [B, H]
bool cell_shapes(at::IntArrayRef gates, at::IntArrayRef state)
{
    return gates.size() == 2 && state.size() == 2 && gates[0] == state[0] && gates[1] == 4 * state[1];
}

// cell(gates, c_in, c_out, h_out, lut, wide) -> (c_out, h_out), or None
PyObject *cell_call(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    HANDLE_TH_ERRORS
    if (nargs != 6 || !ordinary_thread()) Py_RETURN_NONE;
    const bool wide = args[5] == Py_True;
    const Tensor *gates = tensor_of(args[0], kBf16), *c_in = tensor_of(args[1], kF32);
    if (gates == nullptr || c_in == nullptr || gates->dim() != 3 || !cell_shapes(gates->sizes().slice(1), c_in->sizes()))
        Py_RETURN_NONE;
    const int64_t T = gates->size(0), B = c_in->size(0), H = c_in->size(1);
    const Tensor *c_given = nullptr, *h_given = nullptr;
    if (args[2] != Py_None) {
        c_given = tensor_of(args[2], kF32);
        if (c_given == nullptr || c_given->sizes() != c_in->sizes()) Py_RETURN_NONE;
    }
    if (args[3] != Py_None) {
        h_given = tensor_of(args[3], kBf16);
        if (h_given == nullptr || h_given->sizes() != at::IntArrayRef({T, B, H})) Py_RETURN_NONE;
    }
    const TableArgument lut(args[4], wide ? TABLE64 : TABLE32);
    if (!lut.good()) Py_RETURN_NONE;
    Tensor c, h;
    {
        pybind11::gil_scoped_release no_gil;
        c = c_given == nullptr ? at::empty_like(*c_in) : *c_given;
        h = h_given == nullptr ? at::empty({T, B, H}, gates->options()) : *h_given;
        check_status(cell_entry(wide, *gates, *c_in, c, h, (size_t)T, (size_t)B, (size_t)H, lut.pointer()),
                     cell_name(wide));
    }
    return Py_BuildValue("(NN)", THPVariable_Wrap(std::move(c)), THPVariable_Wrap(std::move(h)));
    END_HANDLE_TH_ERRORS
}

// cell_backward(gates, c_prev, dh, dc_next, dgates, dc_prev, lut, wide) -> (dgates, dc_prev), or None
PyObject *cell_backward_call(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    HANDLE_TH_ERRORS
    if (nargs != 8 || !ordinary_thread()) Py_RETURN_NONE;
    const bool wide = args[7] == Py_True;
    const Tensor *gates = tensor_of(args[0], kBf16), *c_prev = tensor_of(args[1], kF32);
    const Tensor *dh = tensor_of(args[2], kBf16), *dc_next = tensor_of(args[3], kF32);
    if (gates == nullptr || c_prev == nullptr || dh == nullptr || dc_next == nullptr ||
        !cell_shapes(gates->sizes(), c_prev->sizes()) || dh->sizes() != c_prev->sizes() ||
        dc_next->sizes() != c_prev->sizes())
        Py_RETURN_NONE;
    const Tensor *dgates_given = nullptr, *dc_given = nullptr;
    if (args[4] != Py_None) {
        dgates_given = tensor_of(args[4], kBf16);
        if (dgates_given == nullptr || dgates_given->sizes() != gates->sizes()) Py_RETURN_NONE;
    }
    if (args[5] != Py_None) {
        dc_given = tensor_of(args[5], kF32);
        if (dc_given == nullptr || dc_given->sizes() != c_prev->sizes()) Py_RETURN_NONE;
    }
    const TableArgument lut(args[6], wide ? TABLE64 : TABLE32);
    if (!lut.good()) Py_RETURN_NONE;
    Tensor dgates, dc;
    {
        pybind11::gil_scoped_release no_gil;
        dgates = dgates_given == nullptr ? at::empty_like(*gates) : *dgates_given;
        dc = dc_given == nullptr ? at::empty_like(*c_prev) : *dc_given;
        check_status(cell_backward_entry(wide, *gates, *c_prev, *dh, *dc_next, dgates, dc, lut.pointer()),
                     cell_backward_name(wide));
    }
    return Py_BuildValue("(NN)", THPVariable_Wrap(std::move(dgates)), THPVariable_Wrap(std::move(dc)));
    END_HANDLE_TH_ERRORS
}

// ---------------------------------------------------------------------------------------- autograd
// The activations by code 2 * {0 TanH, 1 Sigmoid, 2 Swish, 3 GELU} + {0: 32, 1: 64 intervals}; the
// gradients of TanH and Sigmoid read the forward output, those of Swish and GELU the forward input.
struct TrainEntry {
    const char *forward, *backward;
    Unary forward_call;
    Binary backward_call;
    bool from_input;
};
#define TRAIN(fwd, bwd, from_input) {#fwd, #bwd, UnaryOf<&fwd>::call, BinaryOf<&bwd>::call, from_input}
const TrainEntry kTrainBf16[] = {
    TRAIN(ktanh_bf16, ktanh_bf16_backward, false), TRAIN(ktanh64_bf16, ktanh_bf16_backward, false),
    TRAIN(ksigmoid, ksigmoid_backward, false), TRAIN(ksigmoid64, ksigmoid_backward, false),
    TRAIN(kswish, kswish_backward, true), TRAIN(kswish64, kswish64_backward, true),
    TRAIN(kgelu, kgelu_backward, true), TRAIN(kgelu64, kgelu64_backward, true),
};
const TrainEntry kTrainF32[] = {
    TRAIN(ktanh_f32, ktanh_f32_backward, false), TRAIN(ktanh64_f32, ktanh_f32_backward, false),
    TRAIN(ksigmoid_f32, ksigmoid_f32_backward, false), TRAIN(ksigmoid64_f32, ksigmoid_f32_backward, false),
    TRAIN(kswish_f32, kswish_f32_backward, true), TRAIN(kswish64_f32, kswish64_f32_backward, true),
    TRAIN(kgelu_f32, kgelu_f32_backward, true), TRAIN(kgelu64_f32, kgelu64_f32_backward, true),
};
const TrainEntry &train_entry(int64_t code, at::ScalarType type) { return (type == kF32 ? kTrainF32 : kTrainBf16)[code]; }

// What arrives in a backward pass was not looked at by the forward call (a saved-tensor hook or a gradient
// hook may have put something else there): the checks of the Python front-end.
const Tensor &checked(const Tensor &t, at::ScalarType type, const char *what)
{
    TORCH_CHECK(t.defined() && t.has_storage(), what, " must be a tensor with storage");
    TORCH_CHECK_VALUE(t.is_cuda(), what, " must be a CUDA tensor (device memory)");
    TORCH_CHECK_TYPE(t.scalar_type() == type, what, " has dtype ", t.scalar_type(), ", expected ", type);
    TORCH_CHECK_VALUE(t.is_contiguous(), what, " must be contiguous");
    TORCH_CHECK(ordinary(t, type), what, " must be an ordinary tensor on the current device");
    return t;
}

Tensor run_forward(const TrainEntry &entry, const Tensor &x)
{
    const Tensor y = at::empty_like(x);
    check_status(entry.forward_call(x.const_data_ptr(), y.mutable_data_ptr(), (size_t)x.numel(), nullptr,
                                    current_stream()), entry.forward);
    return y;
}

struct Activation : public torch::autograd::Function<Activation> {
    static Tensor forward(AutogradContext *ctx, const Tensor &x, int64_t code)
    {
        const TrainEntry &entry = train_entry(code, x.scalar_type());
        const Tensor y = run_forward(entry, x);
        ctx->save_for_backward({entry.from_input ? x : y});
        ctx->saved_data["code"] = code;
        return y;
    }
    static variable_list backward(AutogradContext *ctx, const variable_list &grads)
    {
        const Tensor saved = ctx->get_saved_variables()[0];
        const at::ScalarType type = grads[0].scalar_type() == kF32 ? kF32 : kBf16;
        const TrainEntry &entry = train_entry(ctx->saved_data["code"].toInt(), type);
        const Tensor dy = grads[0].contiguous();
        checked(dy, type, "dy");
        const Tensor &v = checked(saved, type, "the saved tensor");
        TORCH_CHECK_VALUE(dy.numel() == v.numel(), "dy and the saved tensor differ in size");
        const Tensor dx = at::empty_like(dy);
        check_status(entry.backward_call(dy.const_data_ptr(), v.const_data_ptr(), dx.mutable_data_ptr(),
                                         (size_t)dy.numel(), nullptr, current_stream()), entry.backward);
        return {dx, Tensor()};
    }
};

// h is element 0 of a [1, B, H] tensor, as the multi-step entry point gives it.
variable_list run_cell(const Tensor &gates, const Tensor &c_prev, bool wide)
{
    const int64_t B = c_prev.size(0), H = c_prev.size(1);
    const Tensor c = at::empty_like(c_prev), h = at::empty({1, B, H}, gates.options());
    check_status(cell_entry(wide, gates, c_prev, c, h, 1, (size_t)B, (size_t)H, nullptr), cell_name(wide));
    return {h.select(0, 0), c};
}

struct Cell : public torch::autograd::Function<Cell> {
    static variable_list forward(AutogradContext *ctx, const Tensor &gates, const Tensor &c_prev, bool wide)
    {
        variable_list out = run_cell(gates, c_prev, wide);
        ctx->save_for_backward({gates, c_prev});
        ctx->saved_data["wide"] = wide;
        return out;
    }
    static variable_list backward(AutogradContext *ctx, const variable_list &grads)
    {
        const variable_list saved = ctx->get_saved_variables();
        const bool wide = ctx->saved_data["wide"].toBool();
        const Tensor dh = grads[0].contiguous(), dc_next = grads[1].contiguous();
        const Tensor &gates = checked(saved[0], kBf16, "gates"), &c_prev = checked(saved[1], kF32, "c_prev");
        checked(dh, kBf16, "dh");
        checked(dc_next, kF32, "dc_next");
        TORCH_CHECK_VALUE(cell_shapes(gates.sizes(), c_prev.sizes()) && dh.sizes() == c_prev.sizes() &&
                          dc_next.sizes() == c_prev.sizes(),
                          "gates [B, 4H], c_prev, dh, dc_next [B, H] do not agree");
        const Tensor dgates = at::empty_like(gates), dc_prev = at::empty_like(c_prev);
        check_status(cell_backward_entry(wide, gates, c_prev, dh, dc_next, dgates, dc_prev, nullptr),
                     cell_backward_name(wide));
        return {dgates, dc_prev, Tensor()};
    }
};

bool differentiable(const Tensor &t) { return !t._fw_grad(/*level=*/0).defined(); }

// train(code, x) -> y, or None
PyObject *train_call(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    HANDLE_TH_ERRORS
    if (nargs != 2 || !ordinary_thread()) Py_RETURN_NONE;
    const long code = PyLong_AsLong(args[0]);
    if (code < 0 || code >= (long)std::size(kTrainBf16)) Py_RETURN_NONE;
    const Tensor *x = tensor_of(args[1], kBf16);
    if (x == nullptr) x = tensor_of(args[1], kF32);
    if (x == nullptr || !differentiable(*x)) Py_RETURN_NONE;
    Tensor y;
    {
        pybind11::gil_scoped_release no_gil;
        if (at::GradMode::is_enabled() && x->requires_grad()) y = Activation::apply(*x, (int64_t)code);
        else y = run_forward(train_entry(code, x->scalar_type()), *x);
    }
    return THPVariable_Wrap(std::move(y));
    END_HANDLE_TH_ERRORS
}

// train_cell(gates, c_prev, wide) -> (h, c), or None
PyObject *train_cell_call(PyObject *, PyObject *const *args, Py_ssize_t nargs)
{
    HANDLE_TH_ERRORS
    if (nargs != 3 || !ordinary_thread()) Py_RETURN_NONE;
    const Tensor *gates = tensor_of(args[0], kBf16), *c_prev = tensor_of(args[1], kF32);
    if (gates == nullptr || c_prev == nullptr || !cell_shapes(gates->sizes(), c_prev->sizes()) ||
        !differentiable(*gates) || !differentiable(*c_prev))
        Py_RETURN_NONE;
    const bool wide = args[2] == Py_True;
    variable_list out;
    {
        pybind11::gil_scoped_release no_gil;
        if (at::GradMode::is_enabled() && (gates->requires_grad() || c_prev->requires_grad()))
            out = Cell::apply(*gates, *c_prev, wide);
        else
            out = run_cell(*gates, *c_prev, wide);
    }
    return Py_BuildValue("(NN)", THPVariable_Wrap(std::move(out[0])), THPVariable_Wrap(std::move(out[1])));
    END_HANDLE_TH_ERRORS
}

// ------------------------------------------------------------------------------------------ module
// setup(KtanhLut, KtanhLut64, KtanhError): the classes of binding.py
PyObject *setup_call(PyObject *, PyObject *args)
{
    PyObject *lut32, *lut64, *error;
    if (!PyArg_ParseTuple(args, "OOO", &lut32, &lut64, &error)) return nullptr;
    Py_INCREF(lut32);
    Py_INCREF(lut64);
    Py_INCREF(error);
    Py_XSETREF(g_lut32, lut32);
    Py_XSETREF(g_lut64, lut64);
    Py_XSETREF(g_error, error);
    Py_RETURN_NONE;
}

template <class F> PyCFunction as_method(F f) { return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)); }

PyMethodDef kMethods[] = {
    {"setup", setup_call, METH_VARARGS, nullptr},
    {"cell", as_method(cell_call), METH_FASTCALL, nullptr},
    {"cell_backward", as_method(cell_backward_call), METH_FASTCALL, nullptr},
    {"train", as_method(train_call), METH_FASTCALL, nullptr},
    {"train_cell", as_method(train_cell_call), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyMethodDef g_unary_defs[std::size(kUnary)], g_binary_defs[std::size(kBinary)];
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_ktanh_torch", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

// One function per entry point, under its name, in the dict `calls`; `self` is its index.
template <class Entry, size_t N>
bool add_calls(PyObject *calls, const Entry (&entries)[N], PyMethodDef (&defs)[N], PyCFunction call)
{
    for (size_t i = 0; i < N; ++i) {
        defs[i] = PyMethodDef{entries[i].name, call, METH_FASTCALL, nullptr};
        PyObject *index = PyLong_FromSize_t(i);
        PyObject *fn = index != nullptr ? PyCFunction_New(&defs[i], index) : nullptr;
        Py_XDECREF(index);
        const bool stored = fn != nullptr && PyDict_SetItemString(calls, entries[i].name, fn) == 0;
        Py_XDECREF(fn);
        if (!stored) return false;
    }
    return true;
}

}  // namespace

// Touches nothing of torch: binding.py compares `torch_version` (the one that the headers are of) before the first call.
PyMODINIT_FUNC PyInit__ktanh_torch()
{
    PyObject *module = PyModule_Create(&kModule);
    PyObject *calls = module != nullptr ? PyDict_New() : nullptr;
    if (calls == nullptr || !add_calls(calls, kUnary, g_unary_defs, as_method(unary_call)) ||
        !add_calls(calls, kBinary, g_binary_defs, as_method(binary_call)) ||
        PyModule_AddStringConstant(module, "torch_version", KTANH_TORCH_VERSION) != 0 ||
        PyModule_AddObject(module, "calls", calls) != 0) {
        Py_XDECREF(calls);
        Py_XDECREF(module);
        return nullptr;
    }
    return module;
}
