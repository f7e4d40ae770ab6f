// The ordinary call of every operation, marshalled natively: tensors on the current device, the result allocated here, torch's
// current stream, automatic path.  Checking two tensors attribute by attribute in Python, allocating the result and converting
// sixteen arguments with ctypes took 5 of the 8 us that a call of 2 us of GPU work took, and as much again where a workspace
// is asked for.
//
// Every function returns None for a call that is anything else, or that the library would refuse: the Python function of
// the same name then goes its own way, and raises where something is wrong.  Nothing is decided here that is not decided
// there in the same way.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <stdint.h>

#include "../../../include/ukst.h"

namespace {

decltype(&ukst_workspace_bytes) workspace_bytes;
decltype(&ukst_conv_transpose2d_path) forward_path;
decltype(&ukst_conv_transpose2d_bias_act) forward_bias_act;
decltype(&ukst_conv_transpose2d_ws) forward_ws;
decltype(&ukst_conv_transpose2d_grad_input) grad_input;
decltype(&ukst_conv_transpose2d_grad_weight) grad_weight;
decltype(&ukst_conv_transpose2d_strided) strided;
decltype(&ukst_dilated_conv2d) dilated;

constexpr int64_t kMaxSide = 1 << 28, kMaxGeneralSide = 1 << 24;  // (ukst_output_shape*, and every value below fits an int)

// a plain contiguous 4-D tensor on the current device, float32 or bfloat16; null if it is not
const at::Tensor* operand(PyObject* o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || t.layout() != at::kStrided || !t.is_cuda() || !t.unsafeGetTensorImpl()->has_storage() ||
        t.key_set().has(c10::DispatchKey::FuncTorchBatched) || t.key_set().has(c10::DispatchKey::FuncTorchGradWrapper) ||
        t.key_set().has(c10::DispatchKey::Functionalize) || !t.is_contiguous())
        return nullptr;
    if (t.dim() != 4 || (t.scalar_type() != at::kFloat && t.scalar_type() != at::kBFloat16)) return nullptr;
    for (int64_t s : t.sizes())
        if (s < 1 || s > kMaxSide) return nullptr;
    return &t;
}

bool number(PyObject* o, int64_t lo, int64_t hi, int* v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long long n = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow != 0 || n < lo || n > hi) return false;
    *v = (int)n;
    return true;
}

// the stream of the call; false if the tensors are not on the current device
bool stream_of(const at::Tensor& a, const at::Tensor& b, void** stream)
{
    const c10::DeviceIndex index = a.get_device();
    if (b.get_device() != index || c10::hip::current_device() != index || at::impl::torch_function_mode_enabled()) return false;
    *stream = (void*)c10::hip::getCurrentHIPStream(index).stream();
    return true;
}

at::Tensor result(const at::Tensor& like, at::IntArrayRef sizes, at::ScalarType type)
{
    return at::empty(sizes, at::TensorOptions().dtype(type).device(like.device()));
}

// memory of this call (torch's allocator hands it on to later work of the same stream only)
at::Tensor workspace(const at::Tensor& like, size_t bytes)
{
    return bytes == 0 ? at::Tensor() : result(like, {(int64_t)bytes}, at::kByte);
}
void* address(const at::Tensor& t) { return t.defined() ? t.mutable_data_ptr() : nullptr; }

template <class Call>
int released(Call call)  // without the interpreter lock, as a ctypes call
{
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = call();
    Py_END_ALLOW_THREADS
    return status;
}

// body() -> the result, or an undefined tensor for None
template <class Body>
PyObject* guarded(Body body)
{
    try {
        at::Tensor t = body();
        if (t.defined()) return THPVariable_Wrap(std::move(t));
    } catch (...) {  // (out of memory and the like: raised where the call is made again)
    }
    PyErr_Clear();
    Py_RETURN_NONE;
}

// (x, w, P, bias or None, act or None, out_bf16, with_workspace) -> y
PyObject* forward(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    return guarded([&]() -> at::Tensor {
        if (nargs != 7) return {};
        const at::Tensor *x = operand(args[0]), *w = operand(args[1]), *bias = nullptr;
        int P, act = UKST_ACT_NONE;
        if (!x || !w || !number(args[2], 0, kMaxSide, &P) || x->scalar_type() != w->scalar_type()) return {};
        if (args[4] != Py_None && !number(args[4], UKST_ACT_NONE, UKST_ACT_TANH, &act)) return {};
        const int64_t B = x->size(0), Cin = x->size(1), H = x->size(2), W = x->size(3), Cout = w->size(0), n = w->size(2);
        if (w->size(3) != n || w->size(1) != Cin) return {};
        if (args[3] != Py_None) {
            if (args[4] == Py_None || !THPVariable_CheckExact(args[3])) return {};
            bias = &THPVariable_Unpack(args[3]);
            if (bias->layout() != at::kStrided || !bias->is_cuda() || bias->scalar_type() != at::kFloat || bias->dim() != 1 ||
                bias->size(0) != Cout || !bias->is_contiguous() || bias->get_device() != x->get_device() ||
                !bias->unsafeGetTensorImpl()->has_storage())
                return {};
        }
        const bool f32 = x->scalar_type() == at::kFloat, out16 = args[5] == Py_True;
        if ((!out16 && args[5] != Py_False) || (f32 && out16)) return {};
        const int64_t OH = 2 * H + 2 * (int64_t)P - n, OW = 2 * W + 2 * (int64_t)P - n;
        void* stream;
        if (OH < 1 || OW < 1 || OH > kMaxSide || OW > kMaxSide || !stream_of(*x, *w, &stream)) return {};
        const int dtype = f32 ? UKST_F32 : out16 ? UKST_BF16_BF16 : UKST_BF16_F32;
        at::Tensor y = result(*x, {B, Cout, OH, OW}, out16 ? at::kBFloat16 : at::kFloat), ws;
        const void *xp = x->const_data_ptr(), *wp = w->const_data_ptr();
        const float* bp = bias ? bias->const_data_ptr<float>() : nullptr;
        void* const yp = y.mutable_data_ptr();
        int status;
        if (args[6] == Py_True) {
            const size_t need = workspace_bytes(UKST_OP_FORWARD, B, Cin, Cout, H, W, n, P, dtype);
            ws = workspace(*x, need);
            void* const p = address(ws);
            status = released([&] { return forward_ws(xp, wp, bp, yp, B, Cin, Cout, H, W, n, P, dtype, act, UKST_PATH_AUTO,
                                                      p, need, stream); });
        } else if (args[4] == Py_None) {
            status = released([&] { return forward_path(xp, wp, yp, B, Cin, Cout, H, W, n, P, dtype, UKST_PATH_AUTO, stream); });
        } else {
            status = released([&] { return forward_bias_act(xp, wp, bp, yp, B, Cin, Cout, H, W, n, P, dtype, act,
                                                            UKST_PATH_AUTO, stream); });
        }
        return status == UKST_OK ? y : at::Tensor();
    });
}

// (dy, w, H, W, P) -> dx
PyObject* input_gradient(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    return guarded([&]() -> at::Tensor {
        if (nargs != 5) return {};
        const at::Tensor *dy = operand(args[0]), *w = operand(args[1]);
        int H, W, P;
        if (!dy || !w || dy->scalar_type() != w->scalar_type() || !number(args[2], 1, kMaxSide, &H) ||
            !number(args[3], 1, kMaxSide, &W) || !number(args[4], 0, kMaxSide, &P))
            return {};
        const int64_t B = dy->size(0), Cout = dy->size(1), Cin = w->size(1), n = w->size(2);
        void* stream;
        if (w->size(0) != Cout || w->size(3) != n || dy->size(2) != 2 * (int64_t)H + 2 * (int64_t)P - n ||
            dy->size(3) != 2 * (int64_t)W + 2 * (int64_t)P - n || !stream_of(*dy, *w, &stream))
            return {};
        const int dtype = dy->scalar_type() == at::kFloat ? UKST_F32 : UKST_BF16_F32;
        at::Tensor dx = result(*dy, {B, Cin, H, W}, at::kFloat);
        const size_t need = workspace_bytes(UKST_OP_GRAD_INPUT, B, Cin, Cout, H, W, n, P, dtype);
        const at::Tensor ws = workspace(*dy, need);
        const void *yp = dy->const_data_ptr(), *wp = w->const_data_ptr();
        void *const xp = dx.mutable_data_ptr(), *const p = address(ws);
        const int status = released([&] { return grad_input(yp, wp, xp, B, Cin, Cout, H, W, n, P, dtype, p, need, stream); });
        return status == UKST_OK ? dx : at::Tensor();
    });
}

// (x, dy, n, P) -> dw
PyObject* kernel_gradient(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    return guarded([&]() -> at::Tensor {
        if (nargs != 4) return {};
        const at::Tensor *x = operand(args[0]), *dy = operand(args[1]);
        int n, P;
        if (!x || !dy || x->scalar_type() != dy->scalar_type() || !number(args[2], 1, kMaxSide, &n) ||
            !number(args[3], 0, kMaxSide, &P))
            return {};
        const int64_t B = x->size(0), Cin = x->size(1), H = x->size(2), W = x->size(3), Cout = dy->size(1);
        void* stream;
        if (dy->size(0) != B || dy->size(2) != 2 * H + 2 * (int64_t)P - n || dy->size(3) != 2 * W + 2 * (int64_t)P - n ||
            !stream_of(*x, *dy, &stream))
            return {};
        const int dtype = x->scalar_type() == at::kFloat ? UKST_F32 : UKST_BF16_F32;
        at::Tensor dw = result(*x, {Cout, Cin, n, n}, at::kFloat);
        const size_t need = workspace_bytes(UKST_OP_GRAD_WEIGHT, B, Cin, Cout, H, W, n, P, dtype);
        const at::Tensor ws = workspace(*x, need);
        const void *xp = x->const_data_ptr(), *yp = dy->const_data_ptr();
        void *const wp = dw.mutable_data_ptr(), *const p = address(ws);
        const int status = released([&] { return grad_weight(xp, yp, wp, B, Cin, Cout, H, W, n, P, dtype, p, need, stream); });
        return status == UKST_OK ? dw : at::Tensor();
    });
}

// (x, w, P, step, is_dilated) -> y
PyObject* general(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    return guarded([&]() -> at::Tensor {
        if (nargs != 5) return {};
        const at::Tensor *x = operand(args[0]), *w = operand(args[1]);
        int P, k;
        if (!x || !w || x->scalar_type() != w->scalar_type() || !number(args[2], 0, kMaxGeneralSide, &P) ||
            !number(args[3], 1, UKST_MAX_STEP, &k))
            return {};
        const int64_t B = x->size(0), Cin = x->size(1), H = x->size(2), W = x->size(3), Cout = w->size(0), n = w->size(2);
        if (w->size(3) != n || w->size(1) != Cin || H > kMaxGeneralSide || W > kMaxGeneralSide) return {};
        const bool dil = args[4] == Py_True;
        const int64_t OH = dil ? H + 2 * (int64_t)P - k * (n - 1) : k * (H - 1) + 2 * (int64_t)P - n + 2;
        const int64_t OW = dil ? W + 2 * (int64_t)P - k * (n - 1) : k * (W - 1) + 2 * (int64_t)P - n + 2;
        void* stream;
        if (OH < 1 || OW < 1 || OH > kMaxSide || OW > kMaxSide || !stream_of(*x, *w, &stream)) return {};
        const int dtype = x->scalar_type() == at::kFloat ? UKST_F32 : UKST_BF16_F32;
        at::Tensor y = result(*x, {B, Cout, OH, OW}, at::kFloat);
        const void *xp = x->const_data_ptr(), *wp = w->const_data_ptr();
        void* const yp = y.mutable_data_ptr();
        const int status = released([&] { return (dil ? dilated : strided)(xp, wp, yp, B, Cin, Cout, H, W, n, P, k, dtype,
                                                                           stream); });
        return status == UKST_OK ? y : at::Tensor();
    });
}

// (addresses of the eight library functions, in the order of the pointers above)
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    void* p[8];
    if (nargs != 8) {
        PyErr_SetString(PyExc_TypeError, "eight addresses expected");
        return nullptr;
    }
    for (int i = 0; i < 8; ++i)
        if ((p[i] = PyLong_AsVoidPtr(args[i])) == nullptr) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address");
            return nullptr;
        }
    workspace_bytes = (decltype(workspace_bytes))p[0];
    forward_path = (decltype(forward_path))p[1];
    forward_bias_act = (decltype(forward_bias_act))p[2];
    forward_ws = (decltype(forward_ws))p[3];
    grad_input = (decltype(grad_input))p[4];
    grad_weight = (decltype(grad_weight))p[5];
    strided = (decltype(strided))p[6];
    dilated = (decltype(dilated))p[7];
    Py_RETURN_NONE;
}

#define UKST_METHOD(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {UKST_METHOD(bind), UKST_METHOD(forward), UKST_METHOD(input_gradient), UKST_METHOD(kernel_gradient),
                         UKST_METHOD(general), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ukst_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: the version of torch whose headers this was compiled with
PyMODINIT_FUNC PyInit__ukst_marshal(void)
{
    PyObject* const m = PyModule_Create(&module);
    if (m != nullptr && PyModule_AddStringConstant(m, "built_for", UKST_BUILT_FOR) != 0) {
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
