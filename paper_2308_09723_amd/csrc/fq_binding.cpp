// The calls of the torch-tensor layer that a program makes over and over (products, activation and weight quantiser), in
// native code: argument checks, output allocation, the current stream and the call of the library.
//
// A product of one kernel takes the GPU 4 - 8 us, and issuing it from Python took as long: 6.5 us, of which the launch itself
// is 2.7; here it takes 3.5.  The integer path's two calls: 14.7 us from Python, now 9.7 (which the GPU takes); fq.quantize 9.2
// -> 5.6.
//
// Every function returns None, having launched nothing, where anything is out of the ordinary: objects that are not plain
// CUDA tensors, torch function modes, other types than the listed ones, arguments or a workspace that the library refuses.  fq.py
// then takes its own way, which reports the error or does what it always did.  An error of the runtime (FQ_ERR_HIP) may follow
// launches that were enqueued, so it is raised here and the call is not made again.  Only arguments are looked at; nothing is
// kept between calls.
#include <Python.h>

#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/generated/variable_factories.h>
#include <torch/csrc/autograd/python_variable.h>

#include <limits.h>
#include <string.h>


#include "../../include/fq.h"

namespace {

// the library's functions, as addresses that fq.py hands over (bind): one copy of the library per process
struct {
    decltype(&fq_gemm_sf) gemm_sf;
    decltype(&fq_gemm_workspace_bytes) gemm_workspace_bytes;
    decltype(&fq_gemm_grouped_sf) gemm_grouped_sf;
    decltype(&fq_gemm_w4a8) gemm_w4a8;
    decltype(&fq_gemm_w4a8_workspace_bytes) gemm_w4a8_workspace_bytes;
    decltype(&fq_quantize_act_i8) quantize_act_i8;
    decltype(&fq_quantize_sf) quantize_sf;
    decltype(&fq_quantize_w4a8) quantize_w4a8;
    decltype(&fq_codes_bytes) codes_bytes;
    decltype(&fq_scales_bytes) scales_bytes;
    decltype(&fq_zscale_bytes) zscale_bytes;
} lib;

PyObject* fq_error;       // fq.FqError

struct not_plain {};      // thrown: the Python way
struct runtime_error {    // thrown: FqError(FQ_ERR_HIP, where)
    const char* where;
};

const at::Tensor& tensor(PyObject* o) {
    if (!THPVariable_CheckExact(o)) throw not_plain();
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.layout() != at::kStrided) throw not_plain();
    return t;
}

int integer(PyObject* o) {
    if (!PyLong_CheckExact(o)) throw not_plain();
    int overflow = 0;
    const long v = PyLong_AsLongAndOverflow(o, &overflow);
    if (overflow != 0 || v < INT_MIN || v > INT_MAX) throw not_plain();
    return (int)v;
}

// 0 for binary16, 1 for bfloat16: the library's activation types and its scale formats alike
int type16(at::ScalarType s) {
    if (s == at::kHalf) return 0;
    if (s == at::kBFloat16) return 1;
    throw not_plain();
}

int scalar16(PyObject* o) {
    if (!THPDtype_Check(o)) throw not_plain();
    return type16(reinterpret_cast<THPDtype*>(o)->scalar_type);
}

at::Tensor empty(at::IntArrayRef size, at::ScalarType type, const at::Tensor& like) {
    return torch::empty(size, at::TensorOptions().dtype(type).device(like.device()));
}

void* stream() { return (void*)c10::hip::getCurrentHIPStream(c10::hip::current_device()).stream(); }

void arguments(Py_ssize_t got, Py_ssize_t want) {
    if (got != want || at::impl::torch_function_mode_enabled()) throw not_plain();
}

// runs `f` (a call of the library's function `where`) without the interpreter's lock
template <typename F>
void call(const char* where, F f) {
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = f();
    Py_END_ALLOW_THREADS
    if (status == FQ_ERR_HIP) throw runtime_error{where};
    if (status != FQ_OK) throw not_plain();
}

// a caller's workspace (None: one of `need()` bytes) as address and size
template <typename F>
void* scratch(PyObject* o, const at::Tensor& like, F need, size_t* size, at::Tensor* own) {
    if (o != Py_None) {
        const at::Tensor& t = tensor(o);
        *size = (size_t)t.numel() * t.element_size();
        return t.data_ptr();
    }
    *size = need();
    if (*size == 0) return nullptr;
    *own = empty({(int64_t)*size}, at::kByte, like);
    return own->data_ptr();
}

// the output a caller gave, or a new one
PyObject* result(PyObject* given, at::Tensor&& made) {
    if (given == Py_None) return THPVariable_Wrap(std::move(made));
    Py_INCREF(given);
    return given;
}

template <typename F>
PyObject* guarded(F f) {
    try {
        return f();
    } catch (const runtime_error& e) {
        PyObject* raised = PyObject_CallFunction(fq_error, "is", (int)FQ_ERR_HIP, e.where);
        if (raised) PyErr_SetObject(fq_error, raised);
        Py_XDECREF(raised);
        return nullptr;
    } catch (...) {
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

// gemm(A, codes, scales, bits, group_size, out, workspace)
PyObject* gemm(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        arguments(n, 7);
        const at::Tensor &A = tensor(a[0]), &codes = tensor(a[1]), &scales = tensor(a[2]);
        if (A.dim() != 2 || scales.dim() != 2 || !A.is_contiguous()) throw not_plain();
        const int act = type16(A.scalar_type()), format = type16(scales.scalar_type()), bits = integer(a[3]), g = integer(a[4]);
        const int64_t M = A.size(0), K = A.size(1), N = scales.size(1);
        const void *Ap = A.data_ptr(), *cp = codes.data_ptr(), *sp = scales.data_ptr();
        at::Tensor C = a[5] != Py_None ? tensor(a[5]) : empty({M, N}, A.scalar_type(), A), own;
        size_t size = 0;
        void* ws = scratch(a[6], A, [&] { return lib.gemm_workspace_bytes(M, N, K, bits, g); }, &size, &own);
        void *Cp = C.data_ptr(), *s = stream();
        call("fq_gemm_sf", [&] { return lib.gemm_sf(Ap, act, M, N, K, cp, sp, format, bits, g, Cp, ws, size, s); });
        return result(a[5], std::move(C));
    });
}

// gemm_grouped(A, offsets, codes, scales, bits, group_size, N, out)
PyObject* gemm_grouped(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        arguments(n, 8);
        const at::Tensor &A = tensor(a[0]), &codes = tensor(a[2]), &scales = tensor(a[3]);
        if (A.dim() != 2 || !(PyList_CheckExact(a[1]) || PyTuple_CheckExact(a[1]))) throw not_plain();
        const Py_ssize_t count = PySequence_Fast_GET_SIZE(a[1]);
        if (count < 1 || count > 257) throw not_plain();
        int32_t offsets[257];
        for (Py_ssize_t i = 0; i < count; ++i) offsets[i] = integer(PySequence_Fast_GET_ITEM(a[1], i));
        const int act = type16(A.scalar_type()), format = type16(scales.scalar_type()), bits = integer(a[4]), g = integer(a[5]);
        const int64_t K = A.size(1), N = integer(a[6]);
        const void *Ap = A.data_ptr(), *cp = codes.data_ptr(), *sp = scales.data_ptr();
        at::Tensor C = a[7] != Py_None ? tensor(a[7]) : empty({A.size(0), N}, A.scalar_type(), A);
        void *Cp = C.data_ptr(), *s = stream();
        call("fq_gemm_grouped_sf", [&] {
            return lib.gemm_grouped_sf(Ap, act, offsets, (int)count - 1, N, K, cp, sp, format, bits, g, Cp, nullptr, 0, s);
        });
        return result(a[7], std::move(C));
    });
}

// quantize_act_i8(A)
PyObject* quantize_act_i8(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        arguments(n, 1);
        const at::Tensor& A = tensor(a[0]);
        if (A.dim() != 2 || !A.is_contiguous()) throw not_plain();
        const int act = type16(A.scalar_type());
        const int64_t M = A.size(0), K = A.size(1);
        const void* Ap = A.data_ptr();
        at::Tensor Aq = empty({M, K}, at::kChar, A), alpha = empty({M}, at::kFloat, A);
        int8_t* qp = (int8_t*)Aq.data_ptr();
        float* alp = (float*)alpha.data_ptr();
        void* s = stream();
        call("fq_quantize_act_i8", [&] { return lib.quantize_act_i8(Ap, act, M, K, qp, alp, s); });
        return Py_BuildValue("(NN)", THPVariable_Wrap(std::move(Aq)), THPVariable_Wrap(std::move(alpha)));
    });
}

// gemm_w4a8(Aq, alpha, codes, z, t, group_size, out_dtype, out, workspace)
PyObject* gemm_w4a8(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        arguments(n, 9);
        const at::Tensor &Aq = tensor(a[0]), &alpha = tensor(a[1]), &codes = tensor(a[2]), &z = tensor(a[3]), &t = tensor(a[4]);
        if (Aq.dim() != 2 || t.dim() != 1) throw not_plain();
        const int g = integer(a[5]), type = scalar16(a[6]);
        const int64_t M = Aq.size(0), K = Aq.size(1), N = t.size(0);
        const int8_t* qp = (const int8_t*)Aq.data_ptr();
        const float* alp = (const float*)alpha.data_ptr();
        const void *cp = codes.data_ptr(), *tp = t.data_ptr();
        const uint8_t* zp = (const uint8_t*)z.data_ptr();
        at::Tensor C = a[7] != Py_None ? tensor(a[7]) : empty({M, N}, type == 0 ? at::kHalf : at::kBFloat16, Aq), own;
        size_t size = 0;
        void* ws = scratch(a[8], Aq, [&] { return lib.gemm_w4a8_workspace_bytes(M, N, K, g); }, &size, &own);
        void *Cp = C.data_ptr(), *s = stream();
        call("fq_gemm_w4a8", [&] { return lib.gemm_w4a8(qp, alp, M, N, K, cp, zp, tp, g, Cp, type, ws, size, s); });
        return result(a[7], std::move(C));
    });
}

// quantize(W, bits, group_size, scale_format)
PyObject* quantize(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        arguments(n, 4);
        const at::Tensor& W = tensor(a[0]);
        if (W.dim() != 2 || W.scalar_type() != at::kHalf || !W.is_contiguous()) throw not_plain();
        const int bits = integer(a[1]), g = integer(a[2]), format = integer(a[3]);
        const int64_t K = W.size(0), N = W.size(1);
        const size_t cb = lib.codes_bytes(K, N, bits), sb = lib.scales_bytes(K, N, g);
        if (cb == 0 || sb == 0 || (format != FQ_SCALE_F16 && format != FQ_SCALE_BF16)) throw not_plain();
        const void* Wp = W.data_ptr();
        at::Tensor codes = empty({(int64_t)cb}, at::kByte, W);
        at::Tensor scales = empty({g == 0 ? 1 : K / g, N}, format == FQ_SCALE_BF16 ? at::kBFloat16 : at::kHalf, W);
        void *cp = codes.data_ptr(), *sp = scales.data_ptr(), *s = stream();
        call("fq_quantize_sf", [&] { return lib.quantize_sf(Wp, K, N, bits, g, format, cp, sp, s); });
        return Py_BuildValue("(NN)", THPVariable_Wrap(std::move(codes)), THPVariable_Wrap(std::move(scales)));
    });
}

// quantize_w4a8(W, group_size)
PyObject* quantize_w4a8(PyObject*, PyObject* const* a, Py_ssize_t n) {
    return guarded([&]() -> PyObject* {
        arguments(n, 2);
        const at::Tensor& W = tensor(a[0]);
        if (W.dim() != 2 || W.scalar_type() != at::kHalf || !W.is_contiguous()) throw not_plain();
        const int g = integer(a[1]);
        const int64_t K = W.size(0), N = W.size(1);
        if (lib.zscale_bytes(K, N, g) == 0) throw not_plain();
        const void* Wp = W.data_ptr();
        at::Tensor codes = empty({(int64_t)lib.codes_bytes(K, N, 4)}, at::kByte, W), z = empty({g == 0 ? 1 : K / g, N}, at::kByte, W),
                   t = empty({N}, at::kHalf, W);
        void *cp = codes.data_ptr(), *tp = t.data_ptr(), *s = stream();
        uint8_t* zp = (uint8_t*)z.data_ptr();
        call("fq_quantize_w4a8", [&] { return lib.quantize_w4a8(Wp, K, N, g, cp, zp, tp, s); });
        return Py_BuildValue("(NNN)", THPVariable_Wrap(std::move(codes)), THPVariable_Wrap(std::move(z)), THPVariable_Wrap(std::move(t)));
    });
}

// bind(FqError, addresses of the functions of `lib`, in its order)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
    constexpr Py_ssize_t count = sizeof(lib) / sizeof(void*);
    if (n != 1 + count) {
        PyErr_SetString(PyExc_TypeError, "bind: wrong number of functions");
        return nullptr;
    }
    void* p[count];
    for (Py_ssize_t i = 0; i < count; ++i) {
        p[i] = PyLong_AsVoidPtr(a[1 + i]);
        if (!p[i]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "bind: no address");
            return nullptr;
        }
    }
    memcpy(&lib, p, sizeof(lib));
    Py_INCREF(a[0]);
    Py_XSETREF(fq_error, a[0]);
    Py_RETURN_NONE;
}

#define FQ_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FQ_METHOD(gemm),     FQ_METHOD(gemm_grouped),  FQ_METHOD(quantize_act_i8), FQ_METHOD(gemm_w4a8),
                         FQ_METHOD(quantize), FQ_METHOD(quantize_w4a8), FQ_METHOD(bind),            {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fqcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fqcall(void) { return PyModule_Create(&module); }
