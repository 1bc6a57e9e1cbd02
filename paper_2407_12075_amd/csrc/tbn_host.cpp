// Native form of the binding's everyday calls (module paper_2407_12075_amd._tbn_host).
//
// A call through ctypes costs the host 9 - 11 us (reading a dozen tensor attributes, allocating the output, looking up
// the stream, marshalling), more than the small kernels take.  Here the same checks, allocations and library calls are made on
// the C++ tensors.  Only the plain form of a call is taken: exact torch tensors that pass every check, integer arguments,
// outputs and workspaces left to the call, the current stream, no dispatch or function mode.  Anything else returns None and nothing has
// happened: the Python wrapper then runs its own code, which also words every error.
// One token through a 4096 x 4096 bfloat16 layer, calls in a row: 11.3 us through ctypes, 4.2 here (the kernel takes 3.5).
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <pybind11/pybind11.h>
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>

#include "../../include/tbn.h"

namespace {

PyObject *g_raise = nullptr;   // the binding's _raise(status)

// The library is loaded by the binding; its entry points are handed over as addresses so that there is one instance.
decltype(&tbn_pack_workspace_bytes) p_pack_workspace_bytes;
decltype(&tbn_pack_tile) p_pack_tile;
decltype(&tbn_linear_forward) p_linear_forward;
decltype(&tbn_conv2d_forward) p_conv2d_forward;
decltype(&tbn_linear_coltiled_workspace_bytes) p_coltiled_workspace_bytes;
decltype(&tbn_linear_coltiled_forward) p_coltiled_forward;
decltype(&tbn_sign_pack) p_sign_pack;
decltype(&tbn_linear_forward_binact) p_forward_binact;

constexpr int64_t kMaxElems = int64_t(1) << 40;

// a plain dense tensor on a GPU
const at::Tensor *plain(PyObject *o, int64_t dims = -1) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || (dims >= 0 && t.dim() != dims) || !t.is_contiguous()) return nullptr;
    constexpr c10::DispatchKeySet kWrapped({c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchGradWrapper,
                                            c10::DispatchKey::Functionalize, c10::DispatchKey::Python});
    if (t.key_set().has_any(kWrapped)) return nullptr;
    return &t;
}

const at::Tensor *plain(PyObject *o, at::ScalarType st, const at::Tensor &with) {
    const at::Tensor *t = plain(o);
    return t && t->scalar_type() == st && t->device() == with.device() ? t : nullptr;
}

bool activations(const at::Tensor &x, tbn_dtype &dt) {
    if (x.scalar_type() == at::kBFloat16) dt = TBN_BF16;
    else if (x.scalar_type() == at::kFloat) dt = TBN_F32;
    else return false;
    return true;
}

bool ordinary_context() {
    return !c10::impl::dispatch_mode_enabled() && !at::impl::torch_function_mode_enabled() &&
           !c10::impl::tls_local_dispatch_key_set().included_.has(c10::DispatchKey::FuncTorchDynamicLayerFrontMode);
}

bool integer(PyObject *o, int64_t lo, int64_t hi, int64_t &v) {
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return overflow == 0 && v >= lo && v <= hi;
}

bool pair(PyObject *o, int64_t lo, int64_t hi, int64_t &a, int64_t &b) {
    return PyTuple_CheckExact(o) && PyTuple_GET_SIZE(o) == 2 && integer(PyTuple_GET_ITEM(o, 0), lo, hi, a) &&
           integer(PyTuple_GET_ITEM(o, 1), lo, hi, b);
}

// n weights, n % k == 0 and a tile and alphas that hold them: what the library cannot see behind raw pointers
bool layer(int64_t rows, int64_t row_len, int64_t k, const at::Tensor &tile, const at::Tensor &alpha) {
    int64_t n;
    if (__builtin_mul_overflow(rows, row_len, &n) || n > kMaxElems || n % k != 0) return false;
    return tile.numel() >= (n / k + 31) / 32 && alpha.numel() >= 1 && alpha.numel() <= INT32_MAX;
}

void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

uint32_t *words(const at::Tensor &t) { return static_cast<uint32_t *>(t.data_ptr()); }
float *floats(const at::Tensor &t) { return static_cast<float *>(t.data_ptr()); }

// the wrapper's result, or the binding's exception for this status
PyObject *result(tbn_status st, PyObject *(*make)(const at::Tensor &, const at::Tensor &), const at::Tensor &a, const at::Tensor &b) {
    if (st == TBN_OK) return make(a, b);
    PyObject *r = PyObject_CallFunction(g_raise, "i", static_cast<int>(st));
    Py_XDECREF(r);
    return nullptr;
}
PyObject *one(const at::Tensor &a, const at::Tensor &) { return THPVariable_Wrap(a); }
PyObject *two(const at::Tensor &a, const at::Tensor &b) {
    PyObject *pa = THPVariable_Wrap(a), *pb = THPVariable_Wrap(b);
    PyObject *r = pa && pb ? PyTuple_Pack(2, pa, pb) : nullptr;
    Py_XDECREF(pa);
    Py_XDECREF(pb);
    return r;
}

// (x, tile, alpha, out_features, k, flags)
PyObject *linear_forward(PyObject *, PyObject *const *args, Py_ssize_t n_args) {
    HANDLE_TH_ERRORS
    int64_t out, k, flags;
    tbn_dtype dt;
    if (n_args != 6 || !ordinary_context()) Py_RETURN_NONE;
    const at::Tensor *x = plain(args[0], 2);
    if (!x || !activations(*x, dt)) Py_RETURN_NONE;
    const at::Tensor *tile = plain(args[1], at::kInt, *x), *alpha = plain(args[2], at::kFloat, *x);
    if (!tile || !alpha || !integer(args[3], 1, kMaxElems, out) || !integer(args[4], 1, INT32_MAX, k) ||
        !integer(args[5], 0, UINT32_MAX, flags) || !layer(out, x->size(1), k, *tile, *alpha))
        Py_RETURN_NONE;
    const int64_t M = x->size(0), in = x->size(1);
    at::Tensor y = at::empty({M, out}, x->options());
    tbn_status st;
    {
        pybind11::gil_scoped_release no_gil;
        st = p_linear_forward(x->data_ptr(), y.data_ptr(), dt, M, in, out, words(*tile), static_cast<int32_t>(k), floats(*alpha),
                              static_cast<int32_t>(alpha->numel()), static_cast<uint32_t>(flags), stream());
    }
    return result(st, one, y, y);
    END_HANDLE_TH_ERRORS
}

// (x, tile, alpha, out_channels, kh, kw, k, stride, pad, flags)
PyObject *conv2d_forward(PyObject *, PyObject *const *args, Py_ssize_t n_args) {
    HANDLE_TH_ERRORS
    int64_t O, kh, kw, k, sh, sw, ph, pw, flags;
    tbn_dtype dt;
    constexpr int64_t kSmall = 1 << 20;
    if (n_args != 10 || !ordinary_context()) Py_RETURN_NONE;
    const at::Tensor *x = plain(args[0], 4);
    if (!x || !activations(*x, dt)) Py_RETURN_NONE;
    const at::Tensor *tile = plain(args[1], at::kInt, *x), *alpha = plain(args[2], at::kFloat, *x);
    if (!tile || !alpha || !integer(args[3], 1, 1 << 24, O) || !integer(args[4], 1, 4096, kh) || !integer(args[5], 1, 4096, kw) ||
        !integer(args[6], 1, INT32_MAX, k) || !pair(args[7], 1, kSmall, sh, sw) || !pair(args[8], 0, kSmall, ph, pw) ||
        !integer(args[9], 0, UINT32_MAX, flags))
        Py_RETURN_NONE;
    const int64_t N = x->size(0), C = x->size(1), H = x->size(2), W = x->size(3);
    if (C > (1 << 24) || H + 2 * ph < kh || W + 2 * pw < kw || !layer(O, C * kh * kw, k, *tile, *alpha)) Py_RETURN_NONE;
    at::Tensor y = at::empty({N, O, (H + 2 * ph - kh) / sh + 1, (W + 2 * pw - kw) / sw + 1}, x->options());
    tbn_status st;
    {
        pybind11::gil_scoped_release no_gil;
        st = p_conv2d_forward(x->data_ptr(), y.data_ptr(), dt, N, C, H, W, O, static_cast<int32_t>(kh), static_cast<int32_t>(kw),
                              static_cast<int32_t>(sh), static_cast<int32_t>(sw), static_cast<int32_t>(ph), static_cast<int32_t>(pw),
                              words(*tile), static_cast<int32_t>(k), floats(*alpha), static_cast<int32_t>(alpha->numel()),
                              static_cast<uint32_t>(flags), stream());
    }
    return result(st, one, y, y);
    END_HANDLE_TH_ERRORS
}

// (x, tile, alpha, out_features, k, flags); the workspace is the call's own
PyObject *linear_coltiled_forward(PyObject *, PyObject *const *args, Py_ssize_t n_args) {
    HANDLE_TH_ERRORS
    int64_t out, k, flags;
    tbn_dtype dt;
    if (n_args != 6 || !ordinary_context()) Py_RETURN_NONE;
    const at::Tensor *x = plain(args[0], 2);
    if (!x || !activations(*x, dt)) Py_RETURN_NONE;
    const at::Tensor *tile = plain(args[1], at::kInt, *x), *alpha = plain(args[2], at::kFloat, *x);
    if (!tile || !alpha || !integer(args[3], 1, kMaxElems, out) || !integer(args[4], 1, INT32_MAX, k) ||
        !integer(args[5], 0, UINT32_MAX, flags) || !layer(out, x->size(1), k, *tile, *alpha))
        Py_RETURN_NONE;
    const int64_t M = x->size(0), in = x->size(1);
    const size_t need = std::max<size_t>(p_coltiled_workspace_bytes(dt, M, in, static_cast<int32_t>(k)), 16);
    at::Tensor y = at::empty({M, out}, x->options());
    at::Tensor ws = at::empty({static_cast<int64_t>(need)}, x->options().dtype(at::kByte));
    tbn_status st;
    {
        pybind11::gil_scoped_release no_gil;
        st = p_coltiled_forward(x->data_ptr(), y.data_ptr(), dt, M, in, out, words(*tile), static_cast<int32_t>(k), floats(*alpha),
                                static_cast<int32_t>(alpha->numel()), static_cast<uint32_t>(flags), ws.data_ptr(), need, stream());
    }
    return result(st, one, y, y);
    END_HANDLE_TH_ERRORS
}

// (x)
PyObject *sign_pack(PyObject *, PyObject *const *args, Py_ssize_t n_args) {
    HANDLE_TH_ERRORS
    tbn_dtype dt;
    if (n_args != 1 || !ordinary_context()) Py_RETURN_NONE;
    const at::Tensor *x = plain(args[0], 2);
    if (!x || !activations(*x, dt) || x->size(1) < 1) Py_RETURN_NONE;
    const int64_t M = x->size(0), in = x->size(1);
    at::Tensor bits = at::empty({M, (in + 31) / 32}, x->options().dtype(at::kInt));
    tbn_status st;
    {
        pybind11::gil_scoped_release no_gil;
        st = p_sign_pack(x->data_ptr(), dt, M, in, words(bits), stream());
    }
    return result(st, one, bits, bits);
    END_HANDLE_TH_ERRORS
}

// (xbits, in, tile, alpha, out_features, k, output is bfloat16, flags)
PyObject *linear_forward_binact(PyObject *, PyObject *const *args, Py_ssize_t n_args) {
    HANDLE_TH_ERRORS
    int64_t in, out, k, flags;
    if (n_args != 8 || !ordinary_context()) Py_RETURN_NONE;
    const at::Tensor *bits = plain(args[0], 2);
    if (!bits || bits->scalar_type() != at::kInt || !integer(args[1], 1, kMaxElems, in) || bits->size(1) != (in + 31) / 32)
        Py_RETURN_NONE;
    const at::Tensor *tile = plain(args[2], at::kInt, *bits), *alpha = plain(args[3], at::kFloat, *bits);
    if (!tile || !alpha || !integer(args[4], 1, kMaxElems, out) || !integer(args[5], 1, INT32_MAX, k) ||
        !integer(args[7], 0, UINT32_MAX, flags) || !layer(out, in, k, *tile, *alpha))
        Py_RETURN_NONE;
    const int64_t M = bits->size(0);
    const bool signs = (flags & TBN_FLAG_SIGN_OUT) != 0, bf16 = args[6] == Py_True;
    at::Tensor y = signs ? at::empty({M, (out + 31) / 32}, bits->options())
                         : at::empty({M, out}, bits->options().dtype(bf16 ? at::kBFloat16 : at::kFloat));
    tbn_status st;
    {
        pybind11::gil_scoped_release no_gil;
        st = p_forward_binact(words(*bits), y.data_ptr(), !signs && bf16 ? TBN_BF16 : TBN_F32, M, in, out, words(*tile),
                              static_cast<int32_t>(k), floats(*alpha), static_cast<int32_t>(alpha->numel()), static_cast<uint32_t>(flags),
                              stream());
    }
    return result(st, one, y, y);
    END_HANDLE_TH_ERRORS
}

// (w_real, k, n_alpha); the magnitudes are those of w_real, the outputs and the workspace the call's own
PyObject *pack_tile(PyObject *, PyObject *const *args, Py_ssize_t n_args) {
    HANDLE_TH_ERRORS
    int64_t k, n_alpha;
    if (n_args != 3 || !ordinary_context()) Py_RETURN_NONE;
    const at::Tensor *w = plain(args[0]);
    if (!w || w->scalar_type() != at::kFloat || !integer(args[1], 1, INT32_MAX, k) || !integer(args[2], 1, INT32_MAX, n_alpha))
        Py_RETURN_NONE;
    const int64_t n = w->numel();
    if (n < 1 || n % k != 0 || (n_alpha != 1 && n_alpha != k)) Py_RETURN_NONE;
    at::Tensor tile = at::empty({(n / k + 31) / 32}, w->options().dtype(at::kInt));
    at::Tensor alpha = at::empty({n_alpha}, w->options());
    const size_t need = std::max<size_t>(p_pack_workspace_bytes(n, static_cast<int32_t>(k), static_cast<int32_t>(n_alpha)), 8);
    at::Tensor ws = at::empty({static_cast<int64_t>(need)}, w->options().dtype(at::kByte));
    tbn_status st;
    {
        pybind11::gil_scoped_release no_gil;
        st = p_pack_tile(floats(*w), nullptr, n, static_cast<int32_t>(k), static_cast<int32_t>(n_alpha), words(tile), floats(alpha),
                         ws.data_ptr(), need, stream());
    }
    return result(st, two, tile, alpha);
    END_HANDLE_TH_ERRORS
}

// (raise, {name: address})
PyObject *init(PyObject *, PyObject *args) {
    PyObject *raise, *table;
    if (!PyArg_ParseTuple(args, "OO!", &raise, &PyDict_Type, &table)) return nullptr;
    bool ok = true;
    auto take = [&](auto &fn, const char *name) {
        PyObject *a = PyDict_GetItemString(table, name);
        void *p = a && PyLong_Check(a) ? PyLong_AsVoidPtr(a) : nullptr;
        ok = ok && p;
        fn = reinterpret_cast<std::decay_t<decltype(fn)>>(p);
    };
    take(p_pack_workspace_bytes, "tbn_pack_workspace_bytes");
    take(p_pack_tile, "tbn_pack_tile");
    take(p_linear_forward, "tbn_linear_forward");
    take(p_conv2d_forward, "tbn_conv2d_forward");
    take(p_coltiled_workspace_bytes, "tbn_linear_coltiled_workspace_bytes");
    take(p_coltiled_forward, "tbn_linear_coltiled_forward");
    take(p_sign_pack, "tbn_sign_pack");
    take(p_forward_binact, "tbn_linear_forward_binact");
    if (!ok) {
        PyErr_SetString(PyExc_ImportError, "_tbn_host: an entry point of the library is missing");
        return nullptr;
    }
    Py_INCREF(raise);
    Py_XDECREF(g_raise);
    g_raise = raise;
    Py_RETURN_NONE;
}

#define TBN_FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {TBN_FAST(linear_forward), TBN_FAST(conv2d_forward), TBN_FAST(linear_coltiled_forward), TBN_FAST(sign_pack),
                         TBN_FAST(linear_forward_binact), TBN_FAST(pack_tile), {"init", init, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_tbn_host", "plain calls of the binding on C++ tensors", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__tbn_host(void) { return PyModule_Create(&module); }
