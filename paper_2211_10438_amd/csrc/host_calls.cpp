// The common form of the Python entry points in native code: argument checks, output allocation and the call of the C ABI.
//
// A small layer's kernels take some 3 and 4 us, and a pass through the Python binding's quantizer and linear call took 13.7: attribute
// lookups, a dozen argument conversions of ctypes and two or three torch.empty per call (16 x 768 -> 3072, kernels included; now 8.8).  Here
// a call is one function with the arguments as they are.  It takes only what the binding's general code would pass through unchanged -- plain contiguous GPU tensors of the
// expected types, exact ints and bools, no out= or workspace= -- and returns None for anything else and for every status but
// SQ_OK, whereupon the binding's own code runs, with its checks, messages and exceptions.
// Of the calls that prepare a layer the GPU waits for two, the smoothing factors and the launch behind them: their conversions and
// allocations took some 12 and 8 us (statistics, factors and codes of 5120 x 20480: 188.8 us before, 183.5 with them native).
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/PythonTorchFunctionTLS.h>

#include "sqmi.h"

namespace {

struct Api {
    decltype(&sq_quantize_act) quantize_act;
    decltype(&sq_w8a8_linear) w8a8_linear;
    decltype(&sq_w8a8_linear_q8) w8a8_linear_q8;
    decltype(&sq_w8a8_bmm) w8a8_bmm;
    decltype(&sq_softmax_quant_p) softmax_quant_p;
    decltype(&sq_ln_quantize) ln_quantize;
    decltype(&sq_w8a8_attention) attention, attention_causal;
    decltype(&sq_workspace_bytes) workspace_bytes;
    decltype(&sq_smooth_scales) smooth_scales;
    decltype(&sq_act_absmax_per_channel) act_absmax;
    decltype(&sq_weight_absmax_per_in_channel) weight_absmax;
    decltype(&sq_prepare_weight) prepare_weight;
} api;

// Plain memory: no subclass, no wrapper of a transform, no mode that wants to see the allocation.
const at::Tensor* dense(PyObject* o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.has_storage() || !t.is_contiguous()) return nullptr;
    using K = c10::DispatchKey;
    if (t.key_set().has_any(c10::DispatchKeySet({K::Python, K::FuncTorchBatched, K::FuncTorchGradWrapper, K::Functionalize}))) return nullptr;
    return &t;
}
// ... on the GPU
const at::Tensor* plain(PyObject* o)
{
    const at::Tensor* t = dense(o);
    return t && t->is_cuda() ? t : nullptr;
}
const at::Tensor* plain(PyObject* o, at::ScalarType type)
{
    const at::Tensor* t = plain(o);
    return t && t->scalar_type() == type ? t : nullptr;
}
// None or a tensor of the type; false: neither
bool optional(PyObject* o, at::ScalarType type, const at::Tensor** t)
{
    *t = nullptr;
    if (o == Py_None) return true;
    return (*t = plain(o, type)) != nullptr;
}
bool half_type(at::ScalarType s, sq_dtype* d)
{
    if (s != at::kHalf && s != at::kBFloat16) return false;
    *d = s == at::kHalf ? SQ_F16 : SQ_BF16;
    return true;
}
bool half_dtype(PyObject* o, at::ScalarType* s, sq_dtype* d)
{
    if (!THPDtype_Check(o)) return false;
    *s = reinterpret_cast<THPDtype*>(o)->scalar_type;
    return half_type(*s, d);
}
bool integer(PyObject* o, long* v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    *v = PyLong_AsLongAndOverflow(o, &overflow);
    return !overflow;
}
bool layout_of(PyObject* o, sq_layout* l)
{
    long v;
    if (!integer(o, &v) || (v != SQ_ROW_MAJOR && v != SQ_TILED)) return false;
    *l = (sq_layout)v;
    return true;
}
bool flag(PyObject* o, bool* v)
{
    if (!PyBool_Check(o)) return false;
    *v = o == Py_True;
    return true;
}
bool real(PyObject* o, float* v)
{
    if (!PyFloat_CheckExact(o)) return false;
    *v = (float)PyFloat_AS_DOUBLE(o);
    return true;
}
bool modes() { return c10::impl::TorchDispatchModeTLS::any_modes_set() || at::impl::PythonTorchFunctionTLS::stack_len() > 0; }

at::Tensor empty(at::IntArrayRef sizes, const at::Tensor& like, at::ScalarType type) { return at::empty(sizes, at::TensorOptions().dtype(type).device(like.device())); }
// int8 [rows, k], tiled: padded to whole blocks and seen as its first rows
at::Tensor empty_codes(int64_t rows, int64_t k, sq_layout layout, const at::Tensor& like)
{
    const int64_t padded = layout == SQ_TILED ? (rows + 15) / 16 * 16 : rows;
    at::Tensor t = empty({padded, k}, like, at::kChar);
    return padded == rows ? t : t.narrow(0, 0, rows);
}
const void* ptr(const at::Tensor* t) { return t ? t->const_data_ptr() : nullptr; }
void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

// Workspace of a linear layer: a function of its sizes alone, remembered for the sizes this thread calls with.
size_t linear_workspace(int64_t t, int64_t c_i, int64_t c_o)
{
    struct Entry {
        int64_t t, c_i, c_o;
        size_t bytes;
    };
    static thread_local Entry table[256];
    Entry& e = table[(uint64_t)(t * 31 + c_i * 131 + c_o * 1031) & 255];
    if (e.t != t || e.c_i != c_i || e.c_o != c_o) e = Entry{t, c_i, c_o, api.workspace_bytes(SQ_OP_W8A8_LINEAR, t, c_i, c_o)};
    return e.bytes;
}

// The interpreter's lock is given up while outputs are allocated and kernels launched, as torch.empty and a ctypes call do: a first-time
// allocation can wait for the device, and other Python threads go on meanwhile.
struct Unlocked {
    PyThreadState* state = PyEval_SaveThread();
    Unlocked() = default;
    Unlocked(const Unlocked&) = delete;
    ~Unlocked() { PyEval_RestoreThread(state); }
};
PyObject* pair(const at::Tensor& a, PyObject* b) { return b ? Py_BuildValue("(NN)", THPVariable_Wrap(a), b) : nullptr; }

#define GENERAL Py_RETURN_NONE

// (x, mode, inv_s, static_scale, layout)
PyObject* quantize_act(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    const at::Tensor *x, *inv_s, *step;
    sq_dtype dt;
    sq_layout layout;
    long mode;
    if (n != 5 || modes() || !(x = plain(a[0])) || x->dim() != 2 || !half_type(x->scalar_type(), &dt) || !integer(a[1], &mode) || mode < 0 || mode > 2 ||
        !optional(a[2], at::kFloat, &inv_s) || !layout_of(a[4], &layout))
        GENERAL;
    const int64_t t = x->size(0), c_i = x->size(1);
    if (t <= 0 || c_i <= 0 || (layout == SQ_TILED && c_i % 64)) GENERAL;
    step = nullptr;
    if (mode == SQ_PER_TENSOR_STATIC && !(step = plain(a[3], at::kFloat))) GENERAL;
    at::Tensor xq, scale, ws;
    sq_status status;
    {
        Unlocked u;
        xq = empty_codes(t, c_i, layout, *x);
        if (mode != SQ_PER_TENSOR_STATIC) scale = empty({mode == SQ_PER_TOKEN_DYNAMIC ? t : 1}, *x, at::kFloat);
        size_t bytes = 0;
        if (mode == SQ_PER_TENSOR_DYNAMIC) {
            bytes = api.workspace_bytes(SQ_OP_QUANTIZE_ACT, t, c_i, 0);
            ws = empty({(int64_t)bytes}, *x, at::kByte);
        }
        float* sp = (float*)(step ? step->const_data_ptr() : scale.const_data_ptr());
        status = api.quantize_act(x->const_data_ptr(), dt, t, c_i, c_i, (const float*)ptr(inv_s), (sq_act_mode)mode, sp, (int8_t*)xq.data_ptr(), layout,
                                  bytes ? ws.data_ptr() : nullptr, bytes, stream());
    }
    if (status != SQ_OK) GENERAL;
    if (step) {
        Py_INCREF(a[3]);
        return pair(xq, a[3]);
    }
    return pair(xq, THPVariable_Wrap(scale));
    END_HANDLE_TH_ERRORS
}

struct Linear {
    const at::Tensor *xq, *xs, *wq, *ws, *bias, *res;
    int64_t t, c_i, c_o;
    bool relu, per_channel;
    sq_layout layout;
};
// xq, x_scale, wq, w_scale, bias, residual, relu, layout; residual of type `out`
bool linear_args(PyObject* const* a, at::ScalarType out, Linear* l)
{
    if (!(l->xq = plain(a[0], at::kChar)) || !(l->xs = plain(a[1], at::kFloat)) || !(l->wq = plain(a[2], at::kChar)) || !(l->ws = plain(a[3], at::kFloat)) ||
        !optional(a[4], at::kFloat, &l->bias) || !optional(a[5], out, &l->res) || !flag(a[6], &l->relu) || !layout_of(a[7], &l->layout) ||
        l->xq->dim() != 2 || l->wq->dim() != 2)
        return false;
    l->t = l->xq->size(0);
    l->c_i = l->xq->size(1);
    l->c_o = l->wq->size(0);
    if (l->t <= 0 || l->c_i <= 0 || l->c_o <= 0 || l->wq->size(1) != l->c_i) return false;
    l->per_channel = l->ws->numel() == l->c_o && l->c_o > 1;
    return l->ws->numel() == (l->per_channel ? l->c_o : 1) && (l->xs->numel() == 1 || l->xs->numel() == l->t);
}

// (xq, x_scale, wq, w_scale, bias, residual, relu, layout, out_dtype)
PyObject* w8a8_linear(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    Linear l;
    at::ScalarType type;
    sq_dtype dt;
    if (n != 9 || modes() || !half_dtype(a[8], &type, &dt) || !linear_args(a, type, &l)) GENERAL;
    at::Tensor y, ws;
    sq_status status;
    {
        Unlocked u;
        y = empty({l.t, l.c_o}, *l.xq, type);
        const size_t bytes = linear_workspace(l.t, l.c_i, l.c_o);
        if (bytes) ws = empty({(int64_t)bytes}, *l.xq, at::kByte);
        status = api.w8a8_linear((const int8_t*)ptr(l.xq), (const float*)ptr(l.xs), l.xs->numel() == l.t, (const int8_t*)ptr(l.wq), (const float*)ptr(l.ws),
                                 l.per_channel, (const float*)ptr(l.bias), ptr(l.res), l.relu, y.data_ptr(), dt, l.t, l.c_i, l.c_o, l.layout,
                                 bytes ? ws.data_ptr() : nullptr, bytes, stream());
    }
    if (status != SQ_OK) GENERAL;
    return THPVariable_Wrap(y);
    END_HANDLE_TH_ERRORS
}

// (xq, x_scale, wq, w_scale, bias, residual, relu, layout, mid_dtype, y_step, out_layout)
PyObject* w8a8_linear_q8(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    Linear l;
    at::ScalarType type;
    sq_dtype dt;
    sq_layout out_layout;
    const at::Tensor* step;
    if (n != 11 || modes() || !half_dtype(a[8], &type, &dt) || !linear_args(a, type, &l) || !(step = plain(a[9], at::kFloat)) ||
        !layout_of(a[10], &out_layout) || (out_layout == SQ_TILED && l.c_o % 64))
        GENERAL;
    at::Tensor y, ws;
    sq_status status;
    {
        Unlocked u;
        y = empty_codes(l.t, l.c_o, out_layout, *l.xq);
        const size_t bytes = linear_workspace(l.t, l.c_i, l.c_o);
        if (bytes) ws = empty({(int64_t)bytes}, *l.xq, at::kByte);
        status = api.w8a8_linear_q8((const int8_t*)ptr(l.xq), (const float*)ptr(l.xs), l.xs->numel() == l.t, (const int8_t*)ptr(l.wq),
                                    (const float*)ptr(l.ws), l.per_channel, (const float*)ptr(l.bias), ptr(l.res), l.relu, dt, (const float*)ptr(step),
                                    (int8_t*)y.data_ptr(), out_layout, l.t, l.c_i, l.c_o, l.layout, bytes ? ws.data_ptr() : nullptr, bytes, stream());
    }
    if (status != SQ_OK) GENERAL;
    return THPVariable_Wrap(y);
    END_HANDLE_TH_ERRORS
}

// (a, bm, trans_b, alpha, out_dtype)
PyObject* w8a8_bmm(PyObject*, PyObject* const* a, Py_ssize_t nargs)
{
    HANDLE_TH_ERRORS
    const at::Tensor *x, *y;
    at::ScalarType type;
    sq_dtype dt;
    bool trans;
    float alpha;
    if (nargs != 5 || modes() || !(x = plain(a[0], at::kChar)) || !(y = plain(a[1], at::kChar)) || x->dim() != 3 || y->dim() != 3 || !flag(a[2], &trans) ||
        !real(a[3], &alpha) || !half_dtype(a[4], &type, &dt))
        GENERAL;
    const int64_t b = x->size(0), m = x->size(1), k = x->size(2), n = y->size(trans ? 1 : 2);
    if (b <= 0 || m <= 0 || n <= 0 || k <= 0) GENERAL;
    at::Tensor c;
    sq_status status;
    {
        Unlocked u;
        c = empty({b, m, n}, *x, type);
        status = api.w8a8_bmm((const int8_t*)ptr(x), (const int8_t*)ptr(y), trans, alpha, c.data_ptr(), dt, b, m, n, k, m * k, n * k, m * n, stream());
    }
    if (status != SQ_OK) GENERAL;
    return THPVariable_Wrap(c);
    END_HANDLE_TH_ERRORS
}

// (s)
PyObject* softmax_quant_p(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    const at::Tensor* s;
    sq_dtype dt;
    if (n != 1 || modes() || !(s = plain(a[0])) || s->dim() < 1 || s->numel() <= 0 || !half_type(s->scalar_type(), &dt)) GENERAL;
    const int64_t cols = s->size(-1), rows = s->numel() / cols;
    at::Tensor p;
    sq_status status;
    {
        Unlocked u;
        p = empty(s->sizes(), *s, at::kChar);
        status = api.softmax_quant_p(ptr(s), dt, rows, cols, (int8_t*)p.data_ptr(), stream());
    }
    if (status != SQ_OK) GENERAL;
    return THPVariable_Wrap(p);
    END_HANDLE_TH_ERRORS
}

// (x, gamma, beta, eps, layout)
PyObject* ln_quantize(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    const at::Tensor *x, *g, *b;
    sq_dtype dt;
    float eps;
    sq_layout layout;
    if (n != 5 || modes() || !(x = plain(a[0])) || x->dim() != 2 || !half_type(x->scalar_type(), &dt) || !(g = plain(a[1], at::kFloat)) ||
        !(b = plain(a[2], at::kFloat)) || !real(a[3], &eps) || !layout_of(a[4], &layout))
        GENERAL;
    const int64_t t = x->size(0), c = x->size(1);
    if (t <= 0 || c <= 0 || (layout == SQ_TILED && c % 64)) GENERAL;
    at::Tensor xq, scale;
    sq_status status;
    {
        Unlocked u;
        xq = empty_codes(t, c, layout, *x);
        scale = empty({t}, *x, at::kFloat);
        status = api.ln_quantize(ptr(x), dt, t, c, (const float*)ptr(g), (const float*)ptr(b), eps, (float*)scale.data_ptr(), (int8_t*)xq.data_ptr(), layout, stream());
    }
    if (status != SQ_OK) GENERAL;
    return pair(xq, THPVariable_Wrap(scale));
    END_HANDLE_TH_ERRORS
}

// (q, k, v, alpha1, alpha2, out_dtype, causal)
PyObject* w8a8_attention(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    const at::Tensor *q, *k, *v;
    at::ScalarType type;
    sq_dtype dt;
    float a1, a2;
    bool causal;
    if (n != 7 || modes() || !(q = plain(a[0], at::kChar)) || !(k = plain(a[1], at::kChar)) || !(v = plain(a[2], at::kChar)) || q->dim() != 3 ||
        k->dim() != 3 || k->sizes() != v->sizes() || !real(a[3], &a1) || !real(a[4], &a2) || !half_dtype(a[5], &type, &dt) || !flag(a[6], &causal))
        GENERAL;
    const int64_t b = q->size(0), s_q = q->size(1), d = q->size(2), s_k = k->size(1);
    if (b <= 0 || s_q <= 0 || s_k <= 0 || d <= 0 || k->size(0) != b || k->size(2) != d) GENERAL;
    at::Tensor o;
    sq_status status;
    {
        Unlocked u;
        o = empty({b, s_q, d}, *q, type);
        status = (causal ? api.attention_causal : api.attention)((const int8_t*)ptr(q), (const int8_t*)ptr(k), (const int8_t*)ptr(v), a1, a2, o.data_ptr(),
                                                                 dt, b, s_q, s_k, d, s_q * d, s_k * d, s_k * d, s_q * d, nullptr, stream());
    }
    if (status != SQ_OK) GENERAL;
    return THPVariable_Wrap(o);
    END_HANDLE_TH_ERRORS
}

// (x_absmax, w_absmax, alpha): fp32 in host memory
PyObject* smooth_scales(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    const at::Tensor *x, *w;
    float alpha;
    if (n != 3 || modes() || !(x = dense(a[0])) || !(w = dense(a[1])) || !x->is_cpu() || !w->is_cpu() || x->scalar_type() != at::kFloat ||
        w->scalar_type() != at::kFloat || x->is_neg() || w->is_neg() || x->numel() != w->numel() || !real(a[2], &alpha))
        GENERAL;
    at::Tensor s, inv;
    sq_status status;
    {
        Unlocked u;
        s = empty(x->sizes(), *x, at::kFloat);
        inv = empty(x->sizes(), *x, at::kFloat);
        status = api.smooth_scales((const float*)ptr(x), (const float*)ptr(w), alpha, x->numel(), (float*)s.data_ptr(), (float*)inv.data_ptr());
    }
    if (status != SQ_OK) GENERAL;
    return pair(s, THPVariable_Wrap(inv));
    END_HANDLE_TH_ERRORS
}

// (x) / (w): fp32 maxima of the channels, of the rows
template <bool ROWS> PyObject* absmax(PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    const at::Tensor* x;
    sq_dtype dt;
    if (n != 1 || modes() || !(x = plain(a[0])) || x->dim() != 2 || !half_type(x->scalar_type(), &dt) || x->numel() <= 0) GENERAL;
    at::Tensor m;
    sq_status status;
    {
        Unlocked u;
        m = empty({x->size(ROWS ? 0 : 1)}, *x, at::kFloat);
        status = (ROWS ? api.weight_absmax : api.act_absmax)(ptr(x), dt, x->size(0), x->size(1), (float*)m.data_ptr(), stream());
    }
    if (status != SQ_OK) GENERAL;
    return THPVariable_Wrap(m);
    END_HANDLE_TH_ERRORS
}
PyObject* act_absmax_per_channel(PyObject*, PyObject* const* a, Py_ssize_t n) { return absmax<false>(a, n); }
PyObject* weight_absmax_per_in_channel(PyObject*, PyObject* const* a, Py_ssize_t n) { return absmax<true>(a, n); }

// (w, s, layout, per_channel)
PyObject* prepare_weight(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    const at::Tensor *w, *s;
    sq_dtype dt;
    sq_layout layout;
    bool per_channel;
    if (n != 4 || modes() || !(w = plain(a[0])) || w->dim() != 2 || !half_type(w->scalar_type(), &dt) || !optional(a[1], at::kFloat, &s) ||
        !layout_of(a[2], &layout) || !flag(a[3], &per_channel))
        GENERAL;
    const int64_t c_i = w->size(0), c_o = w->size(1);
    if (c_i <= 0 || c_o <= 0 || (layout == SQ_TILED && c_i % 64) || (s && s->numel() != c_i)) GENERAL;
    at::Tensor wq, scale, ws;
    sq_status status;
    {
        Unlocked u;
        wq = empty_codes(c_o, c_i, layout, *w);
        scale = empty({per_channel ? c_o : 1}, *w, at::kFloat);
        const size_t bytes = api.workspace_bytes(SQ_OP_PREPARE_WEIGHT, 0, c_i, c_o);
        ws = empty({(int64_t)bytes}, *w, at::kByte);
        status = api.prepare_weight(ptr(w), dt, (const float*)ptr(s), c_i, c_o, (int8_t*)wq.data_ptr(), layout, (float*)scale.data_ptr(), per_channel,
                                    ws.data_ptr(), bytes, stream());
    }
    if (status != SQ_OK) GENERAL;
    return pair(wq, THPVariable_Wrap(scale));
    END_HANDLE_TH_ERRORS
}

// Addresses of the library's functions, in the order of Api.
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    constexpr int N = 13;
    void* addr[N];
    if (n != N) return PyErr_Format(PyExc_TypeError, "%d addresses expected", N);
    for (int i = 0; i < N; ++i) {
        addr[i] = PyLong_AsVoidPtr(a[i]);
        if (!addr[i]) return PyErr_Occurred() ? nullptr : PyErr_Format(PyExc_ValueError, "null address");
    }
    static_assert(sizeof(Api) == sizeof(addr), "one address for each function");
    memcpy(&api, addr, sizeof(api));
    Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(bind), FAST(quantize_act), FAST(w8a8_linear), FAST(w8a8_linear_q8), FAST(w8a8_bmm), FAST(softmax_quant_p),
                         FAST(ln_quantize), FAST(w8a8_attention), FAST(smooth_scales), FAST(act_absmax_per_channel),
                         FAST(weight_absmax_per_in_channel), FAST(prepare_weight), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host_calls", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host_calls() { return PyModule_Create(&module); }
