// The short way from a Python call to the C ABI: checks, output extents, the output tensor and the call in one native function.
//
// run(op, x, w, bias, scale, integers and flags ...) returns the output tensor, a status code other than SW_OK, or None for whatever
// it does not take (other types, layouts, devices, arguments out of range): the caller then goes the long way, which takes it or says
// why not.  Nothing is kept between calls but the entry points' addresses.
//
// Measured on one 256 x 256 image under a 3 x 3 filter, whose kernel takes 3.7 us in a graph, calls one after the other: 4.4 to 4.9 us a call,
// 7.05 in Python through ctypes (2.3 of which the checks, 1.4 torch.empty, 0.6 ctypes).
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ops/empty.h>
#include <c10/hip/HIPStream.h>

#include "../../../include/swconv.h"

namespace {

enum Op { kConv1d, kPool1d, kPool2d, kConv2d, kBiasRelu, kDilated, kDepthwise, kDepthwiseBiasRelu, kDepthwiseBf16, kS8, kS8Requant, kS8Nhwc, kNhwc, kOps };

struct Entries {
    decltype(&sw_conv1d) conv1d;
    decltype(&sw_pool1d) pool1d;
    decltype(&sw_pool2d) pool2d;
    decltype(&sw_conv2d) conv2d;
    decltype(&sw_conv2d_bias_relu) bias_relu;
    decltype(&sw_conv2d_dilated) dilated;
    decltype(&sw_conv2d_depthwise) depthwise;
    decltype(&sw_conv2d_depthwise_bias_relu) depthwise_bias_relu;
    decltype(&sw_conv2d_depthwise_bf16) depthwise_bf16;
    decltype(&sw_conv2d_s8) s8;
    decltype(&sw_conv2d_s8_requant) s8_requant;
    decltype(&sw_conv2d_s8_nhwc) s8_nhwc;
    decltype(&sw_conv2d_s8_nhwc_requant) s8_nhwc_requant;
    decltype(&sw_conv2d_nhwc) nhwc;
    decltype(&sw_conv2d_bf16_nhwc) bf16_nhwc;
    decltype(&sw_conv2d_f16_nhwc) f16_nhwc;
};
Entries g_entry;
constexpr int kEntries = sizeof(Entries) / sizeof(void*);
bool g_bound = false;
bool g_host = false;        // bound to entry points that work on host memory, without a stream

// a contiguous tensor on the GPU of that type and number of dimensions, or null
const at::Tensor* tensor(PyObject* o, at::ScalarType type, int dims)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return (g_host ? t.is_cpu() : t.is_cuda()) && t.scalar_type() == type && t.dim() == dims && t.is_contiguous() ? &t : nullptr;
}

// an exact Python integer within int
bool integer(PyObject* o, int* v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    const long long l = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow || l < INT32_MIN || l > INT32_MAX) return false;
    *v = (int)l;
    return true;
}

bool flag(PyObject* o, int* v)
{
    if (o != Py_True && o != Py_False) return false;
    *v = o == Py_True;
    return true;
}

// output positions along one axis, 0 for what has none (as sw_out_dim_dilated)
int64_t extent(int64_t n, int64_t k, int stride, int pad, int dil)
{
    if (n <= 0 || k <= 0 || stride <= 0 || pad < 0 || dil <= 0) return 0;
    const int64_t span = n + 2 * (int64_t)pad - (dil * (k - 1) + 1);
    return span < 0 ? 0 : span / stride + 1;
}

bool fits(const at::Tensor& t)
{
    for (int64_t d : t.sizes())
        if (d > INT32_MAX) return false;
    return true;
}

// without the interpreter's lock, which is taken back however the scope ends
class Unlocked {
    PyThreadState* const state_ = PyEval_SaveThread();

public:
    Unlocked() = default;
    Unlocked(const Unlocked&) = delete;
    ~Unlocked() { PyEval_RestoreThread(state_); }
};

// f(output, stream): the entry point on addresses that were taken before (one that there is not, of a transformed tensor, raises as it is)
template <class F>
PyObject* call(const at::Tensor& x, at::IntArrayRef shape, at::ScalarType type, F&& f)
{
    for (int64_t d : shape)
        if (d <= 0) return nullptr;
    at::Tensor y = at::empty(shape, x.options().dtype(type));
    if (g_host ? !y.is_cpu() : !y.is_cuda()) return nullptr;
    void* const out = y.mutable_data_ptr();
    void* const stream = g_host ? nullptr : static_cast<void*>(c10::hip::getCurrentHIPStream().stream());
    int rc;
    {
        const Unlocked unlocked;
        rc = f(out, stream);
    }
    return rc == SW_OK ? THPVariable_Wrap(std::move(y)) : PyLong_FromLong(rc);
}

// the address of a tensor's memory, whatever an entry point takes it for
struct Address {
    const void* p;
    Address(const at::Tensor* t) : p(t ? t->const_data_ptr() : nullptr) {}
    template <class T>
    operator const T*() const { return static_cast<const T*>(p); }
};

// null: not taken
PyObject* run_op(int op, PyObject* const* a, Py_ssize_t n)
{
    constexpr auto f32 = at::kFloat, bf16 = at::kBFloat16, f16 = at::kHalf, s8 = at::kChar, s32 = at::kInt;
    // a: x, w, bias, scale (None where an op has none), then integers
    if (n < 6) return nullptr;
    PyObject *const px = a[0], *const pw = a[1], *const pb = a[2], *const ps = a[3];
    int i[5] = {0, 0, 0, 0, 0};
    const Py_ssize_t ni = n - 4;
    auto ints = [&](Py_ssize_t want) {
        if (ni < want) return false;
        for (Py_ssize_t k = 0; k < want; ++k)
            if (!integer(a[4 + k], &i[k])) return false;
        return true;
    };
    if (op == kConv1d) {
        const at::Tensor *x = tensor(px, f32, 2), *w = tensor(pw, f32, 1);
        if (!x || !w || !ints(2) || !fits(*w)) return nullptr;
        const int64_t rows = x->size(0), len = x->size(1);
        const int k = (int)w->size(0);
        const Address xa(x), wa(w);
        return call(*x, {rows, extent(len, k, i[0], i[1], 1)}, f32,
                    [&](void* y, void* st) { return g_entry.conv1d(xa, wa, (float*)y, rows, len, k, i[0], i[1], st); });
    }
    if (op == kPool1d) {
        const at::Tensor* x = tensor(px, f32, 2);
        if (!x || !ints(3)) return nullptr;
        const int64_t rows = x->size(0), len = x->size(1);
        const Address xa(x);
        return call(*x, {rows, extent(len, i[0], i[1], 0, 1)}, f32,
                    [&](void* y, void* st) { return g_entry.pool1d(xa, (float*)y, rows, len, i[0], i[1], i[2], st); });
    }
    if (op == kPool2d) {
        const at::Tensor* x = tensor(px, f32, 4);
        if (!x || !ints(5) || !fits(*x)) return nullptr;
        const auto d = x->sizes();
        const Address xa(x);
        return call(*x, {d[0], d[1], extent(d[2], i[0], i[2], i[3], 1), extent(d[3], i[1], i[2], i[3], 1)}, f32, [&](void* y, void* st) {
            return g_entry.pool2d(xa, (float*)y, (int)d[0], (int)d[1], (int)d[2], (int)d[3], i[0], i[1], i[2], i[3], i[4], st);
        });
    }
    if (op == kConv2d || op == kBiasRelu || op == kDilated || op == kS8 || op == kS8Requant) {
        // channel first: x [N,C,H,W], w [K,C,R,S]; integers stride, pad, then relu or dilation
        const bool q = op == kS8 || op == kS8Requant;
        const at::Tensor *x = tensor(px, q ? s8 : f32, 4), *w = tensor(pw, q ? s8 : f32, 4);
        if (!x || !w || !ints(2) || !fits(*x) || !fits(*w)) return nullptr;
        const auto d = x->sizes(), e = w->sizes();
        if (e[1] != d[1]) return nullptr;
        const int N = (int)d[0], C = (int)d[1], H = (int)d[2], W = (int)d[3], K = (int)e[0], R = (int)e[2], S = (int)e[3];
        int relu = 0, dil = 1;
        const at::Tensor *b = nullptr, *sc = nullptr;
        if (op == kDilated) {
            if (ni < 3 || !integer(a[6], &dil)) return nullptr;
        } else if (op != kConv2d && op != kS8) {
            if (ni < 3 || !flag(a[6], &relu)) return nullptr;
            if (pb != Py_None && (!(b = tensor(pb, q ? s32 : f32, 1)) || b->size(0) != K)) return nullptr;
            if (q && (!(sc = tensor(ps, f32, 1)) || sc->size(0) != K)) return nullptr;
        }
        const Address xa(x), wa(w), ba(b), sa(sc);
        return call(*x, {N, K, extent(H, R, i[0], i[1], dil), extent(W, S, i[0], i[1], dil)}, op == kS8 ? s32 : op == kS8Requant ? s8 : f32, [&](void* y, void* st) {
            switch (op) {
            case kConv2d: return g_entry.conv2d(xa, wa, (float*)y, N, C, K, H, W, R, S, i[0], i[1], st);
            case kBiasRelu: return g_entry.bias_relu(xa, wa, ba, (float*)y, N, C, K, H, W, R, S, i[0], i[1], relu, st);
            case kDilated: return g_entry.dilated(xa, wa, (float*)y, N, C, K, H, W, R, S, i[0], i[1], dil, st);
            case kS8: return g_entry.s8(xa, wa, (int32_t*)y, N, C, K, H, W, R, S, i[0], i[1], st);
            default: return g_entry.s8_requant(xa, wa, ba, sa, (int8_t*)y, N, C, K, H, W, R, S, i[0], i[1], relu, st);
            }
        });
    }
    if (op == kDepthwise || op == kDepthwiseBiasRelu || op == kDepthwiseBf16) {
        const auto type = op == kDepthwiseBf16 ? bf16 : f32;
        const at::Tensor *x = tensor(px, type, 4), *w = tensor(pw, f32, 4);
        if (!x || !w || !ints(2) || !fits(*x) || !fits(*w)) return nullptr;
        const auto d = x->sizes(), e = w->sizes();
        if (e[0] != d[1] || e[1] != 1) return nullptr;
        const int N = (int)d[0], C = (int)d[1], H = (int)d[2], W = (int)d[3], R = (int)e[2], S = (int)e[3];
        int relu = 0;
        const at::Tensor* b = nullptr;
        if (op == kDepthwiseBiasRelu) {
            if (ni < 3 || !flag(a[6], &relu)) return nullptr;
            if (pb != Py_None && (!(b = tensor(pb, f32, 1)) || b->size(0) != C)) return nullptr;
        }
        const Address xa(x), wa(w), ba(b);
        return call(*x, {N, C, extent(H, R, i[0], i[1], 1), extent(W, S, i[0], i[1], 1)}, type, [&](void* y, void* st) {
            switch (op) {
            case kDepthwise: return g_entry.depthwise(xa, wa, (float*)y, N, C, H, W, R, S, i[0], i[1], st);
            case kDepthwiseBiasRelu: return g_entry.depthwise_bias_relu(xa, wa, ba, (float*)y, N, C, H, W, R, S, i[0], i[1], relu, st);
            default: return g_entry.depthwise_bf16(xa, wa, (unsigned short*)y, N, C, H, W, R, S, i[0], i[1], st);
            }
        });
    }
    if (op == kS8Nhwc || op == kNhwc) {
        // channel last: x [N,H,W,C], w [K,R,S,C]; integers stride, pad, dilation, relu
        if (!THPVariable_CheckExact(px)) return nullptr;
        const auto type = op == kS8Nhwc ? s8 : THPVariable_Unpack(px).scalar_type();
        if (op == kNhwc && type != f32 && type != bf16 && type != f16) return nullptr;
        const at::Tensor *x = tensor(px, type, 4), *w = tensor(pw, type, 4);
        int relu = 0;
        if (!x || !w || !ints(3) || ni < 4 || !flag(a[7], &relu) || !fits(*x) || !fits(*w)) return nullptr;
        const auto d = x->sizes(), e = w->sizes();
        if (e[3] != d[3]) return nullptr;
        const int N = (int)d[0], H = (int)d[1], W = (int)d[2], C = (int)d[3], K = (int)e[0], R = (int)e[1], S = (int)e[2];
        const at::Tensor *b = nullptr, *sc = nullptr;
        const bool q = op == kS8Nhwc && ps != Py_None;
        if (q && (!(sc = tensor(ps, f32, 1)) || sc->size(0) != K)) return nullptr;
        if ((q || op == kNhwc) && pb != Py_None && (!(b = tensor(pb, q ? s32 : f32, 1)) || b->size(0) != K)) return nullptr;
        const Address xa(x), wa(w), ba(b), sa(sc);
        const auto out = op == kNhwc ? type : q ? s8 : s32;
        return call(*x, {N, extent(H, R, i[0], i[1], i[2]), extent(W, S, i[0], i[1], i[2]), K}, out, [&](void* y, void* st) {
            if (op == kS8Nhwc)
                return q ? g_entry.s8_nhwc_requant(xa, wa, ba, sa, (int8_t*)y, N, H, W, C, K, R, S, i[0], i[1], relu, st)
                         : g_entry.s8_nhwc(xa, wa, (int32_t*)y, N, H, W, C, K, R, S, i[0], i[1], st);
            if (type == f32) return g_entry.nhwc(xa, wa, ba, (float*)y, N, H, W, C, K, R, S, i[0], i[1], i[2], relu, st);
            if (type == bf16) return g_entry.bf16_nhwc(xa, wa, ba, y, N, H, W, C, K, R, S, i[0], i[1], i[2], relu, st);
            return g_entry.f16_nhwc(xa, wa, ba, y, N, H, W, C, K, R, S, i[0], i[1], i[2], relu, st);
        });
    }
    return nullptr;
}

PyObject* run(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    int op;
    if (g_bound && n >= 1 && integer(a[0], &op)) {
        try {
            if (PyObject* y = run_op(op, a + 1, n - 1)) return y;
        } catch (...) {
            // (a tensor without storage, memory that is not there: the long way says it as it always has)
        }
        if (PyErr_Occurred()) PyErr_Clear();
    }
    Py_RETURN_NONE;
}

// bind(addresses of the entry points in the order of Entries, host = False); host: entry points for tensors in host memory, as tests have them
PyObject* bind(PyObject*, PyObject* args)
{
    PyObject* addresses;
    int host = 0;
    if (!PyArg_ParseTuple(args, "O|p", &addresses, &host)) return nullptr;
    if (!PyTuple_CheckExact(addresses) || PyTuple_GET_SIZE(addresses) != kEntries) {
        PyErr_SetString(PyExc_ValueError, "one address per entry point");
        return nullptr;
    }
    void* p[kEntries];
    for (int k = 0; k < kEntries; ++k) {
        p[k] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(addresses, k));
        if (!p[k]) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null entry point");
            return nullptr;
        }
    }
    static_assert(sizeof p == sizeof g_entry, "entries are addresses");
    std::memcpy(&g_entry, p, sizeof g_entry);
    g_host = host != 0;
    g_bound = true;
    Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"run", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(run)), METH_FASTCALL, nullptr},
    {"bind", bind, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_swnative", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__swnative(void) { return PyModule_Create(&kModule); }
