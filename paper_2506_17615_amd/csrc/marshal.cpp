// The binding's ordinary call, in native code: a torch tensor's checks, its pointer and the current stream are a few
// nanoseconds here and 0.2-0.3 us per tensor through the interpreter, where a call with 16 partial sums spent 11 us
// before its first launch (5 us with two; a launch itself takes the host 2.4 us).
//
// Every function takes the arguments of the Python function of its name, positionally, and returns the status of the C
// call it made, or -1 if it made none.  It makes the call only for arguments that the Python function would accept and
// hand on as they are: plain torch.Tensor objects on a GPU, of the expected type, contiguous and long enough, plain ints
// in range.  Everything else -- subclasses, wrappers without memory, anything to be refused -- is -1, and
// the caller goes through the checks in Python, which also word the errors.  Nothing is kept between calls.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "equarx.h"

namespace {

constexpr int kNotPlain = -1;
constexpr auto kBF16 = at::ScalarType::BFloat16;
constexpr auto kInt8 = at::ScalarType::Char;
constexpr auto kFloat = at::ScalarType::Float;

// The library's entry points, as binding.load() found them.
struct Library {
#define EQUARX_CALLS(X)                                                                                              \
    X(equarx_quantize) X(equarx_quantize_batch) X(equarx_dequantize) X(equarx_reduce_stage) X(equarx_reduce_quantized) \
    X(equarx_reduce_quantized_static) X(equarx_reduce_quantized_fused_ends) X(equarx_reduce_fused)                   \
    X(equarx_reduce_variant) X(equarx_reduce_variant_hops) X(equarx_reduce_flat) X(equarx_quantize_strided)          \
    X(equarx_dequantize_strided) X(equarx_reduce_stage_strided) X(equarx_reduce_quantized_strided)                   \
    X(equarx_reduce_fused_strided) X(equarx_reduce_variant_strided) X(equarx_reduce_variant_hops_strided)
#define X(name) decltype(&::name) name;
    EQUARX_CALLS(X)
#undef X
} lib;
bool bound = false;

// A tensor whose memory can be handed on as it is.
const at::Tensor *plain(PyObject *o)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor &t = THPVariable_Unpack(o);
    return t.defined() && t.is_cuda() && t.has_storage() && t.is_contiguous() ? &t : nullptr;
}

struct Buffer {
    void *ptr = nullptr;
    int64_t count = 0;
    const at::Tensor *t = nullptr;

    bool of(PyObject *o, at::ScalarType type)
    {
        t = plain(o);
        if (!t || t->scalar_type() != type) return false;
        ptr = t->data_ptr();
        count = t->numel();
        return true;
    }
    bool of(PyObject *o, at::ScalarType type, int64_t at_least) { return of(o, type) && count >= at_least; }
};

// None, or any contiguous device tensor.
struct Workspace {
    void *ptr = nullptr;
    size_t bytes = 0;

    bool of(PyObject *o)
    {
        if (o == Py_None) return true;
        const at::Tensor *t = plain(o);
        if (!t) return false;
        ptr = t->data_ptr();
        bytes = (size_t)t->numel() * t->element_size();
        return true;
    }
};

bool integer(PyObject *o, long long lo, long long hi, long long &v)
{
    if (!PyLong_CheckExact(o)) return false;
    int overflow = 0;
    v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return !overflow && v >= lo && v <= hi;
}

bool a_block(PyObject *o, int32_t &block)
{
    long long v;
    if (!integer(o, 32, 512, v) || (v & (v - 1))) return false;
    block = (int32_t)v;
    return true;
}

bool a_chunks(PyObject *o, int32_t &chunks) { return a_block(o, chunks) && chunks <= 128; }

bool some_flags(PyObject *o, uint32_t &flags)
{
    long long v;
    if (!integer(o, 0, UINT32_MAX, v)) return false;
    flags = (uint32_t)v;
    return true;
}

// A list or tuple of 1..EQUARX_MAX_PARTIALS tensors of one type, each of n elements (n < 0: the first one's length,
// which is then n) or, with `exactly` false, of at least n.
struct Buffers {
    void *ptr[EQUARX_MAX_PARTIALS];
    int32_t count = 0;

    bool of(PyObject *o, at::ScalarType type, int64_t &n, bool exactly = true)
    {
        if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) return false;
        const Py_ssize_t size = PySequence_Fast_GET_SIZE(o);
        if (size < 1 || size > EQUARX_MAX_PARTIALS) return false;
        for (Py_ssize_t i = 0; i < size; ++i) {
            Buffer b;
            if (!b.of(PySequence_Fast_GET_ITEM(o, i), type)) return false;
            if (n < 0) n = b.count;
            if (exactly ? b.count != n : b.count < n) return false;
            ptr[i] = b.ptr;
        }
        count = (int32_t)size;
        return true;
    }
    template <typename T>
    T *const *as() const { return reinterpret_cast<T *const *>(ptr); }
    const void *const *partials() const { return ptr; }
};

void *stream() { return c10::hip::getCurrentHIPStream().stream(); }

int64_t blocks(int64_t n, int32_t block) { return (n + block - 1) / block; }
int64_t row(int64_t n, int64_t multiple) { return (n + multiple - 1) / multiple * multiple; }

template <typename F, typename... A>
int call(F f, A... args)
{
    void *const on = stream();      // may throw: not without the interpreter lock
    int status;
    Py_BEGIN_ALLOW_THREADS
    status = f(args..., on);
    Py_END_ALLOW_THREADS
    return status;
}

// What every chain call starts with: partials, block (or chunks), and an output of their length.
struct Chain {
    Buffers x;
    int64_t n = -1;
    int32_t block = 0;
    Buffer out;

    bool of(PyObject *partials, PyObject *b, PyObject *o, bool strided = false)
    {
        return x.of(partials, kBF16, n) && n > 0 && (strided ? a_chunks(b, block) : a_block(b, block)) && out.of(o, kBF16, n);
    }
};

// The wire a chain call may keep: both arrays or neither.
struct KeptWire {
    Buffer codes, scales;

    bool of(PyObject *c, PyObject *s, const Chain &k)
    {
        if (c == Py_None && s == Py_None) return true;
        return codes.of(c, kInt8, k.x.count * row(k.n, 16)) && scales.of(s, kFloat, k.x.count * row(blocks(k.n, k.block), 4));
    }
};

int quantize(PyObject *const *a, bool strided)
{
    Buffer x, codes, scales;
    int32_t b;
    if (!x.of(a[0], kBF16) || x.count == 0 || !(strided ? a_chunks(a[1], b) : a_block(a[1], b))) return kNotPlain;
    if (!codes.of(a[2], kInt8, x.count)) return kNotPlain;
    if (!scales.of(a[3], kFloat, strided ? x.count / b : blocks(x.count, b))) return kNotPlain;
    return call(strided ? lib.equarx_quantize_strided : lib.equarx_quantize, x.ptr, x.count, b,
                static_cast<int8_t *>(codes.ptr), static_cast<float *>(scales.ptr));
}

int dequantize(PyObject *const *a, bool strided)
{
    Buffer codes, scales, out;
    int32_t b;
    if (!codes.of(a[0], kInt8) || codes.count == 0 || !(strided ? a_chunks(a[2], b) : a_block(a[2], b))) return kNotPlain;
    if (!scales.of(a[1], kFloat, strided ? codes.count / b : blocks(codes.count, b))) return kNotPlain;
    if (!out.of(a[3], kBF16, codes.count)) return kNotPlain;
    return call(strided ? lib.equarx_dequantize_strided : lib.equarx_dequantize, static_cast<const int8_t *>(codes.ptr),
                static_cast<const float *>(scales.ptr), codes.count, b, out.ptr);
}

int reduce_stage(PyObject *const *a, bool strided)
{
    Buffer cin, sin, local, cout, sout;
    int32_t b;
    if (!local.of(a[2], kBF16) || local.count == 0 || !(strided ? a_chunks(a[3], b) : a_block(a[3], b))) return kNotPlain;
    const int64_t n = local.count, ns = strided ? n / b : blocks(n, b);
    if (!cin.of(a[0], kInt8, n) || !cout.of(a[4], kInt8, n)) return kNotPlain;
    if (!sin.of(a[1], kFloat, ns) || !sout.of(a[5], kFloat, ns)) return kNotPlain;
    return call(strided ? lib.equarx_reduce_stage_strided : lib.equarx_reduce_stage, static_cast<const int8_t *>(cin.ptr),
                static_cast<const float *>(sin.ptr), local.ptr, n, b, static_cast<int8_t *>(cout.ptr),
                static_cast<float *>(sout.ptr));
}

int quantize_batch(PyObject *const *a)
{
    Buffers x, codes, scales;
    int64_t n = -1;
    int32_t block;
    if (!x.of(a[0], kBF16, n) || n == 0 || !a_block(a[1], block)) return kNotPlain;
    int64_t nb = blocks(n, block);
    if (!codes.of(a[2], kInt8, n, false) || !scales.of(a[3], kFloat, nb, false)) return kNotPlain;
    if (codes.count != x.count || scales.count != x.count) return kNotPlain;
    return call(lib.equarx_quantize_batch, x.partials(), codes.as<int8_t>(), scales.as<float>(), x.count, n, block);
}

int reduce_quantized(PyObject *const *a)
{
    Chain k;
    Workspace w;
    KeptWire wire;
    if (!k.of(a[0], a[1], a[2]) || !w.of(a[3]) || !wire.of(a[4], a[5], k)) return kNotPlain;
    return call(lib.equarx_reduce_quantized, k.x.partials(), k.x.count, k.n, k.block, k.out.ptr, w.ptr, w.bytes,
                static_cast<int8_t *>(wire.codes.ptr), static_cast<float *>(wire.scales.ptr));
}

int reduce_quantized_static(PyObject *const *a)
{
    Chain k;
    if (!k.of(a[0], a[1], a[2])) return kNotPlain;
    return call(lib.equarx_reduce_quantized_static, k.x.partials(), k.x.count, k.n, k.block, k.out.ptr);
}

int reduce_quantized_fused_ends(PyObject *const *a)
{
    Chain k;
    Workspace w;
    if (!k.of(a[0], a[1], a[2]) || !w.of(a[3])) return kNotPlain;
    return call(lib.equarx_reduce_quantized_fused_ends, k.x.partials(), k.x.count, k.n, k.block, k.out.ptr, w.ptr, w.bytes);
}

int reduce_fused(PyObject *const *a)
{
    Chain k;
    KeptWire wire;
    if (!k.of(a[0], a[1], a[2]) || !wire.of(a[3], a[4], k)) return kNotPlain;
    return call(lib.equarx_reduce_fused, k.x.partials(), k.x.count, k.n, k.block, k.out.ptr,
                static_cast<int8_t *>(wire.codes.ptr), static_cast<float *>(wire.scales.ptr));
}

int reduce_variant(PyObject *const *a, bool strided)
{
    Chain k;
    uint32_t flags;
    if (!k.of(a[0], a[1], a[3], strided) || !some_flags(a[2], flags)) return kNotPlain;
    return call(strided ? lib.equarx_reduce_variant_strided : lib.equarx_reduce_variant, k.x.partials(), k.x.count, k.n,
                k.block, flags, k.out.ptr);
}

int reduce_variant_hops(PyObject *const *a, bool strided)
{
    Chain k;
    uint32_t flags;
    Workspace w;
    if (!k.of(a[0], a[1], a[3], strided) || !some_flags(a[2], flags)) return kNotPlain;
    if ((strided && a[4] == Py_None) || !w.of(a[4])) return kNotPlain;
    return call(strided ? lib.equarx_reduce_variant_hops_strided : lib.equarx_reduce_variant_hops, k.x.partials(),
                k.x.count, k.n, k.block, flags, k.out.ptr, w.ptr, w.bytes);
}

int reduce_quantized_strided(PyObject *const *a)
{
    Chain k;
    Workspace w;
    if (!k.of(a[0], a[1], a[2], true) || !w.of(a[3])) return kNotPlain;
    return call(lib.equarx_reduce_quantized_strided, k.x.partials(), k.x.count, k.n, k.block, k.out.ptr, w.ptr, w.bytes);
}

int reduce_fused_strided(PyObject *const *a)
{
    Chain k;
    if (!k.of(a[0], a[1], a[2], true)) return kNotPlain;
    return call(lib.equarx_reduce_fused_strided, k.x.partials(), k.x.count, k.n, k.block, k.out.ptr);
}

int reduce_flat(PyObject *const *a)
{
    Buffer local, out, codes_out, scales_out;
    Buffers codes, scales;
    int32_t block;
    if (!local.of(a[0], kBF16) || local.count == 0 || !a_block(a[3], block)) return kNotPlain;
    int64_t n = local.count, nb = blocks(n, block);
    if (!codes.of(a[1], kInt8, n, false) || !scales.of(a[2], kFloat, nb, false)) return kNotPlain;
    if (codes.count != scales.count) return kNotPlain;
    if (a[4] != Py_None && !out.of(a[4], kBF16, n)) return kNotPlain;
    if (a[5] != Py_None || a[6] != Py_None) {
        if (!codes_out.of(a[5], kInt8, n) || !scales_out.of(a[6], kFloat, nb)) return kNotPlain;
    }
    return call(lib.equarx_reduce_flat, local.ptr, codes.as<const int8_t>(), scales.as<const float>(), codes.count, n, block,
                out.ptr, static_cast<int8_t *>(codes_out.ptr), static_cast<float *>(scales_out.ptr));
}

// The Python-callable form of f: kArgs positional arguments; an exception from torch is "not plain" too.
template <int kArgs, typename F>
PyObject *enter(PyObject *const *a, Py_ssize_t count, F f)
{
    int status = kNotPlain;
    if (!bound) {
        PyErr_SetString(PyExc_RuntimeError, "not bound to a library");
        return nullptr;
    }
    if (count == kArgs) {
        try {
            status = f(a);
        } catch (...) {
            status = kNotPlain;
        }
    }
    return PyLong_FromLong(status);
}

#define ENTRY(args, name, expr)                                                       \
    PyObject *py_##name(PyObject *, PyObject *const *a, Py_ssize_t count)             \
    {                                                                                 \
        return enter<args>(a, count, [](PyObject *const *a) { return expr; });        \
    }
ENTRY(4, equarx_quantize, quantize(a, false))
ENTRY(4, equarx_quantize_batch, quantize_batch(a))
ENTRY(4, equarx_dequantize, dequantize(a, false))
ENTRY(6, equarx_reduce_stage, reduce_stage(a, false))
ENTRY(6, equarx_reduce_quantized, reduce_quantized(a))
ENTRY(3, equarx_reduce_quantized_static, reduce_quantized_static(a))
ENTRY(4, equarx_reduce_quantized_fused_ends, reduce_quantized_fused_ends(a))
ENTRY(5, equarx_reduce_fused, reduce_fused(a))
ENTRY(4, equarx_reduce_variant, reduce_variant(a, false))
ENTRY(5, equarx_reduce_variant_hops, reduce_variant_hops(a, false))
ENTRY(7, equarx_reduce_flat, reduce_flat(a))
ENTRY(4, equarx_quantize_strided, quantize(a, true))
ENTRY(4, equarx_dequantize_strided, dequantize(a, true))
ENTRY(6, equarx_reduce_stage_strided, reduce_stage(a, true))
ENTRY(4, equarx_reduce_quantized_strided, reduce_quantized_strided(a))
ENTRY(3, equarx_reduce_fused_strided, reduce_fused_strided(a))
ENTRY(4, equarx_reduce_variant_strided, reduce_variant(a, true))
ENTRY(5, equarx_reduce_variant_hops_strided, reduce_variant_hops(a, true))
#undef ENTRY

// bind({name: address}): where the library's entry points are.
PyObject *bind(PyObject *, PyObject *table)
{
    Library found;
#define X(name)                                                                       \
    {                                                                                 \
        PyObject *at = PyDict_Check(table) ? PyDict_GetItemString(table, #name) : nullptr; \
        void *p = at ? PyLong_AsVoidPtr(at) : nullptr;                                \
        if (!p) {                                                                     \
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "no address for " #name); \
            return nullptr;                                                           \
        }                                                                             \
        found.name = reinterpret_cast<decltype(&::name)>(p);                          \
    }
    EQUARX_CALLS(X)
#undef X
    lib = found;
    bound = true;
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
#define X(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_##name)), METH_FASTCALL, nullptr},
    EQUARX_CALLS(X)
#undef X
    {"bind", bind, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal()
{
    PyObject *m = PyModule_Create(&module);
    if (m && PyModule_AddStringConstant(m, "torch_version", EQUARX_TORCH) < 0) Py_CLEAR(m);
    return m;
}
