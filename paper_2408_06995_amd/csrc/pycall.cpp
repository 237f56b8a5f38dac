// The calls of the binding that programs make per layer and step, as a CPython extension (_fpqcall): argument
// marshalling only, as in binding.py, without ctypes.
//
// A layer call of a small layer costs what the host needs to make it.  Through ctypes the marshalling took 5.5 us per
// call (2.9 of them torch.cuda.current_stream(), the rest one wrapper object per argument) next to 3.5 us for the C call
// with its launch; here it takes under 1 us: tensors give their address through data_ptr(), the stream comes from the raw
// stream query.  Arguments, names and defaults are those of the Python functions that this replaces; the functions of
// libfpq.so are looked up once through the resolver that binding.py registers, and a status other than FPQ_OK goes to its
// checker, which raises FpqError.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <string.h>

#include "../../include/fpq.h"

namespace {

PyObject* g_resolve = nullptr;      // resolver(name) -> address of the C function
PyObject* g_check = nullptr;        // checker(status, name): raises
PyObject *g_format = nullptr, *g_problem = nullptr, *g_array = nullptr;   // fpq_format_t, fpq_gemm_problem_t, ctypes.Array
PyObject *s_type, *s_data_ptr, *s_numel, *s_element_size, *s_shape;
PyObject *g_get_device = nullptr, *g_get_stream = nullptr;

constexpr int kBad = 1;             // a Python error is set (statuses of the library are <= 0)

struct Args {
    PyObject* const* a;
    bool bad = false;

    // (after a failure the remaining arguments are not looked at: the first error is the one reported)
    long long integer(int i)
    {
        if (bad) return 0;
        PyObject* o = a[i];
        if (PyLong_CheckExact(o)) {
            const long long v = PyLong_AsLongLong(o);
            if (v == -1 && PyErr_Occurred()) bad = true;
            return v;
        }
        PyObject* n = PyNumber_Long(o);
        if (!n) { bad = true; return 0; }
        const long long v = PyLong_AsLongLong(n);
        Py_DECREF(n);
        if (v == -1 && PyErr_Occurred()) bad = true;
        return v;
    }
    int i(int k) { return (int)integer(k); }
    // a size: whole numbers only, no conversion
    int64_t l(int k)
    {
        if (bad) return 0;
        if (!PyLong_Check(a[k])) {
            PyErr_Format(PyExc_TypeError, "sizes are ints, not %s", Py_TYPE(a[k])->tp_name);
            bad = true;
            return 0;
        }
        return (int64_t)integer(k);
    }
    int d(int k) { return (int)l(k); }
    float f(int k)
    {
        if (bad) return 0.0f;
        const double v = PyFloat_AsDouble(a[k]);
        if (v == -1.0 && PyErr_Occurred()) bad = true;
        return (float)v;
    }
    // data_ptr() of a tensor; None: null
    void* ptr_of(PyObject* o)
    {
        if (bad || o == Py_None) return nullptr;
        PyObject* r = PyObject_CallMethodNoArgs(o, s_data_ptr);
        if (!r) { bad = true; return nullptr; }
        void* p = PyLong_AsVoidPtr(r);
        Py_DECREF(r);
        if (!p && PyErr_Occurred()) bad = true;
        return p;
    }
    void* p(int k) { return ptr_of(a[k]); }
    float* fp(int k) { return static_cast<float*>(p(k)); }
    uint8_t* bp(int k) { return static_cast<uint8_t*>(p(k)); }
    size_t method(PyObject* o, PyObject* name)
    {
        if (bad) return 0;
        PyObject* r = PyObject_CallMethodNoArgs(o, name);
        if (!r) { bad = true; return 0; }
        const size_t v = PyLong_AsSize_t(r);
        Py_DECREF(r);
        if (v == (size_t)-1 && PyErr_Occurred()) bad = true;
        return v;
    }
    size_t numel(int k) { return method(a[k], s_numel); }
    size_t bytes(int k) { return a[k] == Py_None ? 0 : method(a[k], s_numel) * method(a[k], s_element_size); }
    // dimension `dim` of a tensor that must have `ndim` (0: any number)
    int64_t size(int k, int dim, int ndim)
    {
        if (bad) return 0;
        PyObject* sh = PyObject_GetAttr(a[k], s_shape);
        if (!sh) { bad = true; return 0; }
        const Py_ssize_t have = PySequence_Size(sh);
        if (have < 0 || (ndim && have != ndim)) {
            if (have >= 0) PyErr_Format(PyExc_ValueError, "a tensor of %d dimensions expected, not %zd", ndim, have);
            Py_DECREF(sh);
            bad = true;
            return 0;
        }
        PyObject* d = PySequence_GetItem(sh, dim);
        Py_DECREF(sh);
        if (!d) { bad = true; return 0; }
        const long long v = PyLong_AsLongLong(d);
        Py_DECREF(d);
        if (v == -1 && PyErr_Occurred()) bad = true;
        return v;
    }
    // the ctypes structure, or anything with four elements (e, m, b, c)
    fpq_format_t fmt(int k)
    {
        fpq_format_t r;
        memset(&r, 0, sizeof r);
        if (bad) return r;
        PyObject* o = a[k];
        if (PyTuple_CheckExact(o) && PyTuple_GET_SIZE(o) == 4) {
            Args t{&PyTuple_GET_ITEM(o, 0)};
            r.ebits = t.i(0); r.mbits = t.i(1); r.bias = t.i(2); r.maxval = t.f(3);
            bad |= t.bad;
            return r;
        }
        const int is = PyObject_IsInstance(o, g_format);
        if (is < 0) { bad = true; return r; }
        if (is) {
            Py_buffer b;
            if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE)) { bad = true; return r; }
            memcpy(&r, b.buf, sizeof r);
            PyBuffer_Release(&b);
            return r;
        }
        PyObject* t = PySequence_Tuple(o);
        if (!t) { bad = true; return r; }
        if (PyTuple_GET_SIZE(t) == 4) {
            Args u{&PyTuple_GET_ITEM(t, 0)};
            r.ebits = u.i(0); r.mbits = u.i(1); r.bias = u.i(2); r.maxval = u.f(3);
            bad |= u.bad;
        } else {
            PyErr_SetString(PyExc_TypeError, "a format is (e, m, b, c)");
            bad = true;
        }
        Py_DECREF(t);
        return r;
    }
    // the current torch stream of the current device
    void* stream()
    {
        if (bad) return nullptr;
        if (!g_get_stream) {
            PyObject* m = PyImport_ImportModule("torch._C");
            if (!m) { bad = true; return nullptr; }
            g_get_device = PyObject_GetAttrString(m, "_cuda_getDevice");
            g_get_stream = PyObject_GetAttrString(m, "_cuda_getCurrentRawStream");
            Py_DECREF(m);
            if (!g_get_device || !g_get_stream) { Py_CLEAR(g_get_stream); bad = true; return nullptr; }
        }
        PyObject* d = PyObject_CallNoArgs(g_get_device);
        if (!d) { bad = true; return nullptr; }
        PyObject* r = PyObject_CallOneArg(g_get_stream, d);
        Py_DECREF(d);
        if (!r) { bad = true; return nullptr; }
        void* p = PyLong_AsVoidPtr(r);
        Py_DECREF(r);
        if (!p && PyErr_Occurred()) bad = true;
        return p;
    }
};

template <typename F>
F resolve(F, const char* name)
{
    PyObject* r = g_resolve ? PyObject_CallFunction(g_resolve, "s", name) : nullptr;
    if (!r) {
        if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, "_fpqcall is not set up");
        return nullptr;
    }
    void* p = PyLong_AsVoidPtr(r);
    Py_DECREF(r);
    return reinterpret_cast<F>(p);
}

// Calls the library with the interpreter released, as ctypes does (a full queue makes a launch wait).
template <typename F, typename... V>
int invoke(const Args& A, F fn, V... v)
{
    if (A.bad) return kBad;
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = fn(v...);
    Py_END_ALLOW_THREADS
    return st;
}

#define FN(name)                                     \
    static decltype(&name) fn = nullptr;             \
    if (!fn && !(fn = resolve(&name, #name))) return kBad

// a: arguments in order, missing trailing ones replaced by their defaults
int do_gemm(Args& A)
{
    FN(fpq_gemm);
    return invoke(A, fn, A.p(0), A.i(1), A.fmt(2), A.f(3), A.fp(4), A.p(5), A.fmt(6), A.fp(7), A.fp(8), A.fp(9), A.l(10), A.l(11),
                  A.l(12), A.i(13), A.p(14), A.bytes(14), A.stream());
}
int do_gemm_noalloc(Args& A)
{
    FN(fpq_gemm_noalloc);
    return invoke(A, fn, A.p(0), A.i(1), A.fmt(2), A.f(3), A.fp(4), A.p(5), A.fmt(6), A.fp(7), A.fp(8), A.fp(9), A.l(10), A.l(11),
                  A.l(12), A.i(13), A.stream());
}
int do_conv2d(Args& A)
{
    FN(fpq_conv2d);
    return invoke(A, fn, A.p(0), A.i(1), A.fmt(2), A.f(3), A.fp(4), A.p(5), A.fmt(6), A.fp(7), A.fp(8), A.fp(9), A.l(10), A.l(11),
                  A.l(12), A.l(13), A.l(14), A.d(15), A.d(16), A.d(17), A.d(18), A.i(19), A.p(20), A.bytes(20), A.stream());
}
int do_gemm_codes_out(Args& A)
{
    FN(fpq_gemm_codes_out);
    return invoke(A, fn, A.p(0), A.i(1), A.fmt(2), A.f(3), A.fp(4), A.p(5), A.fmt(6), A.fp(7), A.fp(8), A.fmt(9), A.f(10), A.fp(11),
                  A.bp(12), A.l(13), A.l(14), A.l(15), A.i(16), A.p(17), A.bytes(17), A.stream());
}
int do_conv2d_codes_out(Args& A)
{
    FN(fpq_conv2d_codes_out);
    return invoke(A, fn, A.p(0), A.i(1), A.fmt(2), A.f(3), A.fp(4), A.p(5), A.fmt(6), A.fp(7), A.fp(8), A.fmt(9), A.f(10), A.fp(11),
                  A.bp(12), A.l(13), A.l(14), A.l(15), A.l(16), A.l(17), A.d(18), A.d(19), A.d(20), A.d(21), A.i(22), A.p(23),
                  A.bytes(23), A.stream());
}
int do_gemm_sparse(Args& A)
{
    FN(fpq_gemm_sparse);
    return invoke(A, fn, A.p(0), A.i(1), A.fmt(2), A.f(3), A.fp(4), A.p(5), A.fmt(6), A.fp(7), A.fp(8), A.fp(9), A.l(10), A.l(11),
                  A.l(12), A.p(13), A.bytes(13), A.stream());
}
int do_conv2d_sparse(Args& A)
{
    FN(fpq_conv2d_sparse);
    return invoke(A, fn, A.p(0), A.i(1), A.fmt(2), A.f(3), A.fp(4), A.p(5), A.fmt(6), A.fp(7), A.fp(8), A.fp(9), A.l(10), A.l(11),
                  A.l(12), A.l(13), A.l(14), A.d(15), A.d(16), A.d(17), A.d(18), A.p(19), A.bytes(19), A.stream());
}
int do_gemm_grouped(Args& A)
{
    FN(fpq_gemm_grouped);
    // the array of gemm_problems() and nothing else that has a buffer: the library reads addresses from it
    PyObject* of = PyObject_IsInstance(A.a[0], g_array) == 1 ? PyObject_GetAttr(A.a[0], s_type) : nullptr;
    const bool problems = of == g_problem;
    Py_XDECREF(of);
    if (!problems) {
        if (!PyErr_Occurred()) PyErr_Format(PyExc_TypeError, "problems: the array of gemm_problems(), not %s", Py_TYPE(A.a[0])->tp_name);
        return kBad;
    }
    Py_buffer b;
    if (PyObject_GetBuffer(A.a[0], &b, PyBUF_SIMPLE)) return kBad;
    const int st = invoke(A, fn, static_cast<const fpq_gemm_problem_t*>(b.buf), (int)(b.len / (Py_ssize_t)sizeof(fpq_gemm_problem_t)),
                          A.i(1), A.fmt(2), A.fmt(3), A.i(4), A.p(5), A.bytes(5), A.stream());
    PyBuffer_Release(&b);
    return st;
}
int do_absmax(Args& A)
{
    FN(fpq_absmax);
    return invoke(A, fn, A.fp(0), A.numel(0), A.f(1), A.fp(2), A.fp(3), A.p(4), A.bytes(4), A.stream());
}
int do_quantize(Args& A)
{
    FN(fpq_quantize);
    return invoke(A, fn, A.fp(0), A.numel(0), A.fmt(1), A.f(2), A.fp(3), A.bp(4), A.stream());
}
int do_quantize_nhwc(Args& A)
{
    FN(fpq_quantize_nhwc);
    return invoke(A, fn, A.fp(0), A.size(0, 0, 4), A.size(0, 1, 4), A.size(0, 2, 4), A.size(0, 3, 4),
                  A.fmt(1), A.f(2), A.fp(3), A.bp(4), A.stream());
}
int do_int_calibrate(Args& A)
{
    FN(fpq_int_calibrate);
    return invoke(A, fn, A.fp(0), A.numel(0), A.i(1), static_cast<fpq_int_params*>(A.p(2)), A.p(3), A.bytes(3), A.stream());
}
int do_int_quantize(Args& A)
{
    FN(fpq_int_quantize);
    return invoke(A, fn, A.fp(0), A.numel(0), A.i(1), A.f(2), (int32_t)A.i(3), static_cast<const fpq_int_params*>(A.p(4)), A.bp(5),
                  A.stream());
}
int do_int_gemm(Args& A)
{
    FN(fpq_int_gemm);
    return invoke(A, fn, A.bp(0), A.f(1), (int32_t)A.i(2), static_cast<const fpq_int_params*>(A.p(3)), A.p(4), A.i(5), A.fp(6),
                  static_cast<const int32_t*>(A.p(7)), A.fp(8), A.fp(9), A.l(10), A.l(11), A.l(12), A.p(13), A.bytes(13), A.stream());
}
int do_rl_step(Args& A)
{
    FN(fpq_rl_step);
    return invoke(A, fn, A.fp(0), A.fp(1), A.size(0, 0, 2), A.size(0, 1, 2), A.fmt(2), A.fp(3), A.fp(4), A.size(4, 0, 0), A.f(5), A.f(6), A.fp(7),
                  A.fp(8), A.p(9), A.bytes(9), A.stream());
}
int do_search_format(Args& A)
{
    FN(fpq_search_format);
    int32_t e[64], m[64];                        // the library takes at most 8 and says so
    int n = 0;
    PyObject* seq = PySequence_Fast(A.a[1], "encodings: a sequence of (e, m)");
    if (!seq) return kBad;
    const Py_ssize_t len = PySequence_Fast_GET_SIZE(seq);
    for (Py_ssize_t k = 0; k < len && k < 64 && !A.bad; ++k, ++n) {
        PyObject* t = PySequence_Tuple(PySequence_Fast_GET_ITEM(seq, k));
        if (!t || PyTuple_GET_SIZE(t) != 2) {
            if (t) PyErr_SetString(PyExc_ValueError, "encodings: a sequence of (e, m)");
            A.bad = true;
        } else {
            Args u{&PyTuple_GET_ITEM(t, 0)};
            e[k] = u.i(0);
            m[k] = u.i(1);
            A.bad |= u.bad;
        }
        Py_XDECREF(t);
    }
    Py_DECREF(seq);
    return invoke(A, fn, A.fp(0), A.numel(0), (const int32_t*)e, (const int32_t*)m, n, A.i(2), A.fp(3),
                  static_cast<fpq_search_result*>(A.p(4)), A.p(5), A.bytes(5), A.stream());
}

// ---- names, parameters and defaults

enum { kMaxParams = 26 };
struct Entry {
    const char* name;
    int (*run)(Args&);
    const char* params;                          // blank-separated
    int required;                                // the others default to 0 ("acc_mode") or None
    int count;
    PyObject* names[kMaxParams];
    PyObject* defaults[kMaxParams];
};

#define LAYER_HEAD "x x_is_fp32 fx sx sx_dev packed_w fw sw bias "
#define SPARSE_HEAD "x x_is_fp32 fx sx sx_dev packed_sparse fw sw bias "
Entry g_entries[] = {
    {"fpq_gemm", do_gemm, LAYER_HEAD "y M N K acc_mode workspace", 13},
    {"fpq_gemm_noalloc", do_gemm_noalloc, LAYER_HEAD "y M N K acc_mode", 13},
    {"fpq_conv2d", do_conv2d, LAYER_HEAD "y B Cin H W Cout kh kw stride pad acc_mode workspace", 19},
    {"fpq_gemm_codes_out", do_gemm_codes_out, LAYER_HEAD "fy sy sy_dev yq M N K acc_mode workspace", 16},
    {"fpq_conv2d_codes_out", do_conv2d_codes_out, LAYER_HEAD "fy sy sy_dev yq B Cin H W Cout kh kw stride pad acc_mode workspace", 22},
    {"fpq_gemm_sparse", do_gemm_sparse, SPARSE_HEAD "y M N K workspace", 13},
    {"fpq_conv2d_sparse", do_conv2d_sparse, SPARSE_HEAD "y B Cin H W Cout kh kw stride pad workspace", 19},
    {"fpq_gemm_grouped", do_gemm_grouped, "problems x_is_fp32 fx fw acc_mode workspace", 4},
    {"fpq_absmax", do_absmax, "x maxval absmax_out scale_out workspace", 5},
    {"fpq_quantize", do_quantize, "x f scale scale_dev codes", 5},
    {"fpq_quantize_nhwc", do_quantize_nhwc, "x f scale scale_dev codes", 5},
    {"fpq_int_calibrate", do_int_calibrate, "x bits params_out workspace", 4},
    {"fpq_int_quantize", do_int_quantize, "x bits scale zero_point params_dev codes", 6},
    {"fpq_int_gemm", do_int_gemm, "xcodes sx zx px_dev packed_w wbits sw zw bias y M N K workspace", 14},
    {"fpq_rl_step", do_rl_step, "w sw f alpha a lr reg_weight loss_out grad_out workspace", 10},
    {"fpq_search_format", do_search_format, "x encodings n_bias mse_out result workspace", 6},
};
constexpr int kEntries = sizeof g_entries / sizeof g_entries[0];

PyObject* call_entry(const Entry& e, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames)
{
    PyObject* a[kMaxParams];
    if (nargs > e.count) return PyErr_Format(PyExc_TypeError, "%s() takes %d arguments, %zd given", e.name, e.count, nargs);
    for (int k = 0; k < e.count; ++k) a[k] = k < nargs ? args[k] : nullptr;
    if (kwnames) {
        const Py_ssize_t nk = PyTuple_GET_SIZE(kwnames);
        for (Py_ssize_t q = 0; q < nk; ++q) {
            PyObject* name = PyTuple_GET_ITEM(kwnames, q);
            int k = 0;
            while (k < e.count && name != e.names[k] && PyUnicode_Compare(name, e.names[k]) != 0) ++k;
            if (k == e.count) return PyErr_Format(PyExc_TypeError, "%s() has no argument %R", e.name, name);
            if (a[k]) return PyErr_Format(PyExc_TypeError, "%s() got argument %R twice", e.name, name);
            a[k] = args[nargs + q];
        }
    }
    for (int k = 0; k < e.count; ++k)
        if (!a[k] && !(a[k] = e.defaults[k])) return PyErr_Format(PyExc_TypeError, "%s() misses argument %R", e.name, e.names[k]);
    Args A{a};
    const int st = e.run(A);
    if (st == kBad) return nullptr;
    if (st != FPQ_OK) return PyObject_CallFunction(g_check, "is", st, e.name);
    Py_RETURN_NONE;
}

template <int I>
PyObject* trampoline(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames)
{
    return call_entry(g_entries[I], args, nargs, kwnames);
}

PyObject* setup(PyObject*, PyObject* args)
{
    PyObject *r, *c, *f, *p, *a;
    if (!PyArg_ParseTuple(args, "OOOOO", &r, &c, &f, &p, &a)) return nullptr;
    PyObject** const to[] = {&g_resolve, &g_check, &g_format, &g_problem, &g_array};
    PyObject* const from[] = {r, c, f, p, a};
    for (int i = 0; i < 5; ++i) {
        Py_INCREF(from[i]);
        Py_XSETREF(*to[i], from[i]);
    }
    Py_RETURN_NONE;
}

PyMethodDef g_methods[kEntries + 2];

template <int I>
void fill_methods()
{
    if constexpr (I < kEntries) {
        g_methods[I] = PyMethodDef{g_entries[I].name, (PyCFunction)(void (*)(void))trampoline<I>, METH_FASTCALL | METH_KEYWORDS,
                                   g_entries[I].params};
        fill_methods<I + 1>();
    }
}

PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_fpqcall", "Native argument marshalling of the libfpq binding.", -1, g_methods,
                        nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fpqcall(void)
{
    s_type = PyUnicode_InternFromString("_type_");
    s_data_ptr = PyUnicode_InternFromString("data_ptr");
    s_numel = PyUnicode_InternFromString("numel");
    s_element_size = PyUnicode_InternFromString("element_size");
    s_shape = PyUnicode_InternFromString("shape");
    PyObject* zero = PyLong_FromLong(0);
    for (int i = 0; i < kEntries; ++i) {
        Entry& e = g_entries[i];
        e.count = 0;
        const char* p = e.params;
        while (*p) {
            const char* q = strchr(p, ' ');
            const size_t len = q ? (size_t)(q - p) : strlen(p);
            PyObject* name = PyUnicode_FromStringAndSize(p, (Py_ssize_t)len);
            PyUnicode_InternInPlace(&name);
            e.names[e.count] = name;
            e.defaults[e.count] = e.count < e.required ? nullptr : (strncmp(p, "acc_mode", 8) == 0 ? zero : Py_None);
            ++e.count;
            p += len + (q ? 1 : 0);
        }
    }
    fill_methods<0>();
    g_methods[kEntries] = PyMethodDef{"setup", setup, METH_VARARGS, "setup(resolver, checker, fpq_format_t, fpq_gemm_problem_t, ctypes.Array)"};
    g_methods[kEntries + 1] = PyMethodDef{nullptr, nullptr, 0, nullptr};
    return PyModule_Create(&g_module);
}
