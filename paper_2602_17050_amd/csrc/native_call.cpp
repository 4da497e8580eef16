// The calls of binding.py that a training or serving loop repeats, from Python arguments to the C ABI of
// include/mpzch.h: checks the tensors, takes their addresses and torch's current stream, and calls the function.
//
// A small call takes the GPU some 4 us, and through ctypes its arguments took the host as long again: every tensor's
// checks and address are attribute look-ups and method calls there.  mpzch_lookup 4.5 -> 2.9 us per call on the host,
// mpzch_remap 5.7 -> 2.9, mpzch_reset_rows 5.2 -> 2.9; launching a kernel is some 2.5 of it.
//
// The library itself is loaded by binding.py (which can be told to load another build); it hands the addresses of the
// functions over with bind().
#include <Python.h>

#include <ATen/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/mpzch.h"

namespace {

struct Functions {
#define MPZCH_CALLS(F)                                                                                              \
    F(mpzch_init_tensors) F(mpzch_remap) F(mpzch_remap_noalloc) F(mpzch_remap_reset) F(mpzch_remap_feature_ttl)      \
    F(mpzch_lookup) F(mpzch_lookup_stats) F(mpzch_lookup_gather) F(mpzch_reset_rows) F(mpzch_reset_rows_multi)       \
    F(mpzch_collect_delta) F(mpzch_gather_rows) F(mpzch_apply_delta) F(mpzch_remap_jagged_feature_ttl)               \
    F(mpzch_lookup_jagged) F(mpzch_reset_rows_jagged)
#define F(name) decltype(&::name) name = nullptr;
    MPZCH_CALLS(F)
#undef F
} g_call;

// An error is a Python exception that has been set.
struct Failed {};

[[noreturn]] void fail(PyObject *type, const char *text)
{
    PyErr_SetString(type, text);
    throw Failed{};
}

const at::Tensor &tensor(PyObject *o)
{
    if (!THPVariable_Check(o)) fail(PyExc_TypeError, "a tensor is expected");
    return THPVariable_Unpack(o);
}

// Dense device tensors, or the strided views of a table kept as 16-byte records (identities: every second int64,
// metadata: every fourth int32).  None: no tensor.
template <typename T>
T *address(PyObject *o, at::ScalarType type)
{
    if (o == Py_None) return nullptr;
    const at::Tensor &t = tensor(o);
    if (!t.is_cuda() || !(t.is_contiguous() || (t.dim() == 1 && (t.stride(0) == 2 || t.stride(0) == 4))))
        fail(PyExc_AssertionError, "device, dense tensors only");
    if (t.scalar_type() != type) fail(PyExc_AssertionError, "tensor of another type expected");
    return (T *)t.data_ptr();
}
int64_t *i64(PyObject *o) { return address<int64_t>(o, at::kLong); }
int32_t *i32(PyObject *o) { return address<int32_t>(o, at::kInt); }
uint8_t *u8(PyObject *o) { return address<uint8_t>(o, at::kByte); }
// entries of a tensor that the call cannot do without, and of one that may be left out
int64_t count(PyObject *o) { return tensor(o).numel(); }
int64_t count_if_given(PyObject *o) { return o == Py_None ? 0 : tensor(o).numel(); }

// whole numbers as a ctypes parameter takes them (numpy integers and the like too; the low bits of what does not fit)
int64_t number(PyObject *o)
{
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
    if (v == ~0ull && PyErr_Occurred()) throw Failed{};
    return (int64_t)v;
}
// ... and as int() makes them
int64_t number_of(PyObject *o)
{
    if (PyLong_CheckExact(o)) return number(o);
    PyObject *i = PyNumber_Long(o);
    if (!i) throw Failed{};
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(i);
    Py_DECREF(i);
    return (int64_t)v;
}
int32_t number32(PyObject *o) { return (int32_t)number(o); }

// A handle: a ctypes.c_void_p (what the create calls return), an address, None, or another pointer of ctypes.  (Not a text,
// which ctypes would pass as the address of its characters.)
PyObject *g_c_void_p = nullptr, *g_cast = nullptr;           // ctypes.c_void_p, ctypes.cast

void *value_of(PyObject *o)
{
    static PyObject *const name = PyUnicode_InternFromString("value");
    PyObject *v = PyObject_GetAttr(o, name);
    if (!v) throw Failed{};
    void *p = v == Py_None ? nullptr : PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    if (!p && PyErr_Occurred()) throw Failed{};
    return p;
}
void *pointer(PyObject *o)
{
    if (o == Py_None) return nullptr;
    if ((PyObject *)Py_TYPE(o) == g_c_void_p) return value_of(o);
    if (PyLong_Check(o)) {
        void *p = PyLong_AsVoidPtr(o);
        if (!p && PyErr_Occurred()) throw Failed{};
        return p;
    }
    if (!g_cast || PyUnicode_Check(o) || PyBytes_Check(o)) fail(PyExc_TypeError, "a handle is expected");
    PyObject *v = PyObject_CallFunctionObjArgs(g_cast, o, g_c_void_p, nullptr);
    if (!v) throw Failed{};
    struct Release {
        PyObject *o;
        ~Release() { Py_DECREF(o); }
    } release{v};
    return value_of(v);
}
template <typename T>
T *handle(PyObject *o) { return (T *)pointer(o); }

void *stream() { return (void *)c10::hip::getCurrentHIPStream().stream(); }

// a 2-D device tensor whose rows are dense (where host memory that the device can reach will do too: pinned_too,
// init_pinned_too)
mpzch_rows_t rows_of(PyObject *o, PyObject *init, bool pinned_too = false, bool init_pinned_too = false)
{
    const at::Tensor &t = tensor(o);
    if (t.dim() != 2 || t.stride(1) != 1 || !(t.is_cuda() || pinned_too)) fail(PyExc_AssertionError, "rows: 2-D device tensor with dense rows");
    const int64_t size = (int64_t)t.element_size();
    mpzch_rows_t r;
    r.rows = t.data_ptr();
    r.num_rows = t.size(0);
    r.row_bytes = t.size(1) * size;
    r.row_stride_bytes = t.stride(0) * size;
    r.init_row = nullptr;
    if (init != Py_None) {
        const at::Tensor &i = tensor(init);
        if (!(i.is_cuda() || (init_pinned_too && i.is_pinned())) || !i.is_contiguous() || i.numel() * (int64_t)i.element_size() != r.row_bytes)
            fail(PyExc_AssertionError, "init_row: one dense row on the device");
        r.init_row = i.data_ptr();
    }
    return r;
}

// a Python list or tuple
struct Sequence {
    PyObject *o;
    Py_ssize_t n;
    explicit Sequence(PyObject *s) : o(PySequence_Fast(s, "a list is expected"))
    {
        if (!o) throw Failed{};
        n = PySequence_Fast_GET_SIZE(o);
    }
    ~Sequence() { Py_DECREF(o); }
    Sequence(const Sequence &) = delete;
    Sequence &operator=(const Sequence &) = delete;
    PyObject *operator[](Py_ssize_t k) const { return PySequence_Fast_GET_ITEM(o, k); }
};

// Several tensors with the initial row of each.  The tensors beyond a list of initial rows that is shorter have no entry
// (rows == NULL: the reset of several tensors refuses it, the one of a group leaves that table alone); what a longer
// list holds beyond the tensors is not looked at.
struct RowsList {
    mpzch_rows_t v[MPZCH_MAX_GROUP_TABLES] = {};
    RowsList(const Sequence &t, const Sequence &init, bool may_be_none)
    {
        if (t.n > MPZCH_MAX_GROUP_TABLES) fail(PyExc_ValueError, "more tensors than a group has tables");
        for (Py_ssize_t k = 0; k < t.n && k < init.n; ++k)
            if (!(may_be_none && t[k] == Py_None)) v[k] = rows_of(t[k], init[k], false, true);
    }
};

// what the group calls take per table.  The library reads as many as the group has tables, which may be more than the list
// has: those are null, and it refuses them.
struct Tables {
    void *p[MPZCH_MAX_GROUP_TABLES] = {};
    Tables(PyObject *list, Py_ssize_t n)
    {
        const Sequence s(list);
        if (s.n != n || n > MPZCH_MAX_GROUP_TABLES) fail(PyExc_ValueError, "one tensor per table of the group");
        for (Py_ssize_t k = 0; k < n; ++k) p[k] = tensor(s[k]).data_ptr();
    }
};
Py_ssize_t length(PyObject *list)
{
    const Py_ssize_t n = PySequence_Size(list);
    if (n < 0) throw Failed{};
    return n;
}
// n + 1 of them; what a shorter list leaves out is zero
struct Offsets {
    int64_t v[MPZCH_MAX_GROUP_TABLES + 1] = {};
    Offsets(PyObject *list, Py_ssize_t n)
    {
        const Sequence s(list);
        if (s.n > n + 1 || n > MPZCH_MAX_GROUP_TABLES) fail(PyExc_IndexError, "one offset per table of the group and one more");
        for (Py_ssize_t k = 0; k < s.n; ++k) v[k] = number_of(s[k]);
    }
};

// Calls without the interpreter lock (as ctypes does): some calls wait for the device.
template <typename Fn, typename... A>
PyObject *call(Fn *fn, A... a)
{
    if (!fn) fail(PyExc_RuntimeError, "the library has not been loaded");
    mpzch_status_t st;
    Py_BEGIN_ALLOW_THREADS
    st = fn(a...);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong((long)st);
}

// a is the list of arguments, in the order in which binding.py passes them
PyObject *init_tensors(PyObject *const *a)
{
    return call(g_call.mpzch_init_tensors, handle<const mpzch_table_t>(a[0]), i64(a[1]), i32(a[2]), stream());
}
PyObject *remap(PyObject *const *a)
{
    return call(g_call.mpzch_remap, handle<mpzch_table_t>(a[0]), i64(a[1]), i32(a[2]), (const int64_t *)i64(a[3]), count(a[3]),
                number32(a[4]), i64(a[5]), i64(a[6]), count_if_given(a[6]), i64(a[7]), i64(a[8]), stream());
}
PyObject *remap_noalloc(PyObject *const *a)
{
    return call(g_call.mpzch_remap_noalloc, handle<const mpzch_table_t>(a[0]), i64(a[1]), i32(a[2]), (const int64_t *)i64(a[3]),
                count(a[3]), number32(a[4]), i64(a[5]), i64(a[6]), count_if_given(a[6]), i64(a[7]), i64(a[8]), stream());
}
PyObject *remap_feature_ttl(PyObject *const *a)
{
    if (a[4] != Py_None && count(a[4]) != count(a[3])) fail(PyExc_AssertionError, "one ttl per id");
    return call(g_call.mpzch_remap_feature_ttl, handle<mpzch_table_t>(a[0]), i64(a[1]), i32(a[2]), (const int64_t *)i64(a[3]),
                (const int32_t *)i32(a[4]), count(a[3]), number32(a[5]), i64(a[6]), i64(a[7]), count_if_given(a[7]), i64(a[8]), i64(a[9]),
                stream());
}
PyObject *remap_reset(PyObject *const *a)
{
    const mpzch_rows_t r = rows_of(a[9], a[10]);
    const int64_t num_rows = a[11] == Py_None ? r.num_rows : number(a[11]);
    return call(g_call.mpzch_remap_reset, handle<mpzch_table_t>(a[0]), i64(a[1]), i32(a[2]), (const int64_t *)i64(a[3]), count(a[3]),
                number32(a[4]), i64(a[5]), i64(a[6]), count_if_given(a[6]), i64(a[7]), i64(a[8]), r.rows, num_rows, r.row_bytes,
                r.row_stride_bytes, r.init_row, stream());
}
PyObject *lookup(PyObject *const *a)
{
    return call(g_call.mpzch_lookup, handle<const mpzch_table_t>(a[0]), (const int64_t *)i64(a[1]), (const int64_t *)i64(a[2]),
                count(a[2]), i64(a[3]), u8(a[4]), stream());
}
PyObject *lookup_stats(PyObject *const *a)
{
    return call(g_call.mpzch_lookup_stats, handle<mpzch_table_t>(a[0]), (const int64_t *)i64(a[1]), (const int64_t *)i64(a[2]),
                count(a[2]), i64(a[3]), u8(a[4]), i64(a[5]), stream());
}
PyObject *lookup_gather(PyObject *const *a)
{
    const mpzch_rows_t r = rows_of(a[3], Py_None);
    const at::Tensor &out = tensor(a[4]);
    if (!out.is_contiguous() || out.numel() * (int64_t)out.element_size() != count(a[2]) * r.row_bytes)
        fail(PyExc_AssertionError, "out_rows: one dense row per id");
    return call(g_call.mpzch_lookup_gather, handle<const mpzch_table_t>(a[0]), (const int64_t *)i64(a[1]), (const int64_t *)i64(a[2]),
                count(a[2]), (const void *)r.rows, r.num_rows, r.row_bytes, r.row_stride_bytes, out.data_ptr(), i64(a[5]),
                u8(a[6]), stream());
}
PyObject *reset_rows(PyObject *const *a)
{
    const mpzch_rows_t r = rows_of(a[2], a[3], true);
    const int64_t num_rows = a[4] == Py_None ? r.num_rows : number(a[4]);
    return call(g_call.mpzch_reset_rows, (const int64_t *)i64(a[0]), (const int64_t *)i64(a[1]), count(a[0]), r.rows, num_rows,
                r.row_bytes, r.row_stride_bytes, r.init_row, stream());
}
PyObject *reset_rows_multi(PyObject *const *a)
{
    const Sequence t(a[2]), init(a[3]);
    const RowsList r(t, init, false);
    return call(g_call.mpzch_reset_rows_multi, (const int64_t *)i64(a[0]), (const int64_t *)i64(a[1]), count(a[0]),
                (const mpzch_rows_t *)r.v, (int32_t)t.n, stream());
}
PyObject *collect_delta(PyObject *const *a)
{
    return call(g_call.mpzch_collect_delta, handle<const mpzch_table_t>(a[0]), (const int64_t *)i64(a[1]), (const int32_t *)i32(a[2]),
                number32(a[3]), i64(a[4]), i64(a[5]), count(a[4]), i64(a[6]), stream());
}
PyObject *gather_rows(PyObject *const *a)
{
    const mpzch_rows_t r = rows_of(a[2], Py_None);
    const at::Tensor &out = tensor(a[3]);
    if (!out.is_contiguous()) fail(PyExc_AssertionError, "out_rows: dense rows");
    return call(g_call.mpzch_gather_rows, (const int64_t *)i64(a[0]), (const int64_t *)i64(a[1]), count(a[0]), (const void *)r.rows,
                r.num_rows, r.row_bytes, r.row_stride_bytes, out.data_ptr(), stream());
}
PyObject *apply_delta(PyObject *const *a)
{
    mpzch_rows_t r{};
    const void *delta = nullptr;
    if (a[4] != Py_None) {
        r = rows_of(a[4], Py_None);
        delta = tensor(a[5]).data_ptr();
    }
    return call(g_call.mpzch_apply_delta, i64(a[0]), count(a[0]), (const int64_t *)i64(a[1]), (const int64_t *)i64(a[2]),
                (const int64_t *)i64(a[3]), count(a[1]), r.rows, r.num_rows, r.row_bytes, r.row_stride_bytes, delta, stream());
}
PyObject *remap_jagged(PyObject *const *a)
{
    const Py_ssize_t n = length(a[1]);
    Tables identities(a[1], n), metadata(a[2], n);
    const Offsets evicted(a[9], n);
    return call(g_call.mpzch_remap_jagged_feature_ttl, handle<mpzch_group_t>(a[0]), (int64_t *const *)identities.p,
                (int32_t *const *)metadata.p, (const int64_t *)i64(a[3]), (const int32_t *)i32(a[4]), (const int64_t *)i64(a[5]),
                count(a[3]), number32(a[6]), i64(a[7]), i64(a[8]), (const int64_t *)evicted.v, i64(a[10]), i64(a[11]), stream());
}
PyObject *lookup_jagged(PyObject *const *a)
{
    const Tables identities(a[1], length(a[1]));
    return call(g_call.mpzch_lookup_jagged, handle<mpzch_group_t>(a[0]), (const int64_t *const *)identities.p,
                (const int64_t *)i64(a[2]), (const int64_t *)i64(a[3]), count(a[2]), i64(a[4]), u8(a[5]), stream());
}
PyObject *reset_rows_jagged(PyObject *const *a)
{
    const Sequence t(a[4]), init(a[5]);
    const RowsList r(t, init, true);
    const Offsets evicted(a[2], t.n);
    return call(g_call.mpzch_reset_rows_jagged, handle<mpzch_group_t>(a[0]), (const int64_t *)i64(a[1]), (const int64_t *)evicted.v,
                (const int64_t *)i64(a[3]), (const mpzch_rows_t *)r.v, stream());
}

template <PyObject *(*FN)(PyObject *const *), int N>
PyObject *entry(PyObject *, PyObject *const *a, Py_ssize_t n)
{
    try {
        if (n != N) fail(PyExc_TypeError, "wrong number of arguments");
        return FN(a);
    } catch (const Failed &) {
        return nullptr;
    } catch (const std::exception &e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    }
}

// bind({name: address of the library's function})
PyObject *bind(PyObject *, PyObject *functions)
{
#define F(name)                                                                        \
    {                                                                                  \
        PyObject *v = PyDict_GetItemString(functions, #name);                          \
        void *p = v ? PyLong_AsVoidPtr(v) : nullptr;                                   \
        if (!p) {                                                                      \
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_KeyError, #name);             \
            return nullptr;                                                            \
        }                                                                              \
        g_call.name = (decltype(&::name))p;                                            \
    }
    MPZCH_CALLS(F)
#undef F
    if (!g_cast) {
        PyObject *ctypes = PyImport_ImportModule("ctypes");
        if (!ctypes) return nullptr;
        g_c_void_p = PyObject_GetAttrString(ctypes, "c_void_p");
        g_cast = g_c_void_p ? PyObject_GetAttrString(ctypes, "cast") : nullptr;
        Py_DECREF(ctypes);
        if (!g_cast) return nullptr;
    }
    Py_RETURN_NONE;
}

#define METHOD(name, n) {#name, (PyCFunction)(void (*)(void)) & entry<name, n>, METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {
    {"bind", bind, METH_O, nullptr},
    METHOD(init_tensors, 3), METHOD(remap, 9), METHOD(remap_noalloc, 9), METHOD(remap_feature_ttl, 10), METHOD(remap_reset, 12),
    METHOD(lookup, 5), METHOD(lookup_stats, 6), METHOD(lookup_gather, 7), METHOD(reset_rows, 5), METHOD(reset_rows_multi, 4),
    METHOD(collect_delta, 7), METHOD(gather_rows, 4), METHOD(apply_delta, 6), METHOD(remap_jagged, 12), METHOD(lookup_jagged, 6),
    METHOD(reset_rows_jagged, 6), {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&g_module); }
