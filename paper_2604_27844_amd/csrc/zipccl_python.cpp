/*
 * The calls of binding.py that a training or serving loop makes for every tensor, as a CPython module: what ctypes does
 * for them, without building a Python object per argument.  On small tensors the host's part of a call is what it lasts: of
 * the 5.5 us that a decompress of 200 003 values in 8 pieces took through ctypes, 2 were the conversion of its arguments
 * and 2.8 the launch.  Every function takes its arguments by position, releases the interpreter lock around the library's
 * call and returns its status.
 *
 * Device buffers are torch tensors: contiguous, on the GPU, or None.  A plain torch.Tensor or Parameter is looked at
 * directly; anything else is asked through its attributes, as Python would.
 */
#include <Python.h>

#include <exception>

#include <torch/csrc/autograd/python_variable.h>

#include "zipccl.h"

namespace {

PyObject* table_type;          /* binding.zipccl_table_t */
PyObject* host_array;          /* binding._host_array: anything with an element count per chunk -> uint64 array */
PyObject* resolve_stream;      /* binding._raw_stream_functions */
PyObject *raw_stream, *current_device;      /* what that returned, once asked */

/* Throughout: false = a Python exception is set. */

bool as_u64(PyObject* o, uint64_t* v)
{
    if (PyLong_CheckExact(o)) {
        *v = PyLong_AsUnsignedLongLongMask(o);
    } else {
        PyObject* i = PyNumber_Long(o);
        if (!i) return false;
        *v = PyLong_AsUnsignedLongLongMask(i);
        Py_DECREF(i);
    }
    return !(*v == (uint64_t)-1 && PyErr_Occurred());
}

/* an enum or a count that C takes as an int: no floats, as with ctypes */
bool as_int(PyObject* o, int* v)
{
    PyObject* i = PyNumber_Index(o);
    if (!i) return false;
    *v = (int)PyLong_AsUnsignedLongMask(i);
    Py_DECREF(i);
    return true;
}

bool as_buffer(PyObject* o, void** p, uint64_t* bytes)
{
    *p = nullptr;
    if (o == Py_None) {
        if (!bytes) return true;
    } else if (THPVariable_CheckExact(o)) {
        try {
            const at::Tensor& t = THPVariable_Unpack(o);
            if (!t.is_cuda() || !t.is_contiguous()) {
                PyErr_SetString(PyExc_ValueError, "device buffers must be contiguous tensors on the GPU");
                return false;
            }
            *p = t.data_ptr();
            if (bytes) *bytes = t.nbytes();
            return true;
        } catch (const std::exception& e) {
            PyErr_SetString(PyExc_RuntimeError, e.what());
            return false;
        }
    }
    auto truth = [](PyObject* r) { const int t = r ? PyObject_IsTrue(r) : -1; Py_XDECREF(r); return t; };
    const int cuda = truth(PyObject_GetAttrString(o, "is_cuda"));
    const int whole = cuda > 0 ? truth(PyObject_CallMethod(o, "is_contiguous", nullptr)) : cuda;
    if (whole < 0) return false;
    if (whole == 0) {
        PyErr_SetString(PyExc_ValueError, "device buffers must be contiguous tensors on the GPU");
        return false;
    }
    uint64_t v = 0;
    PyObject* r = PyObject_CallMethod(o, "data_ptr", nullptr);
    bool ok = r && as_u64(r, &v);
    Py_XDECREF(r);
    *p = reinterpret_cast<void*>(v);
    if (ok && bytes) {
        r = PyObject_GetAttrString(o, "nbytes");
        ok = r && as_u64(r, bytes);
        Py_XDECREF(r);
    }
    return ok;
}

bool as_stream(PyObject* o, void** p)
{
    uint64_t v = 0;
    PyObject* r = nullptr;
    if (o == Py_None) {
        if (!raw_stream) {
            PyObject* both = PyObject_CallNoArgs(resolve_stream);
            if (!both) return false;
            if (!PyArg_ParseTuple(both, "OO", &raw_stream, &current_device)) { Py_DECREF(both); raw_stream = nullptr; return false; }
            Py_INCREF(raw_stream);
            Py_INCREF(current_device);
            Py_DECREF(both);
        }
        PyObject* device = PyObject_CallNoArgs(current_device);
        if (!device) return false;
        r = PyObject_CallOneArg(raw_stream, device);
        Py_DECREF(device);
    } else if (PyLong_CheckExact(o)) {
        Py_INCREF(o);
        r = o;
    } else {
        r = PyObject_GetAttrString(o, "cuda_stream");
        if (!r && PyErr_ExceptionMatches(PyExc_AttributeError)) {
            PyErr_Clear();
            r = PyNumber_Long(o);
        }
    }
    const bool ok = r && as_u64(r, &v);
    Py_XDECREF(r);
    *p = reinterpret_cast<void*>(v);
    return ok;
}

/* A view of some object's bytes for the length of a call. */
struct View {
    Py_buffer b = {};
    ~View() { if (b.obj) PyBuffer_Release(&b); }
};

bool as_table(PyObject* o, View& view, const zipccl_table_t** p)
{
    const int is = PyObject_IsInstance(o, table_type);
    if (is <= 0) {
        if (is == 0) PyErr_Format(PyExc_TypeError, "a zipccl_table_t is needed, not %s", Py_TYPE(o)->tp_name);
        return false;
    }
    if (PyObject_GetBuffer(o, &view.b, PyBUF_SIMPLE) != 0) return false;
    *p = static_cast<const zipccl_table_t*>(view.b.buf);
    return true;
}

/* element counts, one per chunk at least: None, or a C-contiguous array of uint64; anything else is made one first */
bool as_counts(PyObject* o, uint32_t chunks, View& view, const uint64_t** p)
{
    *p = nullptr;
    if (o == Py_None) return true;
    auto all_there = [&] {
        if ((uint64_t)view.b.len / 8u >= chunks) {
            *p = static_cast<const uint64_t*>(view.b.buf);
            return true;
        }
        PyErr_Format(PyExc_ValueError, "%zd element counts for %u chunks", view.b.len / 8, (unsigned)chunks);
        return false;
    };
    if (PyObject_CheckBuffer(o) && PyObject_GetBuffer(o, &view.b, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT) == 0) {
        const char* f = view.b.format;
        if (view.b.itemsize == 8 && f && (f[0] == 'L' || f[0] == 'Q') && f[1] == 0) return all_there();
        PyBuffer_Release(&view.b);
    }
    PyErr_Clear();
    PyObject* a = PyObject_CallOneArg(host_array, o);
    if (!a) return false;
    const int rc = PyObject_GetBuffer(a, &view.b, PyBUF_C_CONTIGUOUS);        /* keeps the array */
    Py_DECREF(a);
    return rc == 0 && all_there();
}

bool as_bytes(PyObject* o, uint64_t* bytes)          /* None: leave what the buffer holds */
{
    return o == Py_None || as_u64(o, bytes);
}

bool arity(Py_ssize_t got, Py_ssize_t want)
{
    if (got == want) return true;
    PyErr_Format(PyExc_TypeError, "%zd arguments, %zd are needed", got, want);
    return false;
}

struct Shape {
    uint64_t n = 0, chunks = 0;
    int dt = 0;
    View counts_view;
    const uint64_t* counts = nullptr;

    bool read(PyObject* n_, PyObject* dt_, PyObject* chunks_, PyObject* counts_)
    {
        return as_u64(n_, &n) && as_int(dt_, &dt) && as_u64(chunks_, &chunks) && as_counts(counts_, (uint32_t)chunks, counts_view, &counts);
    }
};

#define CALL(expr)                    \
    zipccl_status_t rc;               \
    Py_BEGIN_ALLOW_THREADS            \
    rc = (expr);                      \
    Py_END_ALLOW_THREADS              \
    return PyLong_FromLong((long)rc)

/* d_in, n, dt, chunks, counts, table, d_out, capacity, d_chunk_bytes, d_workspace, workspace_bytes, stream; without the
 * two workspace arguments zipccl_compress_static.  The table: a zipccl_table_t, or a tensor with one for all chunks
 * (compress_device_table) or one each (compress_chunk_tables). */
enum Table { kHost, kDevice, kChunks };

template <Table TABLE, bool STATIC>
PyObject* compress(PyObject*, PyObject* const* a, Py_ssize_t n_args)
{
    Shape s;
    View table_view;
    const zipccl_table_t* table = nullptr;
    void *in, *out, *sizes, *ws = nullptr, *stream, *d_table = nullptr;
    uint64_t cap = 0, ws_bytes = 0;
    if (!arity(n_args, STATIC ? 10 : 12) || !as_buffer(a[0], &in, nullptr) || !s.read(a[1], a[2], a[3], a[4]) ||
        !(TABLE == kHost ? as_table(a[5], table_view, &table) : as_buffer(a[5], &d_table, nullptr)) ||
        !as_buffer(a[6], &out, a[7] == Py_None ? &cap : nullptr) || !as_bytes(a[7], &cap) || !as_buffer(a[8], &sizes, nullptr) ||
        (!STATIC && (!as_buffer(a[9], &ws, a[10] == Py_None ? &ws_bytes : nullptr) || !as_bytes(a[10], &ws_bytes))) || !as_stream(a[STATIC ? 9 : 11], &stream))
        return nullptr;
    const zipccl_dtype_t dt = (zipccl_dtype_t)s.dt;
    const uint32_t chunks = (uint32_t)s.chunks;
    uint64_t* const cb = static_cast<uint64_t*>(sizes);
    if (STATIC) { CALL(zipccl_compress_static(in, s.n, dt, chunks, s.counts, table, out, cap, cb, stream)); }
    if (TABLE == kHost) { CALL(zipccl_compress(in, s.n, dt, chunks, s.counts, table, out, cap, cb, ws, ws_bytes, stream)); }
    table = static_cast<const zipccl_table_t*>(d_table);
    if (TABLE == kDevice) { CALL(zipccl_compress_device_table(in, s.n, dt, chunks, s.counts, table, out, cap, cb, ws, ws_bytes, stream)); }
    CALL(zipccl_compress_chunk_tables(in, s.n, dt, chunks, s.counts, table, out, cap, cb, ws, ws_bytes, stream));
}

/* d_comp, capacity, d_out, n, dt, chunks, counts, d_status, stream */
PyObject* decompress(PyObject*, PyObject* const* a, Py_ssize_t n_args)
{
    Shape s;
    void *comp, *out, *status, *stream;
    uint64_t cap = 0;
    if (!arity(n_args, 9) || !as_buffer(a[0], &comp, a[1] == Py_None ? &cap : nullptr) || !as_bytes(a[1], &cap) || !as_buffer(a[2], &out, nullptr) ||
        !s.read(a[3], a[4], a[5], a[6]) || !as_buffer(a[7], &status, nullptr) || !as_stream(a[8], &stream))
        return nullptr;
    CALL(zipccl_decompress(comp, cap, out, s.n, (zipccl_dtype_t)s.dt, (uint32_t)s.chunks, s.counts, static_cast<uint32_t*>(status), stream));
}

/* d_comp, capacity, d_out, n, dt, peers, out_dt, d_status, stream */
PyObject* decompress_reduce(PyObject*, PyObject* const* a, Py_ssize_t n_args)
{
    Shape s;
    void *comp, *out, *status, *stream;
    uint64_t cap = 0;
    int out_dt = 0;
    if (!arity(n_args, 9) || !as_buffer(a[0], &comp, a[1] == Py_None ? &cap : nullptr) || !as_bytes(a[1], &cap) || !as_buffer(a[2], &out, nullptr) ||
        !s.read(a[3], a[4], a[5], Py_None) || !as_int(a[6], &out_dt) || !as_buffer(a[7], &status, nullptr) || !as_stream(a[8], &stream))
        return nullptr;
    CALL(zipccl_decompress_reduce(comp, cap, out, s.n, (zipccl_dtype_t)s.dt, (uint32_t)s.chunks, (zipccl_dtype_t)out_dt,
                                  static_cast<uint32_t*>(status), stream));
}

/* d_in, n, dt, d_table, d_sigma, d_workspace, stream */
template <bool ROBUST>
PyObject* estimate(PyObject*, PyObject* const* a, Py_ssize_t n_args)
{
    Shape s;
    void *in, *table, *sigma, *ws, *stream;
    uint64_t ws_bytes = 0;
    if (!arity(n_args, 7) || !as_buffer(a[0], &in, nullptr) || !as_u64(a[1], &s.n) || !as_int(a[2], &s.dt) || !as_buffer(a[3], &table, nullptr) ||
        !as_buffer(a[4], &sigma, nullptr) || !as_buffer(a[5], &ws, &ws_bytes) || !as_stream(a[6], &stream))
        return nullptr;
    CALL((ROBUST ? zipccl_estimate_table_robust : zipccl_estimate_table)(in, s.n, (zipccl_dtype_t)s.dt, static_cast<zipccl_table_t*>(table),
                                                                         static_cast<double*>(sigma), ws, ws_bytes, stream));
}

/* d_in, n, dt, chunks, counts, stride or None, d_tables, d_sigmas, d_workspace, stream */
PyObject* estimate_chunk_tables(PyObject*, PyObject* const* a, Py_ssize_t n_args)
{
    Shape s;
    void *in, *tables, *sigmas, *ws, *stream;
    uint64_t ws_bytes = 0, stride = 0;
    if (!arity(n_args, 10) || !as_buffer(a[0], &in, nullptr) || !s.read(a[1], a[2], a[3], a[4]) || !as_bytes(a[5], &stride) ||
        !as_buffer(a[6], &tables, nullptr) || !as_buffer(a[7], &sigmas, nullptr) || !as_buffer(a[8], &ws, &ws_bytes) || !as_stream(a[9], &stream))
        return nullptr;
    const zipccl_dtype_t dt = (zipccl_dtype_t)s.dt;
    zipccl_table_t* const t = static_cast<zipccl_table_t*>(tables);
    double* const sg = static_cast<double*>(sigmas);
    if (a[5] == Py_None) { CALL(zipccl_estimate_chunk_tables(in, s.n, dt, (uint32_t)s.chunks, s.counts, t, sg, ws, ws_bytes, stream)); }
    CALL(zipccl_estimate_chunk_tables_sampled(in, s.n, dt, (uint32_t)s.chunks, s.counts, (uint32_t)stride, t, sg, ws, ws_bytes, stream));
}

/* table type, host_array, resolve_stream */
PyObject* setup(PyObject*, PyObject* const* a, Py_ssize_t n_args)
{
    if (!arity(n_args, 3)) return nullptr;
    PyObject** const to[3] = {&table_type, &host_array, &resolve_stream};
    for (int i = 0; i < 3; ++i) {
        Py_INCREF(a[i]);
        Py_XSETREF(*to[i], a[i]);
    }
    Py_RETURN_NONE;
}

#define METHOD(name, f) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(static_cast<_PyCFunctionFast>(f))), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    METHOD("setup", setup),
    METHOD("compress", (compress<kHost, false>)),
    METHOD("compress_static", (compress<kHost, true>)),
    METHOD("compress_device_table", (compress<kDevice, false>)),
    METHOD("compress_chunk_tables", (compress<kChunks, false>)),
    METHOD("decompress", decompress),
    METHOD("decompress_reduce", decompress_reduce),
    METHOD("estimate_table", estimate<false>),
    METHOD("estimate_table_robust", estimate<true>),
    METHOD("estimate_chunk_tables", estimate_chunk_tables),
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "zipccl_python", "Calls of libzipccl.so for binding.py.", -1, methods, nullptr, nullptr, nullptr, nullptr};

} // namespace

PyMODINIT_FUNC PyInit_zipccl_python(void) { return PyModule_Create(&module); }
