// Python module _stepq_args: the argument checks of the binding's device calls
// (stepq.py) in native code, followed by the C call.
//
// A small decode step is bound by its launch: checking eight tensors from
// Python and marshalling twelve arguments through ctypes took 9 of the 12 us
// of a one-request step (the kernel 5): 12.4 -> 5.2 us here; export + import
// with FP16 rows of 32 requests (four calls) 35.2 -> 26.4 us.  Each function here checks what
// stepq.py's own path checks (device, dtype, shape, contiguity) and makes the
// call, or returns -1 without calling anything when an argument is not plainly
// what the call takes: stepq.py then goes through its own path, which raises
// the error or handles the case.  Nothing is kept between calls.
#include <Python.h>

#include <type_traits>

#include <ATen/core/Tensor.h>
#include <torch/csrc/autograd/python_variable.h>

#include "stepq.h"

namespace {

struct Entry {
    decltype(&stepq_decode_step_ex) step;
    decltype(&stepq_pool_load) load;
    decltype(&stepq_pool_import) import;
    decltype(&stepq_pool_export) exprt;
    decltype(&stepq_pool_dequant) dequant;
    decltype(&stepq_pool_export_pivots) export_pivots;
    decltype(&stepq_pool_import_pivots) import_pivots;
    int (*get_device)(int *);                  // the runtime's current device
    PyObject *raw_stream, *stream_type;        // torch's raw current-stream query and stream class
} g{};

struct Plain {
    stepq_pool *pool;
    int device;
    int64_t Hv, Hqk, dk, dv;
};

// The tensor's data if it is a plain tensor of this device, type and shape.
bool take(PyObject *o, const Plain &p, at::ScalarType dt, at::IntArrayRef shape, void **out)
{
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (!t.is_cuda() || t.get_device() != p.device || t.scalar_type() != dt || t.layout() != at::kStrided ||
        t.sizes() != shape || !t.is_contiguous())
        return false;
    *out = t.data_ptr();
    return true;
}

bool take_ids(PyObject *o, const Plain &p, int64_t *n, void **out)
{
    if (!THPVariable_CheckExact(o)) return false;
    const at::Tensor &t = THPVariable_Unpack(o);
    if (t.dim() != 1) return false;
    *n = t.size(0);
    return *n <= INT32_MAX && take(o, p, at::kInt, {*n}, out);
}

// None: torch's current stream, which is the current device's (not the pool's);
// an int: the stream itself; a torch stream.
bool take_stream(PyObject *o, void **out)
{
    PyObject *v = nullptr;
    if (o == Py_None) {
        int device;
        if (g.get_device(&device) != 0) return false;
        if (PyObject *d = PyLong_FromLong(device)) {
            v = PyObject_CallOneArg(g.raw_stream, d);
            Py_DECREF(d);
        }
    } else if (PyLong_CheckExact(o)) {
        v = o;
        Py_INCREF(v);
    } else {
        const int is = PyObject_IsInstance(o, g.stream_type);
        if (is == 0) return false;
        if (is > 0) v = PyObject_GetAttrString(o, "cuda_stream");
    }
    if (!v) {
        PyErr_Clear();
        return false;
    }
    *out = PyLong_AsVoidPtr(v);
    Py_DECREF(v);
    if (PyErr_Occurred()) {
        PyErr_Clear();
        return false;
    }
    return true;
}

const Plain *plain_of(PyObject *o)
{
    if (!PyCapsule_CheckExact(o)) return nullptr;
    return static_cast<const Plain *>(PyCapsule_GetPointer(o, "stepq.plain"));
}

void free_plain(PyObject *cap) { delete static_cast<Plain *>(PyCapsule_GetPointer(cap, "stepq.plain")); }

// plain(handle, device, Hv, Hqk, dk, dv): what the checks compare with.
PyObject *py_plain(PyObject *, PyObject *args)
{
    unsigned long long handle;
    int device;
    long long Hv, Hqk, dk, dv;
    if (!PyArg_ParseTuple(args, "KiLLLL", &handle, &device, &Hv, &Hqk, &dk, &dv)) return nullptr;
    auto *p = new Plain{reinterpret_cast<stepq_pool *>(handle), device, Hv, Hqk, dk, dv};
    return PyCapsule_New(p, "stepq.plain", free_plain);
}

// bind(step_ex, load, import, export, dequant, export_pivots, import_pivots, get_device, raw_stream, stream_type)
PyObject *py_bind(PyObject *, PyObject *args)
{
    unsigned long long f[8];
    PyObject *rs, *st;
    if (!PyArg_ParseTuple(args, "KKKKKKKKOO", &f[0], &f[1], &f[2], &f[3], &f[4], &f[5], &f[6], &f[7], &rs, &st))
        return nullptr;
    auto set = [&f](auto &fn, int i) { fn = reinterpret_cast<std::remove_reference_t<decltype(fn)>>(f[i]); };
    set(g.step, 0);
    set(g.load, 1);
    set(g.import, 2);
    set(g.exprt, 3);
    set(g.dequant, 4);
    set(g.export_pivots, 5);
    set(g.import_pivots, 6);
    set(g.get_device, 7);
    Py_INCREF(rs);
    Py_XSETREF(g.raw_stream, rs);
    Py_INCREF(st);
    Py_XSETREF(g.stream_type, st);
    Py_RETURN_NONE;
}

template <class F>
PyObject *guarded(F &&f)
{
    long st = -1;
    try {
        st = f();
    } catch (...) {
        st = -1;      // e.g. a tensor without data: the binding's own path says so
    }
    return PyLong_FromLong(st);
}

// decode(plain, slot_ids, q, k, v, gate, beta, o, stream, flags) -> status or -1
PyObject *py_decode(PyObject *, PyObject *const *a, Py_ssize_t n_args)
{
    return guarded([&]() -> long {
        const Plain *p = n_args == 10 ? plain_of(a[0]) : nullptr;
        if (!p || !g.step || !PyLong_CheckExact(a[9]) || !THPVariable_CheckExact(a[2])) return -1;
        const unsigned long flags = PyLong_AsUnsignedLong(a[9]);
        if (PyErr_Occurred()) {
            PyErr_Clear();
            return -1;
        }
        const at::ScalarType dt = THPVariable_Unpack(a[2]).scalar_type();
        if (dt != at::kFloat && dt != at::kBFloat16) return -1;
        int64_t n;
        void *ids, *q, *k, *v, *gate, *beta, *o, *s;
        if (!take_ids(a[1], *p, &n, &ids) || !take(a[2], *p, dt, {n, p->Hqk, p->dk}, &q) ||
            !take(a[3], *p, dt, {n, p->Hqk, p->dk}, &k) || !take(a[4], *p, dt, {n, p->Hv, p->dv}, &v) ||
            !((flags & STEPQ_STEP_KDA_GATE) ? take(a[5], *p, dt, {n, p->Hv, p->dk}, &gate)
                                            : take(a[5], *p, dt, {n, p->Hv}, &gate)) ||
            !take(a[6], *p, dt, {n, p->Hv}, &beta) || !take(a[7], *p, at::kFloat, {n, p->Hv, p->dv}, &o) ||
            !take_stream(a[8], &s))
            return -1;
        stepq_status st;
        Py_BEGIN_ALLOW_THREADS;
        st = g.step(p->pool, static_cast<const int32_t *>(ids), static_cast<int32_t>(n), q, k, v, gate, beta,
                    dt == at::kFloat ? STEPQ_F32 : STEPQ_BF16, static_cast<uint32_t>(flags), static_cast<float *>(o), s);
        Py_END_ALLOW_THREADS;
        return st;
    });
}

enum { kLoad, kImport, kExport };

// scaled(op, plain, slot_ids, rows, r, c, stream): load (0), import (1), export (2)
PyObject *py_scaled(PyObject *, PyObject *const *a, Py_ssize_t n_args)
{
    return guarded([&]() -> long {
        const Plain *p = n_args == 7 ? plain_of(a[1]) : nullptr;
        if (!p || !g.load || !PyLong_CheckExact(a[0])) return -1;
        const long op = PyLong_AsLong(a[0]);
        int64_t n;
        void *ids, *x, *r, *c, *s;
        if (!take_ids(a[2], *p, &n, &ids) ||
            !take(a[3], *p, op == kLoad ? at::kFloat : at::kChar, {n, p->Hv, p->dk, p->dv}, &x) ||
            !take(a[4], *p, at::kFloat, {n, p->Hv, p->dk}, &r) || !take(a[5], *p, at::kFloat, {n, p->Hv, p->dv}, &c) ||
            !take_stream(a[6], &s))
            return -1;
        const auto *id = static_cast<const int32_t *>(ids);
        const auto m = static_cast<int32_t>(n);
        auto *rf = static_cast<float *>(r), *cf = static_cast<float *>(c);
        stepq_status st;
        Py_BEGIN_ALLOW_THREADS;
        st = op == kLoad     ? g.load(p->pool, id, m, static_cast<const float *>(x), rf, cf, s)
             : op == kImport ? g.import(p->pool, id, m, static_cast<const int8_t *>(x), rf, cf, s)
                             : g.exprt(p->pool, id, m, static_cast<int8_t *>(x), rf, cf, s);
        Py_END_ALLOW_THREADS;
        return st;
    });
}

enum { kDequant, kExportPivots, kImportPivots };

// tiles(op, plain, slot_ids, rows, stream): dequant (0), export (1) and import (2) of the pivot rows
PyObject *py_tiles(PyObject *, PyObject *const *a, Py_ssize_t n_args)
{
    return guarded([&]() -> long {
        const Plain *p = n_args == 5 ? plain_of(a[1]) : nullptr;
        if (!p || !g.dequant || !PyLong_CheckExact(a[0])) return -1;
        const long op = PyLong_AsLong(a[0]);
        int64_t n;
        void *ids, *x, *s;
        if (!take_ids(a[2], *p, &n, &ids)) return -1;
        const int64_t shape[4] = {n, p->Hv, p->dk, p->dv};
        const bool ok = op == kDequant ? take(a[3], *p, at::kFloat, shape, &x)
                                       : take(a[3], *p, at::kShort, shape, &x) || take(a[3], *p, at::kUInt16, shape, &x);
        if (!ok || !take_stream(a[4], &s)) return -1;
        const auto *id = static_cast<const int32_t *>(ids);
        const auto m = static_cast<int32_t>(n);
        stepq_status st;
        Py_BEGIN_ALLOW_THREADS;
        st = op == kDequant        ? g.dequant(p->pool, id, m, static_cast<float *>(x), s)
             : op == kExportPivots ? g.export_pivots(p->pool, id, m, static_cast<uint16_t *>(x), s)
                                   : g.import_pivots(p->pool, id, m, static_cast<const uint16_t *>(x), s);
        Py_END_ALLOW_THREADS;
        return st;
    });
}

PyMethodDef methods[] = {
    {"bind", py_bind, METH_VARARGS, "addresses of the C calls, torch's raw stream query and stream class"},
    {"plain", py_plain, METH_VARARGS, "a pool's handle, device and sizes"},
    {"decode", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(py_decode)), METH_FASTCALL, "one decode step"},
    {"scaled", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(py_scaled)), METH_FASTCALL,
     "load, import or export"},
    {"tiles", reinterpret_cast<PyCFunction>(reinterpret_cast<void *>(py_tiles)), METH_FASTCALL,
     "dequant, export or import of pivot rows"},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_stepq_args", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__stepq_args(void) { return PyModule_Create(&module); }
