// Native marshalling of the calls a program makes once per tensor: binding.observe_into and PreparedObserve.
//
// A small capture takes the GPU two to four microseconds and hipLaunchKernel about as long; reading a tensor's address and layout
// through Python attributes, packing the argument structs and the foreign call itself cost 1.2 us of Python per
// observe_into and 0.8 us per prepared observe on top (with it a call of 4 rows x 256 takes 8.1 us, with this 6.5).  Only the plain case is handled: exact torch
// tensors, a C-contiguous uint32 table, ints.  Whatever else comes -- other types, subclasses, wrong or missing
// arguments, tensors without storage -- is handed to the Python function of the same meaning, which converts or refuses
// it as it always has.  The library's entry points come in as addresses, so this module loads without libdmi.so; and what reads
// tensors (dmi_python_torch.cpp) comes in when there is one to read, so that it loads without torch too.
#include "dmi_python.h"

namespace {

typedef dmi_status_t (*into_fn)(uint32_t, const dmi_tensor_t *, const dmi_selection_t *, const dmi_transform_t *, uint64_t,
                                uint64_t, uint32_t, void *, uint64_t, uint64_t *, void *);
typedef dmi_status_t (*observe_fn)(dmi_ring_t *, uint32_t, const void *, const dmi_selection_t *, const dmi_transform_t *,
                                   uint64_t, void *);

into_fn g_into = nullptr;
PyObject *g_general = nullptr;      // binding's own observe_into: everything but the plain case
PyObject *g_check = nullptr;        // binding._check(code, allow)
PyObject *g_module = nullptr;       // binding's namespace, where _into_fn may name another foreign function
PyObject *g_load = nullptr;         // called once a tensor may be at hand: has set_reader() called, or not
dmi_py_reader g_reader = nullptr;
PyObject *g_names[12];              // observe_into's parameters, interned
PyObject *g_into_name = nullptr;
const char *const kNames[12] = {"point_id", "tensor", "reqs", "out", "seq", "step_id", "rank_tag", "out_dtype", "summary_mask",
                                "keep_mask", "row_index", "stream"};

bool as_u64(PyObject *o, uint64_t *v)       // an int's low 64 bits, as ctypes takes them
{
    if (!PyLong_Check(o)) return false;
    *v = PyLong_AsUnsignedLongLongMask(o);
    return !(*v == (uint64_t)-1 && PyErr_Occurred());
}

bool optional_address(PyObject *o, const void **p)
{
    *p = nullptr;
    if (!o || o == Py_None) return true;
    dmi_py_tensor t;
    if (!g_reader(o, &t)) return false;
    *p = t.data;
    return true;
}

// The plain case; false: it is not one (no Python error is left behind).
bool plain_into(PyObject *const (&v)[12], Py_buffer *table, bool *have_table, dmi_tensor_t *t, dmi_selection_t *sel,
                dmi_transform_t *xf, uint64_t (&n)[4], void **out, uint64_t *out_bytes)
{
    dmi_py_tensor x, dst;
    if (!g_reader(v[1], &x) || !g_reader(v[3], &dst) || x.dim != 2 || !x.dtype) return false;
    t->dtype = x.dtype;
    uint64_t od = 0, mask = 0, stream = 0;
    if (!as_u64(v[0], &n[0]) || !as_u64(v[4], &n[1]) || !as_u64(v[5], &n[2])) return false;
    n[3] = 0;
    if (v[6] && !as_u64(v[6], &n[3])) return false;
    if (v[7] && v[7] != Py_None) { if (!as_u64(v[7], &od)) return false; } else od = t->dtype;
    if (v[8] && !as_u64(v[8], &mask)) return false;
    if (v[11] && !as_u64(v[11], &stream)) return false;
    const void *keep, *index;
    if (!optional_address(v[9], &keep) || !optional_address(v[10], &index)) return false;
    if (PyObject_GetBuffer(v[2], table, PyBUF_ND | PyBUF_FORMAT) != 0) { PyErr_Clear(); return false; }
    *have_table = true;
    if (table->ndim != 2 || table->shape[1] != 5 || table->itemsize != 4 || !table->format || table->format[0] != 'I' ||
        table->format[1] || table->shape[0] > 0x7FFFFFFF)
        return false;
    t->data = x.data;
    for (int i = 0; i < 2; i++) { t->shape[i] = x.shape[i]; t->stride[i] = x.stride[i]; }
    sel->n_reqs = (uint32_t)table->shape[0];
    sel->reqs = static_cast<const dmi_req_sel_t *>(table->buf);
    sel->keep_mask_dev = static_cast<const uint8_t *>(keep);
    sel->row_index_dev = static_cast<const int32_t *>(index);
    xf->out_dtype = (uint32_t)od;
    xf->summary_mask = (uint32_t)mask;
    *out = dst.data;
    *out_bytes = dst.bytes;
    n[0] = (uint32_t)n[0];
    n[3] = (uint32_t)n[3];
    return true;
}

PyObject *observe_into(PyObject *, PyObject *const *args, Py_ssize_t n_args, PyObject *kw)
{
    PyObject *v[12] = {}, *allow = nullptr;
    const Py_ssize_t n_kw = kw ? PyTuple_GET_SIZE(kw) : 0;
    bool plain = g_into && n_args <= 4;
    for (Py_ssize_t i = 0; plain && i < n_args; i++) v[i] = args[i];
    for (Py_ssize_t i = 0; plain && i < n_kw; i++) {
        PyObject *name = PyTuple_GET_ITEM(kw, i);
        int k = 0;
        while (k < 12 && name != g_names[k]) k++;
        if (k < 12 && !v[k]) v[k] = args[n_args + i];
        else if (k == 12 && PyUnicode_CompareWithASCIIString(name, "allow") == 0 && !allow) allow = args[n_args + i];
        else plain = false;
    }
    for (int k = 0; plain && k < 6; k++) plain = v[k] != nullptr;
    if (plain) {
        PyObject *other = PyDict_GetItem(g_module, g_into_name);        // (borrowed)
        plain = other == nullptr || other == Py_None;
    }
    if (plain && !g_reader) {
        if (PyObject *r = g_load && g_load != Py_None ? PyObject_CallNoArgs(g_load) : nullptr) Py_DECREF(r);
        if (PyErr_Occurred()) return nullptr;
        plain = g_reader != nullptr && g_into != nullptr;
    }
    if (plain) {
        Py_buffer table;
        bool have_table = false, failed = false;
        dmi_tensor_t t = {};
        dmi_selection_t sel = {};
        dmi_transform_t xf = {};
        uint64_t n[4], out_bytes = 0, record = 0;
        void *out = nullptr;
        dmi_status_t code = DMI_OK;
        plain = plain_into(v, &table, &have_table, &t, &sel, &xf, n, &out, &out_bytes);
        if (plain) {
            uint64_t stream = 0;
            if (v[11]) as_u64(v[11], &stream);
            Py_BEGIN_ALLOW_THREADS
            code = g_into((uint32_t)n[0], &t, &sel, &xf, n[1], n[2], (uint32_t)n[3], out, out_bytes, &record,
                          reinterpret_cast<void *>(stream));
            Py_END_ALLOW_THREADS
        }
        if (have_table) PyBuffer_Release(&table);
        if (plain) {
            if (code < 0) {
                PyObject *c = PyLong_FromLong(code);
                PyObject *r = c ? (allow ? PyObject_CallFunctionObjArgs(g_check, c, allow, nullptr)
                                         : PyObject_CallFunctionObjArgs(g_check, c, nullptr)) : nullptr;
                failed = r == nullptr;
                Py_XDECREF(r);
                Py_XDECREF(c);
            }
            return failed ? nullptr : PyLong_FromUnsignedLongLong(record);
        }
        if (PyErr_Occurred()) PyErr_Clear();
    }
    if (!g_general) {
        PyErr_SetString(PyExc_RuntimeError, "the binding has not set this module up");
        return nullptr;
    }
    return PyObject_Vectorcall(g_general, args, (size_t)n_args, kw);
}

// ------------------------------------------------------------------ a prepared observe
struct Prepared {
    PyObject_HEAD
    observe_fn fn;
    dmi_ring_t *ring;
    const void *src;
    const dmi_selection_t *sel;
    const dmi_transform_t *xf;
    uint32_t point;
};

PyObject *prepared_bind(PyObject *self, PyObject *args)
{
    unsigned long long a[6];
    if (!PyArg_ParseTuple(args, "KKKKKK", &a[0], &a[1], &a[2], &a[3], &a[4], &a[5])) return nullptr;
    Prepared *p = reinterpret_cast<Prepared *>(self);
    p->fn = reinterpret_cast<observe_fn>(a[0]);
    p->ring = reinterpret_cast<dmi_ring_t *>(a[1]);
    p->point = (uint32_t)a[2];
    p->src = reinterpret_cast<const void *>(a[3]);
    p->sel = reinterpret_cast<const dmi_selection_t *>(a[4]);
    p->xf = reinterpret_cast<const dmi_transform_t *>(a[5]);
    Py_RETURN_NONE;
}

PyObject *prepared_call(PyObject *self, PyObject *args, PyObject *kw)
{
    Prepared *p = reinterpret_cast<Prepared *>(self);
    uint64_t step = 0, stream = 0;
    if (p->fn && !kw && PyTuple_GET_SIZE(args) == 2 && as_u64(PyTuple_GET_ITEM(args, 0), &step) &&
        as_u64(PyTuple_GET_ITEM(args, 1), &stream)) {
        dmi_status_t code;
        Py_BEGIN_ALLOW_THREADS
        code = p->fn(p->ring, p->point, p->src, p->sel, p->xf, step, reinterpret_cast<void *>(stream));
        Py_END_ALLOW_THREADS
        return PyLong_FromLong(code);
    }
    if (PyErr_Occurred()) PyErr_Clear();
    PyObject *f = PyObject_GetAttrString(self, "_call");
    if (!f) return nullptr;
    PyObject *r = PyObject_Call(f, args, kw);
    Py_DECREF(f);
    return r;
}

PyMethodDef prepared_methods[] = {{"_bind", prepared_bind, METH_VARARGS, "entry point, ring, point, source, selection, transform: addresses"},
                                  {nullptr, nullptr, 0, nullptr}};
PyTypeObject prepared_type = {PyVarObject_HEAD_INIT(nullptr, 0)};

PyObject *setup(PyObject *, PyObject *args)
{
    PyObject *general, *check, *module, *load;
    if (!PyArg_ParseTuple(args, "OOO!O", &general, &check, &PyDict_Type, &module, &load)) return nullptr;
    Py_INCREF(general); Py_INCREF(check); Py_INCREF(module); Py_INCREF(load);
    Py_XSETREF(g_load, load);
    Py_XSETREF(g_general, general);
    Py_XSETREF(g_check, check);
    Py_XSETREF(g_module, module);
    Py_RETURN_NONE;
}

PyObject *bind_into(PyObject *, PyObject *arg)
{
    const unsigned long long a = PyLong_AsUnsignedLongLong(arg);
    if (PyErr_Occurred()) return nullptr;
    g_into = reinterpret_cast<into_fn>(a);
    Py_RETURN_NONE;
}

PyObject *set_reader(PyObject *, PyObject *arg)
{
    void *p = PyCapsule_GetPointer(arg, DMI_PY_READER);
    if (!p) return nullptr;
    g_reader = reinterpret_cast<dmi_py_reader>(p);
    Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"observe_into", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(observe_into)), METH_FASTCALL | METH_KEYWORDS,
     "observe_into(point_id, tensor, reqs, out, *, seq, step_id, rank_tag=0, out_dtype=None, summary_mask=0, keep_mask=None, "
     "row_index=None, stream=0, allow=())\n--\n\n"
     "dmi_observe_into: one record into `out` (a uint8 device tensor), no ring, no allocation.\n"
     "Returns the record's size (an upper bound if a keep vector is given)."},
    {"setup", setup, METH_VARARGS, "the binding's general observe_into, its status check, its namespace, what loads the tensor reader"},
    {"set_reader", set_reader, METH_O, "capsule with the function that reads torch tensors"},
    {"bind_into", bind_into, METH_O, "address of dmi_observe_into"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_dmi_python", "native marshalling of per-tensor calls", -1, methods,
                          nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__dmi_python(void)
{
    for (int k = 0; k < 12; k++)
        if (!(g_names[k] = PyUnicode_InternFromString(kNames[k]))) return nullptr;
    if (!(g_into_name = PyUnicode_InternFromString("_into_fn"))) return nullptr;
    prepared_type.tp_name = "paper_2605_11093_amd._dmi_python.Prepared";
    prepared_type.tp_basicsize = sizeof(Prepared);
    prepared_type.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_BASETYPE;
    prepared_type.tp_new = PyType_GenericNew;
    prepared_type.tp_call = prepared_call;
    prepared_type.tp_methods = prepared_methods;
    if (PyType_Ready(&prepared_type) < 0) return nullptr;
    PyObject *m = PyModule_Create(&module_def);
    if (!m) return nullptr;
    if (PyModule_AddIntConstant(m, "INTERFACE", 2) < 0) { Py_DECREF(m); return nullptr; }      // (of this module to binding.py)
    if (PyModule_AddObject(m, "HEADER_DIGEST", PyLong_FromUnsignedLongLong(DMI_HEADER_DIGEST)) < 0) { Py_DECREF(m); return nullptr; }
    Py_INCREF(&prepared_type);
    if (PyModule_AddObject(m, "Prepared", reinterpret_cast<PyObject *>(&prepared_type)) < 0) { Py_DECREF(m); return nullptr; }
    return m;
}
