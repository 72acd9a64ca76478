// The short way from Python into mnn_conv_run and mnn_conv_run_static: what ctypes and a chain of attribute look-ups cost a small layer is longer than
// its kernel (16 -> 16 channels on 32 x 32: 5.2 us per call on the host, 3.1 here, of which 2.45 are the launch; with three states in turn, whose operands come from
// memory, the device bounds it at 4.0, 5.7 before).  Only the usual call is taken here -- plain float32 tensors
// of the right shapes on the GPU, the weight tensor of the call before, unchanged; whatever else comes, the caller is told to take its general
// path, which also words all errors.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <new>
#include <vector>
#include "mnn_conv.h"

namespace {

typedef int (*run_fn)(mnn_conv_plan_t, const float*, const float*, const float*, float*, void*);
typedef int (*static_fn)(const mnn_conv_shape*, const mnn_conv_geom*, int32_t, const float*, const float*, const float*, float*, void*);

#ifndef FAST_CALL_ON_CPU
bool on_device(const at::Tensor& t) { return t.is_cuda(); }
// The stream that torch works on, of the current device
void* current_stream() { return c10::hip::getCurrentHIPStream().stream(); }
#else       // for tests without a GPU, which call functions of their own
bool on_device(const at::Tensor& t) { return t.is_cpu(); }
void* current_stream() { return nullptr; }
#endif

// Address of a tensor of these sizes as the kernels take it, or null
float* plain(PyObject* o, const std::vector<int64_t>* sizes)
{
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !on_device(t) || t.layout() != c10::kStrided || t.scalar_type() != c10::kFloat || t.unsafeGetTensorImpl()->is_python_dispatch() ||
        !t.has_storage())
        return nullptr;
    if (sizes && (!t.sizes().equals(*sizes) || !t.is_contiguous())) return nullptr;
    return static_cast<float*>(t.mutable_data_ptr());
}

// The call, without the GIL and with it again whatever happens.  False if an exception came out.
template <class F>
bool without_gil(F call, int* rc)
{
    bool ok = true;
    PyThreadState* const state = PyEval_SaveThread();
    try {
        *rc = call();
    } catch (...) {
        ok = false;
    }
    PyEval_RestoreThread(state);
    return ok;
}

struct Runner {
    PyObject_HEAD
    vectorcallfunc call;
    run_fn fn;
    mnn_conv_plan_t plan;
    std::vector<int64_t>* sizes;             // input, weight, bias, output
    PyObject* weight;                        // of the call before: kept, so that no other object takes its place
    const void* weight_ptr;
    int64_t weight_version;
};

// (x, w, b, y) -> the library's return code, or None: the general path
PyObject* runner_call(PyObject* self, PyObject* const* args, size_t nargsf, PyObject* kw)
{
    Runner* r = reinterpret_cast<Runner*>(self);
    if (PyVectorcall_NARGS(nargsf) != 4 || kw || !r->plan || args[1] != r->weight) Py_RETURN_NONE;
    int rc = 0;
    try {
        const float* x = plain(args[0], &r->sizes[0]);
        const float* w = plain(args[1], &r->sizes[1]);
        const float* b = args[2] == Py_None ? nullptr : plain(args[2], &r->sizes[2]);
        float* y = plain(args[3], &r->sizes[3]);
        if (!x || !w || !y || (!b && args[2] != Py_None)) Py_RETURN_NONE;
        const at::Tensor& wt = THPVariable_Unpack(args[1]);
        if (wt.is_inference() || w != r->weight_ptr || (int64_t)wt._version() != r->weight_version) Py_RETURN_NONE;
        void* s = current_stream();
        if (!without_gil([&] { return r->fn(r->plan, x, w, b, y, s); }, &rc)) Py_RETURN_NONE;
    } catch (...) {
        Py_RETURN_NONE;
    }
    return PyLong_FromLong(rc);
}

// Holds another weight tensor, or none.  Letting go of the one before may run Python code: last.
void hold(Runner* r, PyObject* w)
{
    PyObject* const before = r->weight;
    Py_XINCREF(w);
    r->weight = w;
    Py_XDECREF(before);
}

// remember(weight): the general path has just run with this tensor; remember(None): forget it
PyObject* runner_remember(PyObject* self, PyObject* w)
{
    Runner* r = reinterpret_cast<Runner*>(self);
    try {
        const float* p = plain(w, &r->sizes[1]);
        if (p && !THPVariable_Unpack(w).is_inference()) {
            const int64_t version = (int64_t)THPVariable_Unpack(w)._version();
            r->weight_ptr = p;
            r->weight_version = version;
            hold(r, w);
            Py_RETURN_NONE;
        }
    } catch (...) {
    }
    hold(r, nullptr);
    Py_RETURN_NONE;
}

// forget the plan, which is about to be destroyed
PyObject* runner_close(PyObject* self, PyObject*)
{
    Runner* r = reinterpret_cast<Runner*>(self);
    r->plan = nullptr;
    hold(r, nullptr);
    Py_RETURN_NONE;
}

// A weight tensor can hold the plan that holds the runner
int runner_traverse(PyObject* self, visitproc visit, void* arg)
{
    Py_VISIT(reinterpret_cast<Runner*>(self)->weight);
    return 0;
}

int runner_clear(PyObject* self)
{
    hold(reinterpret_cast<Runner*>(self), nullptr);
    return 0;
}

void runner_dealloc(PyObject* self)
{
    Runner* r = reinterpret_cast<Runner*>(self);
    PyObject_GC_UnTrack(self);
    hold(r, nullptr);
    delete[] r->sizes;
    Py_TYPE(self)->tp_free(self);
}

bool read_sizes(PyObject* t, std::vector<int64_t>* out)
{
    if (!PyTuple_Check(t)) { PyErr_SetString(PyExc_TypeError, "shapes are tuples"); return false; }
    for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(t); ++i) out->push_back(PyLong_AsLongLong(PyTuple_GET_ITEM(t, i)));
    return !PyErr_Occurred();
}

// Runner(address of mnn_conv_run, plan handle, input, weight, bias and output shape)
PyObject* runner_new(PyTypeObject* type, PyObject* args, PyObject*)
{
    unsigned long long fn, plan;
    PyObject* shape[4];
    if (!PyArg_ParseTuple(args, "KKOOOO", &fn, &plan, &shape[0], &shape[1], &shape[2], &shape[3])) return nullptr;
    Runner* r = reinterpret_cast<Runner*>(type->tp_alloc(type, 0));
    if (!r) return nullptr;
    r->call = runner_call;
    r->fn = reinterpret_cast<run_fn>(fn);
    r->plan = reinterpret_cast<mnn_conv_plan_t>(plan);
    r->weight = nullptr;
    r->sizes = new (std::nothrow) std::vector<int64_t>[4];
    bool ok = r->sizes != nullptr;
    for (int i = 0; i < 4 && ok; ++i) ok = read_sizes(shape[i], &r->sizes[i]);
    if (!ok) {
        if (!PyErr_Occurred()) PyErr_NoMemory();
        Py_DECREF(r);
        return nullptr;
    }
    return reinterpret_cast<PyObject*>(r);
}

PyMethodDef runner_methods[] = {{"remember", runner_remember, METH_O, nullptr}, {"close", runner_close, METH_NOARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyTypeObject RunnerType = {PyVarObject_HEAD_INIT(nullptr, 0)};

PyObject* names[10];                         // n, c_in, h, w, c_out, kh, kw; stride, pad, dil

// One or two numbers, as the general path reads them: a number for both axes, or a pair
bool pair_of(PyObject* o, int32_t* a, int32_t* b)
{
    if (PyLong_CheckExact(o)) { *a = *b = (int32_t)PyLong_AsLong(o); return !PyErr_Occurred(); }
    if (!PyTuple_CheckExact(o) || PyTuple_GET_SIZE(o) != 2 || !PyLong_CheckExact(PyTuple_GET_ITEM(o, 0)) || !PyLong_CheckExact(PyTuple_GET_ITEM(o, 1))) return false;
    *a = (int32_t)PyLong_AsLong(PyTuple_GET_ITEM(o, 0));
    *b = (int32_t)PyLong_AsLong(PyTuple_GET_ITEM(o, 1));
    return !PyErr_Occurred();
}

// run_static(address of mnn_conv_run_static, layer, tile, x, w, b, y) -> return code, or None
PyObject* run_static(PyObject*, PyObject* const* args, Py_ssize_t nargs)
{
    if (nargs != 7) Py_RETURN_NONE;
    const static_fn fn = reinterpret_cast<static_fn>(PyLong_AsUnsignedLongLong(args[0]));
    mnn_conv_shape shape;
    mnn_conv_geom geom;
    int32_t* const one[7] = {&shape.n, &shape.c_in, &shape.h, &shape.w, &shape.c_out, &shape.kh, &shape.kw};
    int32_t* const two[6] = {&geom.stride_h, &geom.stride_w, &geom.pad_h, &geom.pad_w, &geom.dil_h, &geom.dil_w};
    bool ok = fn && PyLong_CheckExact(args[2]);
    for (int i = 0; i < 10 && ok; ++i) {
        PyObject* v = PyObject_GetAttr(args[1], names[i]);
        if (!v) ok = false;
        else if (i < 7) {
            ok = PyLong_CheckExact(v);
            if (ok) *one[i] = (int32_t)PyLong_AsLong(v);
        } else ok = pair_of(v, two[2 * (i - 7)], two[2 * (i - 7) + 1]);
        Py_XDECREF(v);
    }
    const int32_t tile = ok ? (int32_t)PyLong_AsLong(args[2]) : 0;
    if (PyErr_Occurred()) { PyErr_Clear(); ok = false; }
    if (!ok) Py_RETURN_NONE;
    int rc = 0;
    try {
        const float* x = plain(args[3], nullptr);
        const float* w = plain(args[4], nullptr);
        const float* b = args[5] == Py_None ? nullptr : plain(args[5], nullptr);
        float* y = plain(args[6], nullptr);
        if (!x || !w || !y || (!b && args[5] != Py_None)) Py_RETURN_NONE;
        void* s = current_stream();
        if (!without_gil([&] { return fn(&shape, &geom, tile, x, w, b, y, s); }, &rc)) Py_RETURN_NONE;
    } catch (...) {
        Py_RETURN_NONE;
    }
    return PyLong_FromLong(rc);
}

PyMethodDef module_methods[] = {{"run_static", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(run_static)), METH_FASTCALL, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_fast_call", nullptr, -1, module_methods};

}  // namespace

PyMODINIT_FUNC PyInit__fast_call()
{
    static const char* const attr[10] = {"n", "c_in", "h", "w", "c_out", "kh", "kw", "stride", "pad", "dil"};
    for (int i = 0; i < 10; ++i)
        if (!(names[i] = PyUnicode_InternFromString(attr[i]))) return nullptr;
    RunnerType.tp_name = "_fast_call.Runner";
    RunnerType.tp_basicsize = sizeof(Runner);
    RunnerType.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL | Py_TPFLAGS_HAVE_GC;
    RunnerType.tp_traverse = runner_traverse;
    RunnerType.tp_clear = runner_clear;
    RunnerType.tp_free = PyObject_GC_Del;
    RunnerType.tp_new = runner_new;
    RunnerType.tp_dealloc = runner_dealloc;
    RunnerType.tp_methods = runner_methods;
    RunnerType.tp_vectorcall_offset = offsetof(Runner, call);
    RunnerType.tp_call = PyVectorcall_Call;
    if (PyType_Ready(&RunnerType) < 0) return nullptr;
    PyObject* m = PyModule_Create(&module_def);
    if (!m) return nullptr;
    Py_INCREF(&RunnerType);
    if (PyModule_AddObject(m, "Runner", reinterpret_cast<PyObject*>(&RunnerType)) < 0) { Py_DECREF(&RunnerType); Py_DECREF(m); return nullptr; }
    return m;
}
