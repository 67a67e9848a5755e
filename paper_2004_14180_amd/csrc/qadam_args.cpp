// The common form of the binding's calls without Python work per buffer: every tensor is checked here for type, device, layout and
// size, and the library is called with the addresses.  Any other form (another type of tensor or number, a wrong size, a missing
// buffer) makes the function return None before anything is called, and the binding's own path takes or refuses the call.
//
// A step of a short vector is bound by the host: 51 k parameters and 4 workers, 21 buffers, 13.0 us of its 20.0 us per step were the
// checks in Python.
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/qadam.h"

namespace {

constexpr char kPlanName[] = "qadam plan";

struct Plan {
    qadam_handle_t h;
    Py_ssize_t workers;
    int64_t params, segments, code_bytes, wcode_bytes;
    bool weight_ef;
    decltype(&qadam_worker_quantize) worker_quantize;
    decltype(&qadam_server_step) server_step;
    decltype(&qadam_weight_quantize) weight_quantize;
    decltype(&qadam_step_fused) step_fused;
    decltype(&qadam_step_fused_w) step_fused_w;
};

enum class Kind { f32, integers };

// Arguments in order; ok becomes false with the first one that is not of the common form.
struct Args {
    PyObject* const* next;
    bool ok;

    int64_t integer()
    {
        PyObject* o = *next++;
        if (!ok || !PyLong_Check(o)) { ok = false; return 0; }
        const long long v = PyLong_AsLongLong(o);
        if (v == -1 && PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        return v;
    }

    float number()
    {
        PyObject* o = *next++;
        if (!ok || !(PyFloat_Check(o) || PyLong_Check(o))) { ok = false; return 0.0f; }
        const double v = PyFloat_AsDouble(o);
        if (v == -1.0 && PyErr_Occurred()) { PyErr_Clear(); ok = false; }
        return (float)v;
    }

    void* address(PyObject* o, Kind kind, int64_t need, int64_t device, bool optional = false)
    {
        if (!ok || (optional && o == Py_None)) return nullptr;
        ok = false;
        if (!THPVariable_CheckExact(o)) return nullptr;
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.has_storage() || !t.is_cuda() || t.get_device() != device || !t.is_contiguous()) return nullptr;
        if (kind == Kind::f32 ? t.scalar_type() != at::kFloat || t.numel() < need
                              : !at::isIntegralType(t.scalar_type(), true) || t.numel() * (int64_t)t.element_size() < need)
            return nullptr;
        void* p = t.data_ptr();
        ok = true;
        return p;
    }

    void* tensor(Kind kind, int64_t need, int64_t device, bool optional = false)
    {
        return address(*next++, kind, need, device, optional);
    }

    template <typename T>
    void tensors(T* (&out)[QADAM_MAX_WORKERS], Py_ssize_t count, Kind kind, int64_t need, int64_t device)
    {
        PyObject* o = *next++;
        if (!(PyList_Check(o) || PyTuple_Check(o)) || PySequence_Fast_GET_SIZE(o) != count) ok = false;
        for (Py_ssize_t i = 0; ok && i < count; ++i) out[i] = static_cast<T*>(address(PySequence_Fast_GET_ITEM(o, i), kind, need, device));
    }
};

template <typename F>
PyObject* call(const Args& a, F&& f)
{
    if (!a.ok) Py_RETURN_NONE;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = f();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
}

// body(args, plan, device, stream): the arguments behind the plan, the device and the stream
template <typename F>
PyObject* planned(PyObject* const* argv, Py_ssize_t argc, Py_ssize_t expected, F&& body)
{
    if (argc != expected) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    if (argv[0] == Py_None) Py_RETURN_NONE;
    const Plan* plan = static_cast<const Plan*>(PyCapsule_GetPointer(argv[0], kPlanName));
    if (!plan) return nullptr;
    try {
        Args a{argv + 1, true};
        const int64_t device = a.integer();
        void* stream = reinterpret_cast<void*>(a.integer());
        return body(a, *plan, device, stream);
    } catch (const std::exception&) {
        Py_RETURN_NONE;
    }
}

PyObject* worker_quantize(PyObject*, PyObject* const* argv, Py_ssize_t argc)
{
    return planned(argv, argc, 9, [](Args& a, const Plan& p, int64_t device, void* stream) {
        const int64_t worker = a.integer(), step = a.integer();
        if (worker < 0 || worker >= p.workers) a.ok = false;
        const float* grad = static_cast<float*>(a.tensor(Kind::f32, p.params, device));
        float* err = static_cast<float*>(a.tensor(Kind::f32, p.params, device));
        void* codes = a.tensor(Kind::integers, p.code_bytes, device);
        float* scales = static_cast<float*>(a.tensor(Kind::f32, p.segments, device));
        return call(a, [&] { return p.worker_quantize(p.h, (int32_t)worker, step, grad, err, codes, scales, stream); });
    });
}

PyObject* server_step(PyObject*, PyObject* const* argv, Py_ssize_t argc)
{
    return planned(argv, argc, 11, [](Args& a, const Plan& p, int64_t device, void* stream) {
        const int64_t step = a.integer();
        const float lr = a.number(), beta2 = a.number();
        void* codes[QADAM_MAX_WORKERS];
        float* scales[QADAM_MAX_WORKERS];
        a.tensors(codes, p.workers, Kind::integers, p.code_bytes, device);
        a.tensors(scales, p.workers, Kind::f32, p.segments, device);
        float* s[3];
        for (float*& t : s) t = static_cast<float*>(a.tensor(Kind::f32, p.params, device));
        return call(a, [&] { return p.server_step(p.h, step, lr, beta2, codes, scales, s[0], s[1], s[2], stream); });
    });
}

PyObject* weight_quantize(PyObject*, PyObject* const* argv, Py_ssize_t argc)
{
    return planned(argv, argc, 7, [](Args& a, const Plan& p, int64_t device, void* stream) {
        const int64_t step = a.integer();
        const float* x = static_cast<float*>(a.tensor(Kind::f32, p.params, device));
        float* werr = static_cast<float*>(a.tensor(Kind::f32, p.params, device, !p.weight_ef));
        void* wcodes = a.tensor(Kind::integers, p.wcode_bytes, device);
        return call(a, [&] { return p.weight_quantize(p.h, step, x, werr, wcodes, stream); });
    });
}

PyObject* step_fused(PyObject*, PyObject* const* argv, Py_ssize_t argc)
{
    return planned(argv, argc, 15, [](Args& a, const Plan& p, int64_t device, void* stream) {
        const int64_t step = a.integer();
        const float lr = a.number(), beta2 = a.number();
        float *grads[QADAM_MAX_WORKERS], *errs[QADAM_MAX_WORKERS], *scales[QADAM_MAX_WORKERS];
        void* codes[QADAM_MAX_WORKERS];
        a.tensors(grads, p.workers, Kind::f32, p.params, device);
        a.tensors(errs, p.workers, Kind::f32, p.params, device);
        a.tensors(codes, p.workers, Kind::integers, p.code_bytes, device);
        a.tensors(scales, p.workers, Kind::f32, p.segments, device);
        float* s[3];
        for (float*& t : s) t = static_cast<float*>(a.tensor(Kind::f32, p.params, device));
        float* werr = static_cast<float*>(a.tensor(Kind::f32, p.params, device, !p.weight_ef));
        void* wcodes = a.tensor(Kind::integers, p.wcode_bytes, device);
        return call(a, [&] {
            return p.step_fused(p.h, step, lr, beta2, grads, errs, codes, scales, s[0], s[1], s[2], werr, wcodes, stream);
        });
    });
}

PyObject* step_fused_w(PyObject*, PyObject* const* argv, Py_ssize_t argc)
{
    return planned(argv, argc, 15, [](Args& a, const Plan& p, int64_t device, void* stream) {
        const int64_t step = a.integer();
        const float lr = a.number(), beta2 = a.number();
        float *grads[QADAM_MAX_WORKERS], *mw[QADAM_MAX_WORKERS], *vw[QADAM_MAX_WORKERS], *errs[QADAM_MAX_WORKERS],
            *scales[QADAM_MAX_WORKERS];
        void* codes[QADAM_MAX_WORKERS];
        a.tensors(grads, p.workers, Kind::f32, p.params, device);
        a.tensors(mw, p.workers, Kind::f32, p.params, device);
        a.tensors(vw, p.workers, Kind::f32, p.params, device);
        a.tensors(errs, p.workers, Kind::f32, p.params, device);
        a.tensors(codes, p.workers, Kind::integers, p.code_bytes, device);
        a.tensors(scales, p.workers, Kind::f32, p.segments, device);
        float* x = static_cast<float*>(a.tensor(Kind::f32, p.params, device));
        float* werr = static_cast<float*>(a.tensor(Kind::f32, p.params, device, !p.weight_ef));
        void* wcodes = a.tensor(Kind::integers, p.wcode_bytes, device);
        return call(a, [&] { return p.step_fused_w(p.h, step, lr, beta2, grads, mw, vw, errs, codes, scales, x, werr, wcodes, stream); });
    });
}

// (the address of qadam_quantize_segment_noalloc, device, stream, k_g, n, grad, err, codes, scale); the sizes of the buffers are the
// caller's word, as in the binding
PyObject* quantize_segment(PyObject*, PyObject* const* argv, Py_ssize_t argc)
{
    if (argc != 9) {
        PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
        return nullptr;
    }
    try {
        Args a{argv, true};
        const auto fn = reinterpret_cast<decltype(&qadam_quantize_segment_noalloc)>(a.integer());
        (void)a.integer();
        void* stream = reinterpret_cast<void*>(a.integer());
        const int64_t k_g = a.integer(), n = a.integer();
        if (k_g < INT32_MIN || k_g > INT32_MAX) a.ok = false;
        void* t[4] = {};
        for (void*& p : t) {
            PyObject* o = *a.next++;
            if (!a.ok) break;
            a.ok = false;
            if (!THPVariable_CheckExact(o)) break;
            const at::Tensor& v = THPVariable_Unpack(o);
            if (!v.has_storage() || !v.is_cuda() || !v.is_contiguous()) break;
            p = v.data_ptr();
            a.ok = true;
        }
        return call(a, [&] {
            return fn((int32_t)k_g, n, static_cast<float*>(t[0]), static_cast<float*>(t[1]), t[2], static_cast<float*>(t[3]), stream);
        });
    } catch (const std::exception&) {
        Py_RETURN_NONE;
    }
}

void free_plan(PyObject* capsule) { delete static_cast<Plan*>(PyCapsule_GetPointer(capsule, kPlanName)); }

// (handle, workers, params, segments, code bytes, weight code bytes, weight_ef, addresses of the five entry points)
PyObject* plan(PyObject*, PyObject* const* argv, Py_ssize_t argc)
{
    Args a{argv, argc == 12};
    int64_t v[12];
    for (Py_ssize_t i = 0; i < 12 && a.ok; ++i) v[i] = a.integer();
    if (!a.ok || v[1] < 1 || v[1] > QADAM_MAX_WORKERS) {
        PyErr_SetString(PyExc_TypeError, "twelve integers expected");
        return nullptr;
    }
    Plan* p = new Plan{reinterpret_cast<qadam_handle_t>(v[0]), (Py_ssize_t)v[1], v[2], v[3], v[4], v[5], v[6] != 0,
                       reinterpret_cast<decltype(&qadam_worker_quantize)>(v[7]), reinterpret_cast<decltype(&qadam_server_step)>(v[8]),
                       reinterpret_cast<decltype(&qadam_weight_quantize)>(v[9]), reinterpret_cast<decltype(&qadam_step_fused)>(v[10]),
                       reinterpret_cast<decltype(&qadam_step_fused_w)>(v[11])};
    PyObject* capsule = PyCapsule_New(p, kPlanName, free_plan);
    if (!capsule) delete p;
    return capsule;
}

#define QADAM_FUNCTION(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}

PyMethodDef kFunctions[] = {QADAM_FUNCTION(plan), QADAM_FUNCTION(worker_quantize), QADAM_FUNCTION(server_step),
                            QADAM_FUNCTION(weight_quantize), QADAM_FUNCTION(step_fused), QADAM_FUNCTION(step_fused_w),
                            QADAM_FUNCTION(quantize_segment), {nullptr, nullptr, 0, nullptr}};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_args", "Calls of the library with tensors of the common form.", -1, kFunctions,
                       nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__args(void)
{
    PyObject* m = PyModule_Create(&kModule);
    // tensors are read through inlined code of this version
    if (m && PyModule_AddStringConstant(m, "torch_version", QADAM_TORCH_VERSION) < 0) { Py_DECREF(m); return nullptr; }
    return m;
}
