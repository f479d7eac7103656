// The Python binding's calls on torch tensors, in C++: a plan's execute, its
// adjoint and the fused loss, and their autograd functions.
//
// A small transform takes the GPU 3-7 us.  Marshalled in Python with ctypes
// api.fft took 8.6 us of host time, a plan's execute 6.9, and a forward with
// its backward 100, much of it the autograd engine's thread waiting for the
// interpreter; from here 3.9, 3.1 and 46 us (hipLaunchKernel itself is about
// 2.5, the engine's hand-over to its thread most of the 46).
//
// Every entry handles the ordinary case only -- plain dense GPU tensors of
// the right type and size, no tensor subclass, dispatch mode, functorch
// transform, tracing or forward-mode gradient -- and returns NotImplemented
// for anything else, which the Python code then handles (or refuses) itself.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/jit/frontend/tracer.h>
#include <torch/custom_class.h>

#include "../../include/mifft.h"

namespace {

using at::Tensor;

// Entry points of the library that the binding has loaded, and its
// status-to-exception function.
struct Calls {
    int (*execute)(fft_plan, const void*, void*, void*) = nullptr;
    int (*adjoint)(fft_plan, const void*, void*, void*) = nullptr;
    int (*loss_grad)(fft_plan, const void*, const float*, void*, float*, void*) = nullptr;
    int (*loss_grad_to_scale)(fft_plan, const void*, const float*, void*, float*, void*) = nullptr;
    int (*scaled)(fft_plan, const void*, const int32_t*, void*, int32_t*, void*) = nullptr;
    int (*scale)(const void*, const float*, void*, int64_t, void*) = nullptr;
    void (*destroy)(fft_plan) = nullptr;
    PyObject* check = nullptr;
};
Calls g_calls;

// A plan handle, shared by the Python plan object and by the graphs that
// will run its adjoint: destroyed when closed or when the last of them goes.
struct PlanRef : torch::CustomClassHolder {
    fft_plan h;
    int dtype, sign;
    int64_t n, batch;
    PlanRef(fft_plan h_, int dtype_, int sign_, int64_t n_, int64_t batch_)
        : h(h_), dtype(dtype_), sign(sign_), n(n_), batch(batch_)
    {
    }
    void close()
    {
        if (h)
            g_calls.destroy(h);
        h = nullptr;
    }
    ~PlanRef() override { close(); }
    // whether an execute (or adjoint) of an FFT_R32 plan reads reals
    bool to_bins(bool adj) const { return (sign < 0) != adj; }
    bool reads_reals(bool adj) const { return dtype == FFT_R32 && to_bins(adj); }
    at::ScalarType type(bool input, bool adj) const
    {
        switch (dtype) {
        case FFT_R32: return to_bins(adj) == input ? at::kFloat : at::kComplexFloat;
        case FFT_C16: return at::kHalf;
        case FFT_CBF16: return at::kBFloat16;
        default: return at::kComplexFloat;
        }
    }
    // values per transform of one side
    int64_t values(bool input, bool adj) const
    {
        if (dtype == FFT_R32)
            return to_bins(adj) == input ? n : n / 2 + 1;
        return dtype == FFT_C32 ? n : 2 * n;
    }
};
using Plan = c10::intrusive_ptr<PlanRef>;

constexpr const char* kCapsule = "mifft.plan";

Plan* plan_of(PyObject* o)
{
    return PyCapsule_CheckExact(o) ? static_cast<Plan*>(PyCapsule_GetPointer(o, kCapsule)) : nullptr;
}

// Raises the binding's exception for status rc from a thread that need not
// hold the interpreter lock.
[[noreturn]] void raise_status(int rc)
{
    const PyGILState_STATE g = PyGILState_Ensure();
    PyObject* r = PyObject_CallFunction(g_calls.check, "i", rc);
    Py_XDECREF(r);
    python_error e;
    if (!PyErr_Occurred())
        PyErr_SetString(PyExc_RuntimeError, "mifft call failed");
    e.persist();
    PyGILState_Release(g);
    throw e;
}

// Nothing that would see this call otherwise than as a kernel launch.
bool plain_context()
{
    return !c10::impl::TorchDispatchModeTLS::any_modes_set() && at::impl::PythonTorchFunctionTLS::stack_len() == 0 &&
           !c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode) &&
           !torch::jit::tracer::isTracing();
}

bool dense(const Tensor& t, at::ScalarType type)
{
    return t.is_cuda() && t.layout() == at::kStrided && t.has_storage() && t.is_contiguous() && !t.is_conj() && !t.is_neg() &&
           t.scalar_type() == type;
}

bool side_ok(const Tensor& t, const PlanRef& p, bool input, bool adj)
{
    return dense(t, p.type(input, adj)) && t.numel() == p.values(input, adj) * p.batch;
}

// Whether a call without an output given has one of the plan's shape.
bool shape_ok(const Tensor& x, const PlanRef& p, bool adj)
{
    return p.dtype != FFT_R32 || (x.dim() >= 1 && x.size(-1) == p.values(true, adj));
}

Tensor new_output(const Tensor& x, const PlanRef& p, bool adj)
{
    if (p.dtype != FFT_R32)
        return at::empty_like(x);
    auto sizes = x.sizes().vec();
    sizes.back() = p.values(false, adj);
    return at::empty(sizes, x.options().dtype(p.type(false, adj)));
}

// The call itself, on the current stream; without the interpreter lock.
void launch(const PlanRef& p, const Tensor& x, const Tensor& out, bool adj)
{
    const int rc =
        (adj ? g_calls.adjoint : g_calls.execute)(p.h, x.data_ptr(), out.data_ptr(),
                                                  c10::hip::getCurrentHIPStream().stream());
    if (rc != FFT_OK)
        raise_status(rc);
}

Tensor transform(const PlanRef& p, const Tensor& x, bool adj)
{
    Tensor out = new_output(x, p, adj);
    launch(p, x, out, adj);
    return out;
}

Plan saved_plan(torch::autograd::AutogradContext* ctx)
{
    return c10::static_intrusive_pointer_cast<PlanRef>(ctx->saved_data["plan"].toCapsule());
}

// A linear map and its adjoint.
struct LinearFn : torch::autograd::Function<LinearFn> {
    static Tensor forward(torch::autograd::AutogradContext* ctx, const Tensor& x, const Plan& plan)
    {
        ctx->saved_data["plan"] = c10::IValue::make_capsule(plan);
        return transform(*plan, x, false);
    }
    static torch::autograd::tensor_list backward(torch::autograd::AutogradContext* ctx,
                                                 torch::autograd::tensor_list grads)
    {
        const Plan plan = saved_plan(ctx);
        const Tensor g = grads[0].to(plan->type(true, true)).resolve_conj().resolve_neg().contiguous();
        TORCH_CHECK(side_ok(g, *plan, true, true) && shape_ok(g, *plan, true),
                    "the gradient does not fit the plan that made the output");
        return {transform(*plan, g, true), Tensor()};
    }
};

// L = sum_b sum_k w |(A x_b)_k|^2 with the gradient from the same kernel.
struct LossFn : torch::autograd::Function<LossFn> {
    // to_scale: a backward will follow
    static Tensor forward(torch::autograd::AutogradContext* ctx, const Tensor& x, const Tensor& w, const Plan& plan,
                          bool to_scale)
    {
        Tensor grad = at::empty_like(x);
        Tensor loss = at::empty({plan->batch}, x.options().dtype(at::kFloat));
        const int rc = (to_scale ? g_calls.loss_grad_to_scale : g_calls.loss_grad)(
            plan->h, x.data_ptr(), static_cast<const float*>(w.data_ptr()), grad.data_ptr(),
            static_cast<float*>(loss.data_ptr()), c10::hip::getCurrentHIPStream().stream());
        if (rc != FFT_OK)
            raise_status(rc);
        ctx->save_for_backward({grad});
        return loss.sum();
    }
    static torch::autograd::tensor_list backward(torch::autograd::AutogradContext* ctx,
                                                 torch::autograd::tensor_list grads)
    {
        const Tensor grad = ctx->get_saved_variables()[0], g = grads[0].to(at::kFloat);
        // a plain product of what forward saved, with no graph of its own
        if (plain_context() && !(at::GradMode::is_enabled() && g.requires_grad()) && dense(grad, at::kComplexFloat) &&
            dense(g, at::kFloat) && g.numel() == 1 && g.device() == grad.device() && grad.numel() > 0) {
            Tensor out = at::empty_like(grad);
            if (g_calls.scale(grad.data_ptr(), static_cast<const float*>(g.data_ptr()), out.data_ptr(), grad.numel(),
                              c10::hip::getCurrentHIPStream().stream()) == 0)
                return {out, Tensor(), Tensor(), Tensor()};
        }
        return {grad * g, Tensor(), Tensor(), Tensor()};
    }
};

// ------------------------------------------------------------------ Python
const Tensor* plain_tensor(PyObject* o)
{
    if (!THPVariable_CheckExact(o))
        return nullptr;
    const Tensor& t = THPVariable_Unpack(o);
    return t.defined() && !t._fw_grad(0).defined() ? &t : nullptr;
}

PyObject* not_implemented()
{
    Py_INCREF(Py_NotImplemented);
    return Py_NotImplemented;
}

template <class F>
PyObject* guarded(F fn)
{
    HANDLE_TH_ERRORS
    return fn();
    END_HANDLE_TH_ERRORS
}

// plan(handle, dtype, sign, n, batch) -> capsule
PyObject* py_plan(PyObject*, PyObject* args)
{
    unsigned long long h;
    int dtype, sign;
    long long n, batch;
    if (!PyArg_ParseTuple(args, "KiiLL", &h, &dtype, &sign, &n, &batch))
        return nullptr;
    return guarded([&]() -> PyObject* {
        auto* p = new Plan(c10::make_intrusive<PlanRef>(reinterpret_cast<fft_plan>(h), dtype, sign, n, batch));
        return PyCapsule_New(p, kCapsule, [](PyObject* o) {
            delete static_cast<Plan*>(PyCapsule_GetPointer(o, kCapsule));
        });
    });
}

PyObject* py_close(PyObject*, PyObject* capsule)
{
    Plan* p = plan_of(capsule);
    if (!p)
        return PyErr_Format(PyExc_TypeError, "not a plan");
    (*p)->close();
    Py_RETURN_NONE;
}

// run(capsule, x, out or None, adjoint) -> tensor or NotImplemented
PyObject* py_run(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (n != 4)
        return PyErr_Format(PyExc_TypeError, "run takes 4 arguments");
    return guarded([&]() -> PyObject* {
        Plan* plan = plan_of(a[0]);
        const bool adj = a[3] == Py_True;
        const Tensor* x = plain_tensor(a[1]);
        if (!plan || !x || !plain_context() || !side_ok(*x, **plan, true, adj))
            return not_implemented();
        const Plan keep = *plan;
        if (a[2] == Py_None) {
            if (!shape_ok(*x, *keep, adj))
                return not_implemented();
            Tensor out;
            {
                pybind11::gil_scoped_release nogil;
                out = transform(*keep, *x, adj);
            }
            return THPVariable_Wrap(std::move(out));
        }
        const Tensor* out = plain_tensor(a[2]);
        if (!out || !side_ok(*out, *keep, false, adj))
            return not_implemented();
        {
            const Tensor xi = *x, oi = *out;
            pybind11::gil_scoped_release nogil;
            launch(*keep, xi, oi, adj);
        }
        Py_INCREF(a[2]);
        return a[2];
    });
}

// The cached plan for x: cache[(device, n, batch, sign, kind)], n the last
// axis or, if `bins`, the length given for n / 2 + 1 bins; for `ndim` > 0 axes
// cache[(device, "nd", shape, batch, sign)].
Plan* cached(PyObject* cache, const Tensor& x, int sign, PyObject* kind, int64_t ndim, bool bins, int64_t n)
{
    static PyObject* const nd = PyUnicode_InternFromString("nd");
    static PyObject* const attr = PyUnicode_InternFromString("_ref");
    if (!PyDict_CheckExact(cache) || x.dim() < 1 || !x.is_cuda() || ndim > x.dim())
        return nullptr;
    const int64_t last = x.size(-1);
    if (last < 1)
        return nullptr;
    PyObject* key;
    if (ndim > 0) {
        int64_t points = 1;
        PyObject* shape = PyTuple_New(ndim);
        for (int64_t i = 0; i < ndim; i++) {
            const int64_t d = x.size(x.dim() - ndim + i);
            points *= d;
            PyTuple_SET_ITEM(shape, i, PyLong_FromLongLong(d));
        }
        key = points < 1 ? nullptr
                         : Py_BuildValue("(iOOLi)", (int)x.get_device(), nd, shape, (long long)(x.numel() / points), sign);
        Py_DECREF(shape);
    } else {
        if (bins && (n < 2 || n / 2 + 1 != last))
            return nullptr;
        key = Py_BuildValue("(iLLiO)", (int)x.get_device(), (long long)(bins ? n : last),
                            (long long)(x.numel() / last), sign, kind);
    }
    if (!key) {
        PyErr_Clear();
        return nullptr;
    }
    PyObject* p = PyDict_GetItemWithError(cache, key);  // borrowed
    Py_DECREF(key);
    if (!p) {
        PyErr_Clear();
        return nullptr;
    }
    PyObject* ref = PyObject_GetAttr(p, attr);
    if (!ref) {
        PyErr_Clear();
        return nullptr;
    }
    Plan* plan = plan_of(ref);  // kept by the plan object, which the cache holds
    Py_DECREF(ref);
    PyErr_Clear();
    return plan;
}

// call(cache, x, sign, kind, ndim, n or None, differentiable) -> tensor or
// NotImplemented (no cached plan, or not the ordinary case); n: the length
// that bins transform to
PyObject* py_call(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (n != 7)
        return PyErr_Format(PyExc_TypeError, "call takes 7 arguments");
    return guarded([&]() -> PyObject* {
        const Tensor* xp = plain_tensor(a[1]);
        if (!xp || !plain_context() || !PyLong_CheckExact(a[2]) || !PyLong_CheckExact(a[4]) ||
            !(a[5] == Py_None || PyLong_CheckExact(a[5])))
            return not_implemented();
        const long sign = PyLong_AsLong(a[2]);
        const bool bins = a[5] != Py_None;
        const long long ndim = PyLong_AsLongLong(a[4]), len = bins ? PyLong_AsLongLong(a[5]) : 0;
        if (PyErr_Occurred()) {
            PyErr_Clear();
            return not_implemented();
        }
        Plan* plan = cached(a[0], *xp, (int)sign, a[3], ndim, bins, len);
        if (!plan || !side_ok(*xp, **plan, true, false) || !shape_ok(*xp, **plan, false))
            return not_implemented();
        const Plan keep = *plan;
        const Tensor x = *xp;
        const bool diff = a[6] == Py_True;
        Tensor out;
        {
            pybind11::gil_scoped_release nogil;
            out = diff ? LinearFn::apply(x, keep) : transform(*keep, x, false);
        }
        return THPVariable_Wrap(std::move(out));
    });
}

// loss(cache, x, w, sign) -> the summed loss, or NotImplemented
PyObject* py_loss(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    static PyObject* const c32 = PyUnicode_InternFromString("c32");
    if (n != 4)
        return PyErr_Format(PyExc_TypeError, "loss takes 4 arguments");
    return guarded([&]() -> PyObject* {
        const Tensor *xp = plain_tensor(a[1]), *wp = plain_tensor(a[2]);
        if (!xp || !wp || !plain_context() || !PyLong_CheckExact(a[3]))
            return not_implemented();
        const long sign = PyLong_AsLong(a[3]);
        if (PyErr_Occurred()) {
            PyErr_Clear();
            return not_implemented();
        }
        Plan* plan = cached(a[0], *xp, (int)sign, c32, 0, false, 0);
        if (!plan || (*plan)->n > 2048 || !side_ok(*xp, **plan, true, false))
            return not_implemented();
        if (!dense(*wp, at::kFloat) || wp->numel() != xp->numel())
            return not_implemented();
        const Plan keep = *plan;
        const Tensor x = *xp, w = *wp;
        const bool to_scale = at::GradMode::is_enabled() && x.requires_grad();
        Tensor out;
        {
            pybind11::gil_scoped_release nogil;
            out = LossFn::apply(x, w, keep, to_scale);
        }
        return THPVariable_Wrap(std::move(out));
    });
}

// scaled(capsule, x) -> (tensor, exponents) or NotImplemented
PyObject* py_scaled(PyObject*, PyObject* const* a, Py_ssize_t n)
{
    if (n != 2)
        return PyErr_Format(PyExc_TypeError, "scaled takes 2 arguments");
    return guarded([&]() -> PyObject* {
        Plan* plan = plan_of(a[0]);
        const Tensor* x = plain_tensor(a[1]);
        if (!plan || !x || !plain_context() || ((*plan)->dtype != FFT_C16 && (*plan)->dtype != FFT_CBF16) ||
            !side_ok(*x, **plan, true, false))
            return not_implemented();
        const Plan keep = *plan;
        Tensor out, exponents;
        {
            pybind11::gil_scoped_release nogil;
            out = at::empty_like(*x);
            exponents = at::empty({keep->batch}, x->options().dtype(at::kInt));
            const int rc = g_calls.scaled(keep->h, x->data_ptr(), nullptr, out.data_ptr(),
                                          static_cast<int32_t*>(exponents.data_ptr()),
                                          c10::hip::getCurrentHIPStream().stream());
            if (rc != FFT_OK)
                raise_status(rc);
        }
        return Py_BuildValue("(NN)", THPVariable_Wrap(std::move(out)), THPVariable_Wrap(std::move(exponents)));
    });
}

// bind(execute, adjoint, loss_grad, loss_grad_to_scale, scaled, scale, destroy, check)
PyObject* py_bind(PyObject*, PyObject* args)
{
    unsigned long long e, d, l, t, s, c, x;
    PyObject* check;
    if (!PyArg_ParseTuple(args, "KKKKKKKO", &e, &d, &l, &t, &s, &c, &x, &check))
        return nullptr;
    g_calls.execute = reinterpret_cast<decltype(g_calls.execute)>(e);
    g_calls.adjoint = reinterpret_cast<decltype(g_calls.adjoint)>(d);
    g_calls.loss_grad = reinterpret_cast<decltype(g_calls.loss_grad)>(l);
    g_calls.loss_grad_to_scale = reinterpret_cast<decltype(g_calls.loss_grad_to_scale)>(t);
    g_calls.scaled = reinterpret_cast<decltype(g_calls.scaled)>(s);
    g_calls.scale = reinterpret_cast<decltype(g_calls.scale)>(c);
    g_calls.destroy = reinterpret_cast<decltype(g_calls.destroy)>(x);
    Py_INCREF(check);
    g_calls.check = check;
    Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"bind", py_bind, METH_VARARGS, nullptr},
    {"plan", py_plan, METH_VARARGS, nullptr},
    {"close", py_close, METH_O, nullptr},
    {"run", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_run)), METH_FASTCALL, nullptr},
    {"scaled", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_scaled)), METH_FASTCALL, nullptr},
    {"call", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_call)), METH_FASTCALL, nullptr},
    {"loss", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(py_loss)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_mifft_torch", nullptr, -1, kMethods,
                       nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__mifft_torch() { return PyModule_Create(&kModule); }
