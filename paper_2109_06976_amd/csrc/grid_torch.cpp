// The torch-facing calls in native code (module _gridtorch): grid.fd_grad_torch,
// autograd.forward_dynamics and the launches on device buffers, for plain tensors.
//
// In Python the allocation of four outputs, the checks and the argument conversion of one gradient
// call take 13 us beside a 4 us kernel, and an autograd function whose backward is Python makes
// the engine's device thread take the interpreter lock, fetch the stream and allocate there. Here
// the outputs are at::empty, the checks read the tensors' fields, and the backward node is C++.
//
// Each entry point takes only what it can run exactly as the Python code would: torch.Tensor
// objects (no subclass) that are contiguous float32 and large enough, on the model's device. It
// returns None for anything else, and the caller then takes the Python path, which converts or
// raises. The tensors that the backward step gets back are checked like arguments. The library's functions
// come as addresses from the ctypes binding, so both sides call the library that is loaded.
#include <torch/extension.h>

#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>

#include <map>
#include <string>

namespace {

using Handle = void*;
using Vec7 = int32_t (*)(Handle, int32_t, const float*, const float*, const float*, float*, float*,
                         float*, float*, void*);
using Fd = int32_t (*)(Handle, int32_t, const float*, const float*, const float*, float*, void*);
using Vjp = int32_t (*)(Handle, int32_t, const float*, const float*, const float*, const float*,
                        float*, float*, float*, void*);

struct Library {
    Vec7 fd_grad = nullptr;
    Fd fd = nullptr;
    Vjp vjp = nullptr, vjp_adjoint = nullptr;
};
// set once when the module is loaded, before any call; `fail` raises the binding's GridError (these
// stay for the process, like the module)
Library g_lib;
PyObject* g_fail = nullptr;
PyObject* g_dev = nullptr;   // the binding's own check of a buffer (raises, or returns its address)

// with the interpreter lock held: the binding's own exception
void check(int32_t status)
{
    if (status != 0)
        py::reinterpret_borrow<py::object>(g_fail)(status);
}

// with the interpreter lock held and a Python exception set: carries it out of the autograd
// engine's thread
[[noreturn]] void raise_set()
{
    python_error e;
    e.persist();
    throw e;
}

// on the autograd engine's threads: the same exception (the library's message is this thread's)
void check_unlocked(int32_t status)
{
    if (status == 0)
        return;
    py::gil_scoped_acquire gil;
    Py_XDECREF(PyObject_CallFunction(g_fail, "i", (int)status));
    raise_set();
}

// a library call without the interpreter lock: a launch waits when the hardware queue is full
template <class F>
int32_t unlocked(const F& call)
{
    py::gil_scoped_release released;
    return call();
}

// the handle of a grid.Model (a ctypes pointer object; None once the model is closed)
Handle handle_of(const py::object& model)
{
    const py::object h = model.attr("_h");
    if (h.is_none())
        return nullptr;
    const py::object v = h.attr("value");
    return v.is_none() ? nullptr : reinterpret_cast<Handle>(v.cast<uintptr_t>());
}

void* stream_of(const at::Tensor& t)
{
    return (void*)c10::hip::getCurrentHIPStreamMasqueradingAsCUDA(t.device().index()).stream();
}

bool fits(const at::Tensor& t, int64_t device)
{
    return t.is_cuda() && t.scalar_type() == at::kFloat && t.layout() == at::kStrided &&
           t.is_contiguous() && t.device().index() == device && !t.is_neg();
}

// a contiguous float32 tensor on GPU `device` (not a subclass of torch.Tensor but its Parameter)
const at::Tensor* plain(PyObject* o, int64_t device)
{
    if (!THPVariable_CheckExact(o))
        return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    return fits(t, device) ? &t : nullptr;
}

float* data(const at::Tensor& t)
{
    return static_cast<float*>(t.mutable_data_ptr());
}
const float* cdata(const at::Tensor& t)
{
    return static_cast<const float*>(t.const_data_ptr());
}

// The address of a tensor that the backward step was handed with at least `need` elements. A saved
// tensor is whatever the caller's unpack hook returned, if one is set, so it is checked like an
// argument; one that does not fit goes to the binding's own check, which raises.
const float* checked(const at::Tensor& t, int64_t device, int64_t need, const char* what)
{
    if (t.defined() && fits(t, device) && t.numel() >= need)
        return cdata(t);
    py::gil_scoped_acquire gil;
    PyObject* a = PyObject_CallFunction(g_dev, "NLLs", py::cast(t).release().ptr(),
                                        (long long)need, (long long)device, what);
    if (!a)
        raise_set();
    const py::object address = py::reinterpret_steal<py::object>(a);
    return address.is_none() ? nullptr : reinterpret_cast<const float*>(address.cast<uintptr_t>());
}

struct Outputs {
    at::Tensor qdd, Minv, dq, dqd;
};

Outputs run_fd_grad(Handle h, const at::Tensor& q, const at::Tensor& qd, const at::Tensor& tau,
                    void* stream)
{
    const int64_t N = q.size(0), n = q.size(1);
    const auto opt = q.options().requires_grad(false);
    Outputs o{at::empty({N, n}, opt), at::empty({N, n, n}, opt), at::empty({N, n, n}, opt),
              at::empty({N, n, n}, opt)};
    check(unlocked([&] {
        return g_lib.fd_grad(h, (int32_t)N, cdata(q), cdata(qd), cdata(tau), data(o.qdd),
                             data(o.Minv), data(o.dq), data(o.dqd), stream);
    }));
    return o;
}

// a reference to the model that may be dropped by any thread
struct Held : torch::CustomClassHolder {
    explicit Held(const py::object& o) : object(o.ptr()) { Py_INCREF(object); }
    ~Held() override
    {
        if (Py_IsInitialized()) {
            py::gil_scoped_acquire gil;
            Py_DECREF(object);
        }
    }
    PyObject* object;
};

struct Dynamics : torch::autograd::Function<Dynamics> {
    static at::Tensor forward(torch::autograd::AutogradContext* ctx, const at::Tensor& q,
                              const at::Tensor& qd, const at::Tensor& tau,
                              const c10::IValue& model, bool jacobians)
    {
        at::AutoDispatchBelowADInplaceOrView below;
        const auto held = c10::static_intrusive_pointer_cast<Held>(model.toCapsule());
        const Handle h = handle_of(py::reinterpret_borrow<py::object>(held->object));
        ctx->saved_data["model"] = model;
        ctx->saved_data["jacobians"] = jacobians;
        void* stream = stream_of(q);
        if (jacobians) {
            Outputs o = run_fd_grad(h, q, qd, tau, stream);
            ctx->save_for_backward({o.Minv, o.dq, o.dqd});
            return o.qdd;
        }
        at::Tensor qdd = at::empty_like(q);
        check(unlocked([&] {
            return g_lib.fd(h, (int32_t)q.size(0), cdata(q), cdata(qd), cdata(tau), data(qdd), stream);
        }));
        ctx->save_for_backward({q, qd, qdd});
        return qdd;
    }

    static torch::autograd::variable_list backward(torch::autograd::AutogradContext* ctx,
                                                   torch::autograd::variable_list grads)
    {
        // first, and outside any dispatch guard: an unpack hook may run the caller's graph again
        // (checkpointing without re-entrant autograd recomputes its region there)
        const auto saved = ctx->get_saved_variables();
        at::AutoDispatchBelowADInplaceOrView below;
        const at::Tensor g = grads[0].contiguous().to(at::kFloat);
        at::Tensor a = at::empty_like(g), b = at::empty_like(g), c = at::empty_like(g);
        const auto held =
            c10::static_intrusive_pointer_cast<Held>(ctx->saved_data["model"].toCapsule());
        Handle h;
        {
            py::gil_scoped_acquire gil;   // the model may have been closed since
            h = handle_of(py::reinterpret_borrow<py::object>(held->object));
        }
        void* stream = stream_of(g);
        const int32_t N = (int32_t)g.size(0);
        const int64_t device = g.device().index(), vec = g.numel(), mat = vec * g.size(1);
        const float* x[3];
        if (ctx->saved_data["jacobians"].toBool()) {
            const char* const names[3] = {"Minv", "dqdd_dq", "dqdd_dqd"};
            for (int k = 0; k < 3; ++k)
                x[k] = checked(saved[k], device, mat, names[k]);
            check_unlocked(g_lib.vjp(h, N, x[1], x[2], x[0], checked(g, device, vec, "gbar"), data(a),
                                     data(b), data(c), stream));
        } else {
            const char* const names[3] = {"q", "qd", "qdd"};
            for (int k = 0; k < 3; ++k)
                x[k] = checked(saved[k], device, vec, names[k]);
            check_unlocked(g_lib.vjp_adjoint(h, N, x[0], x[1], x[2], checked(g, device, vec, "gbar"),
                                             data(a), data(b), data(c), stream));
        }
        return {a, b, c, at::Tensor(), at::Tensor()};
    }
};

// q, qd, tau: [N][n] each
bool inputs(int64_t n, int64_t device, const py::object (&o)[3], const at::Tensor* (&t)[3])
{
    for (int k = 0; k < 3; ++k) {
        t[k] = plain(o[k].ptr(), device);
        if (!t[k] || t[k]->dim() != 2 || t[k]->size(1) != n || t[k]->size(0) != t[0]->size(0))
            return false;
    }
    return t[0]->size(0) <= INT32_MAX;
}

py::object fd_grad(const py::object& model, int64_t n, int64_t device, const py::object& q,
                   const py::object& qd, const py::object& tau)
{
    const py::object o[3] = {q, qd, tau};
    const at::Tensor* t[3];
    if (!inputs(n, device, o, t))
        return py::none();
    const Outputs y = run_fd_grad(handle_of(model), *t[0], *t[1], *t[2], stream_of(*t[0]));
    py::dict d;
    d["qdd"] = y.qdd;
    d["Minv"] = y.Minv;
    d["dqdd_dq"] = y.dq;
    d["dqdd_dqd"] = y.dqd;
    return d;
}

py::object forward_dynamics(const py::object& model, int64_t n, int64_t device,
                            const py::object& q, const py::object& qd, const py::object& tau,
                            bool jacobians)
{
    const py::object o[3] = {q, qd, tau};
    const at::Tensor* t[3];
    if (!inputs(n, device, o, t))
        return py::none();
    const c10::IValue held = c10::IValue::make_capsule(c10::make_intrusive<Held>(model));
    return py::cast(Dynamics::apply(*t[0], *t[1], *t[2], held, jacobians));
}

// A launch on the caller's buffers: fn is the address of a library function that takes a model,
// N, the buffers' addresses (as many as `bufs`, each with at least need[k] elements) and a stream.
// None: some buffer is not a plain tensor.
py::object launch(uintptr_t fn, const py::object& model, int64_t device, int64_t N,
                  const py::tuple& bufs, const py::tuple& need, const py::object& stream)
{
    const size_t count = bufs.size();
    if (count > 7 || N > INT32_MAX || N < INT32_MIN)
        return py::none();
    void* p[7];
    for (size_t k = 0; k < count; ++k) {
        const at::Tensor* t = plain(PyTuple_GET_ITEM(bufs.ptr(), k), device);
        if (!t || t->numel() < PyLong_AsLongLong(PyTuple_GET_ITEM(need.ptr(), k)))
            return py::none();
        p[k] = t->data_ptr();
    }
    void* s = nullptr;
    if (!stream.is_none())
        s = reinterpret_cast<void*>(
            (PyLong_Check(stream.ptr()) ? stream : stream.attr("cuda_stream")).cast<uintptr_t>());
    Handle h = handle_of(model);
    const int32_t n = (int32_t)N;
    using V = void*;
    if (count != 2 && count != 4 && count != 5 && count != 7)
        return py::none();
    check(unlocked([&]() -> int32_t {
        switch (count) {
        case 2:
            return reinterpret_cast<int32_t (*)(V, int32_t, V, V, V)>(fn)(h, n, p[0], p[1], s);
        case 4:
            return reinterpret_cast<int32_t (*)(V, int32_t, V, V, V, V, V)>(fn)(h, n, p[0], p[1],
                                                                               p[2], p[3], s);
        case 5:
            return reinterpret_cast<int32_t (*)(V, int32_t, V, V, V, V, V, V)>(fn)(
                h, n, p[0], p[1], p[2], p[3], p[4], s);
        default:
            return reinterpret_cast<int32_t (*)(V, int32_t, V, V, V, V, V, V, V, V)>(fn)(
                h, n, p[0], p[1], p[2], p[3], p[4], p[5], p[6], s);
        }
    }));
    return py::bool_(true);
}

}  // namespace

PYBIND11_MODULE(_gridtorch, m)
{
    m.def("bind", [](const std::map<std::string, uintptr_t>& f, py::object fail, py::object dev) {
        g_fail = fail.release().ptr();
        g_dev = dev.release().ptr();
        g_lib.fd_grad = reinterpret_cast<Vec7>(f.at("grid_fd_grad"));
        g_lib.fd = reinterpret_cast<Fd>(f.at("grid_fd"));
        g_lib.vjp = reinterpret_cast<Vjp>(f.at("grid_fd_vjp"));
        g_lib.vjp_adjoint = reinterpret_cast<Vjp>(f.at("grid_fd_vjp_adjoint"));
    });
    m.def("fd_grad", &fd_grad);
    m.def("forward_dynamics", &forward_dynamics);
    m.def("launch", &launch);
}
