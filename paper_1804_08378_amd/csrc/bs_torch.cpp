// The binding's common calls without an interpreter in the way: a planned stack bound to torch tensors (module _bs_torch).
//
// One call of a small stack is a launch of a few microseconds; reading shapes, asking for memory and passing pointers through ctypes took
// three times that (Stack.run 10.3 us, run and backward 21 us, the module under autograd 85 to 95 us, whatever the kernels).  Here the same
// checks, allocations and calls are made natively for the plain case -- dense tensors of the plan's shape, type, memory order and device on
// the current stream -- and every method returns None for anything else, which the Python code then handles (or refuses) as it always does.
//
// The library is reached through the function addresses the Python side has loaded: this file links against torch only.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/core/PythonFallbackKernel.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <c10/util/SmallVector.h>
#include <torch/csrc/Device.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/python_variable.h>

#include <array>
#include <cstdint>
#include <map>
#include <memory>
#include <mutex>
#include <utility>
#include <vector>

namespace {

using Shape = std::array<int64_t, 4>;
using RunFn = int (*)(const void *, const void *, int64_t, const void *const *, void *, int64_t, int32_t *const *, void *, uint64_t, void *);
using BackwardFn = int (*)(const void *, const void *, int64_t, const void *const *, const int32_t *const *, const void *, int64_t, void *, int64_t,
                           void *const *, void *, uint64_t, void *);
using DestroyFn = void (*)(void *);

// A failed library call, raised in Python as the binding's own error (the binding sets the class).
PyObject *g_error = nullptr;
struct CallFailed : std::exception {
    int status;
    const char *where;
    CallFailed(int s, const char *w) : status(s), where(w) {}
    const char *what() const noexcept override { return where; }
};

PyObject *failed(const CallFailed &e)
{
    if (g_error) {
        PyObject *err = PyObject_CallFunction(g_error, "is", e.status, e.where);
        if (err) {
            PyErr_SetObject(reinterpret_cast<PyObject *>(Py_TYPE(err)), err);
            Py_DECREF(err);
        }
    } else {
        PyErr_SetString(PyExc_RuntimeError, e.where);
    }
    return nullptr;
}

// What a planned stack's handle needs beside it.  Shared between the Python object and the graph nodes recorded with it; the last one
// destroys the handle, unless it was closed before.
struct Plan {
    void *handle = nullptr;
    RunFn run = nullptr;
    BackwardFn backward = nullptr;
    DestroyFn destroy = nullptr;
    Shape in{}, out{};
    std::vector<Shape> res, idx;
    at::ScalarType dtype = at::kFloat;
    at::MemoryFormat mf = at::MemoryFormat::Contiguous;
    uint64_t ws_bytes = 0, bwd_ws_bytes = 0;
    bool bwd_planned = false, bwd_reads_picks = true;
    std::mutex mutex;
    // one workspace per (device, stream) and direction: runs on different streams may overlap
    using Buffers = std::map<std::pair<int, void *>, at::Tensor>;
    Buffers ws[2];

    ~Plan()
    {
        if (handle) destroy(handle);
    }
    // Closed or planned anew: the handle is the Python object's again, nothing runs here any more.
    void *release()
    {
        Buffers old[2];
        std::lock_guard<std::mutex> lock(mutex);
        void *h = handle;
        handle = nullptr;
        for (int i = 0; i < 2; ++i) old[i].swap(ws[i]);
        return h;
    }
    // Nothing is allocated or freed under the mutex: the allocator may call into the interpreter, whose lock the thread that waits for the
    // mutex may hold.
    at::Tensor workspace(bool bwd, const at::Device &dev, void *stream)
    {
        const uint64_t n = bwd ? bwd_ws_bytes : ws_bytes;
        if (!n) return {};
        const Buffers::key_type key{dev.index(), stream};
        {
            std::lock_guard<std::mutex> lock(mutex);
            const auto it = ws[bwd].find(key);
            if (it != ws[bwd].end()) return it->second;
        }
        const at::Tensor t = at::empty({(int64_t)n}, at::TensorOptions().dtype(at::kByte).device(dev));
        std::lock_guard<std::mutex> lock(mutex);
        return ws[bwd].emplace(key, t).first->second;  // (another thread's, if it was faster)
    }
    at::TensorOptions options(const at::Tensor &like) const { return at::TensorOptions().dtype(dtype).device(like.device()); }
};

// A dense tensor of this shape in the plan's memory order, on `dev`, whose memory can be addressed.
bool plain(const Plan &p, const at::Tensor &t, const Shape &shape, at::ScalarType dtype, const at::Device *dev)
{
    return t.defined() && t.is_cuda() && t.scalar_type() == dtype && t.dim() == 4 && t.sizes() == at::IntArrayRef(shape.data(), 4) && t.has_storage() &&
           (!dev || t.device() == *dev) && t.is_contiguous(p.mf);
}

// Elements between the images of a tensor that the library can read in place: dense (0), or a channel slice of a dense tensor whose
// images (channels-last: pixels) keep the alignment; -1: neither.
int64_t slice_stride(const Plan &p, const at::Tensor &t)
{
    if (reinterpret_cast<uintptr_t>(t.data_ptr()) % 16 != 0) return -1;
    if (t.is_contiguous(p.mf)) return 0;
    const int64_t n = t.size(0), c = t.size(1), h = t.size(2), w = t.size(3), es = (int64_t)t.element_size();
    const int64_t sn = t.stride(0), sc = t.stride(1), sh = t.stride(2), sw = t.stride(3);
    if (p.mf == at::MemoryFormat::Contiguous) {
        const bool slice = (w == 1 || sw == 1) && (h == 1 || sh == w) && (c == 1 || sc == h * w) && (n == 1 || sn >= c * h * w);
        const int64_t stride = n > 1 ? sn : c * h * w;
        return slice && stride * es % 16 == 0 ? stride : -1;
    }
    const int64_t ct = w > 1 ? sw : h > 1 ? sh : n > 1 ? sn : c;  // channels of the larger tensor
    const bool slice = ct >= c && (c == 1 || sc == 1) && (w == 1 || sw == ct) && (h == 1 || sh == w * ct) && (n == 1 || sn == h * w * ct);
    return slice && ct * es % 16 == 0 ? h * w * ct : -1;
}

bool modes_active() { return c10::impl::dispatch_mode_enabled(); }

// out and (if wanted) picks for x; the launch.  The caller has checked the operands.
void run_forward(Plan &p, const at::Tensor &x, const std::vector<at::Tensor> &res, at::Tensor &out, std::vector<at::Tensor> &picks, bool want_picks = true)
{
    out = at::empty(at::IntArrayRef(p.out.data(), 4), p.options(x).memory_format(p.mf));
    picks.clear();
    if (want_picks)
        for (const Shape &s : p.idx) picks.push_back(at::empty(at::IntArrayRef(s.data(), 4), p.options(x).dtype(at::kInt).memory_format(p.mf)));
    void *stream = c10::hip::getCurrentHIPStream(x.device().index()).stream();
    const at::Tensor ws = p.workspace(false, x.device(), stream);
    c10::SmallVector<const void *, 4> rp;
    c10::SmallVector<int32_t *, 4> ip;
    for (const at::Tensor &r : res) rp.push_back(r.data_ptr());
    for (const at::Tensor &t : picks) ip.push_back(static_cast<int32_t *>(t.data_ptr()));
    const int rc = p.run(p.handle, x.data_ptr(), 0, res.empty() ? nullptr : rp.data(), out.data_ptr(), 0, picks.empty() ? nullptr : ip.data(),
                         ws.defined() ? ws.data_ptr() : nullptr, ws.defined() ? (uint64_t)ws.numel() : 0, stream);
    if (rc != 0) throw CallFailed(rc, "bs_stack_run");
}

// `need`: input, then residuals.
void run_backward(Plan &p, const at::Tensor &x, const std::vector<at::Tensor> &res, const at::Tensor &dy, int64_t dy_stride, const std::vector<at::Tensor> &picks,
                  const std::vector<bool> &need, at::Tensor &gx, std::vector<at::Tensor> &gres)
{
    if (need[0]) gx = at::empty(at::IntArrayRef(p.in.data(), 4), p.options(x).memory_format(p.mf));
    gres.assign(res.size(), at::Tensor());
    for (size_t i = 0; i < res.size(); ++i)
        if (need[i + 1]) gres[i] = at::empty(at::IntArrayRef(p.res[i].data(), 4), p.options(x).memory_format(p.mf));
    void *stream = c10::hip::getCurrentHIPStream(x.device().index()).stream();
    const at::Tensor ws = p.workspace(true, x.device(), stream);
    c10::SmallVector<const void *, 4> rp;
    c10::SmallVector<void *, 4> gp;
    c10::SmallVector<const int32_t *, 4> ip;
    for (size_t i = 0; i < res.size(); ++i) {
        rp.push_back(res[i].data_ptr());
        gp.push_back(gres[i].defined() ? gres[i].data_ptr() : nullptr);
    }
    for (const at::Tensor &t : picks) ip.push_back(t.defined() ? static_cast<const int32_t *>(t.data_ptr()) : nullptr);
    const int rc = p.backward(p.handle, x.data_ptr(), 0, res.empty() ? nullptr : rp.data(), picks.empty() ? nullptr : ip.data(), dy.data_ptr(), dy_stride,
                              gx.defined() ? gx.data_ptr() : nullptr, 0, res.empty() ? nullptr : gp.data(), ws.defined() ? ws.data_ptr() : nullptr,
                              ws.defined() ? (uint64_t)ws.numel() : 0, stream);
    if (rc != 0) throw CallFailed(rc, "bs_stack_backward");
}

// The stack as one node of the autograd graph: keeps its operands (through torch's saved variables) and the picks.
struct StackNode : torch::autograd::Function<StackNode> {
    struct Held : torch::CustomClassHolder {
        std::shared_ptr<Plan> plan;
        std::vector<at::Tensor> picks;
    };
    static at::Tensor forward(torch::autograd::AutogradContext *ctx, const std::shared_ptr<Plan> &plan, const at::Tensor &x, at::TensorList residuals)
    {
        auto held = c10::make_intrusive<Held>();
        held->plan = plan;
        const std::vector<at::Tensor> res = residuals.vec();
        at::Tensor out;
        {
            pybind11::gil_scoped_release no_gil;
            run_forward(*plan, x, res, out, held->picks, plan->bwd_reads_picks);
        }
        torch::autograd::variable_list saved{x};
        saved.insert(saved.end(), res.begin(), res.end());
        ctx->save_for_backward(std::move(saved));
        ctx->saved_data["held"] = c10::IValue::make_capsule(std::move(held));
        return out;
    }
    static torch::autograd::variable_list backward(torch::autograd::AutogradContext *ctx, torch::autograd::variable_list grads)
    {
        const auto held = c10::static_intrusive_pointer_cast<Held>(ctx->saved_data["held"].toCapsule());
        Plan &p = *held->plan;
        const auto saved = ctx->get_saved_variables();
        const at::Tensor &x = saved[0];
        const std::vector<at::Tensor> res(saved.begin() + 1, saved.end());
        TORCH_CHECK(p.handle, "the stack of this graph was closed, or its parameters were read again, before the backward pass");
        std::vector<bool> need(1 + res.size());
        for (size_t i = 0; i < need.size(); ++i) need[i] = ctx->needs_input_grad(i);
        // the upstream gradient has the output's shape and type and is read in place when it is dense or a channel slice
        at::Tensor dy = grads[0];
        int64_t stride = slice_stride(p, dy);
        if (stride < 0) {
            dy = dy.contiguous(p.mf);
            stride = 0;
        }
        at::Tensor gx;
        std::vector<at::Tensor> gres;
        try {
            run_backward(p, x, res, dy, stride, held->picks, need, gx, gres);
        } catch (const CallFailed &e) {  // raised in Python as the binding's error
            pybind11::gil_scoped_acquire gil;
            failed(e);
            python_error err;
            err.persist();
            throw err;
        }
        torch::autograd::variable_list all{at::Tensor(), gx};  // (the plan has no gradient)
        all.insert(all.end(), gres.begin(), gres.end());
        return all;
    }
};

// ---------------------------------------------------------------------------------------------------- Python type
struct PlanObject {
    PyObject_HEAD
    std::shared_ptr<Plan> *plan;
};

bool read_shape(PyObject *o, Shape &s)
{
    PyObject *f = PySequence_Fast(o, "shape");
    if (!f) return false;
    const bool four = PySequence_Fast_GET_SIZE(f) == 4;
    if (!four) PyErr_SetString(PyExc_ValueError, "a shape has four dimensions");
    for (int i = 0; four && i < 4; ++i) s[i] = PyLong_AsLongLong(PySequence_Fast_GET_ITEM(f, i));
    Py_DECREF(f);
    return four && !PyErr_Occurred();
}
bool read_shapes(PyObject *o, std::vector<Shape> &v)
{
    PyObject *f = PySequence_Fast(o, "shapes");
    if (!f) return false;
    bool ok = true;
    for (Py_ssize_t i = 0; ok && i < PySequence_Fast_GET_SIZE(f); ++i) {
        Shape s;
        ok = read_shape(PySequence_Fast_GET_ITEM(f, i), s);
        if (ok) v.push_back(s);
    }
    Py_DECREF(f);
    return ok;
}

// Plan(addresses (run, backward, destroy), handle, in_shape, out_shape, dtype 0 / 1 / 2, channels_last, residual shapes, index shapes, workspace bytes)
PyObject *plan_new(PyTypeObject *type, PyObject *args, PyObject *)
{
    HANDLE_TH_ERRORS
    unsigned long long run, backward, destroy, handle, ws;
    PyObject *in, *out, *res, *idx;
    int dtype, nhwc;
    if (!PyArg_ParseTuple(args, "(KKK)KOOipOOK", &run, &backward, &destroy, &handle, &in, &out, &dtype, &nhwc, &res, &idx, &ws)) return nullptr;
    auto p = std::make_shared<Plan>();
    p->run = reinterpret_cast<RunFn>(run);
    p->backward = reinterpret_cast<BackwardFn>(backward);
    p->destroy = reinterpret_cast<DestroyFn>(destroy);
    p->dtype = dtype == 0 ? at::kFloat : dtype == 1 ? at::kBFloat16 : at::kHalf;
    p->mf = nhwc ? at::MemoryFormat::ChannelsLast : at::MemoryFormat::Contiguous;
    p->ws_bytes = ws;
    if (!read_shape(in, p->in) || !read_shape(out, p->out) || !read_shapes(res, p->res) || !read_shapes(idx, p->idx)) return nullptr;
    PlanObject *self = reinterpret_cast<PlanObject *>(type->tp_alloc(type, 0));
    if (!self) return nullptr;
    p->handle = reinterpret_cast<void *>(handle);
    self->plan = new std::shared_ptr<Plan>(std::move(p));
    return reinterpret_cast<PyObject *>(self);
    END_HANDLE_TH_ERRORS
}

void plan_dealloc(PyObject *o)
{
    PlanObject *self = reinterpret_cast<PlanObject *>(o);
    delete self->plan;
    PyTypeObject *type = Py_TYPE(o);
    type->tp_free(o);
    Py_DECREF(type);
}

Plan &plan_of(PyObject *o) { return **reinterpret_cast<PlanObject *>(o)->plan; }

const at::Tensor *tensor_of(PyObject *o)
{
    return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr;  // (subclasses: Python)
}

// x and a tuple or list of residuals, checked; false: not the plain case (no error set)
bool operands(Plan &p, PyObject *xo, PyObject *ro, const at::Tensor *&x, std::vector<at::Tensor> &res)
{
    x = tensor_of(xo);
    if (!p.handle || !x || modes_active() || !plain(p, *x, p.in, p.dtype, nullptr)) return false;
    if (!PyTuple_Check(ro) && !PyList_Check(ro)) return false;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(ro);
    if ((size_t)n != p.res.size()) return false;
    const at::Device dev = x->device();
    for (Py_ssize_t i = 0; i < n; ++i) {
        const at::Tensor *r = tensor_of(PySequence_Fast_GET_ITEM(ro, i));
        if (!r || !plain(p, *r, p.res[i], p.dtype, &dev)) return false;
        res.push_back(*r);
    }
    return true;
}

PyObject *wrap_list(std::vector<at::Tensor> &v)
{
    PyObject *l = PyList_New((Py_ssize_t)v.size());
    if (!l) return nullptr;
    for (size_t i = 0; i < v.size(); ++i) {
        PyObject *t = nullptr;
        if (v[i].defined()) t = THPVariable_Wrap(std::move(v[i]));
        else t = Py_NewRef(Py_None);
        if (!t) {
            Py_DECREF(l);
            return nullptr;
        }
        PyList_SET_ITEM(l, (Py_ssize_t)i, t);
    }
    return l;
}

// (first, list) with references stolen
PyObject *pair_of(PyObject *a, PyObject *b)
{
    PyObject *t = a && b ? PyTuple_New(2) : nullptr;
    if (!t) {
        Py_XDECREF(a);
        Py_XDECREF(b);
        return nullptr;
    }
    PyTuple_SET_ITEM(t, 0, a);
    PyTuple_SET_ITEM(t, 1, b);
    return t;
}

// run(x, residuals) -> (out, [index outputs]) or None
PyObject *plan_run(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 2) Py_RETURN_NONE;
    const std::shared_ptr<Plan> p = *reinterpret_cast<PlanObject *>(self)->plan;
    const at::Tensor *x;
    std::vector<at::Tensor> res, idx;
    if (!operands(*p, args[0], args[1], x, res)) Py_RETURN_NONE;
    const at::Tensor xs = *x;
    at::Tensor out;
    try {
        pybind11::gil_scoped_release no_gil;
        run_forward(*p, xs, res, out, idx);
    } catch (const CallFailed &e) {
        return failed(e);
    }
    return pair_of(THPVariable_Wrap(std::move(out)), wrap_list(idx));
    END_HANDLE_TH_ERRORS
}

// infer(x, residuals) -> out or None: as run, for plans without index outputs
PyObject *plan_infer(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 2) Py_RETURN_NONE;
    const std::shared_ptr<Plan> p = *reinterpret_cast<PlanObject *>(self)->plan;
    const at::Tensor *x;
    std::vector<at::Tensor> res, idx;
    if (!p->idx.empty() || !operands(*p, args[0], args[1], x, res)) Py_RETURN_NONE;
    const at::Tensor xs = *x;
    at::Tensor out;
    try {
        pybind11::gil_scoped_release no_gil;
        run_forward(*p, xs, res, out, idx);
    } catch (const CallFailed &e) {
        return failed(e);
    }
    return THPVariable_Wrap(std::move(out));
    END_HANDLE_TH_ERRORS
}

// backward(x, residuals, grad_out, indices or None) -> (grad_x, [residual gradients]) or None
PyObject *plan_backward(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 4) Py_RETURN_NONE;
    const std::shared_ptr<Plan> p = *reinterpret_cast<PlanObject *>(self)->plan;
    const at::Tensor *x;
    std::vector<at::Tensor> res, idx, gres;
    if (!p->bwd_planned || !operands(*p, args[0], args[1], x, res)) Py_RETURN_NONE;
    const at::Tensor *dy = tensor_of(args[2]);
    const at::Device dev = x->device();
    if (!dy || !plain(*p, *dy, p->out, p->dtype, &dev)) Py_RETURN_NONE;
    if (args[3] != Py_None) {
        if (!PyTuple_Check(args[3]) && !PyList_Check(args[3])) Py_RETURN_NONE;
        const Py_ssize_t m = PySequence_Fast_GET_SIZE(args[3]);
        if ((size_t)m != p->idx.size()) Py_RETURN_NONE;
        for (Py_ssize_t i = 0; i < m; ++i) {
            const at::Tensor *t = tensor_of(PySequence_Fast_GET_ITEM(args[3], i));
            if (!t || !plain(*p, *t, p->idx[i], at::kInt, &dev)) Py_RETURN_NONE;
            idx.push_back(*t);
        }
    }
    const at::Tensor xs = *x, dys = *dy;
    at::Tensor gx;
    try {
        pybind11::gil_scoped_release no_gil;
        run_backward(*p, xs, res, dys, 0, idx, std::vector<bool>(1 + res.size(), true), gx, gres);
    } catch (const CallFailed &e) {
        return failed(e);
    }
    return pair_of(THPVariable_Wrap(std::move(gx)), wrap_list(gres));
    END_HANDLE_TH_ERRORS
}

// record(x, residuals) -> out with its node in the autograd graph, or None
PyObject *plan_record(PyObject *self, PyObject *const *args, Py_ssize_t n)
{
    HANDLE_TH_ERRORS
    if (n != 2) Py_RETURN_NONE;
    const std::shared_ptr<Plan> p = *reinterpret_cast<PlanObject *>(self)->plan;
    const at::Tensor *x;
    std::vector<at::Tensor> res;
    if (!p->bwd_planned || !operands(*p, args[0], args[1], x, res)) Py_RETURN_NONE;
    // forward-mode and functorch levels see the Python function's own answers
    if (x->_fw_grad(0).defined()) Py_RETURN_NONE;
    for (const at::Tensor &r : res)
        if (r._fw_grad(0).defined()) Py_RETURN_NONE;
    if (at::functorch::functorchTLSAccessor()) Py_RETURN_NONE;
    const at::Tensor xs = *x;
    try {
        return THPVariable_Wrap(StackNode::apply(p, xs, at::TensorList(res)));
    } catch (const CallFailed &e) {
        return failed(e);
    }
    END_HANDLE_TH_ERRORS
}

// set_backward(workspace bytes, reads picks): the backward pass is planned
PyObject *plan_set_backward(PyObject *self, PyObject *args)
{
    unsigned long long n;
    int reads;
    if (!PyArg_ParseTuple(args, "Kp", &n, &reads)) return nullptr;
    Plan &p = plan_of(self);
    {
        Plan::Buffers old;
        std::lock_guard<std::mutex> lock(p.mutex);
        p.bwd_ws_bytes = n;
        p.bwd_planned = true;
        p.bwd_reads_picks = reads != 0;
        old.swap(p.ws[1]);
    }
    Py_RETURN_NONE;
}

// workspace(backward?, device, raw stream) -> the buffer that calls on this stream hand intermediate tensors through, or None
PyObject *plan_workspace(PyObject *self, PyObject *args)
{
    HANDLE_TH_ERRORS
    int bwd;
    PyObject *dev;
    unsigned long long stream;
    if (!PyArg_ParseTuple(args, "pO!K", &bwd, &THPDeviceType, &dev, &stream)) return nullptr;
    const at::Tensor t = plan_of(self).workspace(bwd != 0, reinterpret_cast<THPDevice *>(dev)->device, reinterpret_cast<void *>(stream));
    if (!t.defined()) Py_RETURN_NONE;
    return THPVariable_Wrap(t);
    END_HANDLE_TH_ERRORS
}

// release() -> handle: nothing runs through this object any more, and the caller destroys the handle (0: released before)
PyObject *plan_release(PyObject *self, PyObject *) { return PyLong_FromVoidPtr(plan_of(self).release()); }

PyObject *set_error(PyObject *, PyObject *cls)
{
    Py_XDECREF(g_error);
    g_error = Py_NewRef(cls);
    Py_RETURN_NONE;
}

PyMethodDef plan_methods[] = {
    {"run", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(plan_run)), METH_FASTCALL, "(x, residuals) -> (out, indices) or None"},
    {"infer", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(plan_infer)), METH_FASTCALL, "(x, residuals) -> out or None"},
    {"backward", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(plan_backward)), METH_FASTCALL,
     "(x, residuals, grad_out, indices or None) -> (grad_x, residual gradients) or None"},
    {"record", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(plan_record)), METH_FASTCALL, "(x, residuals) -> out in the autograd graph, or None"},
    {"set_backward", plan_set_backward, METH_VARARGS, "(workspace bytes, reads picks)"},
    {"workspace", plan_workspace, METH_VARARGS, "(backward, device, raw stream) -> buffer or None"},
    {"release", plan_release, METH_NOARGS, "-> handle"},
    {nullptr, nullptr, 0, nullptr}};

PyType_Slot plan_slots[] = {{Py_tp_new, reinterpret_cast<void *>(plan_new)},
                            {Py_tp_dealloc, reinterpret_cast<void *>(plan_dealloc)},
                            {Py_tp_methods, plan_methods},
                            {0, nullptr}};
PyType_Spec plan_spec = {"_bs_torch.Plan", sizeof(PlanObject), 0, Py_TPFLAGS_DEFAULT, plan_slots};

PyMethodDef module_methods[] = {{"set_error", set_error, METH_O, "(class): raised as class(status, where)"}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_bs_torch", nullptr, -1, module_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: what the file was compiled for; read from the file before it is loaded
extern "C" __attribute__((visibility("default"))) PyObject *PyInit__bs_torch(void)
{
    PyObject *m = PyModule_Create(&module_def);
    if (!m) return nullptr;
    PyObject *t = PyType_FromSpec(&plan_spec);
    if (!t || PyModule_AddStringConstant(m, "built_for", BS_TORCH_TAG) != 0 || PyModule_AddObject(m, "Plan", t) != 0) {
        Py_XDECREF(t);
        Py_DECREF(m);
        return nullptr;
    }
    return m;
}
