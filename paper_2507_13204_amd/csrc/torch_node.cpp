// The autograd node of the objectives' Functions (host code).
//
// A training step on a small objective is bound by the host: a Python
// autograd.Function takes some 20 us to go forward and its backward runs
// Python on the engine's thread.  Measured, a whole step (forward, backward)
// on a 61^3 hex mesh: 84 us through the Function, 51 us through the node (of
// which some 30 are the engine's); the forward alone 22.7 and 5.5.  The node
// here does what the Function's
// forward and backward do -- the same library calls on the same tensors, the
// same tensors saved (through SavedVariable, so saved-tensor hooks and the
// checks of in-place changes and second backwards apply) -- without either.
// It takes plain device tensors that need a gradient; everything else (tensor
// subclasses, functorch transforms, forward-mode, tracing, dispatch and
// function modes, wrong devices) is left to the Python Function: apply() then returns None.
#include <ATen/PythonTorchFunctionTLS.h>
#include <ATen/core/LegacyTypeDispatch.h>
#include <c10/core/impl/TorchDispatchModeTLS.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/function.h>
#include <torch/csrc/autograd/functions/utils.h>
#include <torch/csrc/autograd/saved_variable.h>
#include <torch/csrc/autograd/variable.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/jit/frontend/tracer.h>
#include <torch/extension.h>

#include "pgrad.h"

namespace {

using at::Tensor;
using torch::autograd::SavedVariable;
using torch::autograd::variable_list;

pg_stream current_stream() { return c10::hip::getCurrentHIPStream().stream(); }

// Raises the binding's PgError for a status that is not PG_OK (any thread).
void check(PyObject* py_check, int status, const char* where) {
    if (status == PG_OK) return;
    pybind11::gil_scoped_acquire gil;
    PyObject* r = PyObject_CallFunction(py_check, "is", status, where);
    Py_XDECREF(r);
    throw python_error();
}

// What the binding checks of every operand: a hook may hand back another
// tensor than the one that was saved or passed on.
bool operand(const Tensor& t) { return t.is_cuda() && t.is_contiguous(); }
// Raises as the binding does for operands that are not (any thread).
[[noreturn]] void refuse(PyObject* py_check, const char* fn, const Tensor& a, const Tensor& b) {
    pybind11::gil_scoped_acquire gil;
    try {
        pybind11::dict binding = pybind11::handle(py_check).attr("__globals__");
        binding[fn](a);
        binding[fn](b);
        binding["check"]((int)PG_EINVAL, "backward");  // it found nothing: still not to be used
    } catch (pybind11::error_already_set& e) {
        e.restore();
    }
    throw python_error();
}

enum Policy { GRADIENT = 0, STORE = 1 };

struct ObjectiveNode : public torch::autograd::Node {
    std::string label;
    int policy = GRADIENT;
    SavedVariable first, second;  // the gradient; or the tape and x
    std::vector<int64_t> f_sizes, x_sizes;
    c10::TensorOptions f_options, x_options;
    int64_t tape_bytes = 0;
    PyObject* obj = nullptr;  // owns the plan
    PyObject* py_check = nullptr;

    ~ObjectiveNode() override {
        if (!Py_IsInitialized()) return;
        pybind11::gil_scoped_acquire gil;
        Py_XDECREF(obj);
        Py_XDECREF(py_check);
    }
    std::string name() const override { return label; }
    void release_variables() override {
        std::lock_guard<std::mutex> lock(mutex_);
        first.reset_data();
        second.reset_data();
    }

    variable_list apply(variable_list&& grads) override {
        std::lock_guard<std::mutex> lock(mutex_);
        const Tensor a = first.unpack();
        if (policy == STORE) second.unpack();  // for its checks; only its shape is needed
        at::AutoDispatchBelowADInplaceOrView below;
        Tensor seed = grads[0].defined() ? grads[0] : at::zeros(f_sizes, f_options);
        if (seed.scalar_type() != at::kDouble) seed = seed.to(at::kDouble);
        seed = seed.contiguous();
        const bool enough = seed.numel() >= c10::multiply_integers(f_sizes) &&
                            (policy == GRADIENT || (int64_t)a.nbytes() >= tape_bytes);
        if (!operand(seed) || !operand(a) || !enough) refuse(py_check, "_need_cuda", seed, a);
        const double* fbar = seed.const_data_ptr<double>();
        if (policy == GRADIENT) {
            if (a.scalar_type() != at::kDouble && a.scalar_type() != at::kFloat)
                refuse(py_check, "_dtype_code", a, a);
            Tensor y = at::empty_like(a);
            check(py_check,
                  pg_scale(a.scalar_type() == at::kDouble ? PG_F64 : PG_F32, a.numel(), fbar,
                           a.const_data_ptr(), y.mutable_data_ptr(), current_stream()),
                  "pg_scale");
            return {y};
        }
        Tensor y = at::empty(x_sizes, x_options);
        check(py_check,
              pg_adjoint_tape(plan_of(obj), fbar, a.const_data_ptr(), y.mutable_data_ptr(),
                              current_stream()),
              "pg_adjoint_tape");
        return {y};
    }

    // The plan as the object holds it now (NULL once it was closed).
    static pg_plan plan_of(PyObject* obj) {
        pybind11::gil_scoped_acquire gil;
        pybind11::object v = pybind11::handle(obj).attr("_plan").attr("value");
        return v.is_none() ? nullptr : reinterpret_cast<pg_plan>(v.cast<uintptr_t>());
    }
};

// A launch may wait for the device's queue: other threads go on meanwhile.
template <class F>
int unlocked(F&& call) {
    pybind11::gil_scoped_release off;
    return call();
}

bool plain(const Tensor& x) {
    // the keys of a strided device tensor (autocast's is always among them)
    constexpr c10::DispatchKeySet known({c10::DispatchKey::CUDA, c10::DispatchKey::AutogradCUDA,
                                         c10::DispatchKey::ADInplaceOrView,
                                         c10::DispatchKey::AutocastCUDA});
    if (!x.is_cuda() || (x.key_set() | known) != known) return false;
    if (x.scalar_type() != at::kDouble && x.scalar_type() != at::kFloat) return false;
    if (c10::impl::tls_is_dispatch_key_included(c10::DispatchKey::FuncTorchDynamicLayerFrontMode) ||
        c10::impl::TorchDispatchModeTLS::any_modes_set() || at::impl::torch_function_mode_enabled() ||
        torch::jit::tracer::isTracing())
        return false;
    return !x._fw_grad(0).defined();
}

// f of x with its node, or None where the Python Function has to take over.
// plan, policy and label are the objective's and the Function's; n_f is the
// number of objectives (-1: a scalar); tape_doubles the tape's size.
pybind11::object apply(const Tensor& x, pybind11::object obj, uintptr_t plan, int policy,
                       int64_t n_f, int64_t tape_doubles, const char* label,
                       pybind11::object py_check) {
    if (plan == 0 || !plain(x)) return pybind11::none();
    auto node = std::shared_ptr<ObjectiveNode>(new ObjectiveNode(), torch::autograd::deleteNode);
    Tensor f, a, xc;
    {
        at::AutoDispatchBelowADInplaceOrView below;
        xc = x.contiguous();
        node->f_options = x.options().dtype(at::kDouble);
        node->x_options = x.options();
        node->x_sizes = x.sizes().vec();
        node->tape_bytes = 8 * tape_doubles;
        if (n_f >= 0) node->f_sizes.push_back(n_f);
        f = at::empty(node->f_sizes, node->f_options);
        pg_plan p = reinterpret_cast<pg_plan>(plan);
        if (policy == GRADIENT) {
            a = at::empty(xc.sizes(), xc.options());
            check(py_check.ptr(), unlocked([&] {
                      return pg_gradient(p, xc.const_data_ptr(), a.mutable_data_ptr(),
                                         f.mutable_data_ptr<double>(), current_stream());
                  }),
                  "pg_gradient");
        } else {
            a = at::empty({tape_doubles}, node->f_options);
            check(py_check.ptr(), unlocked([&] {
                      return pg_objective_tape(p, xc.const_data_ptr(), f.mutable_data_ptr<double>(),
                                               a.mutable_data_ptr(), current_stream());
                  }),
                  "pg_objective_tape");
        }
    }
    node->label = label;
    node->policy = policy;
    node->obj = obj.release().ptr();
    node->py_check = py_check.release().ptr();
    node->set_next_edges(torch::autograd::collect_next_edges(x));
    torch::autograd::set_history(f, node);
    node->first = SavedVariable(a, false);
    if (policy == STORE) node->second = SavedVariable(xc.is_same(x) ? x.detach() : xc, false);
    return pybind11::cast(f);
}

}  // namespace

PYBIND11_MODULE(_pgrad_torch, m) { m.def("apply", &apply); }
