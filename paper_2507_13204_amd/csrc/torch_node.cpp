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
#include <torch/csrc/autograd/python_cpp_function.h>
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
    // What was saved, as the Function's context gives it.
    variable_list saved() {
        std::lock_guard<std::mutex> lock(mutex_);
        variable_list v{first.unpack()};
        if (policy == STORE) v.push_back(second.unpack());
        return v;
    }
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

// One node class, and Python type of f.grad_fn, per Function.
constexpr const char* kLabels[] = {"MeshFnBackward", "DenseFnBackward", "BatchedDenseFnBackward",
                                   "MeshBatchFnBackward"};
constexpr int kNLabels = 4;
template <int L>
struct LabelledNode final : ObjectiveNode {
    std::string name() const override { return kLabels[L]; }
};

std::shared_ptr<ObjectiveNode> new_node(int label) {
    ObjectiveNode* n = label == 0   ? (ObjectiveNode*)new LabelledNode<0>()
                       : label == 1 ? (ObjectiveNode*)new LabelledNode<1>()
                       : label == 2 ? (ObjectiveNode*)new LabelledNode<2>()
                                    : (ObjectiveNode*)new LabelledNode<3>();
    return std::shared_ptr<ObjectiveNode>(n, torch::autograd::deleteNode);
}

// The attributes of the Function's context that f.grad_fn had.
ObjectiveNode& node_of(PyObject* self) {
    return static_cast<ObjectiveNode&>(*reinterpret_cast<torch::autograd::THPCppFunction*>(self)->cdata);
}
PyObject* get_saved_tensors(PyObject* self, void*) {
    HANDLE_TH_ERRORS
    variable_list v;
    {
        pybind11::gil_scoped_release off;  // the engine may hold the node while a hook waits for this
        v = node_of(self).saved();
    }
    pybind11::tuple t(v.size());
    for (size_t i = 0; i < v.size(); ++i) t[i] = pybind11::cast(v[i]);
    return t.release().ptr();
    END_HANDLE_TH_ERRORS
}
PyObject* get_needs_input_grad(PyObject*, void*) { return Py_BuildValue("(OOO)", Py_True, Py_False, Py_False); }
PyObject* get_obj(PyObject* self, void*) {
    PyObject* o = node_of(self).obj;
    Py_INCREF(o);
    return o;
}
PyObject* get_policy(PyObject* self, void*) {
    return PyUnicode_FromString(node_of(self).policy == STORE ? "store" : "gradient");
}

template <int L>
void register_type() {
    using namespace torch::autograd;
    static PyMethodDef methods[] = {{"_register_hook_dict", THPCppFunction_register_hook_dict, METH_O, nullptr},
                                    {"register_hook", THPCppFunction_register_hook, METH_O, nullptr},
                                    {"register_prehook", THPCppFunction_register_prehook, METH_O, nullptr},
                                    {"name", THPCppFunction_name, METH_NOARGS, nullptr},
                                    {"_sequence_nr", THPCppFunction_sequence_nr, METH_NOARGS, nullptr},
                                    {nullptr, nullptr, 0, nullptr}};
    static PyGetSetDef properties[] = {
        {"next_functions", THPCppFunction_next_functions, nullptr, nullptr, nullptr},
        {"requires_grad", THPCppFunction_requires_grad, nullptr, nullptr, nullptr},
        {"metadata", THPCppFunction_metadata, nullptr, nullptr, nullptr},
        {"_input_metadata", THPCppFunction_input_metadata, nullptr, nullptr, nullptr},
        {"saved_tensors", get_saved_tensors, nullptr, nullptr, nullptr},
        {"needs_input_grad", get_needs_input_grad, nullptr, nullptr, nullptr},
        {"obj", get_obj, nullptr, nullptr, nullptr},
        {"policy", get_policy, nullptr, nullptr, nullptr},
        {nullptr, nullptr, nullptr, nullptr, nullptr}};
    static PyTypeObject type{};
    torch::autograd::_initFunctionPyTypeObject(type, kLabels[L], properties, methods);
    torch::autograd::registerCppFunction(typeid(LabelledNode<L>), &type);
}

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
// plan, policy and label (of kLabels) are the objective's and the Function's; n_f is the
// number of objectives (-1: a scalar); tape_doubles the tape's size.
pybind11::object apply(const Tensor& x, pybind11::object obj, uintptr_t plan, int policy,
                       int64_t n_f, int64_t tape_doubles, int label,
                       pybind11::object py_check) {
    if (plan == 0 || label < 0 || label >= kNLabels || !plain(x)) return pybind11::none();
    auto node = new_node(label);
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

PYBIND11_MODULE(_pgrad_torch, m) {
    register_type<0>();
    register_type<1>();
    register_type<2>();
    register_type<3>();
    m.def("apply", &apply);
}
