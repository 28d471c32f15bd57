// Autograd nodes of the binding: render and pose as C++ functions over the C
// ABI.  A pass of a small scene is a few dozen microseconds of kernels, as long
// as a Python autograd function takes to marshal its arguments, so the nodes
// run without the interpreter and without its lock.  Memory,
// streams and error classes are the Python binding's: the caller's tensors are
// checked and used as they are, outputs come from torch's allocator, work goes
// to the current stream.
#include <c10/util/intrusive_ptr.h>
#include <torch/csrc/Exceptions.h>
#include <torch/extension.h>

#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>

#include <string>
#include <utility>

#include "dsm.h"

namespace {

using torch::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::Variable;
using torch::autograd::variable_list;

// The plan as the nodes hold it: a reference to the Python object that owns the
// library's plan (and refers to nothing: Python's collector does not see this
// reference), released under the interpreter's lock (a graph may be freed on any
// thread).
struct PlanRef : torch::CustomClassHolder {
    PyObject *owner;
    dsm_plan *plan;
    dsm_plan_info info;
    PlanRef(PyObject *o, dsm_plan *p) : owner(o), plan(p) {
        Py_INCREF(owner);
        const dsm_status st = dsm_plan_info_get(plan, &info);
        TORCH_CHECK(st == DSM_OK, "dsm_plan_info_get failed: ", dsm_status_string(st));
    }
    ~PlanRef() override {
        if (!Py_IsInitialized()) return;
        pybind11::gil_scoped_acquire gil;
        Py_DECREF(owner);
    }
};

c10::intrusive_ptr<PlanRef> plan_of(AutogradContext *ctx) {
    return c10::static_intrusive_pointer_cast<PlanRef>(ctx->saved_data["plan"].toCapsule());
}

// A failed call raises the package's DSMError(function, status).
void check(const char *fn, dsm_status st) {
    if (st == DSM_OK) return;
    pybind11::gil_scoped_acquire gil;
    try {
        const pybind11::object cls = pybind11::module_::import("paper_2308_10896_amd._lib").attr("DSMError");
        const pybind11::object err = cls(fn, (int)st);
        PyErr_SetObject(cls.ptr(), err.ptr());
    } catch (pybind11::error_already_set &e) {
        e.restore();
    }
    python_error raised;
    raised.persist();
    throw raised;
}

void need_cuda_f32(const char *name, const Tensor &t) {
    TORCH_CHECK_VALUE(t.is_cuda() && t.scalar_type() == at::kFloat && t.is_contiguous(), name,
                      " must be a contiguous float32 CUDA tensor");
}

dsm_stream current_stream() { return (dsm_stream)c10::hip::getCurrentHIPStreamMasqueradingAsCUDA().stream(); }

const float *in(const Tensor &t) { return (const float *)t.const_data_ptr(); }
float *out(Tensor &t) { return (float *)t.mutable_data_ptr(); }

struct Render : torch::autograd::Function<Render> {
    static Tensor forward(AutogradContext *ctx, const c10::intrusive_ptr<PlanRef> &plan, const Tensor &verts,
                          const Tensor &light_params, const Tensor &albedo, const Tensor &scratch) {
        need_cuda_f32("verts", verts);
        need_cuda_f32("light_params", light_params);
        need_cuda_f32("albedo", albedo);
        const dsm_plan_info &info = plan->info;
        Tensor saved = at::empty({info.saved_bytes}, verts.options().dtype(at::kByte));
        Tensor images = at::empty({info.image_floats}, verts.options());
        check("dsm_forward",
              dsm_forward(plan->plan, in(verts), in(light_params), in(albedo), saved.mutable_data_ptr(),
                          (size_t)saved.numel(), scratch.mutable_data_ptr(), (size_t)scratch.numel(), out(images),
                          current_stream()));
        ctx->saved_data["plan"] = c10::IValue::make_capsule(plan);
        ctx->saved_data["scratch"] = scratch;
        ctx->save_for_backward({verts, light_params, albedo, saved});
        return images;
    }

    static variable_list backward(AutogradContext *ctx, variable_list grads) {
        const auto plan = plan_of(ctx);
        const variable_list held = ctx->get_saved_variables();
        const Tensor &verts = held[0], &light_params = held[1], &albedo = held[2], &saved = held[3];
        const Tensor scratch = ctx->saved_data["scratch"].toTensor(), g = grads[0].contiguous();
        need_cuda_f32("grad_images", g);
        Tensor gv = at::empty_like(verts), gl = at::empty_like(light_params), ga;
        if (ctx->needs_input_grad(2)) ga = at::empty_like(albedo);
        check("dsm_backward",
              dsm_backward(plan->plan, in(verts), in(light_params), in(albedo), saved.const_data_ptr(),
                           (size_t)saved.numel(), scratch.mutable_data_ptr(), (size_t)scratch.numel(), in(g), out(gv),
                           out(gl), ga.defined() ? out(ga) : nullptr, current_stream()));
        return {Variable(), gv, gl, ga, Variable()};
    }
};

struct Pose : torch::autograd::Function<Pose> {
    static Tensor forward(AutogradContext *ctx, const c10::intrusive_ptr<PlanRef> &plan, const Tensor &local,
                          const Tensor &poses) {
        need_cuda_f32("local", local);
        need_cuda_f32("poses", poses);
        Tensor world = at::empty_like(local);
        check("dsm_pose_forward", dsm_pose_forward(plan->plan, in(local), in(poses), out(world), current_stream()));
        ctx->saved_data["plan"] = c10::IValue::make_capsule(plan);
        ctx->save_for_backward({local, poses});
        return world;
    }

    static variable_list backward(AutogradContext *ctx, variable_list grads) {
        const auto plan = plan_of(ctx);
        const variable_list held = ctx->get_saved_variables();
        const Tensor g = grads[0].contiguous();
        Tensor gp = at::empty_like(held[1]);
        check("dsm_pose_backward",
              dsm_pose_backward(plan->plan, in(held[0]), in(held[1]), in(g), out(gp), current_stream()));
        return {Variable(), Variable(), gp};
    }
};

// What Plan keeps for the calls below.  It refers to the owner of the library's
// plan without owning it (the Plan owns both); each node takes a reference of
// its own.
struct PlanHandle {
    PyObject *owner;
    dsm_plan *plan;
    c10::intrusive_ptr<PlanRef> ref() const { return c10::make_intrusive<PlanRef>(owner, plan); }
};

// The call without the interpreter's lock, as the raw calls run: launching can
// take as long as a full queue takes to drain, and other threads go on meanwhile.
template <class Node, class... Args>
Tensor call(const PlanHandle &p, const Args &...args) {
    const c10::intrusive_ptr<PlanRef> ref = p.ref();
    const pybind11::gil_scoped_release unlocked;
    return Node::apply(ref, args...);
}

}  // namespace

PYBIND11_MODULE(_dsm_torch, m) {
    pybind11::class_<PlanHandle>(m, "PlanHandle").def(pybind11::init([](pybind11::handle owner, uintptr_t plan) {
        return PlanHandle{owner.ptr(), reinterpret_cast<dsm_plan *>(plan)};
    }));
    m.def("render", &call<Render, Tensor, Tensor, Tensor, Tensor>);     // verts, light_params, albedo, scratch
    m.def("pose", &call<Pose, Tensor, Tensor>);                         // local, poses
}
