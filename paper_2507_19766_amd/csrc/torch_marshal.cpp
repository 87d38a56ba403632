// Argument marshalling between torch tensors and the C entry points of libulorl, as a Python extension module: checks,
// output tensors, raw pointers, the current stream, and the two autograd nodes.  No arithmetic of the method; the
// objective's scalars and launch options come as addresses of the C structs.
//
// Why it is native: the small calls are bound by the host.  A call on 2048 x 4096 logits took 41 us of host time for
// 27 us of GPU work, 26 of them here (checks, ten output tensors, thirty converted arguments); forward and backward of
// a small lm_head 189 us for 70, because the backward ran Python on autograd's device thread.
#include <ATen/ATen.h>
#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/utils/pybind.h>

#include <array>
#include <exception>
#include <optional>
#include <string>
#include <vector>

#include "ulorl.h"

namespace py = pybind11;
using at::Tensor;
using OptTensor = std::optional<Tensor>;

namespace {

void* ptr(const Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; }
void* ptr(const OptTensor& t) { return t.has_value() ? ptr(*t) : nullptr; }
template <class T, class X>
T* as(const X& t)
{
    return static_cast<T*>(ptr(t));
}

// The current stream of a GPU.  (Asked for a device without an index, as the CPU is, torch answers for the current GPU.)
void* stream_of(const at::Device& dev)
{
    TORCH_CHECK_VALUE(dev.is_cuda(), "Expected a cuda device, but got: ", dev.str());
    return c10::hip::getCurrentHIPStreamMasqueradingAsCUDA(dev.index()).stream();
}

// The Python class of a failed status; lives as long as the interpreter.
PyObject* status_error = nullptr;

// Raises UlorlError(rc, where) in Python, from any thread.
void check(int32_t rc, const char* where)
{
    if (rc == ULORL_OK) return;
    py::gil_scoped_acquire gil;
    PyObject* e = PyObject_CallFunction(status_error, "is", (int)rc, where);
    if (e != nullptr) {
        PyErr_SetObject(status_error, e);
        Py_DECREF(e);
    }
    python_error err;
    err.persist();
    throw err;
}

const char* type_name(at::ScalarType t)
{
    return t == at::kFloat ? "torch.float32" : t == at::kInt ? "torch.int32" : "torch.uint8";
}

// A contiguous vector of n elements on the device, or nothing.
void check_vector(const OptTensor& t, at::ScalarType type, int64_t n, const char* name, const at::Device& dev)
{
    if (!t.has_value()) return;
    TORCH_CHECK_VALUE(t->device() == dev && t->scalar_type() == type && t->dim() == 1 && t->size(0) == n && t->is_contiguous(),
                      name, " must be a contiguous ", type_name(type), "[", n, "] tensor on ", dev.str());
}

// n elements that a kernel can read one after the other, in whatever shape (a mask of either one-byte type), or nothing.
void check_elements(const OptTensor& t, at::ScalarType type, int64_t n, const char* name, const at::Device& dev)
{
    if (!t.has_value()) return;
    const bool same = t->scalar_type() == type || (type == at::kByte && t->scalar_type() == at::kBool);
    TORCH_CHECK_VALUE(t->device() == dev && same && t->numel() >= n && t->is_contiguous(),
                      name, " must hold ", n, " contiguous elements of ", type_name(type), " on ", dev.str());
}

struct Logits {
    int32_t dt;
    int64_t N, V, stride;
    at::Device dev;
};

Logits check_logits(const Tensor& z)
{
    TORCH_CHECK(z.is_cuda(), "libulorl runs on the GPU only: logits must be a device tensor");
    TORCH_CHECK_VALUE(z.dim() == 2 && z.stride(1) == 1, "logits must be [N, V] with unit stride along V");
    TORCH_CHECK_TYPE(z.scalar_type() == at::kFloat || z.scalar_type() == at::kBFloat16, "logits must be float32 or bfloat16, got ", z.scalar_type());
    return Logits{z.scalar_type() == at::kFloat ? 0 : 1, z.size(0), z.size(1), z.stride(0), z.device()};
}

Tensor empty(int64_t n, at::ScalarType type, const at::Device& dev) { return at::empty({n}, at::TensorOptions().dtype(type).device(dev)); }
Tensor empty_rows(int64_t n, at::ScalarType type, const at::Device& dev)
{
    return n > 0 ? empty(n, type, dev) : empty(1, type, dev).narrow(0, 0, 0);
}

// The fields of FwdResult, in its order.  given: they are the caller's, whose tensors are never replaced; what is missing among them is
// a null pointer, which the library refuses where it needs one.
enum { LOSS, LOGP, ENTROPY, LSE, GCOEF, MASK, RATIO, SEGMENT, RESP_ENTROPY, RESP_GATE, COUNTERS, FIELDS };
struct Fields : std::array<Tensor, FIELDS> {
    bool given = false;
};

void allocate_rows(Fields& f, int64_t N, const at::Device& dev)
{
    if (f.given) return;
    for (int i : {LOGP, ENTROPY, LSE}) f[i] = empty(N, at::kFloat, dev);
}
// complete: a caller's result has to be whole; otherwise one without a loss (that of a stats-only pass) gets the rest.
void allocate_objective(Fields& f, int64_t N, int64_t R, const at::Device& dev, bool complete)
{
    allocate_rows(f, N, dev);
    if (f.given && (complete || f[LOSS].defined())) return;
    f[LOSS] = empty(1, at::kFloat, dev);
    f[GCOEF] = empty(N, at::kFloat, dev);
    f[MASK] = empty(N, at::kByte, dev);
    f[RATIO] = empty(N, at::kFloat, dev);
    f[SEGMENT] = empty(N, at::kInt, dev);
    f[RESP_ENTROPY] = empty_rows(R, at::kFloat, dev);
    f[RESP_GATE] = empty_rows(R, at::kByte, dev);
    f[COUNTERS] = empty(4, at::kLong, dev);
}

Tensor workspace_or(const OptTensor& given, size_t need, const at::Device& dev)
{
    return given.has_value() ? *given : empty((int64_t)(need > 256 ? need : 256), at::kByte, dev);
}

// Per-segment diagnostics: count, ratio_sum, ratio_max, clipped, kl_sum, ent_sum, masked, out_of_range, workspace.
using Segments = std::vector<Tensor>;
Segments segment_tensors(int64_t K, int64_t N, const at::Device& dev)
{
    auto i64 = [&](int64_t n) { return empty(n, at::kLong, dev); };
    auto f64 = [&](int64_t n) { return empty(n, at::kDouble, dev); };
    return {i64(K), f64(K), empty(K, at::kFloat, dev), i64(K), f64(K), f64(K), i64(K), i64(1),
            workspace_or(std::nullopt, ulorl_segment_diagnostics_workspace_bytes(N, (int32_t)K), dev)};
}
ulorl_segment_stats segment_struct(const Segments& s, int64_t K)
{
    ulorl_segment_stats c = {};
    c.K = (int32_t)K;
    c.count = as<int64_t>(s[0]);
    c.ratio_sum = as<double>(s[1]);
    c.ratio_max = as<float>(s[2]);
    c.clipped = as<int64_t>(s[3]);
    c.kl_sum = as<double>(s[4]);
    c.ent_sum = as<double>(s[5]);
    c.masked = as<int64_t>(s[6]);
    c.out_of_range = as<int64_t>(s[7]);
    c.workspace = ptr(s[8]);
    c.workspace_bytes = s[8].numel();
    return c;
}

// Inputs of the objective that every forward call takes.
struct Objective {
    OptTensor token_ids, cu, advantages, old_logp, segment_ids;
    const ulorl_params* params;
    const ulorl_launch* launch;
    int64_t R = 0;

    void check_rows(int64_t N, const at::Device& dev) const
    {
        check_vector(token_ids, at::kInt, N, "token_ids", dev);
        check_vector(advantages, at::kFloat, N, "advantages", dev);
        check_vector(old_logp, at::kFloat, N, "old_logp", dev);
        check_vector(segment_ids, at::kInt, N, "segment_ids", dev);
    }
    void check_lengths(const at::Device& dev)
    {
        TORCH_CHECK_VALUE(cu.has_value() && cu->device() == dev && cu->scalar_type() == at::kInt && cu->is_contiguous(),
                          "cu_seqlens must be a contiguous int32 device tensor");
        R = cu->size(0) - 1;
    }
};

void check_gradient(const Tensor& d, const Tensor& z)
{
    TORCH_CHECK_VALUE(d.sizes() == z.sizes() && d.scalar_type() == z.scalar_type() && d.device() == z.device() && d.strides() == z.strides(),
                      "dlogits must match logits in shape, dtype, strides and device");
}
Tensor gradient_for(const Tensor& z, const OptTensor& given, bool inplace)
{
    if (inplace) return z;
    const Tensor d = given.has_value() ? *given : at::empty_strided({z.size(0), z.size(1)}, {z.stride(0), 1}, z.options());
    check_gradient(d, z);
    return d;
}

// ulorl_token_loss_fwd; without advantages the stats-only pass.
void token_loss_fwd(const Tensor& z, Objective o, Fields& f, Segments& seg, int64_t K, const OptTensor& workspace)
{
    const Logits l = check_logits(z);
    if (!o.advantages.has_value()) {
        check_vector(o.token_ids, at::kInt, l.N, "token_ids", l.dev);
        allocate_rows(f, l.N, l.dev);
        const Tensor ws = workspace.has_value() ? *workspace : empty(ulorl_token_loss_workspace_bytes(l.N, l.V, 1), at::kByte, l.dev);
        check(ulorl_token_loss_fwd(ptr(z), l.dt, l.N, l.V, l.stride, as<int32_t>(o.token_ids), nullptr, 0, nullptr, nullptr, nullptr, nullptr,
                                   nullptr, as<float>(f[LOGP]), as<float>(f[ENTROPY]), as<float>(f[LSE]), nullptr, nullptr, nullptr, nullptr,
                                   nullptr, nullptr, nullptr, nullptr, ptr(ws), ws.nbytes(), o.launch, stream_of(l.dev)),
              "ulorl_token_loss_fwd");
        return;
    }
    o.check_rows(l.N, l.dev);
    o.check_lengths(l.dev);
    allocate_objective(f, l.N, o.R, l.dev, false);
    const Tensor ws = workspace_or(workspace, ulorl_token_loss_workspace_bytes(l.N, l.V, (int32_t)o.R), l.dev);
    ulorl_segment_stats st;
    if (K > 0) st = segment_struct(seg = segment_tensors(K, l.N, l.dev), K);
    check(ulorl_token_loss_fwd(ptr(z), l.dt, l.N, l.V, l.stride, as<int32_t>(o.token_ids), as<int32_t>(o.cu), (int32_t)o.R,
                               as<int32_t>(o.segment_ids), as<float>(o.old_logp), as<float>(o.advantages), o.params, as<float>(f[LOSS]),
                               as<float>(f[LOGP]), as<float>(f[ENTROPY]), as<float>(f[LSE]), as<float>(f[GCOEF]), as<uint8_t>(f[MASK]),
                               as<float>(f[RATIO]), as<int32_t>(f[SEGMENT]), as<float>(f[RESP_ENTROPY]), as<uint8_t>(f[RESP_GATE]),
                               as<int64_t>(f[COUNTERS]), K > 0 ? &st : nullptr, ptr(ws), ws.nbytes(), o.launch, stream_of(l.dev)),
          "ulorl_token_loss_fwd");
}

// ulorl_token_loss_fwd_bwd, or its form on the static scratch array.
Tensor token_loss_fwd_bwd(const Tensor& z, Objective o, double grad_out, const OptTensor& dlogits, bool inplace, bool on_static, Fields& f,
                          Segments& seg, int64_t K, const OptTensor& workspace)
{
    const Logits l = check_logits(z);
    o.check_rows(l.N, l.dev);
    o.check_lengths(l.dev);
    TORCH_CHECK_VALUE(o.advantages.has_value(), on_static ? "token_loss_fwd_bwd_static" : "token_loss_fwd_bwd", " needs advantages");
    allocate_objective(f, l.N, o.R, l.dev, on_static);
    const Tensor d = gradient_for(z, dlogits, inplace);
    if (on_static) {
        check(ulorl_token_loss_fwd_bwd_static(ptr(z), l.dt, l.N, l.V, l.stride, as<int32_t>(o.token_ids), as<int32_t>(o.cu), (int32_t)o.R,
                                              as<int32_t>(o.segment_ids), as<float>(o.old_logp), as<float>(o.advantages), o.params,
                                              (float)grad_out, as<float>(f[LOSS]), as<float>(f[LOGP]), as<float>(f[ENTROPY]),
                                              as<float>(f[LSE]), as<float>(f[GCOEF]), as<uint8_t>(f[MASK]), as<float>(f[RATIO]),
                                              as<int32_t>(f[SEGMENT]), as<float>(f[RESP_ENTROPY]), as<uint8_t>(f[RESP_GATE]),
                                              as<int64_t>(f[COUNTERS]), nullptr, ptr(d), o.launch, stream_of(l.dev)),
              "ulorl_token_loss_fwd_bwd_static");
        return d;
    }
    const Tensor ws = workspace_or(workspace, ulorl_token_loss_workspace_bytes(l.N, l.V, (int32_t)o.R), l.dev);
    ulorl_segment_stats st;
    if (K > 0) st = segment_struct(seg = segment_tensors(K, l.N, l.dev), K);
    check(ulorl_token_loss_fwd_bwd(ptr(z), l.dt, l.N, l.V, l.stride, as<int32_t>(o.token_ids), as<int32_t>(o.cu), (int32_t)o.R,
                                   as<int32_t>(o.segment_ids), as<float>(o.old_logp), as<float>(o.advantages), o.params, (float)grad_out,
                                   as<float>(f[LOSS]), as<float>(f[LOGP]), as<float>(f[ENTROPY]), as<float>(f[LSE]), as<float>(f[GCOEF]),
                                   as<uint8_t>(f[MASK]), as<float>(f[RATIO]), as<int32_t>(f[SEGMENT]), as<float>(f[RESP_ENTROPY]),
                                   as<uint8_t>(f[RESP_GATE]), as<int64_t>(f[COUNTERS]), K > 0 ? &st : nullptr, ptr(d), ptr(ws), ws.nbytes(),
                                   o.launch, stream_of(l.dev)),
          "ulorl_token_loss_fwd_bwd");
    return d;
}

Tensor token_loss_bwd(const Tensor& z, const OptTensor& token_ids, const OptTensor& lse, const OptTensor& gcoef, double grad_out,
                      const OptTensor& dlogits, bool inplace)
{
    const Logits l = check_logits(z);
    check_vector(token_ids, at::kInt, l.N, "token_ids", l.dev);
    check_vector(lse, at::kFloat, l.N, "lse", l.dev);
    check_vector(gcoef, at::kFloat, l.N, "gcoef", l.dev);
    const Tensor d = gradient_for(z, dlogits, inplace);
    check(ulorl_token_loss_bwd(ptr(z), l.dt, l.N, l.V, l.stride, as<int32_t>(token_ids), as<float>(lse), as<float>(gcoef), (float)grad_out,
                               ptr(d), stream_of(l.dev)),
          "ulorl_token_loss_bwd");
    return d;
}

struct Lmhead {
    int64_t N, Hd, V;
    at::Device dev;
};
Lmhead check_lmhead(const Tensor& h, const Tensor& w)
{
    TORCH_CHECK(h.is_cuda() && w.is_cuda(), "libulorl runs on the GPU only");
    TORCH_CHECK_TYPE(h.scalar_type() == at::kBFloat16 && w.scalar_type() == at::kBFloat16, "hidden and weight must be bfloat16");
    TORCH_CHECK_VALUE(h.dim() == 2 && w.dim() == 2 && h.is_contiguous() && w.is_contiguous(), "hidden [N, Hd] and weight [Hd, V] must be contiguous");
    TORCH_CHECK_VALUE(h.size(1) == w.size(0), "hidden is [N, Hd], weight is [Hd, V]");
    return Lmhead{h.size(0), h.size(1), w.size(1), h.device()};
}

void lmhead_fwd(const Tensor& h, const Tensor& w, Objective o, int64_t chunk, Fields& f, Segments& seg, int64_t K, const OptTensor& workspace)
{
    const Lmhead l = check_lmhead(h, w);
    const bool stats_only = !o.advantages.has_value();
    o.check_rows(l.N, l.dev);
    if (!stats_only && o.cu.has_value()) o.check_lengths(l.dev);
    else o.R = o.cu.has_value() ? o.cu->size(0) - 1 : 1;      // a stats-only pass reads none: their number sizes the workspace
    if (stats_only) allocate_rows(f, l.N, l.dev);
    else allocate_objective(f, l.N, o.R, l.dev, true);
    const Tensor ws = workspace_or(workspace, ulorl_lmhead_workspace_bytes(l.N, l.Hd, l.V, (int32_t)o.R, (int32_t)chunk), l.dev);
    Fields none;
    const Fields& g = stats_only ? none : f;
    ulorl_segment_stats st;
    const bool diagnose = K > 0 && !stats_only;
    if (diagnose) st = segment_struct(seg = segment_tensors(K, l.N, l.dev), K);
    check(ulorl_lmhead_token_loss_fwd(ptr(h), ptr(w), l.N, l.Hd, l.V, (int32_t)chunk, as<int32_t>(o.token_ids), as<int32_t>(o.cu), (int32_t)o.R,
                                      stats_only ? nullptr : as<int32_t>(o.segment_ids), stats_only ? nullptr : as<float>(o.old_logp),
                                      as<float>(o.advantages), o.params, as<float>(g[LOSS]), as<float>(f[LOGP]), as<float>(f[ENTROPY]),
                                      as<float>(f[LSE]), as<float>(g[GCOEF]), as<uint8_t>(g[MASK]), as<float>(g[RATIO]), as<int32_t>(g[SEGMENT]),
                                      as<float>(g[RESP_ENTROPY]), as<uint8_t>(g[RESP_GATE]), as<int64_t>(g[COUNTERS]), diagnose ? &st : nullptr,
                                      ptr(ws), ws.nbytes(), o.launch, stream_of(l.dev)),
          "ulorl_lmhead_token_loss_fwd");
}

std::pair<Tensor, Tensor> lmhead_bwd(const Tensor& h, const Tensor& w, const OptTensor& token_ids, const OptTensor& lse, const OptTensor& gcoef,
                                     double grad_out, int64_t chunk, const OptTensor& d_hidden, const OptTensor& d_weight,
                                     const OptTensor& workspace, const ulorl_launch* launch)
{
    const Lmhead l = check_lmhead(h, w);
    check_vector(token_ids, at::kInt, l.N, "token_ids", l.dev);
    check_vector(lse, at::kFloat, l.N, "lse", l.dev);
    check_vector(gcoef, at::kFloat, l.N, "gcoef", l.dev);
    const Tensor dh = d_hidden.has_value() ? *d_hidden : at::empty_like(h), dw = d_weight.has_value() ? *d_weight : at::empty_like(w);
    const Tensor ws = workspace_or(workspace, ulorl_lmhead_workspace_bytes(l.N, l.Hd, l.V, 1, (int32_t)chunk), l.dev);
    check(ulorl_lmhead_token_loss_bwd(ptr(h), ptr(w), l.N, l.Hd, l.V, (int32_t)chunk, as<int32_t>(token_ids), as<float>(lse), as<float>(gcoef),
                                      (float)grad_out, ptr(dh), ptr(dw), ptr(ws), ws.nbytes(), launch, stream_of(l.dev)),
          "ulorl_lmhead_token_loss_bwd");
    return {dh, dw};
}

// ------------------------------------------------------------------------------------------ autograd
// The upstream gradient is a 0-dim device tensor; it is multiplied into the saved coefficients on the device (the fp32
// product that the kernels form with a host scalar), so that nothing waits for the GPU.  The objective's float tensors are
// arguments of the nodes, so that one of them that requires a gradient makes the loss require one (it gets none).
using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

struct TokenLossNode : torch::autograd::Function<TokenLossNode> {
    static Tensor forward(AutogradContext* ctx, const Tensor& logits, const OptTensor&, const OptTensor&, const Objective* o, Fields* f)
    {
        Segments none;
        token_loss_fwd(logits, *o, *f, none, 0, std::nullopt);
        ctx->save_for_backward({logits, *o->token_ids, (*f)[LSE], (*f)[GCOEF]});
        return (*f)[LOSS].reshape({});
    }
    static variable_list backward(AutogradContext* ctx, const variable_list& grad)
    {
        const variable_list s = ctx->get_saved_variables();
        return {token_loss_bwd(s[0], s[1], s[2], s[3] * grad[0], 1.0, std::nullopt, false), Tensor(), Tensor(), Tensor(), Tensor()};
    }
};

struct LmheadNode : torch::autograd::Function<LmheadNode> {
    static Tensor forward(AutogradContext* ctx, const Tensor& hidden, const Tensor& weight, const OptTensor&, const OptTensor&, const Objective* o,
                          int64_t chunk, Fields* f)
    {
        Segments none;
        lmhead_fwd(hidden, weight, *o, chunk, *f, none, 0, std::nullopt);
        ctx->save_for_backward({hidden, weight, *o->token_ids, (*f)[LSE], (*f)[GCOEF]});
        ctx->saved_data["chunk"] = chunk;
        if (o->launch != nullptr)
            ctx->saved_data["launch"] = std::vector<int64_t>{o->launch->flags, o->launch->sync_spins, o->launch->gemm_tile, o->launch->gemm_group_m};
        return (*f)[LOSS].reshape({});
    }
    static variable_list backward(AutogradContext* ctx, const variable_list& grad)
    {
        const variable_list s = ctx->get_saved_variables();
        ulorl_launch launch = {};
        const bool given = ctx->saved_data.count("launch") != 0;
        if (given) {
            const std::vector<int64_t> v = ctx->saved_data["launch"].toIntVector();
            launch.flags = (uint32_t)v[0];
            launch.sync_spins = (int32_t)v[1];
            launch.gemm_tile = (int32_t)v[2];
            launch.gemm_group_m = (int32_t)v[3];
        }
        const auto d = lmhead_bwd(s[0], s[1], s[2], s[3], s[4] * grad[0], 1.0, ctx->saved_data["chunk"].toInt(), std::nullopt, std::nullopt,
                                  std::nullopt, given ? &launch : nullptr);
        return {d.first, d.second, Tensor(), Tensor(), Tensor(), Tensor(), Tensor()};
    }
};

// ------------------------------------------------------------------------------------------ Python
using Given = std::optional<std::vector<OptTensor>>;      // a caller's FwdResult, field by field

Fields fields_of(const Given& given)
{
    Fields f;
    f.given = given.has_value();
    if (f.given)
        for (int i = 0; i < FIELDS; ++i)
            if ((*given)[i].has_value()) f[i] = *(*given)[i];
    return f;
}
py::list list_of(const Fields& f)
{
    py::list out;
    for (const Tensor& t : f) out.append(t.defined() ? py::cast(t) : py::object(py::none()));
    return out;
}

// Runs f without the interpreter's lock; its errors become the Python classes that torch gives them (OutOfMemoryError, which
// callers catch, among them).
template <class F>
auto unlocked(F f)
{
    try {
        py::gil_scoped_release no_gil;
        return f();
    } catch (const std::exception&) {
        torch::translate_exception_to_python(std::current_exception());
        throw py::error_already_set();
    }
}

Objective objective(OptTensor token_ids, OptTensor cu, OptTensor advantages, OptTensor old_logp, OptTensor segment_ids, uintptr_t params, uintptr_t launch)
{
    Objective o;
    o.token_ids = std::move(token_ids);
    o.cu = std::move(cu);
    o.advantages = std::move(advantages);
    o.old_logp = std::move(old_logp);
    o.segment_ids = std::move(segment_ids);
    o.params = reinterpret_cast<const ulorl_params*>(params);
    o.launch = reinterpret_cast<const ulorl_launch*>(launch);
    return o;
}

}  // namespace

PYBIND11_MODULE(TORCH_EXTENSION_NAME, m)
{
    m.def("set_status_error", [](py::object cls) { status_error = cls.release().ptr(); });

    m.def("token_loss_fwd", [](const Tensor& z, OptTensor y, OptTensor cu, OptTensor adv, OptTensor old, OptTensor ids, uintptr_t params,
                               uintptr_t launch, const Given& out, const OptTensor& ws, int64_t K) {
        Fields f = fields_of(out);
        Segments seg;
        unlocked([&] { token_loss_fwd(z, objective(y, cu, adv, old, ids, params, launch), f, seg, K, ws); });
        return py::make_tuple(list_of(f), seg);
    });
    m.def("token_loss_fwd_bwd", [](const Tensor& z, OptTensor y, OptTensor cu, OptTensor adv, OptTensor old, OptTensor ids, uintptr_t params,
                                   uintptr_t launch, double grad_out, const OptTensor& d, bool inplace, bool on_static, const Given& out,
                                   const OptTensor& ws, int64_t K) {
        Fields f = fields_of(out);
        Segments seg;
        const Tensor dz = unlocked([&] {
            return token_loss_fwd_bwd(z, objective(y, cu, adv, old, ids, params, launch), grad_out, d, inplace, on_static, f, seg, K, ws);
        });
        return py::make_tuple(list_of(f), seg, dz);
    });
    m.def("token_loss_bwd", [](const Tensor& z, const OptTensor& y, const OptTensor& lse, const OptTensor& g, double grad_out, const OptTensor& d,
                               bool inplace) { return unlocked([&] { return token_loss_bwd(z, y, lse, g, grad_out, d, inplace); }); });
    m.def("lmhead_fwd", [](const Tensor& h, const Tensor& w, OptTensor y, OptTensor cu, OptTensor adv, OptTensor old, OptTensor ids,
                           uintptr_t params, uintptr_t launch, int64_t chunk, const Given& out, const OptTensor& ws, int64_t K) {
        Fields f = fields_of(out);
        Segments seg;
        unlocked([&] { lmhead_fwd(h, w, objective(y, cu, adv, old, ids, params, launch), chunk, f, seg, K, ws); });
        return py::make_tuple(list_of(f), seg);
    });
    m.def("lmhead_bwd", [](const Tensor& h, const Tensor& w, const OptTensor& y, const OptTensor& lse, const OptTensor& g, double grad_out,
                           int64_t chunk, const OptTensor& dh, const OptTensor& dw, const OptTensor& ws, uintptr_t launch) {
        return unlocked([&] { return lmhead_bwd(h, w, y, lse, g, grad_out, chunk, dh, dw, ws, reinterpret_cast<const ulorl_launch*>(launch)); });
    });
    m.def("autograd_token_loss", [](const Tensor& z, OptTensor y, OptTensor cu, OptTensor adv, OptTensor old, OptTensor ids, uintptr_t params,
                                    uintptr_t launch, bool want_fields) {
        const Objective o = objective(y, cu, adv, old, ids, params, launch);
        Fields f;
        const Tensor loss = unlocked([&] { return TokenLossNode::apply(z, o.advantages, o.old_logp, &o, &f); });
        return py::make_tuple(loss, want_fields ? list_of(f) : py::list());
    });
    m.def("autograd_lmhead", [](const Tensor& h, const Tensor& w, OptTensor y, OptTensor cu, OptTensor adv, OptTensor old, OptTensor ids,
                                uintptr_t params, uintptr_t launch, int64_t chunk, bool want_fields) {
        const Objective o = objective(y, cu, adv, old, ids, params, launch);
        Fields f;
        const Tensor loss = unlocked([&] { return LmheadNode::apply(h, w, o.advantages, o.old_logp, &o, chunk, &f); });
        return py::make_tuple(loss, want_fields ? list_of(f) : py::list());
    });

    m.def("advantage_prep", [](const Tensor& rewards, const OptTensor& truncated, const Tensor& cu, int64_t group, double eps, bool unbiased) {
        return unlocked([&] {
            TORCH_CHECK(rewards.is_cuda(), "libulorl runs on the GPU only");
            const at::Device dev = rewards.device();
            const int64_t R = rewards.size(0);
            check_vector(rewards, at::kFloat, R, "rewards", dev);
            check_vector(truncated, at::kByte, R, "truncated", dev);
            TORCH_CHECK_VALUE(cu.device() == dev && cu.scalar_type() == at::kInt && cu.size(0) == R + 1,
                              "cu_seqlens must be int32 [R+1] on the same device");
            const int64_t N = cu.select(0, R).item<int32_t>();
            const int64_t groups = R / (group > 1 ? group : 1);
            const Tensor adv = empty(R, at::kFloat, dev), keep = empty(groups > 1 ? groups : 1, at::kByte, dev), tok = empty(N, at::kFloat, dev),
                         kept = empty(1, at::kLong, dev);
            check(ulorl_advantage_prep(as<float>(rewards), as<uint8_t>(truncated), as<int32_t>(cu), (int32_t)R, (int32_t)group, N, (float)eps,
                                       unbiased ? 1 : 0, as<float>(adv), as<uint8_t>(keep), as<float>(tok), as<int64_t>(kept), stream_of(dev)),
                  "ulorl_advantage_prep");
            return std::make_tuple(adv, groups > 0 ? keep : keep.narrow(0, 0, 0), tok, kept);
        });
    });
    m.def("segment_diagnostics", [](int64_t K, const Tensor& ids, const OptTensor& ratio, const OptTensor& logp, const OptTensor& old,
                                    const OptTensor& entropy, const OptTensor& mask, const OptTensor& adv, double eps_low, double eps_high) {
        return unlocked([&] {
            const at::Device dev = ids.device();
            TORCH_CHECK_VALUE(dev.is_cuda(), "Expected a cuda device, but got: ", dev.str());
            const int64_t N = ids.size(0);
            check_elements(ids, at::kInt, N, "segment_ids", dev);
            check_elements(ratio, at::kFloat, N, "ratio", dev);
            check_elements(logp, at::kFloat, N, "logp", dev);
            check_elements(old, at::kFloat, N, "old_logp", dev);
            check_elements(entropy, at::kFloat, N, "entropy", dev);
            check_elements(mask, at::kByte, N, "mpt_mask", dev);
            check_elements(adv, at::kFloat, N, "advantages", dev);
            Segments s = segment_tensors(K, N, dev);
            check(ulorl_segment_diagnostics(N, (int32_t)K, as<int32_t>(ids), as<float>(ratio), as<float>(logp), as<float>(old), as<float>(entropy),
                                            as<uint8_t>(mask), as<float>(adv), (float)eps_low, (float)eps_high, as<int64_t>(s[0]), as<double>(s[1]),
                                            as<float>(s[2]), as<int64_t>(s[3]), as<double>(s[4]), as<double>(s[5]), as<int64_t>(s[6]),
                                            as<int64_t>(s[7]), ptr(s[8]), s[8].nbytes(), stream_of(dev)),
                  "ulorl_segment_diagnostics");
            return s;
        });
    });
    m.def("segment_pool_step", [](const Tensor& prev, const OptTensor& now, const OptTensor& eos, int64_t seg_len, int64_t max_len) {
        return unlocked([&] {
            TORCH_CHECK(prev.is_cuda(), "libulorl runs on the GPU only");
            const at::Device dev = prev.device();
            const int64_t B = prev.size(0);
            check_vector(prev, at::kInt, B, "prev_len", dev);
            check_vector(now, at::kInt, B, "new_len", dev);
            check_vector(eos, at::kByte, B, "hit_eos", dev);
            const Segments s = {empty(B, at::kByte, dev), empty(B, at::kInt, dev), empty(B, at::kInt, dev), empty(B, at::kInt, dev),
                                empty(B, at::kInt, dev), empty(B + 1, at::kInt, dev), empty(B, at::kByte, dev), empty(5, at::kLong, dev)};
            check(ulorl_segment_pool_step((int32_t)B, as<int32_t>(prev), as<int32_t>(now), as<uint8_t>(eos), (int32_t)seg_len, (int32_t)max_len,
                                          as<uint8_t>(s[0]), as<int32_t>(s[1]), as<int32_t>(s[2]), as<int32_t>(s[3]), as<int32_t>(s[4]),
                                          as<int32_t>(s[5]), as<uint8_t>(s[6]), as<int64_t>(s[7]), stream_of(dev)),
                  "ulorl_segment_pool_step");
            return s;
        });
    });
}
