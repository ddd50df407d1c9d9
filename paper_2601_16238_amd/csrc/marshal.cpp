// Marshalling of torch tensors into the C ABI of attn.h and rowops.h: checks, output and workspace
// allocation, and the call, for binding.py, rowops.py and autograd.py.  No arithmetic.  It is native
// because the kernels of a short problem take less time than the same checks take in Python (one
// forward plus backward of two 128-row heads: 45 us of calls for 17 us of kernels), and because an
// autograd backward runs in the engine's thread on another core, where interpreted code is several
// times slower.
#include <torch/extension.h>

#include <ATen/Context.h>
#include <c10/core/DeviceGuard.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPStream.h>
#include <hip/hip_runtime_api.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/jit/frontend/tracer.h>

#include <algorithm>
#include <initializer_list>
#include <optional>
#include <string>
#include <tuple>
#include <vector>

#include "../../include/attn.h"
#include "../../include/rowops.h"

namespace py = pybind11;
using at::Tensor;
using OptTensor = std::optional<Tensor>;
using OptStream = std::optional<uintptr_t>;
using OptStages = std::optional<int64_t>;

namespace {

PyObject *g_error_class = nullptr;  // binding.AttnError, set once on import

void check_status(int rc, const char *where)
{
    if (rc == ATTN_OK) return;
    py::gil_scoped_acquire gil;  // (the autograd engine's threads call without it)
    py::object e = py::reinterpret_borrow<py::object>(g_error_class)(rc, where);
    PyErr_SetObject(g_error_class, e.ptr());
    throw py::error_already_set();
}

void require(bool ok, const char *message)
{
    if (!ok) throw py::value_error(message);
}

// (the interpreter lock is given up for the call: a launch can block while the queue is full)
template <typename Call>
int unlocked(Call call)
{
    if (!PyGILState_Check()) return call();  // an autograd engine's thread
    py::gil_scoped_release nogil;
    return call();
}

// The stream the caller names, else torch's current one.
void *stream_ptr(const OptStream &stream)
{
    return stream ? reinterpret_cast<void *>(*stream)
                  : static_cast<void *>(c10::hip::getCurrentHIPStream().stream());
}

// (the stride of an axis of length 1 is never used and may be anything)
void same_layout(const Tensor &ref, std::initializer_list<const Tensor *> ts)
{
    for (const Tensor *t : ts) {
        bool ok = t->sizes() == ref.sizes() && t->scalar_type() == ref.scalar_type() &&
                  t->device() == ref.device();
        for (int64_t d = 0; ok && d < ref.dim(); ++d) ok = ref.size(d) == 1 || t->stride(d) == ref.stride(d);
        require(ok, "all bf16 tensors must share shape, strides, dtype and device");
    }
}

void check_element_type(const Tensor &q, bool f16_too, const char *what)
{
    const bool ok = q.scalar_type() == at::kBFloat16 || (f16_too && q.scalar_type() == at::kHalf);
    if (ok && q.is_cuda()) return;
    throw py::value_error(std::string(what) + (f16_too ? " must be torch.bfloat16 or torch.float16"
                                                       : " must be torch.bfloat16") + " tensors on the GPU");
}

void check_lse(const Tensor &lse, const Tensor &q)
{
    require(lse.scalar_type() == at::kFloat && lse.is_contiguous() && lse.sizes() == q.sizes().slice(0, 3) &&
                lse.device() == q.device(),
            "LSE must be a contiguous fp32 [B,Hq,Sq] tensor on the tensors' device");
}

Tensor empty_as(const Tensor &t) { return at::empty_strided(t.sizes(), t.strides(), t.options()); }
Tensor bytes_on(size_t bytes, const Tensor &t) { return at::empty({(int64_t)bytes}, t.options().dtype(at::kByte)); }

// Strides of a [B,H,S,D] tensor in elements.  The stride of an axis of length 1 addresses nothing and
// may hold any value: it is replaced by the one a dense tensor would have, which always passes the
// library's stride checks.
void strides3(const Tensor &t, int64_t &sb, int64_t &sh, int64_t &ss)
{
    ss = t.size(2) > 1 ? t.stride(2) : t.size(3);
    sh = t.size(1) > 1 ? t.stride(1) : t.size(2) * ss;
    sb = t.size(0) > 1 ? t.stride(0) : t.size(1) * sh;
}

attn_rect_params_t rect_params(const Tensor &q, const Tensor &k, double scale, bool causal)
{
    for (const Tensor *t : {&q, &k})
        require(t->dim() == 4 && t->stride(3) == 1, "expected [B,H,S,D] tensors with a contiguous D axis");
    require(k.size(0) == q.size(0) && k.size(3) == q.size(3), "K/V must be [B,Hkv,Sk,D] matching Q in B and D");
    attn_rect_params_t p;
    p.B = q.size(0); p.Hq = q.size(1); p.Hkv = k.size(1); p.Sq = q.size(2); p.Sk = k.size(2); p.D = q.size(3);
    strides3(q, p.q_stride_b, p.q_stride_h, p.q_stride_s);
    strides3(k, p.kv_stride_b, p.kv_stride_h, p.kv_stride_s);
    p.scale = (float)scale;
    p.causal = causal;
    return p;
}

// The tensors of a forward call: outputs are allocated where the caller gives none.
void forward_outputs(const Tensor &q, const Tensor &k, const Tensor &v, bool f16_too, Tensor &o, Tensor &lse,
                     const OptTensor &o_in, const OptTensor &lse_in)
{
    check_element_type(q, f16_too, "Q,K,V");
    same_layout(k, {&v});
    require(k.scalar_type() == q.scalar_type() && k.device() == q.device(), "all tensors must share dtype and device");
    if (o_in) { same_layout(q, {&*o_in}); o = *o_in; } else o = empty_as(q);
    if (lse_in) { check_lse(*lse_in, q); lse = *lse_in; }
    else lse = at::empty(q.sizes().slice(0, 3), q.options().dtype(at::kFloat));
}

// Whether a call takes `bytes` more than it needs for the sake of speed.  Not under
// torch.use_deterministic_algorithms: the result would depend on the free memory through the order of its sums.
// Up to 64 MiB always; more only if the allocator has a block of that size idle or if it is at most an eighth of
// what the process may still get, so that no allocation fails for it (before an allocation fails, the allocator waits
// for the device and gives back everything it holds).  Under 1 us, 6 where the device is asked.
constexpr size_t kFreely = (size_t)64 << 20, kShare = 8;
bool to_spare(size_t bytes, const Tensor &x)
{
    if (at::globalContext().deterministicAlgorithms()) return false;
    if (bytes <= kFreely) return true;
    namespace allocator = c10::hip::HIPCachingAllocator;
    const c10::DeviceIndex device = x.get_device();
    try {
        size_t idle = 1;  // (not 0, for which it would ask the device)
        allocator::cacheInfo(device, &idle);
        if (idle >= bytes) return true;
        const c10::DeviceGuard guard(x.device());
        size_t left = 0, total = 0;
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;  // (the question is no part of a captured graph)
        if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) return false;
        const hipError_t rc = hipMemGetInfo(&left, &total);
        if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess || rc != hipSuccess) return false;
        const double may = allocator::getMemoryFraction(device) * (double)total;
        const double held = allocator::getDeviceStats(device).reserved_bytes[0].current;
        return bytes <= std::min((double)left, may - held) / kShare;
    } catch (const c10::Error &) {  // (an allocator that does not answer these questions)
        return false;
    }
}

// What a forward call does about its split over the keys.  spare: the square calls, whose C entry points have
// no workspace; they take one (of the rectangular call) where there is memory to spare.
enum class Split { no, yes, spare };

// The workspace of that split: the caller's, else one of the planned size.
// Square calls of up to 768 keys are not split: it saves at most 6 us there (2 heads of 768 rows, D = 128
// causal), and their rows stay bit for bit those of a rectangular call that is not split.  Above that,
// us, one kernel -> split: one head of 1957 rows D = 128 49 -> 23, 2 of 1287 D = 32 21 -> 13, 3 of 5199 D = 80
// causal 96 -> 43, 4 of 4829 D = 128 causal 111 -> 53, 8 of 4139 D = 32 causal 40 -> 36; over 170 random calls that
// the plan splits 0.62 on average, three of them 2 .. 7 % slower (16 of 1158 D = 80 causal 28 -> 30).
constexpr int kSquareUnsplitKeys = 768;
Tensor forward_workspace(size_t need, const OptTensor &given, Split split, const Tensor &q)
{
    if (split == Split::no) return Tensor();
    if (given) return *given;
    if (!need || (split == Split::spare && !to_spare(need, q))) return Tensor();
    try {
        return bytes_on(need, q);
    } catch (const c10::OutOfMemoryError &) {
        if (split == Split::yes) throw;
    }
    return Tensor();
}

void *data_of(const Tensor &t) { return t.defined() ? t.data_ptr() : nullptr; }

// Bytes of a workspace (none: 0) for a call on x: not more than lie between its first element and the end
// of its storage (an expanded tensor counts elements that it does not have).
size_t bytes_of(const Tensor &ws, const Tensor &x)
{
    if (!ws.defined()) return 0;
    require(ws.device() == x.device(), "the workspace must be on the tensors' device");
    const size_t offset = ws.storage_offset() * ws.itemsize(), end = ws.storage().nbytes();
    return std::min(ws.nbytes(), end > offset ? end - offset : 0);
}

std::tuple<Tensor, Tensor> run_forward(const char *where, const attn_rect_params_t &p, const Tensor &q,
                                       const Tensor &k, const Tensor &v, bool f16_too, const OptTensor &o_in,
                                       const OptTensor &lse_in, const OptTensor &ws_in, Split split,
                                       const OptStream &stream)
{
    Tensor o, lse;
    forward_outputs(q, k, v, f16_too, o, lse, o_in, lse_in);
    const bool plan = !ws_in && (split == Split::yes || (split == Split::spare && p.Sk > kSquareUnsplitKeys));
    const Tensor ws = forward_workspace(plan ? attn_fwd_rect_workspace_bytes(&p) : 0, ws_in, split, q);
    const size_t bytes = bytes_of(ws, q);
    void *const Q = q.data_ptr(), *const K = k.data_ptr(), *const V = v.data_ptr(), *const O = o.data_ptr(),
               *const W = data_of(ws), *const st = stream_ptr(stream);
    float *const L = static_cast<float *>(lse.data_ptr());
    check_status(unlocked([&] {
        return (q.scalar_type() == at::kHalf ? attn_fwd_rect_f16 : attn_fwd_rect)(Q, K, V, O, L, W, bytes, &p, st);
    }), where);
    return {o, lse};
}

using Grads = std::tuple<Tensor, Tensor, Tensor>;

// The workspace of the fastest form (whole backwards), or the plain one where there is no memory to spare for that.
Tensor backward_workspace(const attn_rect_params_t &p, const Tensor &q, bool whole)
{
    const size_t plain = attn_bwd_rect_workspace_bytes(&p), best = whole ? attn_bwd_rect_best_workspace_bytes(&p) : plain;
    if (best > plain && to_spare(best, q)) {
        try {
            return bytes_on(best, q);
        } catch (const c10::OutOfMemoryError &) {
        }
    }
    return bytes_on(plain, q);
}

// cos, sin: the rotary form; stages: restricted to those stages (square problems)
Grads run_backward(const char *where, const attn_rect_params_t &p, const Tensor &q, const Tensor &k,
                   const Tensor &v, const Tensor &o, const Tensor &g, const Tensor &lse, bool f16_too,
                   const OptTensor &dq_in, const OptTensor &dk_in, const OptTensor &dv_in, const OptTensor &ws_in,
                   const OptStream &stream, const Tensor *cos = nullptr, const Tensor *sin = nullptr,
                   const OptStages &stages = {})
{
    check_element_type(q, f16_too, "tensors");
    same_layout(q, {&o, &g});
    same_layout(k, {&v});
    require(k.scalar_type() == q.scalar_type() && k.device() == q.device(), "all tensors must share dtype and device");
    check_lse(lse, q);
    auto out = [](const OptTensor &given, const Tensor &like) {
        if (given) same_layout(like, {&*given});
        return given ? *given : empty_as(like);
    };
    const Tensor dq = out(dq_in, q), dk = out(dk_in, k), dv = out(dv_in, k);
    const Tensor ws = ws_in ? *ws_in : backward_workspace(p, q, !stages);
    const size_t bytes = bytes_of(ws, q);
    void *const Q = q.data_ptr(), *const K = k.data_ptr(), *const V = v.data_ptr(), *const O = o.data_ptr(),
               *const G = g.data_ptr(), *const DQ = dq.data_ptr(), *const DK = dk.data_ptr(),
               *const DV = dv.data_ptr(), *const W = ws.data_ptr(), *const st = stream_ptr(stream);
    const float *const L = static_cast<const float *>(lse.data_ptr());
    const float *const C = cos ? static_cast<const float *>(cos->data_ptr()) : nullptr,
                *const S = sin ? static_cast<const float *>(sin->data_ptr()) : nullptr;
    check_status(unlocked([&] {
        if (cos) return attn_bwd_rope(Q, K, V, O, G, L, C, S, DQ, DK, DV, W, bytes, &p, st);
        if (stages) {
            attn_gqa_params_t s;
            s.B = p.B; s.Hq = p.Hq; s.Hkv = p.Hkv; s.S = p.Sq; s.D = p.D;
            s.q_stride_b = p.q_stride_b; s.q_stride_h = p.q_stride_h; s.q_stride_s = p.q_stride_s;
            s.kv_stride_b = p.kv_stride_b; s.kv_stride_h = p.kv_stride_h; s.kv_stride_s = p.kv_stride_s;
            s.scale = p.scale; s.causal = p.causal;
            return attn_bwd_gqa_stages(Q, K, V, O, G, L, DQ, DK, DV, W, bytes, &s, st, (uint32_t)*stages);
        }
        return (q.scalar_type() == at::kHalf ? attn_bwd_rect_f16 : attn_bwd_rect)(Q, K, V, O, G, L, DQ, DK, DV, W,
                                                                                   bytes, &p, st);
    }), where);
    return {dq, dk, dv};
}

// ---- multi-head: everything [B,H,S,D] with one layout -------------------------------------------

std::tuple<Tensor, Tensor> attn_fwd_(const Tensor &q, const Tensor &k, const Tensor &v, double scale, bool causal,
                                     const OptTensor &o, const OptTensor &lse, const OptStream &stream)
{
    same_layout(q, {&k, &v});
    return run_forward("attn_fwd", rect_params(q, k, scale, causal), q, k, v, false, o, lse, {}, Split::spare,
                       stream);
}

Grads attn_bwd_(const OptStages &stages, const Tensor &q, const Tensor &k, const Tensor &v, const Tensor &o, const Tensor &g,
                const Tensor &lse, double scale, bool causal, const OptTensor &dq, const OptTensor &dk,
                const OptTensor &dv, const OptTensor &ws, const OptStream &stream)
{
    same_layout(q, {&k, &v});
    return run_backward("attn_bwd", rect_params(q, k, scale, causal), q, k, v, o, g, lse, false, dq, dk, dv, ws,
                        stream, nullptr, nullptr, stages);
}

// ---- grouped-query heads, square ----------------------------------------------------------------

attn_rect_params_t gqa_params(const Tensor &q, const Tensor &k, double scale, bool causal)
{
    const attn_rect_params_t p = rect_params(q, k, scale, causal);
    require(p.Sq == p.Sk, "K/V must be [B,Hkv,S,D] matching Q in B, S and D");
    return p;
}

std::tuple<Tensor, Tensor> attn_fwd_gqa_(const Tensor &q, const Tensor &k, const Tensor &v, double scale, bool causal,
                                         const OptTensor &o, const OptTensor &lse, const OptStream &stream)
{
    return run_forward("attn_fwd_gqa", gqa_params(q, k, scale, causal), q, k, v, false, o, lse, {}, Split::spare,
                       stream);
}

Grads attn_bwd_gqa_(const OptStages &stages, const Tensor &q, const Tensor &k, const Tensor &v, const Tensor &o,
                    const Tensor &g, const Tensor &lse, double scale, bool causal, const OptTensor &dq,
                    const OptTensor &dk, const OptTensor &dv, const OptTensor &ws, const OptStream &stream)
{
    return run_backward("attn_bwd_gqa", gqa_params(q, k, scale, causal), q, k, v, o, g, lse, false, dq, dk, dv, ws,
                        stream, nullptr, nullptr, stages);
}

// ---- rectangular --------------------------------------------------------------------------------

std::tuple<Tensor, Tensor> attn_fwd_rect_(const Tensor &q, const Tensor &k, const Tensor &v, double scale, bool causal,
                                          const OptTensor &o, const OptTensor &lse, const OptTensor &ws, bool split,
                                          const OptStream &stream)
{
    return run_forward("attn_fwd_rect", rect_params(q, k, scale, causal), q, k, v, true, o, lse, ws,
                       split ? Split::yes : Split::no, stream);
}

Grads attn_bwd_rect_(const Tensor &q, const Tensor &k, const Tensor &v, const Tensor &o, const Tensor &g,
                     const Tensor &lse, double scale, bool causal, const OptTensor &dq, const OptTensor &dk,
                     const OptTensor &dv, const OptTensor &ws, const OptStream &stream)
{
    return run_backward("attn_bwd_rect", rect_params(q, k, scale, causal), q, k, v, o, g, lse, true, dq, dk, dv, ws,
                        stream);
}

// ---- rotary embedding fused into the calls ------------------------------------------------------

void check_tables(const Tensor &cos, const Tensor &sin, const Tensor &k)
{
    for (const Tensor *t : {&cos, &sin})
        require(t->scalar_type() == at::kFloat && t->device() == k.device() && t->is_contiguous() && t->dim() == 2 &&
                    t->size(0) == k.size(2) && t->size(1) == k.size(3) / 2,
                "cos/sin tables must be contiguous fp32 [Sk, D/2] tensors on the tensors' device");
}

std::tuple<Tensor, Tensor, OptTensor> attn_fwd_rope_(const Tensor &q, const Tensor &k, const Tensor &v,
                                                     const Tensor &cos, const Tensor &sin, double scale, bool causal,
                                                     const OptTensor &o_in, const OptTensor &lse_in,
                                                     const OptTensor &qrot_in, bool want_q_rot, bool split,
                                                     const OptStream &stream)
{
    const attn_rect_params_t p = rect_params(q, k, scale, causal);
    check_tables(cos, sin, k);
    Tensor o, lse;
    forward_outputs(q, k, v, false, o, lse, o_in, lse_in);
    OptTensor qrot = qrot_in;
    if (qrot) same_layout(q, {&*qrot});
    else if (want_q_rot) qrot = empty_as(q);
    const Tensor ws = forward_workspace(split ? attn_fwd_rope_workspace_bytes(&p) : 0, {}, split ? Split::yes : Split::no, q);
    void *const Q = q.data_ptr(), *const K = k.data_ptr(), *const V = v.data_ptr(), *const O = o.data_ptr(),
               *const R = qrot ? qrot->data_ptr() : nullptr, *const W = data_of(ws), *const st = stream_ptr(stream);
    float *const L = static_cast<float *>(lse.data_ptr());
    const float *const C = static_cast<const float *>(cos.data_ptr()), *const S = static_cast<const float *>(sin.data_ptr());
    check_status(unlocked([&] { return attn_fwd_rope(Q, K, V, C, S, O, L, R, W, bytes_of(ws, q), &p, st); }),
                 "attn_fwd_rope");
    return {o, lse, qrot};
}

Grads attn_bwd_rope_(const Tensor &q, const Tensor &k, const Tensor &v, const Tensor &o, const Tensor &g,
                     const Tensor &lse, const Tensor &cos, const Tensor &sin, double scale, bool causal,
                     const OptTensor &dq, const OptTensor &dk, const OptTensor &dv, const OptTensor &ws,
                     const OptStream &stream)
{
    const attn_rect_params_t p = rect_params(q, k, scale, causal);
    check_tables(cos, sin, k);
    return run_backward("attn_bwd_rope", p, q, k, v, o, g, lse, false, dq, dk, dv, ws, stream, &cos, &sin);
}

// ---- the autograd function's two halves ---------------------------------------------------------

// Layouts the library takes: unit stride along D, other strides multiples of 8 elements, 16-byte
// aligned base.  Anything else is copied to a contiguous tensor.
Tensor dense(const Tensor &t)
{
    const bool ok = t.stride(3) == 1 && t.stride(0) % 8 == 0 && t.stride(1) % 8 == 0 && t.stride(2) % 8 == 0 &&
                    reinterpret_cast<uintptr_t>(t.data_ptr()) % 16 == 0;
    return ok ? t : t.contiguous();
}

// t with the shape, strides and type of ref (copied only if it differs)
Tensor like(const Tensor &ref, const Tensor &t)
{
    if (t.scalar_type() == ref.scalar_type() && t.strides() == ref.strides()) return t;
    Tensor out = empty_as(ref);
    out.copy_(t);
    return out;
}

std::tuple<Tensor, Tensor, Tensor, Tensor, Tensor> fused_forward(const Tensor &q_, const Tensor &k_, const Tensor &v_,
                                                                 double scale, bool causal)
{
    // (layouts the library does not take are copied to ones it does; what is saved is what ran)
    const Tensor q = dense(q_), k = dense(k_), v = like(k, dense(v_));
    auto [o, lse] = run_forward("attn_fwd_rect", rect_params(q, k, scale, causal), q, k, v, true, {}, {}, {},
                                Split::yes, {});
    return {q, k, v, o, lse};
}

Grads fused_backward(const Tensor &q, const Tensor &k, const Tensor &v, const Tensor &o, const Tensor &lse,
                     const Tensor &g, double scale, bool causal)
{
    return run_backward("attn_bwd_rect", rect_params(q, k, scale, causal), q, k, v, o, like(o, g), lse, true, {}, {},
                        {}, {}, {});
}

// A native node: the backward runs in the engine's thread without the interpreter (us per step, Python
// function -> this: 128 x 6 heads of 65 rows 77 -> 61, 8 x 8 of 1024 rows causal 79 -> 69, D = 64).
struct FusedAttention : torch::autograd::Function<FusedAttention> {
    static Tensor forward(torch::autograd::AutogradContext *ctx, const Tensor &q_, const Tensor &k_, const Tensor &v_,
                          double scale, bool causal)
    {
        auto [q, k, v, o, lse] = fused_forward(q_, k_, v_, scale, causal);
        ctx->save_for_backward({q, k, v, o, lse});
        ctx->saved_data["scale"] = scale;
        ctx->saved_data["causal"] = causal;
        return o;
    }

    static torch::autograd::variable_list backward(torch::autograd::AutogradContext *ctx,
                                                   torch::autograd::variable_list grads)
    {
        const torch::autograd::variable_list saved = ctx->get_saved_variables();
        const double scale = ctx->saved_data["scale"].toDouble();
        const bool causal = ctx->saved_data["causal"].toBool();
        // (Python's exceptions to the form in which the engine carries them over to its caller; it would
        // make a RuntimeError of any other)
        auto carried = [](const auto &set_error) {
            py::gil_scoped_acquire gil;
            set_error();
            python_error err;
            err.persist();
            return err;
        };
        try {
            auto [dq, dk, dv] = fused_backward(saved[0], saved[1], saved[2], saved[3], saved[4], grads[0], scale, causal);
            return {dq, dk, dv, Tensor(), Tensor()};
        } catch (py::error_already_set &e) {
            throw carried([&] { e.restore(); });
        } catch (const py::builtin_exception &e) {
            throw carried([&] { e.set_error(); });
        }
    }
};

// (none while a tracer records: it would keep the allocations and not the kernels)
OptTensor fused_attention(const Tensor &q, const Tensor &k, const Tensor &v, double scale, bool causal)
{
    if (torch::jit::tracer::isTracing()) return {};
    for (const Tensor *t : {&q, &k, &v})
        TORCH_CHECK_NOT_IMPLEMENTED(!t->_fw_grad(0).defined(), "fused_attention has no rule for forward mode");
    return FusedAttention::apply(q, k, v, scale, causal);
}

// ---- row-wise kernels ---------------------------------------------------------------------------

const Tensor &rows_of(const Tensor &t, const char *name)
{
    if (t.scalar_type() != at::kBFloat16 || !t.is_cuda() || t.dim() != 2 || t.stride(1) != 1)
        throw py::value_error(std::string(name) + " must be a bf16 [rows, cols] GPU tensor with contiguous rows");
    return t;
}

// An output of the caller's: the library gets only x's rows and columns and writes that many, so there
// has to be room for them.
const Tensor &rows_for(const Tensor &x, const Tensor &t, const char *name)
{
    rows_of(t, name);
    if (t.size(0) < x.size(0) || t.size(1) < x.size(1) || t.device() != x.device())
        throw py::value_error(std::string(name) + " must hold x's rows and columns, on x's device");
    return t;
}

const Tensor &f32_of(const Tensor &x, const Tensor &t, at::IntArrayRef shape, const char *name)
{
    if (t.scalar_type() != at::kFloat || t.device() != x.device() || !t.is_contiguous() || t.sizes() != shape) {
        std::string s = std::string(name) + " must be a contiguous fp32 GPU tensor of shape (";
        for (int64_t n : shape) s += std::to_string(n) + ", ";
        throw py::value_error(s + ") on x's device");
    }
    return t;
}

float *floats(const Tensor &t) { return static_cast<float *>(t.data_ptr()); }

Tensor rmsnorm_fwd(const Tensor &x, const Tensor &w, double eps, const OptTensor &y_in, const OptStream &stream)
{
    rows_of(x, "x");
    const int64_t rows = x.size(0), cols = x.size(1);
    f32_of(x, w, {cols}, "w");
    const Tensor y = y_in ? rows_for(x, *y_in, "y") : at::empty_like(x);
    void *const X = x.data_ptr(), *const Y = y.data_ptr(), *const st = stream_ptr(stream);
    check_status(unlocked([&, W = floats(w)] {
        return rowops_rmsnorm_fwd(X, W, Y, rows, cols, x.stride(0), y.stride(0), (float)eps, st);
    }), "rowops_rmsnorm_fwd");
    return y;
}

std::tuple<Tensor, Tensor, Tensor> layernorm_fwd(const Tensor &x, const Tensor &w, const Tensor &b, double eps,
                                                 const OptTensor &y_in, const OptTensor &mean_in,
                                                 const OptTensor &rstd_in, const OptStream &stream)
{
    rows_of(x, "x");
    const int64_t rows = x.size(0), cols = x.size(1);
    f32_of(x, w, {cols}, "w");
    f32_of(x, b, {cols}, "b");
    const Tensor y = y_in ? rows_for(x, *y_in, "y") : at::empty_like(x);
    auto stat = [&](const OptTensor &t, const char *name) {
        return t ? f32_of(x, *t, {rows}, name) : at::empty({rows}, x.options().dtype(at::kFloat));
    };
    const Tensor mean = stat(mean_in, "mean"), rstd = stat(rstd_in, "rstd");
    void *const X = x.data_ptr(), *const Y = y.data_ptr(), *const st = stream_ptr(stream);
    check_status(unlocked([&, W = floats(w), B = floats(b), M = floats(mean), R = floats(rstd)] {
        return rowops_layernorm_fwd(X, W, B, Y, M, R, rows, cols, x.stride(0), y.stride(0), (float)eps, st);
    }), "rowops_layernorm_fwd");
    return {y, mean, rstd};
}

Grads layernorm_bwd(const Tensor &dy, const Tensor &x, const Tensor &w, const Tensor &mean, const Tensor &rstd,
                    const OptTensor &dx_in, const OptTensor &dw_in, const OptTensor &db_in, const OptTensor &ws_in,
                    const OptStream &stream)
{
    rows_of(x, "x");
    rows_of(dy, "dy");
    const int64_t rows = x.size(0), cols = x.size(1);
    require(dy.sizes() == x.sizes() && dy.device() == x.device(), "dy and x must have one shape and device");
    f32_of(x, w, {cols}, "w");
    f32_of(x, mean, {rows}, "mean");
    f32_of(x, rstd, {rows}, "rstd");
    const Tensor dx = dx_in ? rows_for(x, *dx_in, "dx") : at::empty_like(x);
    auto column = [&](const OptTensor &t, const char *name) {
        return t ? f32_of(x, *t, {cols}, name) : at::empty({cols}, x.options().dtype(at::kFloat));
    };
    const Tensor dw = column(dw_in, "dw"), db = column(db_in, "db");
    const Tensor ws = ws_in ? *ws_in : bytes_on(rowops_layernorm_bwd_workspace_bytes(rows, cols), x);
    const size_t ws_bytes = bytes_of(ws, x);
    void *const DY = dy.data_ptr(), *const X = x.data_ptr(), *const DX = dx.data_ptr(), *const WS = ws.data_ptr(),
               *const st = stream_ptr(stream);
    check_status(unlocked([&, W = floats(w), M = floats(mean), R = floats(rstd), DW = floats(dw), DB = floats(db)] {
        return rowops_layernorm_bwd(DY, X, W, M, R, DX, DW, DB, WS, ws_bytes, rows, cols, dy.stride(0),
                                    x.stride(0), dx.stride(0), st);
    }), "rowops_layernorm_bwd");
    return {dx, dw, db};
}

Tensor rotary_fwd(const Tensor &x, const Tensor &cos, const Tensor &sin, const OptTensor &y_in, const OptStream &stream)
{
    require(x.scalar_type() == at::kBFloat16 && x.is_cuda() && x.dim() == 4 && x.stride(3) == 1,
            "x must be a bf16 [B,H,S,D] GPU tensor with a contiguous D axis");
    const int64_t B = x.size(0), H = x.size(1), S = x.size(2), D = x.size(3);
    f32_of(x, cos, {S, D / 2}, "cos");
    f32_of(x, sin, {S, D / 2}, "sin");
    if (y_in) require(y_in->sizes() == x.sizes() && y_in->scalar_type() == x.scalar_type() &&
                          y_in->device() == x.device() && y_in->stride(3) == 1,
                      "y must match x in shape, type and device");
    const Tensor y = y_in ? *y_in : empty_as(x);
    void *const X = x.data_ptr(), *const Y = y.data_ptr(), *const st = stream_ptr(stream);
    check_status(unlocked([&, C = floats(cos), N = floats(sin)] {
        return rowops_rotary_fwd(X, C, N, Y, B, H, S, D, x.stride(0), x.stride(1), x.stride(2), y.stride(0),
                                 y.stride(1), y.stride(2), st);
    }), "rowops_rotary_fwd");
    return y;
}

}  // namespace

PYBIND11_MODULE(_marshal, m)
{
    m.def("set_error_class", [](py::object cls) { g_error_class = cls.release().ptr(); });
    m.def("attn_fwd", &attn_fwd_);
    m.def("attn_bwd", &attn_bwd_);
    m.def("attn_fwd_gqa", &attn_fwd_gqa_);
    m.def("attn_bwd_gqa", &attn_bwd_gqa_);
    m.def("attn_fwd_rect", &attn_fwd_rect_);
    m.def("attn_bwd_rect", &attn_bwd_rect_);
    m.def("attn_fwd_rope", &attn_fwd_rope_);
    m.def("attn_bwd_rope", &attn_bwd_rope_);
    m.def("fused_attention", &fused_attention);
    m.def("fused_forward", &fused_forward);
    m.def("fused_backward", &fused_backward);
    m.def("rmsnorm_fwd", &rmsnorm_fwd);
    m.def("layernorm_fwd", &layernorm_fwd);
    m.def("layernorm_bwd", &layernorm_bwd);
    m.def("rotary_fwd", &rotary_fwd);
}
