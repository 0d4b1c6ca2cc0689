// Native half of the Python binding: tensors in, C-ABI calls (moga.h), tensors out.
//
// Nothing is computed here.  Each function allocates its outputs and its workspace from torch's caching
// allocator and makes one C-ABI call on the current stream (or the one given), so that a call costs its
// kernel launches and little more.  Host time at a few hundred tokens, with ctypes and with this: the four
// forward calls 72 and 32 us, the four backward calls 70 and 31 us, a training step through autograd 346 and
// 101 us (its backward now runs in the engine's thread without the interpreter).
#include <ATen/ATen.h>
#include <c10/core/StreamGuard.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/utils/pybind.h>

#include <optional>
#include <tuple>
#include <vector>

#include "moga.h"

namespace py = pybind11;
using at::Tensor;
using OptTensor = std::optional<Tensor>;
using OptStream = std::optional<int64_t>;   // hipStream_t as an integer; none: the current stream

namespace {

// Python exceptions are raised with the interpreter lock held: the calls themselves run without it.
[[noreturn]] void raise(PyObject* type, const std::string& text) {
  py::gil_scoped_acquire gil;
  PyErr_SetString(type, text.c_str());
  throw py::error_already_set();
}

void check(const char* fn, int status) {
  if (status == MOGA_OK) return;
  py::gil_scoped_acquire gil;
  py::object cls = py::module_::import("paper_2510_18692_amd.binding").attr("MogaError");
  PyErr_SetObject(cls.ptr(), cls(fn, status).ptr());
  throw py::error_already_set();
}

int dt(const Tensor& t) {
  if (t.scalar_type() == at::kFloat) return MOGA_F32;
  if (t.scalar_type() == at::kBFloat16) return MOGA_BF16;
  raise(PyExc_TypeError, std::string("unsupported dtype ") + c10::toString(t.scalar_type()));
}

void* ptr(const Tensor& t) {
  if (!t.is_cuda() || !t.is_contiguous()) raise(PyExc_AssertionError, "device-resident contiguous tensors only");
  return t.data_ptr();
}
void* ptr(const OptTensor& t) { return t ? ptr(*t) : nullptr; }
template <typename T> T* as(const Tensor& t) { return static_cast<T*>(ptr(t)); }
template <typename T> T* as(const OptTensor& t) { return static_cast<T*>(ptr(t)); }

// Every function checks its tensors before anything touches the GPU.
template <typename... T>
void require(const T&... t) { (ptr(t), ...); }

void need_dims(const Tensor& t, int64_t n) {
  if (t.dim() != n) raise(PyExc_ValueError, "expected a tensor of " + std::to_string(n) + " dimensions");
}

size_t bytes_of(const OptTensor& ws) { return ws ? (size_t)ws->numel() : 0; }

// The stream of a call and what is allocated for it.  Memory comes from the pool of torch's current stream.  Where the
// kernels run on another stream, every tensor is recorded as used there: a workspace or an intermediate result is dropped on
// the host while they may still run, and its memory must not go to the current stream before they are done.  (The stream must
// outlive these tensors, as for Tensor.record_stream.)
class Call {
 public:
  explicit Call(const OptStream& given) {
    const auto current = c10::hip::getCurrentHIPStream();
    handle_ = given ? reinterpret_cast<hipStream_t>(*given) : current.stream();
    if (handle_ != current.stream()) {   // torch's tensors are on "cuda" devices
      const auto s = c10::hip::getStreamFromExternal(handle_, current.device_index());
      other_ = c10::Stream(c10::Stream::UNSAFE, c10::Device(c10::kCUDA, current.device_index()), s.id());
    }
  }
  void* stream() const { return handle_; }
  const std::optional<c10::Stream>& other() const { return other_; }

  Tensor make(at::IntArrayRef size, const Tensor& like, at::ScalarType type) const {
    Tensor t = at::empty(size, like.options().dtype(type));
    if (other_) t.record_stream(*other_);
    return t;
  }
  Tensor make(at::IntArrayRef size, const Tensor& like) const { return make(size, like, like.scalar_type()); }
  Tensor workspace(size_t bytes, const Tensor& like) const { return make({std::max<int64_t>((int64_t)bytes, 16)}, like, at::kByte); }

  // Workspace of an attention call: what it runs fastest with if the device has it, else what it needs; on another stream
  // than torch's current one no more than it needs.  Without the room no last round is split, and the rounding of those
  // rows differs (moga.h): a call that finds the device full gives its result all the same, not the same bits.
  OptTensor attn_workspace(int op, int64_t N, int64_t Nk, int64_t H, int64_t D, int64_t M, const Tensor& like) const {
    const size_t need = moga_workspace_bytes(op, N, (int)H, (int)D, (int)M, 0, dt(like));
    const size_t preferred = moga_workspace_preferred_bytes(op, N, Nk, (int)H, (int)D, (int)M, 0, dt(like));
    if (preferred > need && !other_) {
      try {
        return workspace(preferred, like);
      } catch (const c10::OutOfMemoryError&) {
      }
    }
    if (need == 0) return std::nullopt;
    return workspace(need, like);
  }

 private:
  hipStream_t handle_;
  std::optional<c10::Stream> other_;   // the call's stream, if it is not torch's current one
};

std::tuple<Tensor, Tensor, OptTensor, OptTensor> route(const Tensor& x, const Tensor& w, const OptTensor& bias,
                                                       bool want_probs, bool want_logits, const OptStream& stream) {
  require(x, w, bias);
  const Call call(stream);
  need_dims(x, 2);
  const int64_t N = x.size(0), d = x.size(1), M = w.size(0);
  Tensor group = call.make({N}, x, at::kInt), gate = call.make({N}, x, at::kFloat);
  OptTensor probs, logits;
  if (want_probs) probs = call.make({N, M}, x, at::kFloat);
  if (want_logits) logits = call.make({N, M}, x, at::kFloat);
  check("moga_route", moga_route(ptr(x), dt(x), as<float>(w), as<float>(bias), N, (int)d, (int)M, as<int32_t>(group),
                                 as<float>(gate), as<float>(probs), as<float>(logits), nullptr, 0, call.stream()));
  return {group, gate, probs, logits};
}

struct Permuted {
  Tensor counts, cu_seqlens, max_seqlen, perm, inv_perm;
  OptTensor qh, kh, vh;
};

Permuted permute(const Tensor& group, int64_t M, const OptTensor& q, const OptTensor& k, const OptTensor& v,
                 const OptStream& stream) {
  require(group, q, k, v);
  const Call call(stream);
  const int64_t N = group.size(0);
  Permuted p;
  p.counts = call.make({M}, group, at::kInt);
  p.cu_seqlens = call.make({M + 1}, group, at::kInt);
  p.max_seqlen = call.make({1}, group, at::kInt);
  p.perm = call.make({N}, group, at::kInt);
  p.inv_perm = call.make({N}, group, at::kInt);
  int64_t H = 0, D = 0;
  int type = MOGA_F32;
  if (q) {
    need_dims(*q, 3);
    H = q->size(1);
    D = q->size(2);
    type = dt(*q);
    p.qh = call.make({H, N, D}, *q);
    p.kh = call.make({H, N, D}, k ? *k : *q);
    p.vh = call.make({H, N, D}, v ? *v : *q);
  }
  Tensor ws = call.workspace(moga_workspace_bytes(MOGA_OP_PERMUTE, N, (int)H, (int)D, (int)M, 0, type), group);
  check("moga_permute", moga_permute(as<int32_t>(group), N, (int)M, ptr(q), ptr(k), ptr(v), type, (int)H, (int)D,
                                     as<int32_t>(p.counts), as<int32_t>(p.cu_seqlens), as<int32_t>(p.max_seqlen),
                                     as<int32_t>(p.perm), as<int32_t>(p.inv_perm), ptr(p.qh), ptr(p.kh), ptr(p.vh),
                                     ptr(ws), ws.numel(), call.stream()));
  return p;
}

std::tuple<Tensor, Tensor> group_attn_fwd(const Tensor& qh, const Tensor& kh, const Tensor& vh, const Tensor& cu,
                                          double scale, const OptStream& stream, const OptTensor& out, const OptTensor& lse_out) {
  require(qh, kh, vh, cu, out, lse_out);
  const Call call(stream);
  need_dims(qh, 3);
  const int64_t H = qh.size(0), N = qh.size(1), D = qh.size(2), M = cu.size(0) - 1;
  Tensor oh = out ? *out : call.make({H, N, D}, qh);
  Tensor lse = lse_out ? *lse_out : call.make({H, N}, qh, at::kFloat);
  OptTensor ws = call.attn_workspace(MOGA_OP_ATTN_FWD, N, N, H, D, M, qh);
  check("moga_group_attn_fwd",
        moga_group_attn_fwd_ws(ptr(qh), ptr(kh), ptr(vh), dt(qh), N, (int)H, (int)D, as<int32_t>(cu), (int)M, (float)scale, ptr(oh),
                               as<float>(lse), ptr(ws), bytes_of(ws), call.stream()));
  return {oh, lse};
}

std::tuple<Tensor, Tensor, Tensor> group_attn_fwd_tokens(const Tensor& qh, const Tensor& kh, const Tensor& vh, const Tensor& cu, double scale,
                                                         const Tensor& perm, const Tensor& gate, const OptStream& stream) {
  require(qh, kh, vh, cu, perm, gate);
  const Call call(stream);
  need_dims(qh, 3);
  const int64_t H = qh.size(0), N = qh.size(1), D = qh.size(2), M = cu.size(0) - 1;
  Tensor oh = call.make({H, N, D}, qh), lse = call.make({H, N}, qh, at::kFloat), o = call.make({N, H, D}, qh);
  OptTensor ws = call.attn_workspace(MOGA_OP_ATTN_FWD, N, N, H, D, M, qh);
  check("moga_group_attn_fwd_tokens",
        moga_group_attn_fwd_tokens(ptr(qh), ptr(kh), ptr(vh), dt(qh), N, (int)H, (int)D, as<int32_t>(cu), (int)M, (float)scale,
                                   as<int32_t>(perm), as<float>(gate), ptr(oh), as<float>(lse), ptr(o), ptr(ws), bytes_of(ws), call.stream()));
  return {oh, lse, o};
}

Tensor unpermute(const Tensor& oh, const Tensor& perm, const OptTensor& gate, const OptStream& stream, const OptTensor& out) {
  require(oh, perm, gate, out);
  const Call call(stream);
  need_dims(oh, 3);
  const int64_t H = oh.size(0), N = oh.size(1), D = oh.size(2);
  Tensor o = out ? *out : call.make({N, H, D}, oh);
  check("moga_unpermute", moga_unpermute(ptr(oh), dt(oh), as<int32_t>(perm), as<float>(gate), N, (int)H, (int)D, ptr(o), call.stream()));
  return o;
}

std::tuple<Tensor, Tensor> unpermute_bwd(const Tensor& d_o, const Tensor& oh, const Tensor& perm, const Tensor& gate,
                                         const OptStream& stream) {
  require(d_o, oh, perm, gate);
  const Call call(stream);
  need_dims(oh, 3);
  const int64_t H = oh.size(0), N = oh.size(1), D = oh.size(2);
  Tensor d_oh = call.make({H, N, D}, oh), d_gate = call.make({N}, oh, at::kFloat);
  check("moga_unpermute_bwd", moga_unpermute_bwd(ptr(d_o), ptr(oh), dt(oh), as<int32_t>(perm), as<float>(gate), N, (int)H, (int)D,
                                                 ptr(d_oh), as<float>(d_gate), call.stream()));
  return {d_oh, d_gate};
}

std::tuple<Tensor, Tensor, Tensor> group_attn_bwd(const Tensor& d_oh, const Tensor& qh, const Tensor& kh, const Tensor& vh,
                                                  const Tensor& oh, const Tensor& lse, const Tensor& cu, double scale,
                                                  const OptStream& stream, const OptTensor& ws_in) {
  require(d_oh, qh, kh, vh, oh, lse, cu, ws_in);
  const Call call(stream);
  need_dims(qh, 3);
  const int64_t H = qh.size(0), N = qh.size(1), D = qh.size(2), M = cu.size(0) - 1;
  Tensor d_qh = call.make({H, N, D}, qh), d_kh = call.make(kh.sizes(), kh), d_vh = call.make(vh.sizes(), vh);
  // dQ and dK/dV in one launch where that is the better form, unless the caller brings a workspace of its own
  OptTensor ws = ws_in ? ws_in : call.attn_workspace(MOGA_OP_ATTN_BWD_JOINT, N, N, H, D, M, qh);
  const auto fn = ws_in ? moga_group_attn_bwd : moga_group_attn_bwd_joint;
  check("moga_group_attn_bwd", fn(ptr(d_oh), ptr(qh), ptr(kh), ptr(vh), ptr(oh), as<float>(lse), dt(qh), N, (int)H, (int)D,
                                  as<int32_t>(cu), (int)M, (float)scale, ptr(d_qh), ptr(d_kh), ptr(d_vh), ptr(ws), bytes_of(ws),
                                  call.stream()));
  return {d_qh, d_kh, d_vh};
}

struct TokenGrads {
  Tensor d_oh, d_gate;
  OptTensor d_qh, d_kh, d_vh;   // sorted order, if asked for
  Tensor d_q, d_k, d_v;
};

TokenGrads group_attn_bwd_tokens(const Tensor& d_o, const Tensor& qh, const Tensor& kh, const Tensor& vh, const Tensor& oh, const Tensor& lse,
                                 const Tensor& cu, double scale, const Tensor& perm, const Tensor& gate, bool want_sorted,
                                 const OptStream& stream) {
  require(d_o, qh, kh, vh, oh, lse, cu, perm, gate);
  const Call call(stream);
  need_dims(qh, 3);
  const int64_t H = qh.size(0), N = qh.size(1), D = qh.size(2), M = cu.size(0) - 1;
  TokenGrads g;
  g.d_oh = call.make({H, N, D}, oh);
  g.d_gate = call.make({N}, oh, at::kFloat);
  if (want_sorted) {
    g.d_qh = call.make({H, N, D}, qh);
    g.d_kh = call.make(kh.sizes(), kh);
    g.d_vh = call.make(vh.sizes(), vh);
  }
  g.d_q = call.make({N, H, D}, qh);
  g.d_k = call.make({N, H, D}, kh);
  g.d_v = call.make({N, H, D}, vh);
  OptTensor ws = call.attn_workspace(MOGA_OP_ATTN_BWD_JOINT, N, N, H, D, M, qh);
  check("moga_group_attn_bwd_tokens",
        moga_group_attn_bwd_tokens_joint(ptr(d_o), ptr(qh), ptr(kh), ptr(vh), ptr(oh), as<float>(lse), dt(qh), N, (int)H, (int)D,
                                         as<int32_t>(cu), (int)M, (float)scale, as<int32_t>(perm), as<float>(gate), ptr(g.d_oh),
                                         as<float>(g.d_gate), ptr(g.d_qh), ptr(g.d_kh), ptr(g.d_vh), ptr(g.d_q), ptr(g.d_k), ptr(g.d_v),
                                         ptr(ws), bytes_of(ws), call.stream()));
  return g;
}

std::tuple<Tensor, Tensor, Tensor> permute_bwd(const Tensor& d_qh, const Tensor& d_kh, const Tensor& d_vh, const Tensor& perm,
                                               const OptStream& stream) {
  require(d_qh, d_kh, d_vh, perm);
  const Call call(stream);
  need_dims(d_qh, 3);
  const int64_t H = d_qh.size(0), N = d_qh.size(1), D = d_qh.size(2);
  Tensor d_q = call.make({N, H, D}, d_qh), d_k = call.make({N, H, D}, d_kh), d_v = call.make({N, H, D}, d_vh);
  check("moga_permute_bwd", moga_permute_bwd(ptr(d_qh), ptr(d_kh), ptr(d_vh), dt(d_qh), as<int32_t>(perm), N, (int)H, (int)D, ptr(d_q),
                                             ptr(d_k), ptr(d_v), call.stream()));
  return {d_q, d_k, d_v};
}

// An upstream gradient on the device as an fp32 scalar; a conversion runs in order with the kernel that reads it.
Tensor device_scalar(const Tensor& t, const Call& call) {
  c10::OptionalStreamGuard guard;
  if (call.other()) guard.reset_stream(*call.other());
  return t.reshape({1}).to(at::kFloat);
}

// frac: also the balancing loss's share of the gate's gradient.  dx: the type of d_x, none: not wanted.
std::tuple<Tensor, OptTensor> route_bwd_with(const Tensor& x, const Tensor& w, const Tensor& probs, const Tensor& group, const Tensor& gate,
                                             const Tensor& d_gate, const OptTensor& frac, double alpha, const OptTensor& d_loss,
                                             std::optional<at::ScalarType> dx, const OptStream& stream) {
  require(x, w, probs, group, gate, d_gate, frac);
  const Call call(stream);
  need_dims(x, 2);
  const int64_t N = x.size(0), d = x.size(1), M = w.size(0);
  Tensor d_w = call.make({M, d}, x, at::kFloat);
  OptTensor d_x, dev;
  if (dx) d_x = call.make({N, d}, x, *dx);
  Tensor ws = call.workspace(moga_workspace_bytes(MOGA_OP_ROUTE_BWD, N, 0, 0, (int)M, (int)d, dt(x)), x);
  if (frac) {
    TORCH_CHECK(frac->size(0) == M, "frac of ", frac->size(0), " groups for a router of ", M);
    if (d_loss) dev = device_scalar(*d_loss, call);
  }
  check(frac ? "moga_route_bwd_balanced" : "moga_route_bwd",
        moga_route_bwd_typed(ptr(x), dt(x), as<float>(w), as<float>(probs), as<int32_t>(group), as<float>(gate), as<float>(d_gate),
                             as<float>(frac), (float)alpha, 1.f, as<float>(dev), N, (int)d, (int)M, as<float>(d_w), ptr(d_x),
                             d_x ? dt(*d_x) : MOGA_F32, ptr(ws), ws.numel(), call.stream()));
  return {d_w, d_x};
}

std::optional<at::ScalarType> dx_fp32(bool want_dx) {
  if (want_dx) return at::kFloat;
  return std::nullopt;
}

std::tuple<Tensor, OptTensor> route_bwd(const Tensor& x, const Tensor& w, const Tensor& probs, const Tensor& group, const Tensor& gate,
                                        const Tensor& d_gate, bool want_dx, const OptStream& stream) {
  return route_bwd_with(x, w, probs, group, gate, d_gate, std::nullopt, 0., std::nullopt, dx_fp32(want_dx), stream);
}

std::tuple<Tensor, OptTensor> route_bwd_balanced(const Tensor& x, const Tensor& w, const Tensor& probs, const Tensor& group,
                                                 const Tensor& gate, const Tensor& d_gate, const Tensor& frac, double alpha,
                                                 const Tensor& d_loss, bool want_dx, const OptStream& stream) {
  return route_bwd_with(x, w, probs, group, gate, d_gate, frac, alpha, d_loss, dx_fp32(want_dx), stream);
}

std::tuple<Tensor, Tensor> fused_attn_fwd(const Tensor& q, const Tensor& k, const Tensor& v, const Tensor& perm, const Tensor& gate,
                                          const Tensor& cu, double scale, const OptStream& stream) {
  require(q, k, v, perm, gate, cu);
  const Call call(stream);
  need_dims(q, 3);
  const int64_t N = q.size(0), H = q.size(1), D = q.size(2), M = cu.size(0) - 1;
  Tensor o = call.make({N, H, D}, q), lse = call.make({H, N}, q, at::kFloat);
  check("moga_fused_attn_fwd", moga_fused_attn_fwd(ptr(q), ptr(k), ptr(v), dt(q), N, (int)H, (int)D, as<int32_t>(perm), as<float>(gate),
                                                   as<int32_t>(cu), (int)M, (float)scale, ptr(o), as<float>(lse), call.stream()));
  return {o, lse};
}

std::tuple<Tensor, Tensor, Tensor, Tensor> fused_attn_bwd(const Tensor& d_o, const Tensor& q, const Tensor& k, const Tensor& v,
                                                          const Tensor& o, const Tensor& lse, const Tensor& perm, const Tensor& inv_perm,
                                                          const Tensor& gate, const Tensor& cu, double scale, const OptStream& stream) {
  require(d_o, q, k, v, o, lse, perm, inv_perm, gate, cu);
  const Call call(stream);
  need_dims(q, 3);
  const int64_t N = q.size(0), H = q.size(1), D = q.size(2), M = cu.size(0) - 1;
  Tensor d_q = call.make({N, H, D}, q), d_k = call.make(k.sizes(), k), d_v = call.make(v.sizes(), v), d_gate = call.make({N}, q, at::kFloat);
  Tensor ws = call.workspace(moga_workspace_bytes(MOGA_OP_ATTN_BWD, N, (int)H, (int)D, (int)M, 0, dt(q)), q);
  check("moga_fused_attn_bwd", moga_fused_attn_bwd(ptr(d_o), ptr(q), ptr(k), ptr(v), ptr(o), as<float>(lse), dt(q), N, (int)H, (int)D,
                                                   as<int32_t>(perm), as<int32_t>(inv_perm), as<float>(gate), as<int32_t>(cu), (int)M,
                                                   (float)scale, ptr(d_q), ptr(d_k), ptr(d_v), as<float>(d_gate), ptr(ws), ws.numel(),
                                                   call.stream()));
  return {d_q, d_k, d_v, d_gate};
}

std::tuple<Tensor, Tensor> varlen_attn_fwd(const Tensor& qh, const Tensor& kh, const Tensor& vh, const Tensor& cu_q, const Tensor& cu_k,
                                           double scale, const OptStream& stream) {
  require(qh, kh, vh, cu_q, cu_k);
  const Call call(stream);
  need_dims(qh, 3);
  const int64_t H = qh.size(0), Nq = qh.size(1), D = qh.size(2), Nk = kh.size(1), G = cu_q.size(0) - 1;
  Tensor oh = call.make({H, Nq, D}, qh), lse = call.make({H, Nq}, qh, at::kFloat);
  OptTensor ws = call.attn_workspace(MOGA_OP_VARLEN_ATTN_FWD, Nq, Nk, H, D, G, qh);
  check("moga_varlen_attn_fwd", moga_varlen_attn_fwd(ptr(qh), ptr(kh), ptr(vh), dt(qh), Nq, Nk, (int)H, (int)D, as<int32_t>(cu_q),
                                                     as<int32_t>(cu_k), (int)G, (float)scale, ptr(oh), as<float>(lse), ptr(ws), bytes_of(ws),
                                                     call.stream()));
  return {oh, lse};
}

std::tuple<Tensor, Tensor, Tensor> varlen_attn_bwd(const Tensor& d_oh, const Tensor& qh, const Tensor& kh, const Tensor& vh, const Tensor& oh,
                                                   const Tensor& lse, const Tensor& cu_q, const Tensor& cu_k, double scale,
                                                   const OptStream& stream) {
  require(d_oh, qh, kh, vh, oh, lse, cu_q, cu_k);
  const Call call(stream);
  need_dims(qh, 3);
  const int64_t H = qh.size(0), Nq = qh.size(1), D = qh.size(2), Nk = kh.size(1), G = cu_q.size(0) - 1;
  Tensor d_qh = call.make({H, Nq, D}, qh), d_kh = call.make(kh.sizes(), kh), d_vh = call.make(vh.sizes(), vh);
  OptTensor ws = call.attn_workspace(MOGA_OP_VARLEN_ATTN_BWD, Nq, Nk, H, D, G, qh);
  check("moga_varlen_attn_bwd", moga_varlen_attn_bwd(ptr(d_oh), ptr(qh), ptr(kh), ptr(vh), ptr(oh), as<float>(lse), dt(qh), Nq, Nk, (int)H,
                                                     (int)D, as<int32_t>(cu_q), as<int32_t>(cu_k), (int)G, (float)scale, ptr(d_qh),
                                                     ptr(d_kh), ptr(d_vh), ptr(ws), bytes_of(ws), call.stream()));
  return {d_qh, d_kh, d_vh};
}

// (qh, kh, vh, cu_q, cu_k) of each call -> (oh, lse)
using FwdCallIn = std::tuple<Tensor, Tensor, Tensor, Tensor, Tensor>;
std::vector<std::tuple<Tensor, Tensor>> varlen_attn_fwd_calls(const std::vector<FwdCallIn>& in, double scale, const OptStream& stream) {
  TORCH_CHECK(!in.empty() && in.size() <= MOGA_MAX_CALLS, "one to ", MOGA_MAX_CALLS, " calls");
  const Call call(stream);
  const Tensor& first = std::get<0>(in[0]);
  std::vector<std::tuple<Tensor, Tensor>> out;
  std::vector<OptTensor> ws;
  std::vector<moga_attn_fwd_call> c;
  for (const auto& [qh, kh, vh, cu_q, cu_k] : in) {
    require(qh, kh, vh, cu_q, cu_k);
    need_dims(qh, 3);
    TORCH_CHECK(qh.scalar_type() == first.scalar_type() && qh.size(0) == first.size(0) && qh.size(2) == first.size(2),
                "calls of one type, number of heads and head size");
    const int64_t H = qh.size(0), Nq = qh.size(1), D = qh.size(2), Nk = kh.size(1), G = cu_q.size(0) - 1;
    out.emplace_back(call.make({H, Nq, D}, qh), call.make({H, Nq}, qh, at::kFloat));
    ws.push_back(call.attn_workspace(MOGA_OP_ATTN_FWD_CALL, Nq, Nk, H, D, G, qh));
    c.push_back({ptr(qh), ptr(kh), ptr(vh), as<int32_t>(cu_q), as<int32_t>(cu_k), Nq, Nk, (int)G, ptr(std::get<0>(out.back())),
                 as<float>(std::get<1>(out.back())), ptr(ws.back()), bytes_of(ws.back())});
  }
  check("moga_varlen_attn_fwd_calls", moga_varlen_attn_fwd_calls(c.data(), (int)c.size(), dt(first), (int)first.size(0), (int)first.size(2),
                                                                 (float)scale, call.stream()));
  return out;
}

// (d_oh, qh, kh, vh, oh, lse, cu_q, cu_k, ws) of each call -> (d_qh, d_kh, d_vh)
using BwdCallIn = std::tuple<Tensor, Tensor, Tensor, Tensor, Tensor, Tensor, Tensor, Tensor, Tensor>;
std::vector<std::tuple<Tensor, Tensor, Tensor>> varlen_attn_bwd_rows_calls(const std::vector<BwdCallIn>& in, double scale,
                                                                           const OptStream& stream) {
  TORCH_CHECK(!in.empty() && in.size() <= MOGA_MAX_CALLS, "one to ", MOGA_MAX_CALLS, " calls");
  const Call call(stream);
  const Tensor& first = std::get<1>(in[0]);
  std::vector<std::tuple<Tensor, Tensor, Tensor>> out;
  std::vector<moga_attn_bwd_call> c;
  for (const auto& [d_oh, qh, kh, vh, oh, lse, cu_q, cu_k, ws] : in) {
    require(d_oh, qh, kh, vh, oh, lse, cu_q, cu_k, ws);
    need_dims(qh, 3);
    TORCH_CHECK(qh.scalar_type() == first.scalar_type() && qh.size(0) == first.size(0) && qh.size(2) == first.size(2),
                "calls of one type, number of heads and head size");
    out.emplace_back(call.make(qh.sizes(), qh), call.make(kh.sizes(), kh), call.make(vh.sizes(), vh));
    const auto& [d_qh, d_kh, d_vh] = out.back();
    c.push_back({ptr(d_oh), ptr(qh), ptr(kh), ptr(vh), ptr(oh), as<float>(lse), as<int32_t>(cu_q), as<int32_t>(cu_k), qh.size(1), kh.size(1),
                 (int)cu_q.size(0) - 1, ptr(d_qh), ptr(d_kh), ptr(d_vh), ptr(ws), (size_t)ws.numel()});
  }
  check("moga_varlen_attn_bwd_rows_calls", moga_varlen_attn_bwd_rows_calls(c.data(), (int)c.size(), dt(first), (int)first.size(0),
                                                                           (int)first.size(2), (float)scale, call.stream()));
  return out;
}

Tensor gather_rows(const Tensor& src, const Tensor& index, const OptStream& stream) {
  require(src, index);
  const Call call(stream);
  need_dims(src, 3);
  const int64_t H = src.size(1), D = src.size(2), Nk = index.size(0);
  Tensor dst = call.make({H, Nk, D}, src);
  check("moga_gather_rows", moga_gather_rows(ptr(src), dt(src), as<int32_t>(index), Nk, (int)H, (int)D, ptr(dst), call.stream()));
  return dst;
}

Tensor gather_rows_bwd(const Tensor& d_dst, const Tensor& inv_cu, const Tensor& inv_slots, int64_t N, const OptTensor& into,
                       const OptStream& stream) {
  require(d_dst, inv_cu, inv_slots, into);
  const Call call(stream);
  need_dims(d_dst, 3);
  const int64_t H = d_dst.size(0), Nk = d_dst.size(1), D = d_dst.size(2);
  Tensor d_src = into ? *into : call.make({N, H, D}, d_dst);
  check("moga_gather_rows_bwd", moga_gather_rows_bwd(ptr(d_dst), dt(d_dst), as<int32_t>(inv_cu), as<int32_t>(inv_slots), N, Nk, (int)H, (int)D,
                                                     into ? 1 : 0, ptr(d_src), call.stream()));
  return d_src;
}

py::tuple gather3_fwd(const Tensor& q, const Tensor& k, const Tensor& v, const Tensor& inv_moga, const Tensor& q_slot, const Tensor& inv_cu,
                      const Tensor& inv_slots, const OptTensor& inv_frame, const OptStream& stream) {
  Tensor t[9];
  {
    py::gil_scoped_release nogil;
    require(q, k, v, inv_moga, q_slot, inv_cu, inv_slots, inv_frame);
    const Call call(stream);
    need_dims(q, 3);
    const int64_t N = q.size(0), H = q.size(1), D = q.size(2), Nk = inv_slots.size(0);
    for (int i = 0; i < 9; ++i) t[i] = call.make({H, i == 4 || i == 5 ? Nk : N, D}, i % 3 == 0 ? q : i % 3 == 1 ? k : v);
    check("moga_gather3_fwd", moga_gather3_fwd(ptr(q), ptr(k), ptr(v), dt(q), N, (int)H, (int)D, as<int32_t>(inv_moga), as<int32_t>(q_slot),
                                               as<int32_t>(inv_cu), as<int32_t>(inv_slots), Nk, as<int32_t>(inv_frame), ptr(t[0]), ptr(t[1]),
                                               ptr(t[2]), ptr(t[3]), ptr(t[4]), ptr(t[5]), ptr(t[6]), ptr(t[7]), ptr(t[8]), call.stream()));
  }
  return py::make_tuple(t[0], t[1], t[2], t[3], t[4], t[5], t[6], t[7], t[8]);
}

Tensor gather3_bwd(const Tensor& g_moga, const Tensor& inv_moga, const Tensor& g_stga, const Tensor& inv_cu, const Tensor& inv_slots,
                   const Tensor& g_frame, const OptTensor& inv_frame, const OptStream& stream) {
  require(g_moga, inv_moga, g_stga, inv_cu, inv_slots, g_frame, inv_frame);
  const Call call(stream);
  need_dims(g_moga, 3);
  const int64_t H = g_moga.size(0), N = g_moga.size(1), D = g_moga.size(2), Nk = g_stga.size(1);
  Tensor d_src = call.make({N, H, D}, g_moga);
  check("moga_gather3_bwd", moga_gather3_bwd(ptr(g_moga), as<int32_t>(inv_moga), ptr(g_stga), as<int32_t>(inv_cu), as<int32_t>(inv_slots), Nk,
                                             ptr(g_frame), as<int32_t>(inv_frame), dt(g_moga), N, (int)H, (int)D, ptr(d_src),
                                             call.stream()));
  return d_src;
}

std::tuple<Tensor, Tensor, Tensor> gather3_bwd_qkv(const Tensor& gq_m, const Tensor& gk_m, const Tensor& gv_m, const Tensor& inv_moga,
                                                   const Tensor& gq_s, const Tensor& gk_s, const Tensor& gv_s, const Tensor& q_slot,
                                                   const Tensor& inv_cu, const Tensor& inv_slots, const Tensor& gq_f, const Tensor& gk_f,
                                                   const Tensor& gv_f, const OptTensor& inv_frame, const OptStream& stream) {
  require(gq_m, gk_m, gv_m, inv_moga, gq_s, gk_s, gv_s, q_slot, inv_cu, inv_slots, gq_f, gk_f, gv_f, inv_frame);
  const Call call(stream);
  need_dims(gq_m, 3);
  need_dims(gk_s, 3);
  const int64_t H = gq_m.size(0), N = gq_m.size(1), D = gq_m.size(2), Nk = gk_s.size(1);
  Tensor d_q = call.make({N, H, D}, gq_m), d_k = call.make({N, H, D}, gk_m), d_v = call.make({N, H, D}, gv_m);
  check("moga_gather3_bwd_qkv",
        moga_gather3_bwd_qkv(ptr(gq_m), ptr(gk_m), ptr(gv_m), as<int32_t>(inv_moga), ptr(gq_s), ptr(gk_s), ptr(gv_s), as<int32_t>(q_slot),
                             as<int32_t>(inv_cu), as<int32_t>(inv_slots), Nk, ptr(gq_f), ptr(gk_f), ptr(gv_f), as<int32_t>(inv_frame),
                             dt(gq_m), N, (int)H, (int)D, ptr(d_q), ptr(d_k), ptr(d_v), call.stream()));
  return {d_q, d_k, d_v};
}

Tensor merge3_fwd(const Tensor& a_moga, const Tensor& a_stga, const Tensor& a_frame, const OptTensor& inv_moga, const OptTensor& inv_stga,
                  const OptTensor& inv_frame, const Tensor& gate, const OptStream& stream) {
  require(a_moga, a_stga, a_frame, inv_moga, inv_stga, inv_frame, gate);
  const Call call(stream);
  need_dims(a_moga, 3);
  const int64_t H = a_moga.size(0), N = a_moga.size(1), D = a_moga.size(2);
  Tensor o = call.make({N, H, D}, a_moga);
  check("moga_merge3_fwd", moga_merge3_fwd(ptr(a_moga), ptr(a_stga), ptr(a_frame), dt(a_moga), as<int32_t>(inv_moga), as<int32_t>(inv_stga),
                                           as<int32_t>(inv_frame), as<float>(gate), N, (int)H, (int)D, ptr(o), call.stream()));
  return o;
}

std::tuple<Tensor, Tensor, Tensor, Tensor> merge3_bwd(const Tensor& d_o, const Tensor& a_moga, const OptTensor& inv_moga,
                                                      const OptTensor& inv_stga, const OptTensor& inv_frame, const Tensor& gate,
                                                      const OptStream& stream) {
  require(d_o, a_moga, inv_moga, inv_stga, inv_frame, gate);
  const Call call(stream);
  need_dims(d_o, 3);
  const int64_t N = d_o.size(0), H = d_o.size(1), D = d_o.size(2);
  Tensor d_m = call.make({H, N, D}, d_o), d_s = call.make({H, N, D}, d_o), d_f = call.make({H, N, D}, d_o), d_gate = call.make({N}, d_o, at::kFloat);
  check("moga_merge3_bwd", moga_merge3_bwd(ptr(d_o), ptr(a_moga), dt(d_o), as<int32_t>(inv_moga), as<int32_t>(inv_stga), as<int32_t>(inv_frame),
                                           as<float>(gate), N, (int)H, (int)D, ptr(d_m), ptr(d_s), ptr(d_f), as<float>(d_gate),
                                           call.stream()));
  return {d_m, d_s, d_f, d_gate};
}

using Rows3Out = std::tuple<Tensor, Tensor, Tensor, Tensor, Tensor, Tensor, Tensor>;
Rows3Out merge3_bwd_rows(const Tensor& d_o, const Tensor& a_moga, const Tensor& a_stga, const Tensor& a_frame, const OptTensor& inv_moga,
                         const OptTensor& inv_stga, const OptTensor& inv_frame, const Tensor& gate, const Tensor& lse_moga,
                         const Tensor& lse_stga, const Tensor& lse_frame, double scale, const Tensor& cu_moga, const Tensor& cu_q,
                         int64_t n_keys, const Tensor& cu_frame, bool room, const OptStream& stream) {
  require(d_o, a_moga, a_stga, a_frame, inv_moga, inv_stga, inv_frame, gate, lse_moga, lse_stga, lse_frame, cu_moga, cu_q, cu_frame);
  const Call call(stream);
  need_dims(d_o, 3);
  const int64_t N = d_o.size(0), H = d_o.size(1), D = d_o.size(2);
  Tensor d_m = call.make({H, N, D}, d_o), d_s = call.make({H, N, D}, d_o), d_f = call.make({H, N, D}, d_o), d_gate = call.make({N}, d_o, at::kFloat);
  auto ws = [&](int64_t Nk, const Tensor& cu) {
    const int64_t G = cu.size(0) - 1;
    if (!room) return call.workspace(moga_workspace_bytes(MOGA_OP_VARLEN_ATTN_BWD, N, (int)H, (int)D, (int)G, 0, dt(d_o)), d_o);
    const OptTensor t = call.attn_workspace(MOGA_OP_VARLEN_ATTN_BWD, N, Nk, H, D, G, d_o);
    return t ? *t : call.workspace(0, d_o);   // no rows
  };
  Tensor ws_m = ws(N, cu_moga), ws_s = ws(n_keys, cu_q), ws_f = ws(N, cu_frame);
  const size_t bytes = std::min({ws_m.numel(), ws_s.numel(), ws_f.numel()});
  check("moga_merge3_bwd_rows",
        moga_merge3_bwd_rows(ptr(d_o), ptr(a_moga), ptr(a_stga), ptr(a_frame), dt(d_o), as<int32_t>(inv_moga), as<int32_t>(inv_stga),
                             as<int32_t>(inv_frame), as<float>(gate), as<float>(lse_moga), as<float>(lse_stga), as<float>(lse_frame),
                             (float)scale, N, (int)H, (int)D, ptr(d_m), ptr(d_s), ptr(d_f), as<float>(d_gate), ptr(ws_m), ptr(ws_s), ptr(ws_f),
                             bytes, call.stream()));
  return {d_m, d_s, d_f, d_gate, ws_m, ws_s, ws_f};
}

std::tuple<Tensor, Tensor, Tensor> varlen_attn_bwd_rows(const Tensor& d_oh, const Tensor& qh, const Tensor& kh, const Tensor& vh,
                                                        const Tensor& oh, const Tensor& lse, const Tensor& cu_q, const Tensor& cu_k,
                                                        double scale, const Tensor& ws, const OptStream& stream) {
  require(d_oh, qh, kh, vh, oh, lse, cu_q, cu_k, ws);
  const Call call(stream);
  need_dims(qh, 3);
  const int64_t H = qh.size(0), Nq = qh.size(1), D = qh.size(2), Nk = kh.size(1), G = cu_q.size(0) - 1;
  Tensor d_qh = call.make({H, Nq, D}, qh), d_kh = call.make(kh.sizes(), kh), d_vh = call.make(vh.sizes(), vh);
  check("moga_varlen_attn_bwd_rows",
        moga_varlen_attn_bwd_rows(ptr(d_oh), ptr(qh), ptr(kh), ptr(vh), ptr(oh), as<float>(lse), dt(qh), Nq, Nk, (int)H, (int)D,
                                  as<int32_t>(cu_q), as<int32_t>(cu_k), (int)G, (float)scale, ptr(d_qh), ptr(d_kh), ptr(d_vh), ptr(ws),
                                  (size_t)ws.numel(), call.stream()));
  return {d_qh, d_kh, d_vh};
}

// `loss` [1] or a scalar
std::tuple<Tensor, Tensor> balance_into(const Tensor& loss, const Tensor& group, const Tensor& gate, int64_t M, double alpha,
                                        const OptStream& stream) {
  require(loss, group, gate);
  const Call call(stream);
  const int64_t N = group.size(0);
  Tensor frac = call.make({M}, group, at::kFloat), prob = call.make({M}, group, at::kFloat);
  Tensor ws = call.workspace(moga_workspace_bytes(MOGA_OP_BALANCE_LOSS, N, 0, 0, (int)M, 0, MOGA_F32), group);
  check("moga_balance_loss", moga_balance_loss(as<int32_t>(group), as<float>(gate), N, (int)M, (float)alpha, as<float>(loss), as<float>(frac),
                                               as<float>(prob), ptr(ws), ws.numel(), call.stream()));
  return {frac, prob};
}

std::tuple<Tensor, Tensor, Tensor> balance_loss(const Tensor& group, const Tensor& gate, int64_t M, double alpha, const OptStream& stream) {
  require(group, gate);
  Tensor loss = Call(stream).make({1}, group, at::kFloat);
  auto [frac, prob] = balance_into(loss, group, gate, M, alpha, stream);
  return {loss, frac, prob};
}

Tensor balance_loss_bwd(const Tensor& group, const Tensor& frac, double alpha, double d_loss, const OptTensor& d_loss_dev,
                        const OptTensor& into, const OptStream& stream) {
  require(group, frac, into);
  const Call call(stream);
  const int64_t N = group.size(0), M = frac.size(0);
  Tensor d_gate = into ? *into : call.make({N}, group, at::kFloat);
  OptTensor dev;
  if (d_loss_dev) dev = device_scalar(*d_loss_dev, call);
  check("moga_balance_loss_bwd", moga_balance_loss_bwd(as<int32_t>(group), as<float>(frac), N, (int)M, (float)alpha, (float)d_loss,
                                                       as<float>(dev), into ? 1 : 0, as<float>(d_gate), call.stream()));
  return d_gate;
}

// ---- autograd: Alg. 1 with Eq. 5 and, when alpha is given, the balancing loss of Eqs. 6-8 ----
// Parts of one allocation.  The calls of a step are made directly, with what is small in one tensor (saved for the backward) and what is only needed
// during the pass in another: a step of 1,560 tokens, 4 heads is bound by the host, and an allocation costs 1 us, three in the engine's thread.
class Parts {
 public:
  size_t add(size_t bytes) {
    const size_t at = size_;
    size_ += (bytes + 255) / 256 * 256;
    return at;
  }
  size_t size() const { return size_; }

 private:
  size_t size_ = 0;
};
template <typename T> T* part(const Tensor& t, size_t at) { return reinterpret_cast<T*>(static_cast<char*>(t.data_ptr()) + at); }

struct SavedParts : Parts {   // what the forward leaves for the backward beside the rows
  size_t gate, probs, cu, perm, lse, frac;
  SavedParts(int64_t N, int64_t H, int64_t M)
      : gate(add(4 * N)), probs(add(4 * N * M)), cu(add(4 * (M + 1))), perm(add(4 * N)), lse(add(4 * H * N)), frac(add(4 * M)) {}
};

struct Attention : public torch::autograd::Function<Attention> {
  static torch::autograd::variable_list forward(torch::autograd::AutogradContext* ctx, const Tensor& x, const Tensor& w, const Tensor& q,
                                                const Tensor& k, const Tensor& v, double scale, std::optional<double> alpha, bool grad_x) {
    require(x, w, q, k, v);
    const Call call(std::nullopt);
    need_dims(x, 2);
    need_dims(q, 3);
    const int64_t N = x.size(0), d = x.size(1), M = w.size(0), H = q.size(1), D = q.size(2);
    Tensor group = call.make({N}, x, at::kInt), o = call.make({N, H, D}, q);
    Tensor loss = alpha ? at::empty({}, x.options().dtype(at::kFloat)) : at::zeros({}, x.options().dtype(at::kFloat));
    Tensor qh = call.make({H, N, D}, q), kh = call.make({H, N, D}, k), vh = call.make({H, N, D}, v), oh = call.make({H, N, D}, q);
    const SavedParts at(N, H, M);
    Tensor saved = call.workspace(at.size(), x);
    Parts t;   // of this pass
    const size_t counts = t.add(4 * M), longest = t.add(4), inv_perm = t.add(4 * N), prob = t.add(4 * M);
    const size_t sort_bytes = moga_workspace_bytes(MOGA_OP_PERMUTE, N, (int)H, (int)D, (int)M, 0, dt(q)), sort_ws = t.add(sort_bytes);
    const size_t loss_bytes = alpha ? moga_workspace_bytes(MOGA_OP_BALANCE_LOSS, N, 0, 0, (int)M, 0, MOGA_F32) : 0, loss_ws = t.add(loss_bytes);
    Tensor pass = call.workspace(t.size(), x);
    float *gate = part<float>(saved, at.gate), *lse = part<float>(saved, at.lse);
    int32_t *cu = part<int32_t>(saved, at.cu), *perm = part<int32_t>(saved, at.perm);
    check("moga_route", moga_route(ptr(x), dt(x), as<float>(w), nullptr, N, (int)d, (int)M, as<int32_t>(group), gate,
                                   part<float>(saved, at.probs), nullptr, nullptr, 0, call.stream()));
    check("moga_permute",
          moga_permute(as<int32_t>(group), N, (int)M, ptr(q), ptr(k), ptr(v), dt(q), (int)H, (int)D, part<int32_t>(pass, counts), cu,
                       part<int32_t>(pass, longest), perm, part<int32_t>(pass, inv_perm), ptr(qh), ptr(kh), ptr(vh),
                       part<void>(pass, sort_ws), sort_bytes, call.stream()));
    OptTensor ws = call.attn_workspace(MOGA_OP_ATTN_FWD, N, N, H, D, M, qh);
    check("moga_group_attn_fwd_tokens",
          moga_group_attn_fwd_tokens(ptr(qh), ptr(kh), ptr(vh), dt(qh), N, (int)H, (int)D, cu, (int)M, (float)scale, perm, gate, ptr(oh), lse,
                                     ptr(o), ptr(ws), bytes_of(ws), call.stream()));
    if (alpha)
      check("moga_balance_loss", moga_balance_loss(as<int32_t>(group), gate, N, (int)M, (float)*alpha, as<float>(loss),
                                                   part<float>(saved, at.frac), part<float>(pass, prob), part<void>(pass, loss_ws), loss_bytes,
                                                   call.stream()));
    ctx->save_for_backward({x, w, group, saved, qh, kh, vh, oh});
    ctx->saved_data["args"] = std::vector<double>{scale, alpha.value_or(0.), alpha ? 1. : 0., grad_x ? 1. : 0.};
    ctx->mark_non_differentiable({group});
    ctx->set_materialize_grads(false);
    return {o, loss, group};
  }

  static torch::autograd::variable_list backward(torch::autograd::AutogradContext* ctx, const torch::autograd::variable_list& grads) {
    const auto s = ctx->get_saved_variables();
    const Tensor &x = s[0], &w = s[1], &group = s[2], &saved = s[3], &qh = s[4], &kh = s[5], &vh = s[6], &oh = s[7];
    const std::vector<double> args = ctx->saved_data["args"].toDoubleVector();
    const double scale = args[0];
    const bool balanced = args[2] != 0. && grads[1].defined();
    require(x, w, group, saved, qh, kh, vh, oh);
    const Call call(std::nullopt);
    const int64_t N = x.size(0), d = x.size(1), M = w.size(0), H = qh.size(0), D = qh.size(2);
    const SavedParts at(N, H, M);
    Tensor d_o = grads[0].defined() ? grads[0].contiguous() : at::zeros({N, H, D}, qh.options());
    Tensor d_q = call.make({N, H, D}, qh), d_k = call.make({N, H, D}, kh), d_v = call.make({N, H, D}, vh), d_w = call.make({M, d}, x, at::kFloat);
    Parts t;
    const size_t need = moga_workspace_bytes(MOGA_OP_ATTN_BWD_JOINT, N, (int)H, (int)D, (int)M, 0, dt(qh));
    const bool own_ws = moga_workspace_preferred_bytes(MOGA_OP_ATTN_BWD_JOINT, N, N, (int)H, (int)D, (int)M, 0, dt(qh)) > need;
    const bool own_rows = oh.nbytes() > (64 << 20);   // given back before the router's gradients are made
    const size_t d_gate = t.add(4 * N), attn_ws = t.add(own_ws ? 0 : need);
    const size_t route_bytes = moga_workspace_bytes(MOGA_OP_ROUTE_BWD, N, 0, 0, (int)M, (int)d, dt(x)), route_ws = t.add(route_bytes);
    const size_t rows = t.add(own_rows ? 0 : oh.nbytes());
    Tensor pass = call.workspace(t.size(), x);
    const float *gate = part<float>(saved, at.gate), *lse = part<float>(saved, at.lse);
    const int32_t *cu = part<int32_t>(saved, at.cu), *perm = part<int32_t>(saved, at.perm);
    {
      OptTensor ws, d_oh;
      if (own_ws) ws = call.attn_workspace(MOGA_OP_ATTN_BWD_JOINT, N, N, H, D, M, qh);
      if (own_rows) d_oh = call.make({H, N, D}, oh);
      check("moga_group_attn_bwd_tokens",
            moga_group_attn_bwd_tokens_joint(ptr(d_o), ptr(qh), ptr(kh), ptr(vh), ptr(oh), lse, dt(qh), N, (int)H, (int)D, cu, (int)M,
                                             (float)scale, perm, gate, d_oh ? ptr(*d_oh) : part<void>(pass, rows), part<float>(pass, d_gate),
                                             nullptr, nullptr, nullptr, ptr(d_q), ptr(d_k), ptr(d_v), ws ? ptr(*ws) : part<void>(pass, attn_ws),
                                             ws ? bytes_of(ws) : need, call.stream()));
    }
    Tensor d_x, d_loss;
    if (args[3] != 0.) d_x = call.make({N, d}, x);
    if (balanced) d_loss = grads[1].scalar_type() == at::kFloat ? grads[1] : device_scalar(grads[1], call);
    check("moga_route_bwd",
          moga_route_bwd_typed(ptr(x), dt(x), as<float>(w), part<float>(saved, at.probs), as<int32_t>(group), gate, part<float>(pass, d_gate),
                               balanced ? part<float>(saved, at.frac) : nullptr, (float)args[1], 1.f, balanced ? as<float>(d_loss) : nullptr, N,
                               (int)d, (int)M, as<float>(d_w), d_x.defined() ? ptr(d_x) : nullptr, dt(x), part<void>(pass, route_ws),
                               route_bytes, call.stream()));
    return {d_x, d_w, d_q, d_k, d_v, Tensor(), Tensor(), Tensor()};
  }
};

std::tuple<Tensor, Tensor, Tensor> attention(const Tensor& x, const Tensor& w, const Tensor& q, const Tensor& k, const Tensor& v, double scale,
                                             std::optional<double> alpha, bool grad_x) {
  auto r = Attention::apply(x, w, q, k, v, scale, alpha, grad_x);
  return {r[0], r[1], r[2]};
}

}  // namespace

PYBIND11_MODULE(TORCH_EXTENSION_NAME, m) {
  const auto nogil = py::call_guard<py::gil_scoped_release>();
  m.def("route", &route, nogil);
  m.def(
      "permute",
      [](const Tensor& group, int64_t M, const OptTensor& q, const OptTensor& k, const OptTensor& v, const OptStream& stream) {
        Permuted p = permute(group, M, q, k, v, stream);
        return std::make_tuple(p.counts, p.cu_seqlens, p.max_seqlen, p.perm, p.inv_perm, p.qh, p.kh, p.vh);
      },
      nogil);
  m.def("group_attn_fwd", &group_attn_fwd, nogil);
  m.def("group_attn_fwd_tokens", &group_attn_fwd_tokens, nogil);
  m.def("unpermute", &unpermute, nogil);
  m.def("unpermute_bwd", &unpermute_bwd, nogil);
  m.def("group_attn_bwd", &group_attn_bwd, nogil);
  m.def(
      "group_attn_bwd_tokens",
      [](const Tensor& d_o, const Tensor& qh, const Tensor& kh, const Tensor& vh, const Tensor& oh, const Tensor& lse, const Tensor& cu,
         double scale, const Tensor& perm, const Tensor& gate, bool want_sorted, const OptStream& stream) {
        TokenGrads g = group_attn_bwd_tokens(d_o, qh, kh, vh, oh, lse, cu, scale, perm, gate, want_sorted, stream);
        return std::make_tuple(g.d_oh, g.d_gate, g.d_qh, g.d_kh, g.d_vh, g.d_q, g.d_k, g.d_v);
      },
      nogil);
  m.def("permute_bwd", &permute_bwd, nogil);
  m.def("route_bwd", &route_bwd, nogil);
  m.def("route_bwd_balanced", &route_bwd_balanced, nogil);
  m.def("fused_attn_fwd", &fused_attn_fwd, nogil);
  m.def("fused_attn_bwd", &fused_attn_bwd, nogil);
  m.def("varlen_attn_fwd", &varlen_attn_fwd, nogil);
  m.def("varlen_attn_bwd", &varlen_attn_bwd, nogil);
  m.def("varlen_attn_fwd_calls", &varlen_attn_fwd_calls, nogil);
  m.def("varlen_attn_bwd_rows_calls", &varlen_attn_bwd_rows_calls, nogil);
  m.def("gather_rows", &gather_rows, nogil);
  m.def("gather_rows_bwd", &gather_rows_bwd, nogil);
  m.def("gather3_fwd", &gather3_fwd);
  m.def("gather3_bwd", &gather3_bwd, nogil);
  m.def("gather3_bwd_qkv", &gather3_bwd_qkv, nogil);
  m.def("merge3_fwd", &merge3_fwd, nogil);
  m.def("merge3_bwd", &merge3_bwd, nogil);
  m.def("merge3_bwd_rows", &merge3_bwd_rows, nogil);
  m.def("varlen_attn_bwd_rows", &varlen_attn_bwd_rows, nogil);
  m.def("balance_loss", &balance_loss, nogil);
  m.def("balance_loss_bwd", &balance_loss_bwd, nogil);
  m.def("attention", &attention, nogil);
}
