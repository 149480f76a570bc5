// The differentiable call behind autograd.burst_attention: attention of a query slice against key/value
// chunks as one torch autograd node, in C++.  Argument marshalling and buffers only; every arithmetic
// step is a call into libburst.so (paper Alg. 1 forward, Alg. 2 backward).
// Why native: in Python the two halves of a call ran on two threads (autograd's backward thread is another
// one) and cost 200 us of host time at any size, several times the GPU time of a short sequence.
#include <torch/extension.h>
#include <c10/core/DeviceGuard.h>
#include <c10/hip/HIPGraphsC10Utils.h>
#include <c10/hip/HIPStream.h>

#include <cmath>
#include <optional>
#include <string>
#include <vector>

#include "../../include/burst.h"

namespace {

using torch::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

void check(int status, const char* where) {
  TORCH_CHECK(status == BURST_OK, where, ": ", burst_strerror(status), " (status ", status, ")");
}

// Whether the library can read a [B, H, rows, d] tensor where it lies: last dimension contiguous, the
// other strides and the base address multiples of 16 bytes, rows not overlapping.
bool addressable(const Tensor& t) {
  if (t.dim() != 4 || (t.size(3) != 1 && t.stride(3) != 1)) return false;
  if (reinterpret_cast<uintptr_t>(t.data_ptr()) % 16 != 0) return false;
  const int64_t unit = 16 / (int64_t)t.element_size();
  for (int i = 0; i < 3; i++)
    if (t.size(i) != 1 && (t.stride(i) <= 0 || t.stride(i) % unit != 0)) return false;
  return t.size(2) == 1 || t.stride(2) >= t.size(3);
}

// Strides for the parameter block; all zero for a contiguous tensor.  Dimensions of size 1 (whose stride
// addresses nothing) get the row length.
void set_strides(int64_t (&out)[3], const Tensor& t) {
  const bool dense = t.is_contiguous();
  for (int i = 0; i < 3; i++) out[i] = dense ? 0 : t.size(i) > 1 ? t.stride(i) : t.size(3);
}

// K and V of a chunk as they are if one set of strides addresses both, else contiguous copies.
void pair_in_place(Tensor& k, Tensor& v) {
  bool same = addressable(k) && addressable(v) && k.is_contiguous() == v.is_contiguous() && k.sizes() == v.sizes();
  for (int j = 0; j < 3 && same; j++) same = k.size(j) == 1 || k.stride(j) == v.stride(j);
  if (!same) { k = k.contiguous(); v = v.contiguous(); }
}

// t if it lies in memory like q, else a copy that does.
Tensor lying_like(const Tensor& t, const Tensor& q) {
  return t.strides() == q.strides() ? t : torch::empty_strided(q.sizes(), q.strides(), q.options()).copy_(t);
}

struct Call {                        // what forward and backward have in common
  burst_params p{};
  std::vector<burst_chunk> chunks;
};

// mask_of: for each chunk the place of its block flags in `masks`, -1 = none (empty: no chunk has any).
Call describe(const Tensor& q, const variable_list& ks, const variable_list& vs, const variable_list& masks,
              const std::vector<int64_t>& mask_of, double scale, bool causal, int64_t q_off, int64_t window, int64_t block) {
  Call c;
  burst_params& p = c.p;
  p.B = (int32_t)q.size(0); p.H = (int32_t)q.size(1); p.Nq = (int32_t)q.size(2); p.d = (int32_t)q.size(3);
  p.dtype = q.scalar_type() == torch::kBFloat16 ? BURST_BF16 : BURST_F32;
  p.causal = causal; p.scale = (float)scale; p.q_off = q_off; p.window = window; p.block = (int32_t)block;
  p.kv_heads = ks[0].size(1) != q.size(1) ? (int32_t)ks[0].size(1) : 0;
  set_strides(p.q_strides, q);
  int64_t at = 0;
  c.chunks.resize(ks.size());
  for (size_t i = 0; i < ks.size(); i++) {
    burst_chunk& k = c.chunks[i];
    k = burst_chunk{};
    k.K = ks[i].data_ptr(); k.V = vs[i].data_ptr();
    k.Nc = (int32_t)ks[i].size(2);
    k.k_off = at;
    at += ks[i].size(2);
    set_strides(k.kv_strides, ks[i]);
    if (!mask_of.empty() && mask_of[i] >= 0) {
      const Tensor& m = masks[mask_of[i]];
      const int64_t rows = (q.size(2) + block - 1) / block, cols = (ks[i].size(2) + block - 1) / block;
      const bool one = m.dim() == 2 && m.size(0) == rows && m.size(1) == cols;
      const bool each = m.dim() == 4 && m.size(0) == q.size(0) && m.size(1) == q.size(1) && m.size(2) == rows && m.size(3) == cols;
      TORCH_CHECK_VALUE(m.scalar_type() == torch::kByte && m.is_cuda() && m.is_contiguous(),
                        "block_mask: contiguous uint8 device tensor expected");
      TORCH_CHECK_VALUE(one || each, "block_mask: shape must be [ceil(Nq/block), ceil(Nc/block)], alone or after [B, H]");
      k.block_mask = m.data_ptr<uint8_t>();
      k.block_mask_stride = each ? rows * cols : 0;
    }
  }
  return c;
}

Tensor scratch(const Call& c, int flags, const Tensor& like) {
  const size_t need = burst_walk_workspace_bytes(c.chunks.data(), (int)c.chunks.size(), &c.p, flags);
  return need ? torch::empty({(int64_t)need}, like.options().dtype(torch::kByte)) : Tensor();
}
void* ptr(const Tensor& t) { return t.defined() ? t.data_ptr() : nullptr; }
size_t bytes(const Tensor& t) { return t.defined() ? (size_t)t.nbytes() : 0; }
void* stream_of(const Tensor& t) { return (void*)c10::hip::getCurrentHIPStream(t.device().index()).stream(); }

class Attention : public torch::autograd::Function<Attention> {
 public:
  // kvm: the keys of n chunks, then their values, then the block flags of those that have some (mask_of)
  static variable_list forward(AutogradContext* ctx, const Tensor& q_in, at::TensorList kvm, int64_t n_chunks,
                               const std::vector<int64_t>& mask_of, double scale, bool causal, int64_t q_off, int64_t window,
                               int64_t block) {
    const c10::DeviceGuard on(q_in.device());     // the library launches on the current device
    const size_t n = (size_t)n_chunks;
    const Tensor q = addressable(q_in) ? q_in : q_in.contiguous();
    variable_list ks(kvm.begin(), kvm.begin() + n), vs(kvm.begin() + n, kvm.begin() + 2 * n), masks(kvm.begin() + 2 * n, kvm.end());
    for (size_t i = 0; i < n; i++) pair_in_place(ks[i], vs[i]);
    const Call c = describe(q, ks, vs, masks, mask_of, scale, causal, q_off, window, block);
    Tensor O = torch::empty_strided(q.sizes(), q.strides(), q.options());   // O lies in memory like Q
    Tensor lse = torch::empty({q.size(0), q.size(1), q.size(2)}, q.options().dtype(torch::kFloat));
    const Tensor ws = scratch(c, BURST_WALK_NO_STATE | BURST_WALK_FORWARD, q);
    check(burst_walk_fwd(q.data_ptr(), c.chunks.data(), (int)n, nullptr, nullptr, nullptr, O.data_ptr(), lse.data_ptr<float>(),
                         ptr(ws), bytes(ws), &c.p, stream_of(q)), "burst_walk_fwd");
    variable_list saved = {q, O, lse};
    for (auto* l : {&ks, &vs, &masks}) saved.insert(saved.end(), l->begin(), l->end());
    ctx->save_for_backward(saved);
    ctx->saved_data["n"] = (int64_t)n;
    ctx->saved_data["mask_of"] = mask_of;
    ctx->saved_data["scale"] = scale;
    ctx->saved_data["causal"] = causal;
    ctx->saved_data["q_off"] = q_off;
    ctx->saved_data["window"] = window;
    ctx->saved_data["block"] = block;
    ctx->mark_non_differentiable({lse});
    ctx->set_materialize_grads(false);            // (no zeros for the gradient of lse)
    return {O, lse};
  }

  static variable_list backward(AutogradContext* ctx, variable_list grads) {
    const variable_list s = ctx->get_saved_variables();
    const size_t n = (size_t)ctx->saved_data["n"].toInt();
    variable_list out(1 + (s.size() - 3) + 7);    // q, kvm, and seven arguments that are no tensors
    if (!grads[0].defined()) return out;
    const c10::DeviceGuard on(s[0].device());
    // Hooks on saved tensors may have returned each of them in another layout than it was saved in.
    const Tensor q = addressable(s[0]) ? s[0] : s[0].contiguous(), O = lying_like(s[1], q), lse = s[2].contiguous();
    variable_list ks(s.begin() + 3, s.begin() + 3 + n), vs(s.begin() + 3 + n, s.begin() + 3 + 2 * n), masks(s.begin() + 3 + 2 * n, s.end());
    for (size_t i = 0; i < n; i++) pair_in_place(ks[i], vs[i]);
    Call c = describe(q, ks, vs, masks, ctx->saved_data["mask_of"].toIntVector(), ctx->saved_data["scale"].toDouble(),
                      ctx->saved_data["causal"].toBool(), ctx->saved_data["q_off"].toInt(), ctx->saved_data["window"].toInt(),
                      ctx->saved_data["block"].toInt());
    const Tensor g = lying_like(grads[0].to(q.scalar_type()), q);
    Tensor D = torch::empty(lse.sizes(), lse.options()), dQ = torch::empty(q.sizes(), q.options());
    out[0] = dQ;
    for (size_t i = 0; i < n; i++) {
      out[1 + i] = torch::empty(ks[i].sizes(), ks[i].options());
      out[1 + n + i] = torch::empty(vs[i].sizes(), vs[i].options());
      c.chunks[i].dK = out[1 + i].data_ptr();
      c.chunks[i].dV = out[1 + n + i].data_ptr();
    }
    const Tensor ws = scratch(c, BURST_WALK_HALF_GRADS, q);
    check(burst_walk_bwd(q.data_ptr(), c.chunks.data(), (int)n, O.data_ptr(), g.data_ptr(), lse.data_ptr<float>(),
                         D.data_ptr<float>(), dQ.data_ptr(), 0, 0, 1, ptr(ws), bytes(ws), &c.p, stream_of(q)), "burst_walk_bwd");
    return out;
  }
};

std::vector<Tensor> attention(const Tensor& q, const std::vector<Tensor>& ks, const std::vector<Tensor>& vs,
                              const std::vector<std::optional<Tensor>>& masks, double scale, bool causal, int64_t q_off,
                              int64_t window, int64_t block) {
  TORCH_CHECK_VALUE(!ks.empty() && ks.size() == vs.size(), "one key and one value tensor per chunk, at least one chunk, expected");
  TORCH_CHECK_VALUE(masks.empty() || masks.size() == ks.size(), "one block mask per chunk expected");
  TORCH_CHECK_VALUE(q.dim() == 4 && (q.scalar_type() == torch::kBFloat16 || q.scalar_type() == torch::kFloat),
                    "q: [B, H, Nq, d] of bfloat16 or float32 expected");
  variable_list kvm(ks);
  kvm.insert(kvm.end(), vs.begin(), vs.end());
  for (size_t i = 0; i < ks.size(); i++)
    TORCH_CHECK_VALUE(ks[i].dim() == 4 && ks[i].sizes() == vs[i].sizes(), "the keys and values of a chunk: the same sizes expected");
  for (const Tensor& t : kvm) {
    TORCH_CHECK_VALUE(t.dim() == 4 && t.scalar_type() == q.scalar_type() && t.size(0) == q.size(0) && t.size(1) == ks[0].size(1) &&
                      t.size(3) == q.size(3), "keys and values: [B, Hkv, Nc, d] of the type of q expected");
    TORCH_CHECK_VALUE(t.is_cuda() && t.device() == q.device(), "tensors on one device expected");
  }
  std::vector<int64_t> mask_of;
  for (const auto& m : masks) {
    mask_of.push_back(m.has_value() ? (int64_t)(kvm.size() - 2 * ks.size()) : -1);
    if (m.has_value()) kvm.push_back(*m);
  }
  return Attention::apply(q, at::TensorList(kvm), (int64_t)ks.size(), mask_of, scale, causal, q_off, window, block);
}

// harness.RingWalk's two calls for tensors as they usually are: chunks that lie densely, of the walk's type and sizes and without
// block flags, state and statistics as the walk made them, a workspace that suffices, no capture.  kOther where something
// is not so, with nothing enqueued: the caller's own marshalling then sees to it, and to its errors.  (A pass over four chunks of 256
// rows spent more time in the interpreter than on the GPU: see RingWalk.)
constexpr int kOther = 1;
bool plain_f32(const Tensor& t, const Tensor& q) { return t.is_cuda() && t.device() == q.device() && t.scalar_type() == torch::kFloat && t.is_contiguous(); }
bool like_q(const Tensor& t, const Tensor& q) {
  return t.is_cuda() && t.device() == q.device() && t.scalar_type() == q.scalar_type() && t.sizes() == q.sizes() && t.strides() == q.strides();
}
bool usual(Call& c, const Tensor& q, const std::vector<Tensor>& ks, const std::vector<Tensor>& vs, const std::vector<int64_t>& k_offs, double scale,
           bool causal, int64_t q_off, int64_t window, int64_t kv_heads) {
  if (ks.empty() || vs.size() != ks.size() || k_offs.size() != ks.size() || q.dim() != 4 || !q.is_cuda() || q.numel() == 0) return false;
  if (q.scalar_type() != torch::kBFloat16 && q.scalar_type() != torch::kFloat) return false;
  // (not every stride of a view can go into the parameter block: all of them 0, as of an expanded row, means dense there)
  if (!(q.is_contiguous() || addressable(q)) || q.device().index() != c10::hip::current_device()) return false;
  if (c10::hip::currentStreamCaptureStatusMayInitCtx() != c10::hip::CaptureStatus::None) return false;
  const int64_t heads = kv_heads != 0 ? kv_heads : q.size(1);
  for (size_t i = 0; i < ks.size(); i++) {
    const Tensor &k = ks[i], &v = vs[i];
    if (!k.is_cuda() || !v.is_cuda() || k.device() != q.device() || v.device() != q.device() || k.scalar_type() != q.scalar_type() ||
        v.scalar_type() != q.scalar_type() || k.dim() != 4 || k.sizes() != v.sizes() || !k.is_contiguous() || !v.is_contiguous()) return false;
    if (k.size(0) != q.size(0) || k.size(1) != heads || k.size(3) != q.size(3) || k.size(2) > 0x7fffffff) return false;
  }
  c = describe(q, ks, vs, {}, {}, scale, causal, q_off, window, 0);
  c.p.kv_heads = (int32_t)kv_heads;
  for (size_t i = 0; i < ks.size(); i++) c.chunks[i].k_off = k_offs[i];
  return true;
}
// The walk's workspace, if the call needs one: false where it is too small or belongs to another stream.
bool suffices(const Call& c, int flags, const std::optional<Tensor>& ws, uint64_t ws_stream, void* stream, void*& at, size_t& bytes) {
  const size_t need = burst_walk_workspace_bytes(c.chunks.data(), (int)c.chunks.size(), &c.p, flags);
  at = nullptr; bytes = 0;
  if (need == 0) return true;
  if (!ws.has_value() || (size_t)ws->nbytes() < need || ws_stream != (uint64_t)stream) return false;
  at = ws->data_ptr(); bytes = (size_t)ws->nbytes();
  return true;
}

int walk_forward(const Tensor& q, const std::vector<Tensor>& ks, const std::vector<Tensor>& vs, const std::vector<int64_t>& k_offs, double scale,
                 bool causal, int64_t q_off, int64_t window, int64_t kv_heads, const Tensor& O_acc, const Tensor& m, const Tensor& l,
                 const Tensor& O, const Tensor& lse, const std::optional<Tensor>& ws, uint64_t ws_stream) {
  Call c;
  if (!usual(c, q, ks, vs, k_offs, scale, causal, q_off, window, kv_heads) || !like_q(O, q)) return kOther;
  for (const Tensor* t : {&O_acc, &m, &l, &lse}) if (!plain_f32(*t, q)) return kOther;
  void *at, *const stream = stream_of(q);
  size_t bytes;
  if (!suffices(c, BURST_WALK_FORWARD, ws, ws_stream, stream, at, bytes)) return kOther;
  return burst_walk_fwd(q.data_ptr(), c.chunks.data(), (int)ks.size(), O_acc.data_ptr<float>(), m.data_ptr<float>(), l.data_ptr<float>(),
                        O.data_ptr(), lse.data_ptr<float>(), at, bytes, &c.p, stream);
}

// dQ, dK, dV: new tensors, fp32.
std::tuple<int, Tensor, std::vector<Tensor>, std::vector<Tensor>> walk_backward(
    const Tensor& q, const std::vector<Tensor>& ks, const std::vector<Tensor>& vs, const std::vector<int64_t>& k_offs, double scale, bool causal,
    int64_t q_off, int64_t window, int64_t kv_heads, const Tensor& O, const Tensor& dO, const Tensor& lse, const Tensor& D,
    const std::optional<Tensor>& ws, uint64_t ws_stream) {
  Call c;
  Tensor dQ;
  std::vector<Tensor> dK, dV;
  void *at, *stream = nullptr;
  size_t bytes;
  if (!usual(c, q, ks, vs, k_offs, scale, causal, q_off, window, kv_heads) || !like_q(O, q) || !like_q(dO, q) || !plain_f32(lse, q) || !plain_f32(D, q) ||
      !suffices(c, 0, ws, ws_stream, stream = stream_of(q), at, bytes)) return {kOther, dQ, dK, dV};
  const auto f32 = q.options().dtype(torch::kFloat);
  try {
    dQ = torch::empty(q.sizes(), f32);
    for (size_t i = 0; i < ks.size(); i++) {
      dK.push_back(torch::empty(ks[i].sizes(), f32));
      dV.push_back(torch::empty(vs[i].sizes(), f32));
      c.chunks[i].dK = dK[i].data_ptr();
      c.chunks[i].dV = dV[i].data_ptr();
    }
  } catch (const c10::OutOfMemoryError&) {         // (raised again, as torch's own, by the caller's allocations)
    return {kOther, Tensor(), {}, {}};
  }
  const int st = burst_walk_bwd(q.data_ptr(), c.chunks.data(), (int)ks.size(), O.data_ptr(), dO.data_ptr(), lse.data_ptr<float>(), D.data_ptr<float>(),
                                dQ.data_ptr(), 0, 0, 0, at, bytes, &c.p, stream);
  return {st, dQ, dK, dV};
}

}  // namespace

PYBIND11_MODULE(TORCH_EXTENSION_NAME, m) {
  m.def("attention", &attention, pybind11::call_guard<pybind11::gil_scoped_release>());
  m.def("walk_forward", &walk_forward, pybind11::call_guard<pybind11::gil_scoped_release>());
  m.def("walk_backward", &walk_backward, pybind11::call_guard<pybind11::gil_scoped_release>());
}
