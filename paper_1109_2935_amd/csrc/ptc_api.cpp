// C ABI of the learned preconditioner: weight packing, inference, gradients
// and the Adam update, as host sequences of the kernels in ptc.hip.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdlib>
#include <sstream>
#include <string>
#include <vector>

#include "lqcd_internal.h"
#include "lqcd_ops.h"
#include "lqcd_ptc.h"

using namespace lqcd;

#define TRY(expr)                 \
  do {                            \
    lqcd_status _s = (expr);      \
    if (_s != LQCD_OK) return _s; \
  } while (0)

namespace lqcd {

struct PtcPlan {
  int nl;
  std::vector<PtcLayerDev> layers;
  std::vector<size_t> woff;   // complex-weight offset of each layer in the master array
  std::vector<size_t> poff;   // byte offset of each layer's packed fragments
  size_t nweights = 0, packed_bytes = 0;
};

lqcd_status ptc_plan(lqcd_context *ctx, const lqcd_ptc_shape *sh, PtcPlan *plan) {
  if (!sh) return set_error(ctx, LQCD_ERR_INVALID_ARG, "network shape is NULL");
  if (sh->nlayers < 1 || sh->nlayers > kPtcMaxLayers)
    return set_error(ctx, LQCD_ERR_INVALID_ARG, "network needs 1 to 8 layers");
  if (sh->channels[0] != 1 || sh->channels[sh->nlayers] != 1)
    return set_error(ctx, LQCD_ERR_INVALID_ARG, "network input and output have one channel");
  plan->nl = sh->nlayers;
  plan->layers.clear();
  plan->woff.clear();
  plan->poff.clear();
  size_t w = 0, p = 0;
  for (int l = 0; l < sh->nlayers; ++l) {
    const int cin = sh->channels[l], cout = sh->channels[l + 1];
    if (cin < 1 || cout < 1 || cin > 16 || cout > 16 || (cin > 4 && cin % 4))
      return set_error(ctx, LQCD_ERR_UNSUPPORTED, "channels must be 1..4 or a multiple of 4 up to 16");
    PtcLayerDev L = ptc_layer_desc(cin, cout);
    plan->woff.push_back(w);
    plan->poff.push_back(p);
    w += (size_t)cout * cin * 9 * 16;
    p += ptc_fwd_frag_bytes(L) + ptc_adj_frag_bytes(L);
    plan->layers.push_back(L);
  }
  plan->nweights = w;
  plan->packed_bytes = p;
  return LQCD_OK;
}

static void bind_packed(PtcPlan &plan, const void *packed) {
  for (int l = 0; l < plan.nl; ++l) {
    PtcLayerDev &L = plan.layers[l];
    L.A = (const char *)packed + plan.poff[l];
    L.Aadj = (const char *)packed + plan.poff[l] + ptc_fwd_frag_bytes(L);
  }
}

static lqcd_status ptc_geo(lqcd_context *ctx, const lqcd_operator *op, OpInfo *info, PtcGeo *q) {
  TRY(check_op(ctx, op, info));
  if (op->action != LQCD_WILSON_CLOVER || op->prec != LQCD_F32 || (op->recon != 18 && op->recon != 12))
    return set_error(ctx, LQCD_ERR_UNSUPPORTED, "the network transports with an FP32 Wilson instance (recon 18/12)");
  if (!op->gauge || ((uintptr_t)op->gauge & 15)) return set_error(ctx, LQCD_ERR_INVALID_ARG, "operator gauge missing");
  q->g = info->g;
  q->gauge = (const float *)op->gauge;
  q->recon = op->recon;
  return LQCD_OK;
}

static std::string forward_key(const PtcLayerDev &L, const Geom &g) {
  std::ostringstream key;
  key << "ptc_fwd/" << L.cin << "-" << L.cout << "/" << geom_key(g);
  return key.str();
}

// The form of a 16-input-channel layer: the one for 16 channels, which rounds the
// links to BF16, where the autotuner may choose; the general form, which transports
// with FP32 links, where it may not (LQCD_TUNE=0, whose fallback it has always been)
// or where LQCD_PTC_VARIANT or a saved choice names it (642, 322). The numbers of the
// other forms there have been, all with BF16 links, name the one for 16 channels.
static int forward16_variant(lqcd_context *ctx, const PtcLayerDev &L, const Geom &g, hipStream_t st) {
  const char *forced = std::getenv("LQCD_PTC_VARIANT");
  const int v = forced ? std::atoi(forced) : tune_pick(ctx, forward_key(L, g), {}, 0, false, st, {});
  if (!forced && v == 0) return ctx->tune_enabled && !ctx->tune_frozen ? kPtcForward16 : 642;
  for (int f : {3221, 3231, 3222, 3232, 5031, 5041, 5032, 5042, 5033, 5043, 5034, 5044})
    if (v == f) return kPtcForward16;
  return v;
}

// Forward pass; activation k (input of layer k) is kept in acts[k] (full
// lattice, channel-interleaved BF16), the output y (even sites, FP32 packed
// spinor) goes to y_even.
static lqcd_status ptc_forward_all(lqcd_context *ctx, const PtcPlan &plan, const PtcGeo &q, const OpInfo &info,
                                   const void *in_even, std::vector<void *> &acts, void *y_even, hipStream_t st) {
  const size_t vh = info.vh;
  void *nbr;
  TRY(scratch(ctx, kSlotPtc + kPtcMaxLayers + 5, 2 * 8 * vh * sizeof(int), &nbr));
  // links at the output sites of the layers from 16 channels: the last layer's are
  // even (of a network whose only such layer is the last, 1-16-1 at 24^3 x 48, both
  // parities' table would take 80 us to save the layer 62)
  std::vector<int> variants(plan.nl, 0);
  int npar = 0;
  for (int l = 1; l < plan.nl; ++l) {
    if (plan.layers[l].cin != 16) continue;
    variants[l] = forward16_variant(ctx, plan.layers[l], q.g, st);
    if (variants[l] == kPtcForward16) npar = std::max(npar, l == plan.nl - 1 ? 1 : 2);
  }
  void *links = nullptr;
  if (npar) {
    TRY(scratch(ctx, kSlotPtc + kPtcMaxLayers + 7, ptc_link_bytes(vh, npar), &links));
    TRY(hip_check(ctx, launch_ptc_links(q, npar, (int *)nbr, links, st), "ptc neighbour and link tables"));
  } else {
    TRY(hip_check(ctx, launch_ptc_nbr(q.g, (int *)nbr, st), "ptc neighbour table"));
  }
  // layer-0 input: r on even sites, zero on odd sites
  TRY(hip_check(ctx, launch_ptc_input((int64_t)vh, in_even, acts[0], st), "ptc input"));
  for (int l = 0; l < plan.nl; ++l) {
    const bool last = l == plan.nl - 1;
    const PtcLayerDev &L = plan.layers[l];
    void *out = last ? y_even : acts[l + 1];
    // the layer-0 input (r on even sites) vanishes on odd sites
    const int zero_par = l == 0 ? 1 : -1;
    int variant = variants[l];
    if (L.cin != 16) {
      // sites per workgroup: timed once per layer shape and geometry
      variant = tune_pick(ctx, forward_key(L, q.g), {642, 322}, 642, true, st, [&](int v) {
        return launch_ptc_forward(q, L, (const int *)nbr, links, acts[l], out, last, 0, v, zero_par, st);
      });
    }
    // the last layer's output lives on even sites; 16-channel layers compute
    // both parities in one launch (a third less memory traffic, same time),
    // the first layer (only one path per parity carries data) one per launch
    if (last || zero_par >= 0) {
      for (int par = 0; par < (last ? 1 : 2); ++par)
        TRY(hip_check(ctx, launch_ptc_forward(q, L, (const int *)nbr, links, acts[l], out, last, par, variant, zero_par,
                                              st),
                      "ptc forward"));
    } else {
      TRY(hip_check(ctx, launch_ptc_forward(q, L, (const int *)nbr, links, acts[l], out, last, -1, variant, zero_par,
                                            st),
                    "ptc forward"));
    }
  }
  return LQCD_OK;
}

// Scratch: activation buffers start at slot `slot0` (BF16, both parities); the
// output slot (FP32, even sites) follows them.
static lqcd_status ptc_buffers(lqcd_context *ctx, const PtcPlan &plan, const OpInfo &info, int slot0,
                               std::vector<void *> &acts) {
  acts.assign(plan.nl + 1, nullptr);
  for (int l = 0; l < plan.nl; ++l) {
    const int c = l == 0 ? 1 : plan.layers[l - 1].cout;
    TRY(scratch(ctx, slot0 + l, 2 * info.vh * 24 * c * sizeof(uint16_t), &acts[l]));
  }
  TRY(scratch(ctx, slot0 + plan.nl, info.vh * 24 * sizeof(float), &acts[plan.nl]));
  return LQCD_OK;
}

lqcd_status ptc_apply(lqcd_context *ctx, const lqcd_operator *op, const lqcd_ptc_net *net, void *out_even,
                      const void *in_even, hipStream_t st) {
  if (!net) return set_error(ctx, LQCD_ERR_INVALID_ARG, "network is NULL");
  PtcPlan plan;
  TRY(ptc_plan(ctx, &net->shape, &plan));
  if (!net->packed || ((uintptr_t)net->packed & 15)) return set_error(ctx, LQCD_ERR_INVALID_ARG, "packed weights");
  bind_packed(plan, net->packed);
  OpInfo info;
  PtcGeo q;
  TRY(ptc_geo(ctx, op, &info, &q));
  std::vector<void *> acts;
  TRY(ptc_buffers(ctx, plan, info, kSlotPtc, acts));
  return ptc_forward_all(ctx, plan, q, info, in_even, acts, out_even, st);
}

enum PtcLoss { kLossError, kLossResidual, kLossCotangent };

// Forward pass of the network on r_even, then back-propagation of an output
// cotangent delta = dL/d conj(y) (y = N(r_even), even sites) to the weights:
// grad = dL/d conj(W). The cotangent is
//   kLossError:     (y - e) / |e|^2 for L = |y - e|^2 / |e|^2 (aux = e_even),
//   kLossResidual:  Mhat^+ z / |r|^2, z = Mhat y - r, for L = |z|^2 / |r|^2,
//   kLossCotangent: aux itself (dy_even),
// and *loss (if given) is set for the first two.
static lqcd_status ptc_backprop(lqcd_context *ctx, const lqcd_operator *op, const lqcd_ptc_net *net,
                                const void *r_even, PtcLoss kind, const void *aux, void *grad, double *loss,
                                hipStream_t st) {
  PtcPlan plan;
  TRY(ptc_plan(ctx, &net->shape, &plan));
  bind_packed(plan, net->packed);
  OpInfo info;
  PtcGeo q;
  TRY(ptc_geo(ctx, op, &info, &q));
  const size_t vh = info.vh;
  std::vector<void *> acts;
  TRY(ptc_buffers(ctx, plan, info, kSlotPtc, acts));
  TRY(ptc_forward_all(ctx, plan, q, info, r_even, acts, acts[plan.nl], st));
  int maxc = 1;
  size_t pbytes = 0;
  for (int l = 0; l < plan.nl; ++l) {
    const PtcLayerDev &L = plan.layers[l];
    maxc = std::max(maxc, L.cin);
    pbytes = std::max(pbytes, ptc_weight_partial_bytes(L, vh, l == plan.nl - 1 ? 1 : -1));
  }
  void *dy, *d0, *d1, *part, *nbr;
  TRY(scratch(ctx, kSlotPtc + kPtcMaxLayers + 3, vh * 24 * sizeof(float), &dy));
  TRY(scratch(ctx, kSlotPtc + kPtcMaxLayers + 1, 2 * vh * 24 * maxc * sizeof(uint16_t), &d0));
  TRY(scratch(ctx, kSlotPtc + kPtcMaxLayers + 2, 2 * vh * 24 * maxc * sizeof(uint16_t), &d1));
  TRY(scratch(ctx, kSlotPtc + kPtcMaxLayers + 4, pbytes, &part));
  TRY(scratch(ctx, kSlotPtc + kPtcMaxLayers + 5, 2 * 8 * vh * sizeof(int), &nbr));  // filled by the forward pass
  RedScratch red = red_scratch(ctx);
  const size_t n = vh * 12;  // complex entries of one even field
  float *delta = (float *)dy;  // dL/d conj(y) on even sites
  if (kind == kLossError) {
    // loss = |y - e|^2 / |e|^2 on even sites; delta = dL/d conj(y) = (y - e) / |e|^2
    const void *e_even = aux;
    double en2 = 0, dn2 = 0;
    TRY(hip_check(ctx, blas_norm2(LQCD_F32, e_even, n, red, st), "norm"));
    TRY(read_result(ctx, st, 1, &en2));
    if (!(en2 > 0)) return set_error(ctx, LQCD_ERR_INVALID_ARG, "target has zero norm");
    TRY(hip_check(ctx, hipMemcpyAsync(delta, acts[plan.nl], vh * 24 * sizeof(float), hipMemcpyDeviceToDevice, st),
                  "copy"));
    TRY(hip_check(ctx, blas_axpby(LQCD_F32, e_even, LQCD_F32, delta, n, -1.0, 0.0, 1.0, 0.0, &red, st), "axpby"));
    TRY(read_result(ctx, st, 1, &dn2));
    TRY(hip_check(ctx, blas_convert(LQCD_F32, delta, LQCD_F32, delta, n, 1.0 / en2, st), "scale"));
    if (loss) *loss = dn2 / en2;
  } else if (kind == kLossResidual) {
    // z = Mhat y - r; loss = |z|^2 / |r|^2; delta = Mhat^+ z / |r|^2
    void *z, *tmp;
    TRY(scratch(ctx, kSlotPtc + kPtcMaxLayers + 6, info.spinor_bytes, &z));
    TRY(scratch(ctx, kSlotSchurTmp, info.spinor_bytes, &tmp));
    double rn2 = 0, zn2 = 0;
    TRY(hip_check(ctx, blas_norm2(LQCD_F32, r_even, n, red, st), "norm"));
    TRY(read_result(ctx, st, 1, &rn2));
    if (!(rn2 > 0)) return set_error(ctx, LQCD_ERR_INVALID_ARG, "input has zero norm");
    TRY(schur_apply(ctx, info, info.g, z, acts[plan.nl], tmp, 0, nullptr, st));
    TRY(hip_check(ctx, blas_axpby(LQCD_F32, r_even, LQCD_F32, z, n, -1.0, 0.0, 1.0, 0.0, &red, st), "axpby"));
    TRY(read_result(ctx, st, 1, &zn2));
    TRY(schur_apply(ctx, info, info.g, delta, z, tmp, 1, nullptr, st));
    TRY(hip_check(ctx, blas_convert(LQCD_F32, delta, LQCD_F32, delta, n, 1.0 / rn2, st), "scale"));
    if (loss) *loss = zn2 / rn2;
  } else {
    // the caller's cotangent dL/d conj(y) on even sites
    TRY(hip_check(ctx, hipMemcpyAsync(delta, aux, vh * 24 * sizeof(float), hipMemcpyDeviceToDevice, st), "copy"));
  }
  // backward through the layers; the last layer's cotangent lives on even sites
  void *dcur = d0, *dnext = d1;
  TRY(hip_check(ctx, launch_ptc_delta((int64_t)vh, delta, dcur, st), "ptc delta"));
  for (int l = plan.nl - 1; l >= 0; --l) {
    const PtcLayerDev &L = plan.layers[l];
    const int zero_par = l == plan.nl - 1 ? 1 : -1;
    float *gw = (float *)grad + 2 * plan.woff[l];
    TRY(hip_check(ctx, launch_ptc_bwd_weight(q, L, (const int *)nbr, acts[l], dcur, (float *)part, gw, zero_par, st),
                  "ptc dW"));
    if (l == 0) break;
    TRY(hip_check(ctx, launch_ptc_bwd_data(q, L, (const int *)nbr, dcur, dnext, zero_par, st), "ptc dY"));
    std::swap(dcur, dnext);
  }
  return LQCD_OK;
}

}  // namespace lqcd

extern "C" {

lqcd_status lqcd_ptc_sizes(const lqcd_ptc_shape *shape, size_t *n_weights, size_t *packed_bytes) {
  PtcPlan plan;
  lqcd_status s = ptc_plan(nullptr, shape, &plan);
  if (s) return s;
  if (n_weights) *n_weights = plan.nweights;
  if (packed_bytes) *packed_bytes = plan.packed_bytes;
  return LQCD_OK;
}

lqcd_status lqcd_ptc_pack(lqcd_context *ctx, const lqcd_ptc_shape *shape, const void *weights, void *packed,
                          lqcd_stream stream) {
  if (!ctx) return set_error(ctx, LQCD_ERR_INVALID_ARG, "context is NULL");
  PtcPlan plan;
  TRY(ptc_plan(ctx, shape, &plan));
  if (!weights || !packed || ((uintptr_t)packed & 15)) return set_error(ctx, LQCD_ERR_INVALID_ARG, "bad pointers");
  bind_packed(plan, packed);
  for (int l = 0; l < plan.nl; ++l)
    TRY(hip_check(ctx, launch_ptc_pack(plan.layers[l], (const float *)weights + 2 * plan.woff[l], (hipStream_t)stream),
                  "ptc pack"));
  return LQCD_OK;
}

lqcd_status lqcd_ptc_apply(lqcd_context *ctx, const lqcd_operator *op, const lqcd_ptc_net *net, void *out_even,
                           const void *in_even, lqcd_stream stream) {
  if (!ctx) return set_error(ctx, LQCD_ERR_INVALID_ARG, "context is NULL");
  if (!out_even || !in_even || ((uintptr_t)out_even & 15) || ((uintptr_t)in_even & 15))
    return set_error(ctx, LQCD_ERR_INVALID_ARG, "bad field pointers");
  return ptc_apply(ctx, op, net, out_even, in_even, (hipStream_t)stream);
}

lqcd_status lqcd_ptc_gradient(lqcd_context *ctx, const lqcd_operator *op, const lqcd_ptc_net *net,
                              const void *r_even, const void *e_even, void *grad, double *loss, lqcd_stream stream) {
  if (!ctx) return set_error(ctx, LQCD_ERR_INVALID_ARG, "context is NULL");
  if (!net || !r_even || !e_even || !grad) return set_error(ctx, LQCD_ERR_INVALID_ARG, "NULL argument");
  return ptc_backprop(ctx, op, net, r_even, kLossError, e_even, grad, loss, (hipStream_t)stream);
}

lqcd_status lqcd_ptc_residual_gradient(lqcd_context *ctx, const lqcd_operator *op, const lqcd_ptc_net *net,
                                       const void *r_even, void *grad, double *loss, lqcd_stream stream) {
  if (!ctx) return set_error(ctx, LQCD_ERR_INVALID_ARG, "context is NULL");
  if (!op || !net || !r_even || !grad) return set_error(ctx, LQCD_ERR_INVALID_ARG, "NULL argument");
  TRY(check_fields_internal(ctx, op));
  return ptc_backprop(ctx, op, net, r_even, kLossResidual, nullptr, grad, loss, (hipStream_t)stream);
}

lqcd_status lqcd_ptc_vjp(lqcd_context *ctx, const lqcd_operator *op, const lqcd_ptc_net *net, const void *r_even,
                         const void *dy_even, void *grad, lqcd_stream stream) {
  if (!ctx) return set_error(ctx, LQCD_ERR_INVALID_ARG, "context is NULL");
  if (!net || !r_even || !dy_even || !grad) return set_error(ctx, LQCD_ERR_INVALID_ARG, "NULL argument");
  return ptc_backprop(ctx, op, net, r_even, kLossCotangent, dy_even, grad, nullptr, (hipStream_t)stream);
}

lqcd_status lqcd_ptc_adam(lqcd_context *ctx, const lqcd_ptc_shape *shape, void *weights, void *m, void *v,
                          const void *grad, int32_t step, double lr, lqcd_stream stream) {
  if (!ctx) return set_error(ctx, LQCD_ERR_INVALID_ARG, "context is NULL");
  PtcPlan plan;
  TRY(ptc_plan(ctx, shape, &plan));
  if (!weights || !m || !v || !grad || step < 1 || !(lr > 0))
    return set_error(ctx, LQCD_ERR_INVALID_ARG, "need weights, moments, gradient, step >= 1, lr > 0");
  const float b1 = 0.9f, b2 = 0.999f;
  const float bc1 = 1.f - std::pow(b1, (float)step), bc2 = 1.f - std::pow(b2, (float)step);
  // dL/d(Re W, Im W) = 2 (Re G, Im G) for G = dL/d conj(W)
  return hip_check(ctx, launch_adam((float *)weights, (float *)m, (float *)v, (const float *)grad, 2 * plan.nweights,
                                    (float)lr, b1, b2, 1e-8f, bc1, bc2, 2.f, (hipStream_t)stream),
                   "adam");
}

}  // extern "C"
