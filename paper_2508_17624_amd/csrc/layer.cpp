// One pass of a MoE layer as one host call: router scores -> fused top-k + rerouting + permutation (+ the grouped FFN's
// work plan) -> routed and shared experts -> combine; for few tokens the steps between scores and combine are one launch.  The caller describes the layer once (ew_layer: dimensions, weights,
// work buffers); a pass then costs one crossing from the caller's language instead of four with sixteen arguments each,
// which took longer than the GPU work of a small layer (configuration 0: 119 us of host time per pass, most of it the
// second stream and events that the shared experts' own calls needed).
#include "ew_internal.h"

namespace {

bool aligned256(const void* p) { return p && ((uintptr_t)p & 255) == 0; }

// Whether a pass routes inside the grouped FFN's launch: few tokens, its own router scores (their launch zeroes the plan's counters),
// and arguments that the calls it replaces would take, so that those report what is wrong with any others.  Up to 64 tokens because the
// ranking gives a token a lane, and then wherever the plan fits LDS: it is faster over that whole range (ffn_route.h).
bool routes_itself(const ew_layer* L, const void* x, const int32_t* aid, int T, ew::FfnPlanShape* sh) {
  if (L->dtype != EW_BF16 || T < 1 || T > ew::kRouteTokens || L->k < 1 || L->M < 1 || L->N < 0 || !ew::single_block_permute((long long)T * L->k)) return false;
  if (!x || !aid || !L->Wg || !L->expert_map || !L->w13 || !L->w2 || (L->S > 0 && (!L->w13_shared || !L->w2_shared)) || !L->logits || !L->ids ||
      !L->w || !L->slot || !L->counts || !L->offsets || !L->pair_of_row || !L->row_of_pair || !L->y)
    return false;
  if (!ew::ffn_shape_of_call(L->dtype, T, L->k, L->H, L->I, L->P, L->S, sh) || !ew::ffn_routes(*sh, T, L->M, L->k, L->P, L->S)) return false;
  return aligned256(L->ws_perm) && L->ws_perm_bytes >= moe_reroute_permute_workspace_bytes(T, L->k, L->P) && aligned256(L->ws_ffn) &&
         L->ws_ffn_bytes >= moe_grouped_ffn_workspace_bytes(T, L->k + L->S, L->H, L->I, L->P + L->S, L->dtype);
}

}  // namespace

extern "C" int moe_layer_forward(const ew_layer* L, const void* x, const int32_t* adapter_id, int T, const float* logits,
                                 const void* residual, void* out, void* normed_out, float eps, void* stream) {
  using ew::fail;
  if (!L) return fail(EW_ERR_INVALID_ARG, "moe_layer_forward: layer is NULL");
  if (T < 0 || T > L->T_max) return fail(EW_ERR_INVALID_ARG, "moe_layer_forward: T=%d outside 0..T_max=%d", T, L->T_max);
  if (L->S < 0 || L->k < 1 || L->H < 1 || L->I < 1 || L->P < 1) return fail(EW_ERR_INVALID_ARG, "moe_layer_forward: bad dimensions");
  // (with logits given, the steps before the combine would take any other type for fp32, and count rows in 32 bits)
  if (L->dtype != EW_F32 && L->dtype != EW_BF16) return fail(EW_ERR_INVALID_ARG, "moe_layer_forward: unknown dtype %d", L->dtype);
  if ((long long)T * ((long long)L->k + L->S) >= (1ll << 31)) return fail(EW_ERR_UNSUPPORTED, "moe_layer_forward: the row count must be below 2^31");
  int rc;
  ew::FfnPlanShape sh;
  if (!logits && routes_itself(L, x, adapter_id, T, &sh)) {
    rc = ew::layer_ffn_routed(L, x, adapter_id, T, sh, (hipStream_t)stream);
  } else {
    if (!logits) {
      rc = moe_gate_logits(x, L->dtype, L->Wg, T, L->H, L->M, L->bias ? adapter_id : nullptr, L->bias, L->logits, stream);
      if (rc != EW_OK) return rc;
      logits = L->logits;
    }
    if (L->dtype == EW_BF16) {
      rc = moe_route_reroute_permute_plan(logits, adapter_id, L->expert_map, T, L->M, L->k, L->N, L->P, L->renormalize, L->ids, L->w, L->slot,
                                          L->counts, L->offsets, L->pair_of_row, L->row_of_pair, L->ws_perm, L->ws_perm_bytes, L->H, L->I,
                                          L->S, L->dtype, L->ws_ffn, L->ws_ffn_bytes, stream);
      if (rc != EW_OK) return rc;
      rc = moe_grouped_ffn_planned(x, L->dtype, T, L->k, L->H, L->I, L->P, L->S, L->counts, L->offsets, L->pair_of_row, L->w13, L->w2,
                                   L->w13_shared, L->w2_shared, L->y, L->ws_ffn, L->ws_ffn_bytes, stream);
    } else {
      rc = moe_route_reroute_permute(logits, adapter_id, L->expert_map, T, L->M, L->k, L->N, L->P, L->renormalize, L->ids, L->w, L->slot,
                                     L->counts, L->offsets, L->pair_of_row, L->row_of_pair, L->ws_perm, L->ws_perm_bytes, stream);
      if (rc != EW_OK) return rc;
      rc = ew::grouped_ffn_f32(x, T, L->k, L->H, L->I, L->P, L->S, L->counts, L->offsets, L->pair_of_row, L->w13, L->w2, L->w13_shared,
                               L->w2_shared, L->y, L->ws_ffn, L->ws_ffn_bytes, stream);
    }
  }
  if (rc != EW_OK) return rc;
  const size_t el = L->dtype == EW_BF16 ? 2 : 4;
  const void* shared_out = L->S > 0 ? (const char*)L->y + (size_t)T * L->k * L->H * el : nullptr;
  if (normed_out)
    return moe_unpermute_rmsnorm(L->y, L->row_of_pair, L->w, shared_out, L->S, residual, T, L->k, L->H, L->dtype, out, eps, normed_out, stream);
  return moe_unpermute(L->y, L->row_of_pair, L->w, shared_out, L->S, residual, T, L->k, L->H, L->dtype, out, stream);
}
