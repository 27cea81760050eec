// Internal helpers shared by the translation units of libexpertweave (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdint>
#include <cstdio>

#include "expertweave.h"

#include "ffn_plan.h"

namespace ew {

// Records a printf-style message for ew_last_error() and returns `code`.
int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
void clear_error();

inline int hip_fail(hipError_t e, const char* what) {
  return fail(e == hipErrorOutOfMemory ? EW_ERR_OOM : EW_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

#define EW_HIP(call)                                    \
  do {                                                  \
    hipError_t _e = (call);                             \
    if (_e != hipSuccess) return ::ew::hip_fail(_e, #call); \
  } while (0)

// Checks the launch that was just enqueued.
#define EW_LAUNCH_CHECK(name)                                   \
  do {                                                          \
    hipError_t _e = hipGetLastError();                          \
    if (_e != hipSuccess) return ::ew::hip_fail(_e, "launch " name); \
  } while (0)

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
inline int ilog2_ceil(int v) {  // smallest b with (1<<b) >= v, at least 1
  int b = 1;
  while ((1 << b) < v) ++b;
  return b;
}


// ffn_gemm.hip: LDS-tiled grouped GEMM path of moe_grouped_ffn (bf16, many rows per slot).
size_t ffn_gemm_plan_ints(int rows, int P);
int launch_ffn_gemm(const void* x, int rows, int k, int H, int I, int P, const int32_t* counts, const int32_t* offsets,
                    const int32_t* por, const void* w13, const void* w2, void* act, void* y, int32_t* plan, hipStream_t st);


// ffn_f32.hip: the fp32 path (both products; S shared experts' slots behind the P routed ones, or none).
int launch_ffn_f32(const void* x, int T, int k, int H, int I, int P, int S, const int32_t* counts, const int32_t* offsets,
                   const int32_t* por, const void* w13, const void* w2, const void* w13_sh, const void* w2_sh, void* act, void* y,
                   hipStream_t st);

// ffn.hip: moe_grouped_ffn's fp32 path with shared experts, workspace checked as in the public calls.
int grouped_ffn_f32(const void* x, int T, int k, int H, int I, int P, int S, const int32_t* counts, const int32_t* offsets,
                    const int32_t* pair_of_row, const void* w13, const void* w2, const void* w13_shared, const void* w2_shared,
                    void* y, void* ws, size_t ws_bytes, void* stream);

// ffn_plan.hip: the bf16 path of moe_grouped_ffn (weights and gathered token rows both reach LDS by LDS-direct loads,
// persistent workgroups claim their units from a plan built on the device).
size_t ffn_plan_ints(int T, int rows, int P);
// Plan shape of a call with `rows` rows in all and `slots` slots (shared experts included).  frags, chunk_frags: the tuning
// hook's kernel shape and cap on 32-row fragments per chunk, 0 = automatic; merge: the two products share a launch;
// wait_polls: the tuning hook's limit on a unit's wait, 0 = automatic.
FfnPlanShape ffn_plan_shape(int T, int rows, int slots, int H, int I, int frags, int chunk_frags, bool merge, int wait_polls);
// A layer pass of few tokens routes inside the grouped FFN's launch (ffn_route.h).  What that needs, and hands out: the arguments of
// moe_route_reroute_permute.
constexpr int kRouteTokens = 64, kRoutePairs = 512;
struct FfnRoute {
  const float* logits;
  const int32_t* aid;
  const int32_t* emap;
  int T, E, k, renorm, bits, S;
  int32_t* ids;
  float* w;
  int32_t* slot;
  int32_t* counts;
  int32_t* offsets;
  int32_t* por;
  int32_t* rop;
};
// Whether a plan of this shape can be made there, for these dimensions.
bool ffn_routes(const FfnPlanShape& sh, int T, int E, int k, int P, int S);
// The plan's counters that such a call needs zeroed before its launch: the claim counters and n_done completion counters.
struct FfnCounters {
  int32_t* plan;  // nullptr: none
  int done_off, n_done;
};
// unpermute_gate.hip: moe_gate_logits, whose launch also zeroes the counters (bf16, H % 128 == 0).
int gate_logits(const void* x, int dtype, const float* Wg, int T, int H, int E, const int32_t* adapter_id, const float* bias, float* logits,
                const FfnCounters& zero, hipStream_t st);
// route_permute.hip: whether a call of so many pairs takes the single-block permutation (a tuning hook moves the line).
bool single_block_permute(long long pairs);
// ffn.hip: router scores, routing, routed and shared experts of a layer pass that routes inside the FFN's launch.
int layer_ffn_routed(const ew_layer* L, const void* x, const int32_t* adapter_id, int T, const FfnPlanShape& sh, hipStream_t st);
// The plan kernel alone (what launch_ffn_bf16 runs first unless plan_ready).
int launch_ffn_plan(const int32_t* counts, const int32_t* offsets, int P, int S, int T, int rows_routed, const FfnPlanShape& sh,
                    int32_t* plan, hipStream_t st);
// S > 0: slots P .. P+S-1 are shared experts (weights w13_sh / w2_sh) that every one of the rows_routed / k tokens
// visits; their rows follow the routed ones in act and y, and plan must be sized for all rows and P + S slots.
// H % 128 == 0, I % 128 == 0, rows * max(H, I) * 2 < 2^32 and H * I * 4 < 2^32 are the caller's checks.
int launch_ffn_bf16(const void* x, int rows_routed, int k, int H, int I, int P, int S, const FfnPlanShape& sh, bool plan_ready,
                    const int32_t* counts, const int32_t* offsets, const int32_t* por, const void* w13, const void* w2, const void* w13_sh,
                    const void* w2_sh, void* act, void* y, int32_t* plan, hipStream_t st, const FfnRoute* route = nullptr);

// Whether moe_grouped_ffn / moe_grouped_ffn_with_shared with these dimensions runs those kernels, and
// if so with which plan shape (defined beside the tuning state it depends on).
bool ffn_shape_of_call(int dtype, int T, int k, int H, int I, int P, int S, FfnPlanShape* sh);

}  // namespace ew
