// Device helpers of the router and the permutation that more than one kernel uses: ranking lanes by key, and the top-k of a token
// in sixteen lanes.
#pragma once
#include <cstdint>
#include <hip/hip_runtime.h>

namespace ew {

// Monotone map float -> uint32 (larger float, larger key); -0.0 and +0.0 share one key.
__device__ __forceinline__ uint32_t order_key(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u << 1) == 0u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Lanes in `active` whose `key` (low `bits` bits significant) equals this lane's.
__device__ __forceinline__ unsigned long long match_any(uint32_t key, int bits, unsigned long long active) {
  unsigned long long m = active;
  for (int b = 0; b < bits; ++b) {
    const bool bit = (key >> b) & 1u;
    const unsigned long long vote = __ballot(bit);
    m &= bit ? vote : ~vote;
  }
  return m;
}

__device__ __forceinline__ unsigned long long lanemask_lt() {
  const unsigned lane = threadIdx.x & 63;
  return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// All 16 lanes of a row: the row's maximum / minimum.
template <typename F>
__device__ __forceinline__ uint32_t row_reduce(uint32_t v, F f) {
#define EW_ROR(x, n) (uint32_t) __builtin_amdgcn_update_dpp(0, (int)(x), 0x120 + (n), 0xf, 0xf, false)
  v = f(v, EW_ROR(v, 8));
  v = f(v, EW_ROR(v, 4));
  v = f(v, EW_ROR(v, 2));
  return f(v, EW_ROR(v, 1));
#undef EW_ROR
}
__device__ __forceinline__ uint32_t row_max(uint32_t v) { return row_reduce(v, [](uint32_t a, uint32_t b) { return a > b ? a : b; }); }
__device__ __forceinline__ uint32_t row_min(uint32_t v) { return row_reduce(v, [](uint32_t a, uint32_t b) { return a < b ? a : b; }); }
// All 16 lanes of a row: wave_sum_f32 of 64 values that the row holds R per lane (value r of lane l for wave lane l + 16 r, zero from
// R on), bit for bit: that sum pairs neighbours, then pairs of pairs, inside each row, and the row totals as (3 + 2) + (1 + 0).
template <int R>
__device__ __forceinline__ float row_sum_f32(const float (&part)[R]) {
#define EW_DPP_ADD(ctrl) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xf, 0xf, false))
  float row[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int r = 0; r < R; ++r) {
    float v = part[r];
    EW_DPP_ADD(0xB1);   // quad_perm 1,0,3,2
    EW_DPP_ADD(0x4E);   // quad_perm 2,3,0,1
    EW_DPP_ADD(0x141);  // row_half_mirror
    EW_DPP_ADD(0x140);  // row_mirror
    row[r] = v;
  }
#undef EW_DPP_ADD
  return (row[3] + row[2]) + (row[1] + row[0]);
}

// The value a key stands for (+0.0 for either zero).
__device__ __forceinline__ float key_value(uint32_t key) { return __uint_as_float(key & 0x80000000u ? key & 0x7FFFFFFFu : ~key); }

// Sixteen lanes select the top-k of one token, so a wave does four: lane l of them holds experts l, l + 16, ... (V per lane,
// E <= 16 V, k <= 16).  k rounds of "largest key, lowest index that has it, take it out"; the winner of round j stays in lane j,
// so ids and weights leave in one coalesced store.  REROUTE: maprow is the token's row of the expert map; it is read while the
// selection runs, and the slots ride in the low bits of the index that the rounds reduce, so no lookup follows.  emit(rank, expert,
// slot, weight); weigh false (wave-uniform): the weights are not worked out.  What bounds the selection is the chain of dependent instructions, and the
// wave-wide radix select (wave_topk in route_permute.hip) spends it on one token at a time, through the scalar unit that all waves of a SIMD share: k_hist
// at 8192 tokens of 64 experts, k = 6: 15.8 -> 5.0 us, at 512 tokens 8.0 -> 4.7; top-k alone at 64 tokens 3.8 -> 2.7.
template <int V, bool REROUTE, typename Emit>
__device__ __forceinline__ void group_topk(const float* __restrict__ row, const int32_t* __restrict__ maprow, int E, int k, int renorm, bool weigh, Emit emit) {
  const int l = threadIdx.x & 15;
  float val[V];
  uint32_t key[V], at[V];  // at: expert << 16 | slot
#pragma unroll
  for (int v = 0; v < V; ++v) val[v] = row[min(l + 16 * v, E - 1)];
#pragma unroll
  for (int v = 0; v < V; ++v) at[v] = ((uint32_t)(l + 16 * v) << 16) | (REROUTE ? (uint32_t)maprow[min(l + 16 * v, E - 1)] & 0xFFFFu : 0u);
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const uint32_t o = order_key(val[v]);
    key[v] = l + 16 * v < E ? (o ? o : 1u) : 0u;  // 0: not there, or taken out
  }
  uint32_t my_key = 0u, my_at = 0u, top = 0u;
  for (int j = 0; j < k; ++j) {
    uint32_t m = key[0];
#pragma unroll
    for (int v = 1; v < V; ++v) m = m > key[v] ? m : key[v];
    m = row_max(m);
    uint32_t first = ~0u;
#pragma unroll
    for (int v = V - 1; v >= 0; --v) first = key[v] == m ? at[v] : first;
    first = row_min(first);
#pragma unroll
    for (int v = 0; v < V; ++v) key[v] = first == at[v] ? 0u : key[v];
    if (j == 0) top = m;
    if (j == l) {
      my_key = m;
      my_at = first;
    }
  }
  if (!weigh) {
    if (l < k) emit(l, (int)(my_at >> 16), (int)(my_at & 0xFFFFu), 0.f);
    return;
  }
  // softmax over all E logits: max = the first winner.  Both sums run in the order of wave_topk, so that a weight does not depend
  // on which of the two selected it (one ulp of it flips a bf16 rounding of the layer's output, and the layers behind carry that on).
  const float vmax = key_value(top);
  constexpr int R = V < 4 ? V : 4;
  float part[R] = {}, chosen[R] = {};
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const float ex = l + 16 * v < E ? expf(val[v] - vmax) : 0.f;
    part[v % R] += ex;
    chosen[v % R] += key[v] == 0u ? ex : 0.f;
  }
  const float denom = row_sum_f32(part);
  const float p = l < k ? expf(key_value(my_key) - vmax) / denom : 0.f;
  float scale = 1.f;
  if (renorm) {
#pragma unroll
    for (int r = 0; r < R; ++r) chosen[r] /= denom;
    scale = 1.f / row_sum_f32(chosen);
  }
  if (l < k) emit(l, (int)(my_at >> 16), (int)(my_at & 0xFFFFu), p * scale);
}

}  // namespace ew
