// Routing inside the grouped FFN's launch, for layer passes of few tokens: every workgroup selects the experts of all tokens, ranks
// the pairs by slot and makes its own copy of the work plan in LDS, one of them also writes what the call hands out.
//
// What it replaces is a launch of a single workgroup (selection, permutation and plan, 5 us and the gap behind it) and, in front of
// the first weights, three round trips to memory for what that launch wrote (the plan's size, the unit's entry, its rows).  The
// logits and the token's row of the expert map are two round trips, the rest stays in the CU: the selection is four tokens per wave,
// and the ranking is the scheduling wave's alone, so that one barrier is all there is.  What bounds it is that chain: from the
// kernel's entry 1.2 us to the selected experts (2.8 at 64 tokens), 1.0 (2.0) for the ranking, 0.8 until the first unit is known.
// Whole passes, us, launch of its own / so: 1 token of 64 experts, k = 6, 2048 x 1408 47.3 / 43.6; 13 tokens, 96 experts, k = 4, 1024 x 896
// 54.2 / 49.8; 64 tokens, 64 experts, k = 6, 2048 x 1408 235.0 / 230.7; the least gained where the selection is dearest, 64 tokens of 256
// experts, k = 8, 1024 x 512 138.9 / 137.2.  77 layers of 1 to 64 tokens: 1.10 in the geometric mean, none slower.
#pragma once
#include "ffn_roles.h"
#include "route_select.h"

#include <type_traits>

namespace ew {

constexpr int kRouteScan = 512;    // slots per round of the scan, eight per lane
static_assert(kPlanMaxP % kRouteScan == 0 && kRoutePairs % 256 == 0, "rounds without bounds checks");
constexpr int kRouteShared = 16;   // row chunks of shared experts at most

// What stays in LDS while the units run.
struct RoutePlan {
  uint2 entry[kRoutePairs + kRouteShared];  // chunk: slot | rows << 16, first sorted row
  uint8_t token[kRoutePairs];               // of a sorted row
};

// Ranking wave's scratch, in the rings before anything is loaded into them.
struct __align__(16) RouteScratch {
  unsigned long long tokens[kPlanMaxP];  // of a slot, a bit each
  uint32_t at[kPlanMaxP];                // first row of a slot | its first chunk << 16
  int32_t cnt[kPlanMaxP];                // rows of a slot
  uint32_t pair[kRoutePairs];            // slot | token << 16 | expert << 24
  float weight[kRoutePairs];
  uint16_t rank[kRoutePairs];            // among the pairs of its slot
};

// Selects the experts of all tokens into sc; copies > 1: also into a second one, which the weights go to.  Every thread of the block.
template <int WAVES, int FIRST>
__device__ __forceinline__ void route_select(const FfnRoute& r, int slots, RouteScratch* sc, int copies) {
  const int tid = threadIdx.x;
  for (int i = tid; i < (slots + kRouteScan - 1) / kRouteScan * kRouteScan; i += 64 * WAVES)
    for (int c = 0; c < copies; ++c) sc[c].tokens[i] = 0ull;
  // four tokens per wave; from wave FIRST on, so that the first four waves lie on different SIMDs whichever they are
  const int t0 = 4 * ((__builtin_amdgcn_readfirstlane(tid >> 6) + WAVES - FIRST) % WAVES);
  static_assert(4 * WAVES >= kRouteTokens, "one round of the waves selects for all tokens");
  auto pick = [&](auto v_tag) {
    const int mine = t0 + ((tid & 63) >> 4), t = min(mine, r.T - 1);
    group_topk<decltype(v_tag)::value, true>(r.logits + (size_t)t * r.E, r.emap + (size_t)r.aid[t] * r.E, r.E, r.k, r.renorm, copies > 1,
                                             [&](int rank, int e, int slot, float wt) {
                                               if (mine >= r.T) return;
                                               const int p = t * r.k + rank;
                                               for (int c = 0; c < copies; ++c) sc[c].pair[p] = (uint32_t)slot | (uint32_t)t << 16 | (uint32_t)e << 24;
                                               if (copies > 1) sc[1].weight[p] = wt;
                                             });
  };
  if (t0 >= r.T) return;
  if (r.E <= 16) pick(std::integral_constant<int, 1>{});
  else if (r.E <= 64) pick(std::integral_constant<int, 4>{});
  else if (r.E <= 128) pick(std::integral_constant<int, 8>{});
  else pick(std::integral_constant<int, 16>{});
}

// One wave: rows and chunks before each slot (sc.at), from the bits in sc.tokens or the counts in sc.cnt.  run: rows | chunks << 16
// before slot 0; returns those before slot P.
template <bool COUNTS, int N>
__device__ __forceinline__ uint32_t route_scan_n(int P, int bt, bool one, uint32_t run, RouteScratch& sc) {
  const int lane = threadIdx.x & 63;
  for (int s0 = 0; s0 < P; s0 += 64 * N) {
    const int s = s0 + N * lane;
    uint32_t c[N], mine = 0u;
#pragma unroll
    for (int i = 0; i < N; ++i) c[i] = COUNTS ? (uint32_t)(s + i < P ? sc.cnt[s + i] : 0) : (uint32_t)__popcll(sc.tokens[s + i]);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      c[i] |= (one ? min(c[i], 1u) : (uint32_t)dec_chunks((int)c[i], bt)) << 16;
      mine += c[i];
    }
    const uint32_t incl = wave_incl_scan_u32(mine);
    uint32_t at = run + incl - mine;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      sc.at[s + i] = at;
      at += c[i];
    }
    run += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
  }
  __builtin_amdgcn_wave_barrier();
  return run;
}
template <bool COUNTS>
__device__ __forceinline__ uint32_t route_scan(int P, int bt, bool one, uint32_t run, RouteScratch& sc) {
  if (P <= 128) return route_scan_n<COUNTS, 2>(P, bt, one, run, sc);
  return route_scan_n<COUNTS, kRouteScan / 64>(P, bt, one, run, sc);
}

// One wave: ranks the pairs (ascending inside a slot, as every permutation kernel does) and writes the plan, or with WRITE what the
// call hands out.  P: routed slots; shared experts' chunks, as many each, are the plan's first.  bt: rows per chunk at most.  Returns
// the number of chunks.
// A lane is a token: its slots are distinct, so a bit per token and slot, ORed in LDS, holds a slot's rows in order.  A wave alone on
// its SIMD waits for every LDS access and nearly every instruction, so the accesses go in batches without bounds checks.  (Ranked 64
// pairs at a time by comparing slots bit by bit, as the other kernels do, 384 pairs took 5.2 us, 6 pairs 1.3; that way is left for a
// token with a repeated slot, that is a map that sends two experts to one.)
template <bool WRITE>
__device__ __forceinline__ int route_rank(const FfnRoute& r, int P, int bt, RouteScratch& sc, RoutePlan& plan) {
  const int lane = threadIdx.x & 63, T = r.T, k = r.k, S = r.S, n = T * k;
  if (lane < T)
    for (int j0 = 0; j0 < k; j0 += 4) {
      uint32_t s[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) s[j] = sc.pair[min(lane * k + j0 + j, n - 1)] & (kPlanMaxP - 1);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (j0 + j < k) __hip_atomic_fetch_or(&sc.tokens[s[j]], 1ull << lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  __builtin_amdgcn_wave_barrier();
  const int sh_chunks = T <= bt ? 1 : dec_chunks(T, bt);
  const uint32_t first = (uint32_t)(S * sh_chunks) << 16;
  bool one = sh_chunks == 1;                       // no slot has more rows than a chunk takes
  uint32_t end = route_scan<false>(P, bt, one, first, sc);
  const bool repeated = (int)(end & 0xFFFFu) != n;  // bits that fell together
  if (repeated) {
    one = false;
    for (int s = lane; s < P; s += 64) sc.cnt[s] = 0;
    __builtin_amdgcn_wave_barrier();
    for (int base = 0; base < n; base += 64) {
      const int i = base + lane;
      const bool ok = i < n;
      const uint32_t s = ok ? sc.pair[i] & (kPlanMaxP - 1) : 0u;
      const unsigned long long peers = match_any(s, r.bits, __ballot(ok));
      const int before = __popcll(peers & lanemask_lt()), old = ok ? sc.cnt[s] : 0;
      __builtin_amdgcn_wave_barrier();
      if (ok) {
        sc.rank[i] = (uint16_t)(old + before);
        if (before == 0) sc.cnt[s] = old + __popcll(peers);
      }
      __builtin_amdgcn_wave_barrier();
    }
    end = route_scan<true>(P, bt, false, first, sc);
  }
  for (int i0 = lane; i0 - lane < n; i0 += 256) {
    uint32_t v[4], at[4];
    unsigned long long m[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = sc.pair[i0 + 64 * q];  // (what lies behind the last pair is not used)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      at[q] = sc.at[v[q] & (kPlanMaxP - 1)];
      m[q] = sc.tokens[v[q] & (kPlanMaxP - 1)];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = i0 + 64 * q;
      if (i >= n) continue;
      const uint32_t s = v[q] & (kPlanMaxP - 1), t = (v[q] >> 16) & 63u;
      int c = __popcll(m[q]), rk = __popcll(m[q] & ((1ull << t) - 1ull));
      if (repeated) {
        c = sc.cnt[s];
        rk = sc.rank[i];
      }
      const int row = (int)(at[q] & 0xFFFFu) + rk;
      if constexpr (WRITE) {
        r.ids[i] = (int)(v[q] >> 24);
        r.w[i] = sc.weight[i];
        r.slot[i] = (int)s;
        r.por[row] = i;
        r.rop[i] = row;
      } else {
        plan.token[row] = (uint8_t)t;
        int j = 0, bts = bt;
        if (!one && c > bt) {
          const int nch = dec_chunks(c, bt);
          bts = ((c + nch - 1) / nch + 15) & ~15;
          j = rk / bts;
        }
        if (rk == j * bts) plan.entry[(at[q] >> 16) + j] = make_uint2(s | (uint32_t)min(bts, c - j * bts) << 16, (uint32_t)row);
      }
    }
  }
  if constexpr (WRITE) {
    for (int s = lane; s < P; s += 64) {
      r.counts[s] = repeated ? sc.cnt[s] : __popcll(sc.tokens[s]);
      r.offsets[s] = (int)(sc.at[s] & 0xFFFFu);
    }
    if (lane == 0) r.offsets[P] = n;
  } else if (lane < S * sh_chunks) {
    const int s = one ? lane : lane / sh_chunks, j = lane - s * sh_chunks, bts = one ? bt : ((T + sh_chunks - 1) / sh_chunks + 15) & ~15;
    plan.entry[lane] = make_uint2((uint32_t)(P + s) | (uint32_t)min(bts, T - j * bts) << 16, (uint32_t)(n + s * T + j * bts));
  }
  return (int)(end >> 16);
}

}  // namespace ew
