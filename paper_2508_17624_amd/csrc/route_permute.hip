// Router top-k, batched rerouting and stable token permutation for gfx950 (wave64).
//
// Paper Sec. 2.1 (router top-k; dispatch = replicate, permute, group by expert id), Sec. 4.1
// (TopK'(x) = {Pi[A(x), j] : j in TopK(x)}) and Sec. 4.3 (rerouting fused into one kernel).
//
// Design for CDNA4:
//  * top-k: sixteen lanes per token, so four tokens per wave (up to 256 experts and k = 16); beyond
//    that one wave per token.  Each logit becomes an order-preserving 32-bit key (ties go to the
//    lower index).
//  * rerouting is a lookup in the expert map, fused into whichever kernel first touches the ids: it never costs a launch or a pass over
//    memory of its own.  (The histogram of given ids stages the map in LDS; where the selection is fused the token's row of it is read
//    from L2 while the selection runs.)
//  * permutation is a stable counting sort by slot.  Order inside a slot must be ascending
//    pair index, so no atomic cursors: every wave ranks a contiguous run of pairs 64 at a time
//    with a ballot-built peer mask (rank = popcount of lower peers) and a wave-private LDS
//    counter; runs are stitched by exclusive scans over waves (LDS) and over blocks (global).
//  * small batches (decode): ONE single-block kernel does top-k, lookup, histogram, scan and scatter
//    without leaving the CU (above 64 tokens, and below for many experts, a multi-block top-k + lookup kernel runs first and that
//    block receives slots).  Larger ones use two kernels, per-block histogram (fused with top-k
//    and lookup) and ranked scatter; the largest have a column scan between them.
//  * the grouped FFN's work plan, if asked for, never is a launch of its own: the single block goes
//    on to build it, and the scatter's launch has one more block for it.
#include "ew_internal.h"
#include "route_select.h"

#include <atomic>
#include <type_traits>

namespace {

using ew::group_topk;
using ew::lanemask_lt;
using ew::match_any;
using ew::order_key;

constexpr int kWave = 64;
constexpr int kMaxP = 2048;          // slots supported by the permutation kernels
constexpr int kMaxE = 1024;          // experts supported by the top-k kernels
constexpr int kSmallPairs = 4096;    // single-block path: capacity of its LDS arrays (T*k at most this)
int g_small_pairs = 2048;            // single-block path is used up to this many pairs (tunable, <= kSmallPairs)
constexpr int kSelectTokens = 64;    // single-block path: the selection can join it up to this many tokens (joins_selection)
constexpr int kSmallCnt = 12288;     // single-block path: waves * P at most this (uint16 counters)
constexpr int kBigThreads = 512;     // multi-block path: threads per block
constexpr int kBigWaves = kBigThreads / kWave;
constexpr int kHistThreads = 1024;   // the histogram kernel is a plain stream: more waves per block hide its latency
constexpr int kBigPairs = 12288;     // multi-block path: pairs per block at most this
constexpr int kBigSteps = kBigPairs / kBigWaves / kWave;  // 64-pair steps per wave = 24
constexpr int kDirectPairs = 1 << 18;  // up to this many pairs the scatter sums the histogram's columns itself (chunk_tokens)
constexpr int kDirectBlocks = 128;
constexpr int kMapLds = 8192;        // expert-map entries staged in LDS at most

// ------------------------------------------------------------------------------------------
// wave primitives
// Wave-wide fp32 sum, result broadcast to every lane.  Row-local Hillis-Steele steps with DPP
// row_shr 1/2/4/8 leave each 16-lane row's total in its last lane; row_bcast15 / row_bcast31
// carry the totals across rows into lane 63.  Fixed order, so the sum is deterministic.
__device__ __forceinline__ float wave_sum_f32(float v) {
#define EW_DPP_ADD(ctrl, rmask)                                                                          \
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, rmask, 0xf, false))
  EW_DPP_ADD(0x111, 0xf);  // row_shr:1
  EW_DPP_ADD(0x112, 0xf);  // row_shr:2
  EW_DPP_ADD(0x114, 0xf);  // row_shr:4
  EW_DPP_ADD(0x118, 0xf);  // row_shr:8
  EW_DPP_ADD(0x142, 0xa);  // row_bcast:15 into rows 1 and 3
  EW_DPP_ADD(0x143, 0xc);  // row_bcast:31 into rows 2 and 3
#undef EW_DPP_ADD
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

__device__ __forceinline__ int wave_incl_scan_i32(int v) { return (int)ew::wave_incl_scan_u32((uint32_t)v); }

// The `n` lowest set bits of m (n <= popcount(m)).
__device__ __forceinline__ unsigned long long lowest_bits(unsigned long long m, int n) {
  unsigned long long t = 0;
  for (int i = 0; i < n; ++i) {
    t |= m & (0ull - m);
    m &= m - 1;
  }
  return t;
}

// One wave selects the top-k of one token's E logits and calls emit(rank, expert, weight) once
// per selected expert, from the lane that holds it (rank 0 = largest logit; equal logits rank by
// lower expert index).  Lane l holds experts l, l+64, ... (VPL per lane, E <= 64*VPL).
//
// Selection is a radix select over the 32 bits of the order-preserving key, most significant
// first: a ballot splits the still-tied candidates by the current bit; if the ones alone fill
// what is still needed they become the candidates, otherwise they are all taken.  What is left
// at the end ties exactly with the k-th value and is filled up from the lowest index.  All of
// that is wave-uniform mask arithmetic on the scalar unit: no cross-lane data movement.
template <int VPL, typename Emit>
__device__ __forceinline__ void wave_topk(const float* __restrict__ row, int E, int k, int renorm, Emit emit) {
  const int lane = threadIdx.x & (kWave - 1);
  float val[VPL];
  uint32_t key[VPL];
  unsigned long long cand[VPL], sel[VPL];
#pragma unroll
  for (int v = 0; v < VPL; ++v) {
    const int e = lane + v * kWave;
    const bool ok = e < E;
    val[v] = ok ? row[e] : 0.f;
    key[v] = ok ? order_key(val[v]) : 0u;
    cand[v] = __ballot(ok);
    sel[v] = 0ull;
  }
  int need = k;
  for (int b = 31; b >= 0; --b) {
    unsigned long long ones[VPL];
    int c = 0;
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
      ones[v] = __ballot((key[v] >> b) & 1u) & cand[v];
      c += __popcll(ones[v]);
    }
    if (c >= need) {
#pragma unroll
      for (int v = 0; v < VPL; ++v) cand[v] = ones[v];
    } else {
      need -= c;
#pragma unroll
      for (int v = 0; v < VPL; ++v) {
        sel[v] |= ones[v];
        cand[v] &= ~ones[v];
      }
    }
  }
#pragma unroll
  for (int v = 0; v < VPL; ++v) {  // ties with the k-th value: lowest expert index first
    const int have = __popcll(cand[v]);
    const int take = have < need ? have : need;
    sel[v] |= lowest_bits(cand[v], take);
    need -= take;
  }
  // rank of every selected value among the selected ones
  int rank[VPL];
#pragma unroll
  for (int v = 0; v < VPL; ++v) rank[v] = 0;
#pragma unroll
  for (int u = 0; u < VPL; ++u) {
    unsigned long long m = sel[u];
    while (m) {
      const int src = __ffsll((long long)m) - 1;
      m &= m - 1;
      const uint32_t okey = (uint32_t)__builtin_amdgcn_readlane((int)key[u], src);
      const int oe = src + u * kWave;
#pragma unroll
      for (int v = 0; v < VPL; ++v) {
        const int e = lane + v * kWave;
        rank[v] += (okey > key[v] || (okey == key[v] && oe < e)) ? 1 : 0;
      }
    }
  }
  // softmax over all E logits: max = the rank-0 value
  float vmax = 0.f;
#pragma unroll
  for (int v = 0; v < VPL; ++v) {
    const unsigned long long top = __ballot(((sel[v] >> lane) & 1ull) && rank[v] == 0);
    if (top) vmax = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(val[v]), __ffsll((long long)top) - 1));
  }
  float ex[VPL], part = 0.f, spart = 0.f;
#pragma unroll
  for (int v = 0; v < VPL; ++v) {
    ex[v] = (lane + v * kWave < E) ? expf(val[v] - vmax) : 0.f;
    part += ex[v];
    if ((sel[v] >> lane) & 1ull) spart += ex[v];
  }
  const float denom = wave_sum_f32(part);
  float scale = 1.f;
  if (renorm) scale = 1.f / wave_sum_f32(spart / denom);
#pragma unroll
  for (int v = 0; v < VPL; ++v)
    if ((sel[v] >> lane) & 1ull) emit(rank[v], lane + v * kWave, ex[v] / denom * scale);
}

// Top-k of tokens first, first + 1, ... below end, as many as a wave takes at once: V > 0: sixteen lanes per token with V logits
// each, V < 0: all 64 lanes on one token with -V logits each.  emit(token, rank, expert, slot, weight); REROUTE: the slots come
// from the expert map, otherwise they mean nothing.
template <int V>
constexpr int kTokensPerWave = V > 0 ? 4 : 1;
template <int V, bool REROUTE, typename Emit>
__device__ __forceinline__ void wave_select(const float* __restrict__ logits, const int32_t* __restrict__ aid, const int32_t* __restrict__ emap,
                                            int first, int end, int E, int k, int renorm, Emit emit) {
  if constexpr (V < 0) {
    const int32_t* maprow = REROUTE ? emap + (size_t)aid[first] * E : nullptr;
    wave_topk<-V>(logits + (size_t)first * E, E, k, renorm, [&](int rank, int e, float wt) { emit(first, rank, e, REROUTE ? maprow[e] : 0, wt); });
  } else {
    const unsigned mine = (unsigned)first + ((threadIdx.x & (kWave - 1)) >> 4);  // (may lie past 2^31)
    const int t = (int)mine, row = (int)min(mine, (unsigned)end - 1);
    group_topk<V, REROUTE>(logits + (size_t)row * E, REROUTE ? emap + (size_t)aid[row] * E : nullptr, E, k, renorm, true,
                           [&](int rank, int e, int slot, float wt) {
                             if (mine < (unsigned)end) emit(t, rank, e, slot, wt);
                           });
  }
}

// Stages the expert map in LDS when it fits; returns the pointer lookups should use.
__device__ __forceinline__ const int32_t* stage_map(const int32_t* __restrict__ emap, int32_t* s_map, int entries) {
  if (entries > kMapLds) return emap;
  for (int i = threadIdx.x; i < entries; i += blockDim.x) s_map[i] = emap[i];
  return s_map;
}

// Exclusive scans of two values per thread over the block's kBigThreads threads at once (thread order); ta, tb = the
// totals.  s_w: 2 * kBigWaves ints of LDS.  Contains one barrier; s_w may be reused after the next one.
__device__ __forceinline__ void block_exscan2(int a, int b, int& ea, int& eb, int& ta, int& tb, int32_t* s_w) {
  const int wave = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
  const int ia = wave_incl_scan_i32(a), ib = wave_incl_scan_i32(b);
  if (lane == kWave - 1) {
    s_w[2 * wave] = ia;
    s_w[2 * wave + 1] = ib;
  }
  __syncthreads();
  int pa = 0, pb = 0;
  ta = 0;
  tb = 0;
#pragma unroll
  for (int w = 0; w < kBigWaves; ++w) {
    const int xa = s_w[2 * w], xb = s_w[2 * w + 1];
    if (w < wave) { pa += xa; pb += xb; }
    ta += xa;
    tb += xb;
  }
  ea = pa + ia - a;
  eb = pb + ib - b;
}

// Exclusive scan of one value per thread over the block (thread order).  s_w: an int per wave.  Contains one barrier.  The wave totals
// are read by the lanes at once and scanned there: a loop over them is a chain of LDS round trips, 0.4 to 0.6 us with 16 waves.
__device__ __forceinline__ int block_exscan(int a, int32_t* s_w) {
  const int wave = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1), nwaves = blockDim.x / kWave;
  const int ia = wave_incl_scan_i32(a);
  if (lane == kWave - 1) s_w[wave] = ia;
  __syncthreads();
  const int totals = wave_incl_scan_i32(lane < nwaves ? s_w[lane] : 0);
  const int before = wave ? __builtin_amdgcn_readlane(totals, __builtin_amdgcn_readfirstlane(wave) - 1) : 0;
  return before + ia - a;
}

// Exclusive scan of v[0..P) in place by wave 0 (P <= kMaxP); v[P] = total.  Needs barriers around.
__device__ __forceinline__ void wave0_exscan(int32_t* v, int P) {
  if (threadIdx.x >= kWave) return;
  const int lane = threadIdx.x;
  const int per = (P + kWave - 1) / kWave;
  const int lo = lane * per, hi = min(P, lo + per);
  int sum = 0;
  for (int i = lo; i < hi; ++i) sum += v[i];
  int run = wave_incl_scan_i32(sum) - sum;
  for (int i = lo; i < hi; ++i) {
    const int c = v[i];
    v[i] = run;
    run += c;
  }
  const int total = __shfl(run, kWave - 1, kWave);
  if (lane == 0) v[P] = total;
}

// ------------------------------------------------------------------------------------------
// Router top-k, four waves per block.  REROUTE: with the rerouting fused in (Sec. 4.3: the lookup rides on the kernel that
// produces the ids), over as many blocks as the batch needs: the first half of the decode-sized path, whose second half (k_small
// with slots given) is a single block.  The grid strides over the tokens: a launch takes less than 2^32 threads in a dimension,
// which one wave per token would pass at 2^26 tokens.  The stride is that of the largest grid; a smaller one ends after its first step.
// (gridDim lies behind the 64 bytes of arguments, in a line of its own that every wave would wait for: 0.2 to 0.4 us of 4 to 7.)
constexpr int kRouteBlocks = 1 << 20;
template <int V, bool REROUTE>
__global__ __launch_bounds__(256) void k_route(const float* __restrict__ logits, const int32_t* __restrict__ aid,
                                               const int32_t* __restrict__ emap, int T, int E, int k, int renorm,
                                               int32_t* __restrict__ ids, float* __restrict__ w, int32_t* __restrict__ slot_ids) {
  for (unsigned first = (blockIdx.x * 4 + threadIdx.x / kWave) * kTokensPerWave<V>; first < (unsigned)T; first += kRouteBlocks * 4u * kTokensPerWave<V>)
    wave_select<V, REROUTE>(logits, aid, emap, (int)first, T, E, k, renorm, [&](int t, int rank, int e, int slot, float wt) {
      const size_t p = (size_t)t * k + rank;
      ids[p] = e;
      w[p] = wt;
      if constexpr (REROUTE) slot_ids[p] = slot;
    });
}

// Plan request of a permutation call: the grouped FFN's work plan is written too (plan == nullptr: not asked for).
struct PlanReq {
  int32_t* plan;
  int S;
  ew::FfnPlanShape shape;
};

// Block 0 of a scatter launch that was asked for a plan: builds it from the counts while the other blocks scatter.  Scatter and
// plan, us, as two launches before / now: 512 tokens 5.7 + 3.7 / 5.1; 8192 tokens 7.7 + 10.3 / 9.2.  T tokens, n pairs; a block of 512 threads; lds: the scatter's sorted-pairs array.
__device__ __forceinline__ void plan_block(const int32_t* counts, int T, int n, int P, const PlanReq& fp, int32_t* s_w, void* lds) {
  int rows[4], first[4], sum = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int sl = 4 * (int)threadIdx.x + i;
    rows[i] = sl < P ? counts[sl] : 0;
    sum += rows[i];
  }
  int at = block_exscan(sum, s_w);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    first[i] = at;
    at += rows[i];
  }
  ew::ffn_plan_build(rows, first, P, fp.S, T, n, fp.shape, fp.plan, *reinterpret_cast<ew::FfnPlanLds*>(lds));
}

// ------------------------------------------------------------------------------------------
// Single-block path (decode-sized batches): ids -> slots, ranking, scan, scatter and, if asked for, the FFN's work plan in one
// launch.  V = 0: ids are given (emap == nullptr: they are slots already, written by k_route), otherwise the selection
// (wave_select) runs here too.  What bounds it is the chain of dependent steps, each a memory round trip or a barrier; so only the
// waves that a batch gives 64 pairs rank, the scans run on DPP instead of through LDS, and one scan over all threads makes the
// offsets.  Selection to plan, us, as two launches before / now: 1 token 8.9 / 5.7, 64 tokens 10.2 / 7.7.
// run = pairs per ranking wave, a multiple of 64; nrank = ranking waves, ceil(T k / run); per = slots per thread of the scan (both
// from the host: an integer division is a few dozen dependent instructions).  Ids given, us, with the waves' totals summed in a loop
// and both divisions here / now: 256 tokens of k = 2 on 128 slots 4.4 / 3.6, 1024 6.6 / 5.7; 341 of k = 6 on 384 7.1 / 6.3.
template <int V>
__global__ __launch_bounds__(1024) void k_small(const float* __restrict__ logits, const int32_t* __restrict__ ids_in,
                                                const int32_t* __restrict__ aid, const int32_t* __restrict__ emap,
                                                int T, int E, int k, int P, int renorm, int bits, int run, int nrank, int per,
                                                int32_t* __restrict__ ids_out, float* __restrict__ w_out,
                                                int32_t* __restrict__ slot_ids, int32_t* __restrict__ counts,
                                                int32_t* __restrict__ offsets, int32_t* __restrict__ pair_of_row,
                                                int32_t* __restrict__ row_of_pair, PlanReq fp) {
  struct Perm {
    uint16_t slot[kSmallPairs];
    uint16_t rank[kSmallPairs];
    uint16_t cnt[kSmallCnt];
    int32_t off[kMaxP + 1];
    int32_t w[1024 / kWave];
  };
  __shared__ union Lds {
    Perm perm;
    ew::FfnPlanLds plan;  // after the scatter
  } lds;
  uint16_t (&s_slot)[kSmallPairs] = lds.perm.slot;
  uint16_t (&s_rank)[kSmallPairs] = lds.perm.rank;
  uint16_t (&s_cnt)[kSmallCnt] = lds.perm.cnt;
  int32_t (&s_off)[kMaxP + 1] = lds.perm.off;
  const int tid = threadIdx.x, nthreads = blockDim.x;
  const int wave = tid / kWave, lane = tid & (kWave - 1), nwaves = nthreads / kWave;
  const int n = T * k;

  for (int i = tid; i < nrank * P; i += nthreads) s_cnt[i] = 0;

  // A: ids (top-k or given) -> slots through the expert map
  if constexpr (V != 0) {
    for (int first = wave * kTokensPerWave<V>; first < T; first += nwaves * kTokensPerWave<V>)
      wave_select<V, true>(logits, aid, emap, first, T, E, k, renorm, [&](int t, int rank, int e, int s, float wt) {
        const int p = t * k + rank;
        ids_out[p] = e;
        w_out[p] = wt;
        slot_ids[p] = s;
        s_slot[p] = (uint16_t)s;
      });
  } else {
    for (int p = tid; p < n; p += nthreads) {
      int s;
      if (emap) {
        s = emap[(size_t)aid[p / k] * E + ids_in[p]];
        slot_ids[p] = s;
      } else {
        s = ids_in[p];
      }
      s_slot[p] = (uint16_t)s;
    }
  }
  __syncthreads();

  // B: wave w ranks its run [w*run, (w+1)*run) 64 pairs at a time
  {
    uint16_t* cnt = s_cnt + (size_t)wave * P;
    const int lo = wave * run, hi = min(n, lo + run);
    const unsigned long long lt = lanemask_lt();
    for (int base = lo; base < hi; base += kWave) {
      const int i = base + lane;
      const bool valid = i < hi;
      const uint32_t s = valid ? s_slot[i] : 0u;
      const unsigned long long peers = match_any(s, bits, __ballot(valid));
      const int before = __popcll(peers & lt);
      uint16_t old = 0;
      if (valid) old = cnt[s];
      __builtin_amdgcn_wave_barrier();
      if (valid) {
        s_rank[i] = (uint16_t)(old + before);
        if (before == 0) cnt[s] = (uint16_t)(old + __popcll(peers));
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
  __syncthreads();

  // C: per slot, exclusive scan over the ranking waves (in place); then over the slots, each thread taking `per` of them in a row
  const int s0 = tid * per;
  int mine = 0;
  for (int s = s0; s < min(P, s0 + per); ++s) {
    int tot = 0;
    for (int w = 0; w < nrank; ++w) {
      const int c = s_cnt[(size_t)w * P + s];
      s_cnt[(size_t)w * P + s] = (uint16_t)tot;
      tot += c;
    }
    s_off[s] = tot;
    mine += tot;
  }
  int at = block_exscan(mine, lds.perm.w);
  for (int s = s0; s < min(P, s0 + per); ++s) {
    const int tot = s_off[s];
    s_off[s] = at;
    offsets[s] = at;
    counts[s] = tot;
    at += tot;
  }
  if (tid == 0) {
    s_off[P] = n;
    offsets[P] = n;
  }
  __syncthreads();

  // D: scatter
  for (int p = tid; p < n; p += nthreads) {
    const int s = s_slot[p];
    const int dest = s_off[s] + s_cnt[(size_t)(p / run) * P + s] + s_rank[p];
    pair_of_row[dest] = p;
    if (row_of_pair) row_of_pair[p] = dest;
  }

  // E: the work plan of the grouped FFN call that consumes counts / offsets, if asked for (block of >= 512 threads)
  if (fp.plan) {
    int rows[4] = {0, 0, 0, 0}, first[4] = {0, 0, 0, 0};   // this thread's four slots, taken from LDS before the plan reuses it
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int sl = 4 * tid + i;
      if (tid < 512 && sl < P) {
        first[i] = s_off[sl];
        rows[i] = s_off[sl + 1] - s_off[sl];
      }
    }
    __syncthreads();  // the permutation's LDS arrays are dead
    ew::ffn_plan_build(rows, first, P, fp.S, T, n, fp.shape, fp.plan, lds.plan);
  }
}

// ------------------------------------------------------------------------------------------
// Multi-block path, kernel 1: block b owns tokens [b*cht, (b+1)*cht).  ids (top-k or given) ->
// slots (written out) -> LDS histogram -> hist[b][0..P).
template <int V>
__global__ __launch_bounds__(kHistThreads) void k_hist(const float* __restrict__ logits, const int32_t* __restrict__ ids_in,
                                                      const int32_t* __restrict__ aid, const int32_t* __restrict__ emap,
                                                      int T, int E, int k, int P, int map_entries, int renorm, int cht,
                                                      int32_t* __restrict__ ids_out, float* __restrict__ w_out,
                                                      int32_t* __restrict__ slot_ids, int32_t* __restrict__ hist) {
  __shared__ int32_t s_hist[kMaxP];
  const int tid = threadIdx.x;
  const int t0 = blockIdx.x * cht, t1 = min(T, t0 + cht);
  for (int i = tid; i < P; i += blockDim.x) s_hist[i] = 0;
  if constexpr (V != 0) {
    __syncthreads();
    const int step = blockDim.x / kWave * kTokensPerWave<V>;
    for (int first = t0 + tid / kWave * kTokensPerWave<V>; first < t1; first += step) {
      wave_select<V, true>(logits, aid, emap, first, t1, E, k, renorm, [&](int t, int rank, int e, int s, float wt) {
        const size_t p = (size_t)t * k + rank;
        ids_out[p] = e;
        w_out[p] = wt;
        slot_ids[p] = s;
        atomicAdd(&s_hist[s], 1);
      });
    }
  } else {
    __shared__ int32_t s_map[kMapLds];
    const int32_t* map = stage_map(emap, s_map, map_entries);
    __syncthreads();
    // four pairs per thread and pass, all loads of a pass issued before their first use; the
    // token of local pair q is floor((q + 0.5) / k), exact in fp32 for q < 2^14 and k <= 64
    const size_t p0 = (size_t)t0 * k;
    const int n = (t1 - t0) * k;
    const float inv_k = 1.0f / (float)k;
    for (int q0 = tid; q0 < n; q0 += 4 * kHistThreads) {
      int idv[4], av[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int q = q0 + j * kHistThreads;
        const bool ok = q < n;
        idv[j] = ok ? ids_in[p0 + q] : 0;
        av[j] = ok ? aid[t0 + (int)(((float)q + 0.5f) * inv_k)] : 0;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int q = q0 + j * kHistThreads;
        if (q < n) {
          const int s = map[av[j] * E + idv[j]];
          slot_ids[p0 + q] = s;
          atomicAdd(&s_hist[s], 1);
        }
      }
    }
  }
  __syncthreads();
  int32_t* out = hist + (size_t)blockIdx.x * P;
  for (int i = tid; i < P; i += blockDim.x) out[i] = s_hist[i];
}

// Kernel 2: exclusive scan down the columns of hist[nb][P] in place; counts[s] = column total.
// Block bx owns 16 columns; thread (c = tid%16, g = tid/16) owns rows [g*rpg, (g+1)*rpg) and keeps them in registers
// when there are at most kScanRows of them (nb <= 512), so that the matrix is read once; wave w then scans the 64 group
// sums of column w with lane shuffles.
constexpr int kScanCols = 16;
constexpr int kScanGroups = 64;
constexpr int kScanRows = 8;
static_assert(kScanGroups == kWave && kScanCols * kScanGroups / kWave == kScanCols, "one wave per column in the middle step");
__global__ __launch_bounds__(kScanCols * kScanGroups) void k_colscan(int32_t* __restrict__ hist, int nb, int P,
                                                                     int32_t* __restrict__ counts) {
  __shared__ int32_t s_part[kScanCols][kScanGroups + 1];
  const int c = threadIdx.x % kScanCols, g = threadIdx.x / kScanCols;
  const int col = blockIdx.x * kScanCols + c;
  const int rpg = (nb + kScanGroups - 1) / kScanGroups;
  const int r0 = g * rpg, r1 = min(nb, r0 + rpg);
  const bool in_regs = rpg <= kScanRows;  // block-uniform
  int v[kScanRows];
  int sum = 0;
  if (in_regs) {
#pragma unroll
    for (int j = 0; j < kScanRows; ++j) {
      v[j] = (col < P && r0 + j < r1) ? hist[(size_t)(r0 + j) * P + col] : 0;
      sum += v[j];
    }
  } else if (col < P) {
    for (int r = r0; r < r1; ++r) sum += hist[(size_t)r * P + col];
  }
  s_part[c][g] = sum;
  __syncthreads();
  {
    const int w = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
    const int x = s_part[w][lane];
    const int inc = wave_incl_scan_i32(x);
    s_part[w][lane] = inc - x;
    if (lane == kWave - 1 && blockIdx.x * kScanCols + w < P) counts[blockIdx.x * kScanCols + w] = inc;
  }
  __syncthreads();
  int run = s_part[c][g];
  if (in_regs) {
#pragma unroll
    for (int j = 0; j < kScanRows; ++j) {
      if (col < P && r0 + j < r1) hist[(size_t)(r0 + j) * P + col] = run;
      run += v[j];
    }
  } else if (col < P) {
    for (int r = r0; r < r1; ++r) {
      const int x = hist[(size_t)r * P + col];
      hist[(size_t)r * P + col] = run;
      run += x;
    }
  }
}

// The wave's slot ids, one pair per lane and step (pair lo + 64 i + lane), all loads issued before any is used:
// one memory round trip instead of one per step.
__device__ __forceinline__ void load_pairs(const int32_t* __restrict__ slot_ids, size_t p0, int lo, int hi, int steps,
                                           uint32_t (&packed)[kBigSteps]) {
  const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
  for (int i = 0; i < kBigSteps; ++i) {
    const int idx = lo + i * kWave + lane;
    packed[i] = (i < steps && idx < hi) ? (uint32_t)slot_ids[p0 + idx] : 0u;
  }
}

// Ranks the wave's pairs [lo, hi), 64 consecutive pairs per step: packed[i] = slot on entry and
// slot | rank among the wave's earlier pairs of that slot << 12 | valid << 31 on return.  cnt: the wave's counter per
// slot (zeroed).  MASKS: lanes of a step that hold the same slot find each other through a 64-bit lane mask per slot in
// LDS (`mask`, zeroed): every lane ORs its bit in (commutative, so the result does not depend on the order the
// hardware resolves the conflicts in), reads the mask back, and the first lane of each group clears it again.
// Otherwise the lanes compare keys bit by bit with ballots (about six times the vector instructions).
template <bool MASKS>
__device__ __forceinline__ void rank_pairs(int lo, int hi, int steps, int bits, uint16_t* cnt, unsigned long long* mask,
                                           uint32_t (&packed)[kBigSteps]) {
  const int lane = threadIdx.x & (kWave - 1);
  const unsigned long long lt = lanemask_lt();
#pragma unroll
  for (int i = 0; i < kBigSteps; ++i) {
    if (i >= steps) { packed[i] = 0u; continue; }
    const int idx = lo + i * kWave + lane;
    const bool valid = idx < hi;
    const uint32_t s = packed[i];
    unsigned long long peers;
    if constexpr (MASKS) {
      if (valid) __hip_atomic_fetch_or(&mask[s], 1ull << lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      __builtin_amdgcn_wave_barrier();
      peers = valid ? __hip_atomic_load(&mask[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) : 0ull;
    } else {
      peers = match_any(s, bits, __ballot(valid));
    }
    const int before = __popcll(peers & lt);
    uint32_t old = 0;
    if (valid) old = cnt[s];
    __builtin_amdgcn_wave_barrier();
    if (valid && before == 0) {
      cnt[s] = (uint16_t)(old + __popcll(peers));
      if constexpr (MASKS) mask[s] = 0ull;
    }
    __builtin_amdgcn_wave_barrier();
    packed[i] = s | ((old + before) << 12) | (valid ? 0x80000000u : 0u);
  }
}

// Kernel 3: block b ranks its pairs and scatters them.  base[b][s] (scanned hist) + offsets[s]
// is where block b's first pair of slot s goes.  row_of_pair is written in pair order straight
// from the ranking.  pair_of_row would be a 4-byte store per lane to 64 different cache lines that
// way, so the block first sorts its pairs by slot in LDS and then writes each slot's run with
// consecutive lanes on consecutive addresses.  MAXP sizes the LDS tables (P <= MAXP).
template <int MAXP>
__global__ __launch_bounds__(kBigThreads) void k_scatter(const int32_t* __restrict__ slot_ids, const int32_t* __restrict__ counts,
                                                         const int32_t* __restrict__ base, int T, int k, int P, int bits, int cht,
                                                         int run, int32_t* __restrict__ offsets, int32_t* __restrict__ pair_of_row,
                                                         int32_t* __restrict__ row_of_pair, PlanReq fp) {
  __shared__ uint16_t s_cnt[kBigWaves * MAXP];
  __shared__ int32_t s_off[MAXP + 1];    // first row of the block's pairs of slot s
  __shared__ int32_t s_loc[MAXP + 1];    // first position of slot s in the block's sorted order
  __shared__ __align__(16) uint32_t s_sorted[kBigPairs];  // slot << 16 | pair index inside the block, sorted by slot
  static_assert(sizeof(ew::FfnPlanLds) <= sizeof(s_sorted), "a plan is built in the sorted-pairs array");
  if (fp.plan && blockIdx.x == 0) {
    plan_block(counts, T, T * k, P, fp, s_off, s_sorted);
    return;
  }
  const int block = blockIdx.x - (fp.plan ? 1 : 0);
  const int tid = threadIdx.x;
  const int wave = tid / kWave, lane = tid & (kWave - 1);
  const int t0 = block * cht, t1 = min(T, t0 + cht);
  const size_t p0 = (size_t)t0 * k;
  const int n = (t1 - t0) * k;                                    // pairs of this block, <= kBigPairs
  const int lo = wave * run, hi = min(n, lo + run);               // run: pairs per wave, a multiple of 64
  const int steps = run / kWave;                                  // <= kBigSteps
  uint32_t packed[kBigSteps];                                     // slot | rank << 12 | valid << 31
  load_pairs(slot_ids, p0, lo, hi, steps, packed);
  const int32_t* mybase = base + (size_t)block * P;
  int32_t base_v[MAXP / kBigThreads];                             // this block's row of the scanned histogram
#pragma unroll
  for (int j = 0; j < MAXP / kBigThreads; ++j) {
    const int sl = tid + j * kBigThreads;
    base_v[j] = sl < P ? mybase[sl] : 0;
  }
  // Lanes of a step that hold the same slot find each other through a 64-bit lane mask per (wave,
  // slot) in LDS: every lane ORs its bit in (commutative, so the result does not depend on the
  // order the hardware resolves the conflicts in), reads the mask back, and the first lane of
  // each group clears it again.  It needs waves * P * 8 bytes, which the sorted-pairs array lends
  // while the ranking runs; the table for P > 512 would not fit, there the lanes compare keys bit
  // by bit with ballots instead (about six times the vector instructions).
  constexpr bool kMasks = (size_t)kBigWaves * MAXP * 8 <= sizeof(s_sorted);
  unsigned long long* s_mask = reinterpret_cast<unsigned long long*>(s_sorted);
  for (int i = tid; i < kBigWaves * P; i += kBigThreads) {
    s_cnt[i] = 0;
    if (kMasks) s_mask[i] = 0ull;
  }
  for (int i = tid; i < P; i += kBigThreads) s_off[i] = counts[i];
  __syncthreads();
  wave0_exscan(s_off, P);
  __syncthreads();
  if (block == 0)
    for (int i = tid; i <= P; i += kBigThreads) offsets[i] = s_off[i];

  rank_pairs<kMasks>(lo, hi, steps, bits, s_cnt + (size_t)wave * P, s_mask + (size_t)wave * P, packed);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < MAXP / kBigThreads; ++j) {
    const int s = tid + j * kBigThreads;
    if (s < P) {
      int tot = 0;
#pragma unroll
      for (int w = 0; w < kBigWaves; ++w) {
        const int c = s_cnt[(size_t)w * P + s];
        s_cnt[(size_t)w * P + s] = (uint16_t)tot;
        tot += c;
      }
      s_off[s] += base_v[j];
      s_loc[s] = tot;
    }
  }
  __syncthreads();
  wave0_exscan(s_loc, P);
  __syncthreads();
  const uint16_t* cntx = s_cnt + (size_t)wave * P;
#pragma unroll
  for (int i = 0; i < kBigSteps; ++i) {
    if (packed[i] & 0x80000000u) {
      const uint32_t s = packed[i] & 0xFFFu;
      const int r = (int)cntx[s] + (int)((packed[i] >> 12) & 0x7FFFFu);   // rank among the block's pairs of slot s
      const int idx = lo + i * kWave + lane;
      s_sorted[s_loc[s] + r] = (s << 16) | (uint32_t)idx;
      if (row_of_pair) row_of_pair[p0 + idx] = s_off[s] + r;
    }
  }
  __syncthreads();
  for (int j = tid; j < n; j += kBigThreads) {
    const uint32_t v = s_sorted[j];
    const uint32_t s = v >> 16;
    pair_of_row[s_off[s] + (j - s_loc[s])] = (int32_t)(p0 + (v & 0xFFFFu));
  }
}

// Column s of the histogram matrix hist[nb][P], P <= 512 and a multiple of 4: its sum, and its sum over the rows before `row`, for
// thread s < P of a block of 512 threads.  A thread loads four columns at once from its share of the rows, so that the whole matrix
// is a few loads per thread, all in flight together; the shares meet in s_a (kColumnSumInts ints).  Contains a barrier; s_a may be
// reused after another one.
constexpr int kColumnSumInts = 2 * 4 * kBigThreads;
__device__ __forceinline__ void column_sums(const int32_t* __restrict__ hist, int nb, int P, int row, int32_t* s_a, int& total, int& before) {
  const int lg = P > 256 ? 7 : P > 128 ? 6 : 5, parts = kBigThreads >> lg;  // (groups of columns, threads per group)
  const int tid = threadIdx.x, group = tid & ((1 << lg) - 1), part = tid >> lg;
  const int per = (nb + parts - 1) / parts, r0 = part * per, r1 = min(nb, r0 + per);
  int4 sum = make_int4(0, 0, 0, 0), pre = sum;
  if (4 * group < P) {
    constexpr int kAhead = 8;
    for (int r = r0; r < r1; r += kAhead) {
      int4 v[kAhead];
#pragma unroll
      for (int j = 0; j < kAhead; ++j) v[j] = r + j < r1 ? *reinterpret_cast<const int4*>(hist + (size_t)(r + j) * P + 4 * group) : make_int4(0, 0, 0, 0);
#pragma unroll
      for (int j = 0; j < kAhead; ++j) {
        sum.x += v[j].x; sum.y += v[j].y; sum.z += v[j].z; sum.w += v[j].w;
        if (r + j < row) { pre.x += v[j].x; pre.y += v[j].y; pre.z += v[j].z; pre.w += v[j].w; }
      }
    }
  }
  int32_t* s_b = s_a + 4 * kBigThreads;
  reinterpret_cast<int4*>(s_a)[tid] = sum;
  reinterpret_cast<int4*>(s_b)[tid] = pre;
  __syncthreads();
  total = 0;
  before = 0;
  if (tid < P)
    for (int q = 0; q < parts; ++q) {
      total += s_a[(q << (lg + 2)) + tid];
      before += s_b[(q << (lg + 2)) + tid];
    }
}

// Kernel 3 for 2 <= k <= 8 and P <= 512: the same stable scatter with the ranking done one TOKEN per lane.  A wave
// step then covers 64 tokens = 64 k pairs; a token's k slots are distinct (the ids of a top-k are, and a row of the
// expert map is injective), so a lane's k pairs never meet each other in a slot's lane mask and one mask round ranks
// all of them: the chain of dependent LDS round trips per wave shrinks from one per 64 pairs to one per 64 k pairs
// (the ranking, not memory, bounded the pair-per-lane kernel).  A block that does find a token with a repeated slot
// (ids that no top-k would produce) ranks pair per lane as k_scatter does, so the result is exact for any input.
//   tpw = tokens per wave, a multiple of 64.
// direct: `base` is the blocks' histograms as k_hist left them, and counts is written here; every block sums its columns over
// them instead of a launch in between (us, scan and scatter with plan, before / now: 512 tokens 4.0 + 5.1 / 5.9; 8192 tokens
// 3.8 + 9.2 / 12.9).
template <int K>
__global__ __launch_bounds__(kBigThreads) void k_scatter_tok(const int32_t* __restrict__ slot_ids, int32_t* __restrict__ counts,
                                                             const int32_t* __restrict__ base, int direct, int nb, int T, int P, int bits, int cht,
                                                             int tpw, int run, int32_t* __restrict__ offsets,
                                                             int32_t* __restrict__ pair_of_row, int32_t* __restrict__ row_of_pair,
                                                             PlanReq fp) {
  constexpr int MAXP = 512;
  constexpr int STEPS = ((kBigPairs / K + kBigWaves - 1) / kBigWaves + kWave - 1) / kWave;  // 64-token steps per wave at most
  constexpr int NV = STEPS * K > kBigSteps ? STEPS * K : kBigSteps;                        // values per lane
  __shared__ uint16_t s_cnt[kBigWaves * MAXP];
  __shared__ int32_t s_off[MAXP + 1];    // first row of the block's pairs of slot s
  __shared__ int32_t s_loc[MAXP + 1];    // first position of slot s in the block's sorted order
  __shared__ __align__(16) uint32_t s_sorted[kBigPairs];  // slot << 16 | pair index inside the block, sorted by slot
  __shared__ int32_t s_w[2 * kBigWaves];
  __shared__ int s_dup;
  static_assert((size_t)kBigWaves * MAXP * 8 <= sizeof(s_sorted), "the lane masks borrow the sorted-pairs array");
  static_assert(sizeof(ew::FfnPlanLds) <= sizeof(s_sorted), "a plan is built in the sorted-pairs array");
  static_assert(kColumnSumInts * 4 <= sizeof(s_sorted), "the column sums borrow it too");
  int32_t* s_a = reinterpret_cast<int32_t*>(s_sorted);
  const int tid = threadIdx.x;
  if (fp.plan && blockIdx.x == 0) {
    if (direct) {
      int total, before;
      column_sums(base, nb, P, 0, s_a, total, before);
      if (tid < P) s_off[tid] = total;
      __syncthreads();
    }
    plan_block(direct ? s_off : counts, T, T * K, P, fp, s_w, s_sorted);
    return;
  }
  const int block = blockIdx.x - (fp.plan ? 1 : 0);
  const int wave = tid / kWave, lane = tid & (kWave - 1);
  const int t0 = block * cht, t1 = min(T, t0 + cht);
  const size_t p0 = (size_t)t0 * K;
  const int ntok = t1 - t0, n = ntok * K;                          // pairs of this block, <= kBigPairs
  const int wt0 = wave * tpw, wt1 = min(ntok, wt0 + tpw);          // this wave's tokens
  const int steps = tpw / kWave;                                   // <= STEPS
  uint32_t packed[NV];                                             // slot | rank << 12 | valid << 31; value st*K + j = choice j of token wt0 + 64 st + lane
  bool dup = false;
#pragma unroll
  for (int st = 0; st < STEPS; ++st) {
    const int tok = wt0 + st * kWave + lane;
    const bool valid = st < steps && tok < wt1;
    const int32_t* src = slot_ids + p0 + (size_t)tok * K;
#pragma unroll
    for (int j = 0; j < K; ++j) packed[st * K + j] = valid ? (uint32_t)src[j] : 0u;
  }
#pragma unroll
  for (int i = STEPS * K; i < NV; ++i) packed[i] = 0u;
  int base_v = 0, count_v = 0;                                     // slot tid: pairs in the blocks before this one, in all
  if (direct) {
    column_sums(base, nb, P, block, s_a, count_v, base_v);
    if (block == 0 && tid < P) counts[tid] = count_v;
    __syncthreads();                                               // s_a becomes the lane masks
  } else if (tid < P) {
    base_v = base[(size_t)block * P + tid];                        // the scanned histogram
    count_v = counts[tid];
  }
  unsigned long long* s_mask = reinterpret_cast<unsigned long long*>(s_sorted);
  for (int i = tid; i < kBigWaves * P; i += kBigThreads) {
    s_cnt[i] = 0;
    s_mask[i] = 0ull;
  }
  if (tid == 0) s_dup = 0;
#pragma unroll
  for (int st = 0; st < STEPS; ++st) {
    if (st < steps && wt0 + st * kWave + lane < wt1) {
#pragma unroll
      for (int j = 1; j < K; ++j)
#pragma unroll
        for (int j2 = 0; j2 < j; ++j2) dup = dup || packed[st * K + j] == packed[st * K + j2];
    }
  }
  __syncthreads();
  if (dup) s_dup = 1;
  __syncthreads();
  const bool generic = s_dup != 0;                                 // block-uniform

  uint16_t* cnt = s_cnt + (size_t)wave * P;
  unsigned long long* mask = s_mask + (size_t)wave * P;
  if (!generic) {
    const unsigned long long lt = lanemask_lt();
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
      if (st >= steps) break;
      const bool valid = wt0 + st * kWave + lane < wt1;
      uint32_t sl[K], old[K];
      unsigned long long peers[K];
#pragma unroll
      for (int j = 0; j < K; ++j) {
        sl[j] = packed[st * K + j];
        if (valid) __hip_atomic_fetch_or(&mask[sl[j]], 1ull << lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int j = 0; j < K; ++j) {
        peers[j] = valid ? __hip_atomic_load(&mask[sl[j]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) : 0ull;
        old[j] = valid ? cnt[sl[j]] : 0u;
      }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const int before = __popcll(peers[j] & lt);
        if (valid && before == 0) {
          cnt[sl[j]] = (uint16_t)(old[j] + __popcll(peers[j]));
          mask[sl[j]] = 0ull;
        }
        packed[st * K + j] = sl[j] | ((old[j] + before) << 12) | (valid ? 0x80000000u : 0u);
      }
      __builtin_amdgcn_wave_barrier();
    }
  } else {
    // pair per lane, on the wave's run of `run` consecutive pairs (re-read: the values above are laid out per token)
    const int lo = wave * run, hi = min(n, lo + run);
    uint32_t pk[kBigSteps];
    load_pairs(slot_ids, p0, lo, hi, run / kWave, pk);
    rank_pairs<true>(lo, hi, run / kWave, bits, cnt, mask, pk);
#pragma unroll
    for (int i = 0; i < kBigSteps; ++i) packed[i] = pk[i];
  }
  __syncthreads();
  {
    // thread s: the waves' counts of slot s become running sums; then the block scans the slots' totals (positions in
    // the block's sorted order) and the call's counts (first rows) together
    int tot = 0;
    if (tid < P) {
#pragma unroll
      for (int w = 0; w < kBigWaves; ++w) {
        const int c = s_cnt[(size_t)w * P + tid];
        s_cnt[(size_t)w * P + tid] = (uint16_t)tot;
        tot += c;
      }
    }
    int first_row, first_pos, rows_total, pos_total;
    block_exscan2(count_v, tot, first_row, first_pos, rows_total, pos_total, s_w);
    if (tid < P) {
      s_off[tid] = first_row + base_v;
      s_loc[tid] = first_pos;
      if (block == 0) offsets[tid] = first_row;
    }
    if (tid == 0) {
      s_loc[P] = pos_total;
      if (block == 0) offsets[P] = rows_total;
    }
  }
  __syncthreads();
  if (!generic) {
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
      if (st >= steps) break;
      const int tok = wt0 + st * kWave + lane;
      if (tok < wt1) {
        int32_t rows[K];
#pragma unroll
        for (int j = 0; j < K; ++j) {
          const uint32_t v = packed[st * K + j], s = v & 0xFFFu;
          const int r = (int)cnt[s] + (int)((v >> 12) & 0x7FFFFu);   // rank among the block's pairs of slot s
          s_sorted[s_loc[s] + r] = (s << 16) | (uint32_t)(tok * K + j);
          rows[j] = s_off[s] + r;
        }
        if (row_of_pair) {
          int32_t* dst = row_of_pair + p0 + (size_t)tok * K;        // K consecutive ints per lane
          if constexpr (K % 2 == 0) {
#pragma unroll
            for (int j = 0; j < K; j += 2) *reinterpret_cast<int2*>(dst + j) = make_int2(rows[j], rows[j + 1]);
          } else {
#pragma unroll
            for (int j = 0; j < K; ++j) dst[j] = rows[j];
          }
        }
      }
    }
  } else {
    const int lo = wave * run;
#pragma unroll
    for (int i = 0; i < kBigSteps; ++i) {
      if (packed[i] & 0x80000000u) {
        const uint32_t s = packed[i] & 0xFFFu;
        const int r = (int)cnt[s] + (int)((packed[i] >> 12) & 0x7FFFFu);
        const int idx = lo + i * kWave + lane;
        s_sorted[s_loc[s] + r] = (s << 16) | (uint32_t)idx;
        if (row_of_pair) row_of_pair[p0 + idx] = s_off[s] + r;
      }
    }
  }
  __syncthreads();
  for (int j = tid; j < n; j += kBigThreads) {
    const uint32_t v = s_sorted[j];
    const uint32_t s = v >> 16;
    pair_of_row[s_off[s] + (j - s_loc[s])] = (int32_t)(p0 + (v & 0xFFFFu));
  }
}

__global__ void k_zero_counts(int32_t* counts, int32_t* offsets, int P) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i <= P; i += gridDim.x * blockDim.x) {
    if (i < P) counts[i] = 0;
    offsets[i] = 0;
  }
}

// ------------------------------------------------------------------------------------------
// Tokens per block of the multi-block path: at most kBigPairs pairs, and small enough that a
// batch spreads over about 512 blocks: two 512-thread blocks fit a CU (LDS of k_scatter), so up to
// 2^20 tokens at k = 6 the whole grid is resident at once, and longer chunks mean longer runs per
// slot in the scatter's coalesced writes.
// Up to kDirectPairs pairs of a call that k_scatter_tok takes there are kDirectBlocks blocks at most, few enough for the scatter
// to do without the column scan (direct_sums).  Hist, scan and scatter of 30011 tokens, k = 8, us: 3.4 + 4.0 + 7.2, without the scan
// 3.1 + 7.8, and the call, which takes the host about as long, 20.5 -> 18.0.  More pairs want two blocks on every CU: calls with / without
// the column scan, us, at 2^18 pairs 13.4 / 13.2 (k = 8, 288 slots), 13.6 / 13.6 (4, 512), 11.8 / 10.2 (2, 128); 3 2^17 14.0 / 14.1, 14.4 / 14.5,
// 12.1 / 10.9; 2^19 14.6 / 15.2, 15.2 / 15.2, 12.8 / 12.0; 2^20 17.2 / 22.0, 17.4 / 21.0, 14.6 / 16.5.  (Of 2048 to 4096 tokens on 288 slots and more
// the sums cost as much as the scan did: 10.8 / 11.2.)
inline bool direct_sums(int T, int k, int P) {
  return P <= 512 && P % 4 == 0 && k >= 2 && k <= 8 && (long long)T * k <= kDirectPairs;
}
inline int chunk_tokens(int T, int k, int P) {
  const int cap = kBigPairs / k;  // >= 192 for k <= 64
  int want = ew::ceil_div(T, direct_sums(T, k, P) ? kDirectBlocks : 512);
  if (want < 16) want = 16;
  return want < cap ? want : cap;
}

// f(V) with the selection (wave_select) that E experts and k choices take; sixteen_lanes false: one wave per token in any case.
template <typename F>
int with_selection(int E, int k, bool sixteen_lanes, F f) {
  if (k <= 16 && E <= 256 && sixteen_lanes) {
    if (E <= 16) return f(std::integral_constant<int, 1>{});
    if (E <= 64) return f(std::integral_constant<int, 4>{});
    if (E <= 128) return f(std::integral_constant<int, 8>{});
    return f(std::integral_constant<int, 16>{});
  }
  if (E <= 64) return f(std::integral_constant<int, -1>{});
  if (E <= 128) return f(std::integral_constant<int, -2>{});
  if (E <= 256) return f(std::integral_constant<int, -4>{});
  if (E <= 512) return f(std::integral_constant<int, -8>{});
  return f(std::integral_constant<int, -16>{});
}

// Whether the single block of nwaves waves makes the selection too, sixteen lanes of V logits each per token, or a launch before it
// does on many CUs.  Joined it saves that launch, about 1.4 us, but four waves share a SIMD whose time V k bounds; beyond two waves on
// a SIMD or one round of the waves it has to be cheap.  Selection to plan, us, joined / own launch: 32 tokens, V k = 256 9.5 / 10.4;
// 48 tokens, V k = 96 (128 experts) 9.8 / 10.0, 128 11.0 / 10.7, of 256 experts 64 9.5 / 9.1; 64 tokens, V k = 32 8.1 / 8.1, 48 8.9 /
// 8.6, 128 (256 experts) 13.0 / 10.9; two rounds, V k = 24 12.5 / 12.5, 64 12.5 / 12.0; three rounds, V k = 2 9.5 / 10.0, 24 13.6 / 13.0.
// (256 tokens, four rounds of V k = 24: a stack of layers 2058 / 2033.)
inline bool joins_selection(int V, int T, int k, int nwaves) {
  if (V <= 0 || T > kSelectTokens) return false;
  const int rounds = ew::ceil_div(T, 4 * nwaves), cost = V * k;
  if (cost <= 8) return true;
  if (rounds > 1) return rounds == 2 && V < 16 && cost <= 32;
  return T <= 32 || (V < 16 && cost <= (T <= 48 ? 96 : 32));
}

template <int V>
int launch_permute(const float* logits, const int32_t* ids_in, const int32_t* aid, const int32_t* emap, int T, int E,
                   int k, int N, int P, int renorm, int32_t* ids_out, float* w_out, int32_t* slot_ids, int32_t* counts,
                   int32_t* offsets, int32_t* por, int32_t* rop, void* ws, hipStream_t st, const ew::FfnPlanShape* shape = nullptr,
                   int S = 0, int32_t* plan = nullptr) {
  const long long n = (long long)T * k;
  const int bits = ew::ilog2_ceil(P);
  const int map_entries = (N + 1) * E;
  if (n <= g_small_pairs) {
    int nwaves = kSmallCnt / P;
    // (8 waves are enough for 32 tokens' selection and what the plan needs; its barriers and start are cheaper: 1 token 46.8 ->
    // 46.4 us a pass, 13 tokens 53.9 -> 53.3)
    const int most = T <= 32 ? 8 : 16;
    if (nwaves > most) nwaves = most;
    int run = ((int)n + nwaves - 1) / nwaves;
    run = (run + kWave - 1) / kWave * kWave;
    const int nrank = ew::ceil_div((int)n, run), per = ew::ceil_div(P, nwaves * kWave);  // nrank <= nwaves
    // the FFN plan rides on the single-block kernel when that has the 512 threads the plan needs
    PlanReq fp{nullptr, 0, ew::FfnPlanShape{}};
    const bool fused_plan = plan && nwaves * kWave >= 512;
    if (fused_plan) fp = PlanReq{plan, S, *shape};
    if (joins_selection(V, T, k, nwaves)) {
      hipLaunchKernelGGL(k_small<(V > 0 ? V : 0)>, dim3(1), dim3(nwaves * kWave), 0, st, logits, ids_in, aid, emap, T, E, k, P, renorm, bits,
                         run, nrank, per, ids_out, w_out, slot_ids, counts, offsets, por, rop, fp);
    } else {
      if constexpr (V != 0) {
        hipLaunchKernelGGL((k_route<V, true>), dim3(ew::ceil_div(T, 4 * kTokensPerWave<V>)), dim3(256), 0, st, logits, aid, emap, T, E, k,
                           renorm, ids_out, w_out, slot_ids);
        EW_LAUNCH_CHECK("k_route");
      }
      hipLaunchKernelGGL(k_small<0>, dim3(1), dim3(nwaves * kWave), 0, st, logits, V != 0 ? (const int32_t*)slot_ids : ids_in, aid,
                         V != 0 ? (const int32_t*)nullptr : emap, T, E, k, P, renorm, bits, run, nrank, per, ids_out, w_out, slot_ids, counts,
                         offsets, por, rop, fp);
    }
    EW_LAUNCH_CHECK("k_small");
    if (plan && !fused_plan) return ew::launch_ffn_plan(counts, offsets, P, S, T, (int)n, *shape, plan, st);
    return EW_OK;
  }
  const int cht = chunk_tokens(T, k, P);
  const bool direct = direct_sums(T, k, P);
  const int nb = ew::ceil_div(T, cht);
  const int run = (int)ew::align_up((size_t)ew::ceil_div(cht * k, kBigWaves), kWave);
  int32_t* hist = (int32_t*)ws;
  // with the router fused, a thread for every lane that a block's tokens keep busy
  const int hist_threads = V == 0 ? kHistThreads : (int)ew::align_up((size_t)ew::ceil_div(cht, kTokensPerWave<V>) * kWave, 256);
  hipLaunchKernelGGL((k_hist<V>), dim3(nb), dim3(hist_threads < kHistThreads ? hist_threads : kHistThreads), 0, st, logits, ids_in, aid, emap, T, E, k, P,
                     map_entries, renorm, cht, ids_out, w_out, slot_ids, hist);
  EW_LAUNCH_CHECK("k_hist");
  if (!direct) {
    hipLaunchKernelGGL(k_colscan, dim3(ew::ceil_div(P, kScanCols)), dim3(kScanCols * kScanGroups), 0, st, hist, nb, P, counts);
    EW_LAUNCH_CHECK("k_colscan");
  }
  const int tpw = (int)ew::align_up((size_t)ew::ceil_div(cht, kBigWaves), kWave);  // tokens per wave of the token-per-lane kernel
  const PlanReq fp = plan ? PlanReq{plan, S, *shape} : PlanReq{nullptr, 0, ew::FfnPlanShape{}};
  const int blocks = nb + (plan ? 1 : 0);
#define EW_SCATTER_TOK(KK)                                                                                                      \
  hipLaunchKernelGGL(k_scatter_tok<KK>, dim3(blocks), dim3(kBigThreads), 0, st, slot_ids, counts, hist, (int)direct, nb, T, P, bits, cht, tpw, run, \
                     offsets, por, rop, fp)
  if (P <= 512 && k >= 2 && k <= 8) {
    switch (k) {
      case 2: EW_SCATTER_TOK(2); break;
      case 3: EW_SCATTER_TOK(3); break;
      case 4: EW_SCATTER_TOK(4); break;
      case 5: EW_SCATTER_TOK(5); break;
      case 6: EW_SCATTER_TOK(6); break;
      case 7: EW_SCATTER_TOK(7); break;
      default: EW_SCATTER_TOK(8); break;
    }
  } else if (P <= 512)
    hipLaunchKernelGGL(k_scatter<512>, dim3(blocks), dim3(kBigThreads), 0, st, slot_ids, counts, hist, T, k, P, bits, cht, run,
                       offsets, por, rop, fp);
  else
    hipLaunchKernelGGL(k_scatter<kMaxP>, dim3(blocks), dim3(kBigThreads), 0, st, slot_ids, counts, hist, T, k, P, bits, cht, run,
                       offsets, por, rop, fp);
#undef EW_SCATTER_TOK
  EW_LAUNCH_CHECK("k_scatter");
  return EW_OK;
}

int check_permute_args(const char* who, const int32_t* aid, const int32_t* emap, int T, int k, int E, int N, int P,
                       int32_t* slot_ids, int32_t* counts, int32_t* offsets, int32_t* por, void* ws, size_t ws_bytes) {
  using ew::fail;
  if (T < 0 || k < 1 || E < 1 || N < 0 || P < 1) return fail(EW_ERR_INVALID_ARG, "%s: need T>=0, k>=1, E>=1, N>=0, P>=1", who);
  if (k > 64) return fail(EW_ERR_UNSUPPORTED, "%s: k=%d above the supported 64", who, k);
  if (P > kMaxP) return fail(EW_ERR_UNSUPPORTED, "%s: P=%d above the supported %d", who, P, kMaxP);
  if ((long long)T * k >= (1ll << 31)) return fail(EW_ERR_UNSUPPORTED, "%s: T*k must be below 2^31", who);
  if (!counts || !offsets) return fail(EW_ERR_INVALID_ARG, "%s: counts/offsets is NULL", who);
  if (T == 0) return EW_OK;
  if (!aid || !emap || !slot_ids || !por) return fail(EW_ERR_INVALID_ARG, "%s: NULL device pointer", who);
  const size_t need = moe_reroute_permute_workspace_bytes(T, k, P);
  if (need && (!ws || ((uintptr_t)ws & 255) || ws_bytes < need))
    return fail(EW_ERR_WORKSPACE, "%s: workspace needs %zu bytes aligned to 256 (got %zu at %p)", who, need, ws_bytes, ws);
  return EW_OK;
}

}  // namespace

// ------------------------------------------------------------------------------------------
// Rerouting as separate canonical operators, each a launch and a pass over memory of its own:
// the unfused baseline the paper's fused kernel is compared with (Sec. 5.3, ExpertWeave-SingleOp).
namespace {
__global__ __launch_bounds__(256) void k_so_broadcast(const int32_t* __restrict__ aid, long long n, int k, int32_t* __restrict__ aid_b) {
  for (long long p = (long long)blockIdx.x * 256 + threadIdx.x; p < n; p += (long long)gridDim.x * 256) aid_b[p] = aid[(uint32_t)p / (uint32_t)k];
}
__global__ __launch_bounds__(256) void k_so_offsets(const int32_t* __restrict__ aid_b, const int32_t* __restrict__ ids, long long n,
                                                   int E, int32_t* __restrict__ off) {
  for (long long p = (long long)blockIdx.x * 256 + threadIdx.x; p < n; p += (long long)gridDim.x * 256) off[p] = aid_b[p] * E + ids[p];
}
__global__ __launch_bounds__(256) void k_so_gather(const int32_t* __restrict__ emap, const int32_t* __restrict__ off, long long n,
                                                  int32_t* __restrict__ slot) {
  for (long long p = (long long)blockIdx.x * 256 + threadIdx.x; p < n; p += (long long)gridDim.x * 256) slot[p] = emap[off[p]];
}
}  // namespace

extern "C" size_t moe_reroute_singleop_workspace_bytes(int T, int k) {
  if (T <= 0 || k < 1) return 0;
  return 2 * ew::align_up((size_t)T * k * sizeof(int32_t), 256);
}

extern "C" int moe_reroute_singleop(const int32_t* topk_ids, const int32_t* adapter_id, const int32_t* expert_map, int T, int k,
                                    int E, int N, int32_t* slot_ids, void* ws, size_t ws_bytes, void* stream) {
  using ew::fail;
  if (T < 0 || k < 1 || E < 1 || N < 0) return fail(EW_ERR_INVALID_ARG, "moe_reroute_singleop: need T>=0, k>=1, E>=1, N>=0");
  if ((long long)T * k >= (1ll << 31)) return fail(EW_ERR_UNSUPPORTED, "moe_reroute_singleop: T*k must be below 2^31");
  if (T == 0) return EW_OK;
  if (!topk_ids || !adapter_id || !expert_map || !slot_ids) return fail(EW_ERR_INVALID_ARG, "moe_reroute_singleop: NULL device pointer");
  const size_t need = moe_reroute_singleop_workspace_bytes(T, k);
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < need)
    return fail(EW_ERR_WORKSPACE, "moe_reroute_singleop: workspace needs %zu bytes aligned to 256 (got %zu at %p)", need, ws_bytes, ws);
  hipStream_t st = (hipStream_t)stream;
  const long long n = (long long)T * k;
  int32_t* aid_b = (int32_t*)ws;
  int32_t* off = (int32_t*)((char*)ws + need / 2);
  const int blocks = (int)((n + 255) / 256 < 16384 ? (n + 255) / 256 : 16384);
  hipLaunchKernelGGL(k_so_broadcast, dim3(blocks), dim3(256), 0, st, adapter_id, n, k, aid_b);
  EW_LAUNCH_CHECK("k_so_broadcast");
  hipLaunchKernelGGL(k_so_offsets, dim3(blocks), dim3(256), 0, st, aid_b, topk_ids, n, E, off);
  EW_LAUNCH_CHECK("k_so_offsets");
  hipLaunchKernelGGL(k_so_gather, dim3(blocks), dim3(256), 0, st, expert_map, off, n, slot_ids);
  EW_LAUNCH_CHECK("k_so_gather");
  return EW_OK;
}

// ------------------------------------------------------------------------------------------
// moe_reroute_permute for callers that cannot allocate: the block-histogram table lives in a
// file-scope device array instead of a caller workspace.  Each GPU holds its own copy of the array
// at its own address; the address is looked up once per device, with that device current, and only
// that pointer (never the array's name, which is a host-side stand-in) is handed to kernels.
namespace {
constexpr size_t kStaticScratchBytes = (size_t)4 << 20;
__device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kScratchMaxDev = 64;
std::atomic<void*> g_scratch_ptr[kScratchMaxDev];

int static_scratch(void** out) {
  int dev = 0;
  EW_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kScratchMaxDev) return ew::fail(EW_ERR_UNSUPPORTED, "moe_reroute_permute_static: device index %d above %d", dev, kScratchMaxDev - 1);
  void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!p) {
    EW_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return ew::fail(EW_ERR_HIP, "moe_reroute_permute_static: the scratch array has no device address");
    g_scratch_ptr[dev].store(p, std::memory_order_release);  // racing first calls store the same address
  }
  *out = p;
  return EW_OK;
}
}  // namespace

extern "C" size_t moe_reroute_permute_static_max_bytes(void) { return kStaticScratchBytes; }

extern "C" int moe_reroute_permute_static(const int32_t* topk_ids, const int32_t* adapter_id, const int32_t* expert_map, int T,
                                          int k, int E, int N, int P, int32_t* slot_ids, int32_t* counts, int32_t* offsets,
                                          int32_t* pair_of_row, int32_t* row_of_pair, void* stream) {
  const size_t need = moe_reroute_permute_workspace_bytes(T, k, P);
  if (need > kStaticScratchBytes)
    return ew::fail(EW_ERR_UNSUPPORTED,
                    "moe_reroute_permute_static: T=%d k=%d P=%d needs %zu bytes of scratch, the built-in buffer holds %zu; "
                    "use moe_reroute_permute with a workspace",
                    T, k, P, need, kStaticScratchBytes);
  void* ws = nullptr;
  if (need) {
    int rc = static_scratch(&ws);
    if (rc != EW_OK) return rc;
  }
  // Every block of the histogram kernel writes its whole row of the table before anything reads it,
  // so nothing has to be cleared between calls; the table keeps the last call's contents.
  return moe_reroute_permute(topk_ids, adapter_id, expert_map, T, k, E, N, P, slot_ids, counts, offsets, pair_of_row,
                             row_of_pair, ws, need, stream);
}

bool ew::single_block_permute(long long pairs) { return pairs <= g_small_pairs; }

extern "C" void ew_tune_route(int small_pairs) {
  g_small_pairs = small_pairs < 0 ? 0 : (small_pairs > kSmallPairs ? kSmallPairs : small_pairs);
}

// ==========================================================================================
extern "C" size_t moe_reroute_permute_workspace_bytes(int T, int k, int P) {
  if (T <= 0 || k < 1 || k > 64 || P < 1) return 0;
  // sized for the multi-block path even where the single-block one will run: the switch-over is a tuning knob
  // and never less for more tokens (a workspace made for a largest batch serves the smaller ones): chunk_tokens gives at most 512
  // blocks, of 16 tokens at least, until a block's pairs reach their limit
  const int most = ew::ceil_div(T, 16) < 512 ? ew::ceil_div(T, 16) : 512, full = ew::ceil_div(T, kBigPairs / k);
  return ew::align_up((size_t)(most > full ? most : full) * P * sizeof(int32_t), 256);
}

extern "C" int moe_route_topk(const float* logits, int T, int E, int k, int renormalize, int32_t* topk_ids,
                              float* topk_w, void* stream) {
  using ew::fail;
  if (T < 0 || E < 1 || k < 1 || k > E) return fail(EW_ERR_INVALID_ARG, "moe_route_topk: need T>=0 and 1<=k<=E (T=%d E=%d k=%d)", T, E, k);
  if (E > kMaxE || k > 64) return fail(EW_ERR_UNSUPPORTED, "moe_route_topk: supports E<=%d and k<=64 (E=%d k=%d)", kMaxE, E, k);
  if (T == 0) return EW_OK;
  if (!logits || !topk_ids || !topk_w) return fail(EW_ERR_INVALID_ARG, "moe_route_topk: NULL device pointer");
  hipStream_t st = (hipStream_t)stream;
  // Many choices among many experts are a long chain for sixteen lanes, one wave per token is faster until its tokens fill the chip.
  // us, sixteen lanes / a wave: 512 tokens of 256 experts, k = 14 6.7 / 6.8, k = 16 7.3 / 6.9; of 128, k = 16 5.1 / 5.0; of 256, k = 16,
  // 1024 tokens 7.3 / 6.9, 2048 7.3 / 7.8, 4096 7.4 / 9.9.
  const bool sixteen_lanes = T > 1024 || E <= 128 || k <= 14;
  with_selection(E, k, sixteen_lanes, [&](auto tag) {
    constexpr int V = decltype(tag)::value;
    const int full = (T - 1) / (4 * kTokensPerWave<V>);  // (T up to 2^31 - 1: no rounding up before the division)
    hipLaunchKernelGGL((k_route<V, false>), dim3(full < kRouteBlocks ? full + 1 : kRouteBlocks), dim3(256), 0, st, logits, (const int32_t*)nullptr,
                       (const int32_t*)nullptr, T, E, k, renormalize, topk_ids, topk_w, (int32_t*)nullptr);
    return EW_OK;
  });
  EW_LAUNCH_CHECK("k_route_topk");
  return EW_OK;
}

extern "C" int moe_reroute_permute(const int32_t* topk_ids, const int32_t* adapter_id, const int32_t* expert_map, int T,
                                   int k, int E, int N, int P, int32_t* slot_ids, int32_t* counts, int32_t* offsets,
                                   int32_t* pair_of_row, int32_t* row_of_pair, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_permute_args("moe_reroute_permute", adapter_id, expert_map, T, k, E, N, P, slot_ids, counts, offsets,
                              pair_of_row, ws, ws_bytes);
  if (rc != EW_OK) return rc;
  hipStream_t st = (hipStream_t)stream;
  if (T == 0) {
    hipLaunchKernelGGL(k_zero_counts, dim3(1), dim3(256), 0, st, counts, offsets, P);
    EW_LAUNCH_CHECK("k_zero_counts");
    return EW_OK;
  }
  if (!topk_ids) return ew::fail(EW_ERR_INVALID_ARG, "moe_reroute_permute: topk_ids is NULL");
  return launch_permute<0>(nullptr, topk_ids, adapter_id, expert_map, T, E, k, N, P, 0, nullptr, nullptr, slot_ids, counts,
                           offsets, pair_of_row, row_of_pair, ws, st);
}

namespace {

int route_reroute_permute(const char* who, const float* logits, const int32_t* adapter_id, const int32_t* expert_map, int T, int E,
                          int k, int N, int P, int renormalize, int32_t* topk_ids, float* topk_w, int32_t* slot_ids,
                          int32_t* counts, int32_t* offsets, int32_t* pair_of_row, int32_t* row_of_pair, void* ws, size_t ws_bytes,
                          const ew::FfnPlanShape* shape, int S, int32_t* plan, hipStream_t st) {
  using ew::fail;
  if (k > E) return fail(EW_ERR_INVALID_ARG, "%s: k=%d exceeds E=%d", who, k, E);
  int rc = check_permute_args(who, adapter_id, expert_map, T, k, E, N, P, slot_ids, counts, offsets, pair_of_row, ws, ws_bytes);
  if (rc != EW_OK) return rc;
  if (E > kMaxE) return fail(EW_ERR_UNSUPPORTED, "%s: supports E<=%d (E=%d)", who, kMaxE, E);
  if (T == 0) {
    hipLaunchKernelGGL(k_zero_counts, dim3(1), dim3(256), 0, st, counts, offsets, P);
    EW_LAUNCH_CHECK("k_zero_counts");
    return EW_OK;
  }
  if (!logits || !topk_ids || !topk_w) return fail(EW_ERR_INVALID_ARG, "%s: NULL device pointer", who);
  // Where the selection is a launch of its own and its tokens few, many choices among many experts take a wave per token, as in
  // moe_route_topk: 256 experts, k = 16, us, sixteen lanes / a wave: 64 tokens 12.1 / 11.4, 128 tokens 13.8 / 12.8.
  const bool sixteen_lanes = E <= 128 || k <= 14 || T <= 32 || (long long)T * k > g_small_pairs;
  return with_selection(E, k, sixteen_lanes, [&](auto tag) {
    return launch_permute<decltype(tag)::value>(logits, nullptr, adapter_id, expert_map, T, E, k, N, P, renormalize, topk_ids, topk_w,
                                                slot_ids, counts, offsets, pair_of_row, row_of_pair, ws, st, shape, S, plan);
  });
}

}  // namespace

extern "C" int moe_route_reroute_permute(const float* logits, const int32_t* adapter_id, const int32_t* expert_map, int T,
                                         int E, int k, int N, int P, int renormalize, int32_t* topk_ids, float* topk_w,
                                         int32_t* slot_ids, int32_t* counts, int32_t* offsets, int32_t* pair_of_row,
                                         int32_t* row_of_pair, void* ws, size_t ws_bytes, void* stream) {
  return route_reroute_permute("moe_route_reroute_permute", logits, adapter_id, expert_map, T, E, k, N, P, renormalize, topk_ids,
                               topk_w, slot_ids, counts, offsets, pair_of_row, row_of_pair, ws, ws_bytes, nullptr, 0, nullptr,
                               (hipStream_t)stream);
}

extern "C" int moe_route_reroute_permute_plan(const float* logits, const int32_t* adapter_id, const int32_t* expert_map, int T,
                                              int E, int k, int N, int P, int renormalize, int32_t* topk_ids, float* topk_w,
                                              int32_t* slot_ids, int32_t* counts, int32_t* offsets, int32_t* pair_of_row,
                                              int32_t* row_of_pair, void* ws, size_t ws_bytes, int H, int I, int S, int dtype,
                                              void* ffn_ws, size_t ffn_ws_bytes, void* stream) {
  using ew::fail;
  const char* who = "moe_route_reroute_permute_plan";
  if (T < 0 || k < 1 || P < 1 || H < 1 || I < 1 || S < 0) return fail(EW_ERR_INVALID_ARG, "%s: need T>=0, k>=1, P>=1, H>=1, I>=1, S>=0", who);
  ew::FfnPlanShape shape{};
  int32_t* plan = nullptr;
  if (T > 0) {
    if (!ew::ffn_shape_of_call(dtype, T, k, H, I, P, S, &shape))
      return fail(EW_ERR_UNSUPPORTED, "%s: the grouped FFN of these dimensions takes no plan (needs bf16, H and I multiples of 128, "
                  "P+S <= 2048, T*(k+S)*max(H,I)*2 < 2^32, H*I < 2^30)", who);
    const size_t need = moe_grouped_ffn_workspace_bytes(T, k + S, H, I, P + S, dtype);
    if (!ffn_ws || ((uintptr_t)ffn_ws & 255) || ffn_ws_bytes < need)
      return fail(EW_ERR_WORKSPACE, "%s: the FFN workspace needs %zu bytes aligned to 256 (got %zu at %p)", who, need, ffn_ws_bytes, ffn_ws);
    plan = (int32_t*)ffn_ws;
  }
  return route_reroute_permute(who, logits, adapter_id, expert_map, T, E, k, N, P, renormalize, topk_ids, topk_w, slot_ids, counts,
                               offsets, pair_of_row, row_of_pair, ws, ws_bytes, &shape, S, plan, (hipStream_t)stream);
}
