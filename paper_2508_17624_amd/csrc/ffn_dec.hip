// Grouped SwiGLU expert FFN for calls with few rows per slot on gfx950: one continuous stream of weights through every CU.
//
// With a handful of rows per slot both products are a pure weight stream (17 MB per active expert at the 2048/1408 shape),
// so what counts is that every CU has enough bytes in flight from the first microsecond to the last.
//   * A unit is 64, 128 or 256 weight rows of one slot's chunk of 16 to 160 token rows.  The units of a workgroup form ONE stream of
//     slabs (16 or 32 KB of weights): the LDS rings keep filling across unit boundaries, nothing drains between two units.
//   * Loading and multiplying are different waves.  An LDS-direct load stalls its wave while the CU's queue of outstanding
//     lines is full, which here is most of the time; a wave that also multiplied would multiply late, and with it everyone
//     at the slab's barrier.
//   * A wave that does nothing else claims the units, two ahead, and leaves their description and row map in a small LDS
//     queue.  Claims go to eight lists per product, each with a counter in a cache line of its own that practically only
//     one XCD touches (one counter for all: 39 ns per claim, one after the other, longer than the whole weight stream).  A
//     workgroup takes from its home list, then from the others, and turns to the second product when no list has a
//     first-product unit left, so both products share one launch.
//   * A second-product unit reads activation rows of other workgroups once its chunk's completion counter says that they
//     are stored.  Every such wait ends: a workgroup that waits holds second-product units only, since it claimed the first
//     of them when all first-product units were claimed; a first-product unit is held by a workgroup whose earlier units
//     are first-product too, which wait for nothing, and whose stores are counted before it waits for anything (workgroups
//     that are not resident hold no claims).  A limit on the number of looks makes sure of it, see wait_stored.
//   * Coherence of the activations: agent-scope stores, acknowledged before they are counted; for the loads see kHalfLines.
// Measured (call with plan, one card): 1 token on 8 experts of 2048 x 1408: 76 -> 43 us (kernel alone now 37.4 -> 34.7); 13 tokens
// on 36 of 1024 x 896: 88 -> 47 us (42.2 -> 40.2); 64 tokens on 90: 263 -> 246 us (6.3 TB/s of weights; a bare stream of the same slabs reaches 6.85); 512 tokens on
// 242: 699 -> 682 us; 512 on 150 of 1536 x 640: 182 -> 161 us; 2000 on 194 of those: 328 -> 257 us, with chunks of up to 160 rows
// 257 -> 228.  Calls of layer passes of up to 64 tokens route themselves too (ffn_route.h).
//
// Waves: NW load weights, NT token rows, each into a ring of its own (the vector-memory counter retires in order, so each
// ring is awaited at its own depth), one schedules, eight multiply (v_mfma_f32_16x16x32_bf16).
// LDS rows are 256 or 128 bytes in pieces of 16, the piece index XOR-ed with (a half of) the row: the operand reads of 16
// rows at one logical piece then cover all banks.  The loads apply it on the global side (a lane fetches the piece that
// belongs at its position).
// Fragments: a wave's two weight fragments (i = 0, 1) interleave so that a lane's eight sums belong together.  First
// product: row m = 4 q + r of fragment i is feature 16 pair + 4 q + 2 i + (r & 1), gate for r < 2 and up for r >= 2: a lane
// holds gate and up of four consecutive features, SwiGLU needs no exchange and 8 bytes are stored.  Second product: feature
// 32 pair + 8 q + 4 i + r, 16 bytes.  (With one fragment per wave and half the width the stores alone cost 5 to 8 %.)
#include "ffn_route.h"

namespace ew {

namespace {

// NTF: 16-row token fragments per chunk; MR: weight rows per unit.
template <int NTF, int MR>
struct DecCfg {
  static constexpr int SK = MR == 64 ? 128 : 64;                    // contraction elements per slab
  static constexpr int RB = SK * 2;                                 // bytes of an LDS row
  static constexpr int FRAG = 16 * RB;                              // bytes of a 16-row fragment
  static constexpr int WSLAB = MR * RB;                             // bytes of one weight slab
  static constexpr int TSLAB = NTF * FRAG;                          // bytes of one token slab
  // waves: NW load weights, NT token rows, one schedules, eight multiply.  256-row units keep 64 accumulators per lane, for
  // which there are registers with three waves per SIMD; a slab of theirs lasts long enough for fewer loading waves.
  static constexpr int NW = MR == 256 ? 2 : 4, NT = MR == 256 ? 1 : 2;
  static constexpr int THREADS = 64 * (NW + NT + 1 + 8);
  static constexpr int RPI = 1024 / RB;                             // rows per load instruction
  static constexpr int NWI = MR / (NW * RPI);                       // load instructions per weight wave and slab
  static constexpr int NTI = 16 / (NT * RPI);                       // load instructions per token wave and fragment
  static constexpr int PN = MR / 32;                                // pairs of weight fragments
  static constexpr int QI = 8 + (16 * NTF + 63) / 64 * 64;          // ints of a queue entry: description, source rows, 64 at a time
  static constexpr int LEFT = 160 * 1024 - 4 * QI * 4;
  // ring depths: the token rows come from L2 and need less, the weights take the rest
  static constexpr int DT = TSLAB > 8192 ? 3 : NTF == 1 ? 6 : 5;
  static constexpr int MOST = NTF == 1 ? 6 : 8;                     // (1 and 13 tokens: 8 and 5 slabs 48.2, 54.9 us, 6 and 6 47.6, 54.4)
  static constexpr int DW = (LEFT - DT * TSLAB) / WSLAB < MOST ? (LEFT - DT * TSLAB) / WSLAB : MOST;
  static constexpr int Q_OFF = DW * WSLAB + DT * TSLAB;
  static constexpr int LDS = Q_OFF + 4 * QI * 4;
  static_assert(LDS <= 160 * 1024 && DW * WSLAB >= 80 * 1024, "LDS budget of a CU, bytes in flight");
  static constexpr int FPI = NW * RPI / 16;                         // fragments per round of the weight waves' instructions
  static constexpr bool SPLIT = NTF == 1;                           // units of the first product may come in halves, see whole_units
  static_assert(!SPLIT || (PN / 2 % FPI == 0 && NWI % 2 == 0), "half a unit: whole pairs of fragments, loads for every weight wave");
};

// Where the plan of a call lies that routes itself: behind the rings and the queue.
template <typename C>
struct Routed {
  static constexpr int OFF = C::LDS, LDS = C::LDS + (int)sizeof(RoutePlan);
  static_assert(C::QI > 72 || (C::LDS % 8 == 0 && LDS <= 160 * 1024), "LDS budget of a CU, for the shapes that route themselves");
  static_assert(2 * sizeof(RouteScratch) <= C::Q_OFF, "the ranking's scratch, in the rings");
  int claim = 0, n_chunks = 0;                                      // scheduling wave: its first claim, chunks of the plan
  static __device__ __forceinline__ RoutePlan& plan(unsigned char* s_lds) { return *reinterpret_cast<RoutePlan*>(s_lds + OFF); }
};

// Operands of one k-step (32 elements): MFW weight fragments WS bytes apart and NB token fragments FS bytes apart, issued
// without waiting.
template <int N, int STEP>
__device__ __forceinline__ void read_frags(uint32_t addr, u32x4* v) {
  if constexpr (N == 1)
    asm volatile("ds_read_b128 %0, %1" : "=&v"(v[0]) : "v"(addr));
  else if constexpr (N == 2)
    asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %2 offset:%3" : "=&v"(v[0]), "=&v"(v[1]) : "v"(addr), "n"(STEP));
  else if constexpr (N == 3)
    asm volatile("ds_read_b128 %0, %3\n\tds_read_b128 %1, %3 offset:%4\n\tds_read_b128 %2, %3 offset:%5"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]) : "v"(addr), "n"(STEP), "n"(2 * STEP));
  else {
    asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:%5\n\tds_read_b128 %2, %4 offset:%6\n\tds_read_b128 %3, %4 offset:%7"
                 : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]) : "v"(addr), "n"(STEP), "n"(2 * STEP), "n"(3 * STEP));
    if constexpr (N > 4) read_frags<N - 4, STEP>(addr + 4 * STEP, v + 4);
  }
}
// This wave's operand reads have landed; the registers are named so that nothing uses them earlier.
template <int N>
__device__ __forceinline__ void landed(u32x4* v) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(v[i]));
}

// One slab: KS k-steps of MFW weight fragments times NB token fragments.  All operands are read
// at once where they fit the registers (128 per wave), otherwise one k-step and four token fragments at a time.
template <int MFW, int NB, int KS, int WS, int FS>
__device__ __forceinline__ void mul_slab(uint32_t wa, uint32_t tb, f32x4 (&acc)[MFW][NB]) {
  constexpr int BATCH = MFW * NB + KS * (MFW + NB) <= 22 ? KS : 1, N = NB < 4 ? NB : NB % 4 ? 5 : 4;
  static_assert(NB % N == 0, "whole rounds of token fragments");
#pragma unroll
  for (int j0 = 0; j0 < KS; j0 += BATCH) {
    u32x4 a[BATCH][MFW];
#pragma unroll
    for (int f0 = 0; f0 < NB; f0 += N) {
      u32x4 b[BATCH][N];
#pragma unroll
      for (int j = 0; j < BATCH; ++j) {
        if (f0 == 0) read_frags<MFW, WS>(wa ^ (uint32_t)(64 * (j0 + j)), a[j]);
        read_frags<N, FS>((tb ^ (uint32_t)(64 * (j0 + j))) + f0 * FS, b[j]);
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int j = 0; j < BATCH; ++j) {
        if (f0 == 0) landed<MFW>(a[j]);
        landed<N>(b[j]);
      }
#pragma unroll
      for (int j = 0; j < BATCH; ++j)
#pragma unroll
        for (int f = 0; f < N; ++f)
#pragma unroll
            for (int i = 0; i < MFW; ++i)
              acc[i][f0 + f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[j][i]), __builtin_bit_cast(bf16x8, b[j][f]),
                                                                            acc[i][f0 + f], 0, 0, 0);
    }
  }
}
// First slab of a unit's walk over K: a function of the unit alone (results do not depend on who computes it) that keeps
// workgroups streaming neighbouring units in step off the same memory channels.
__device__ __forceinline__ int first_slab(const FfnUnit& u, int nk) { return (u.slot * 5 + u.g * 3) % nk; }

// ------------------------------------------------------------------------------------------
// A call of a few tokens has one to three units of the first product per workgroup, and the second product waits for the last
// one: where the units beyond the last full round fit one round as halves (of their weight rows), they are split.  1 token: 96
// units beyond 256, a pass 48.9 -> 47.9 us; 13 tokens: 62 beyond 512, 56.9 -> 54.6.  A slab costs about half a microsecond of hand-overs
// between the waves however small it is, so halves cost more than their unit and pay only where the call, `second` units of the second
// product among it, needs no further round for them.  Call with plan, us, whole / halves, at units of both products (rounds): 2048 x 1408
// 572 + 416 (3.9) 75.8 / 81.5, 594 + 432 (4.0) 80.9 / 81.4, 638 + 464 (4.3) 87.6 / 84.0; 1024 x 896 574 + 328 (3.5) 47.7 / 46.0, 602 + 344 (3.7)
// 47.7 / 51.8; 1536 x 768 336 + 336 (2.6) 45.1 / 42.7, 348 + 348 (2.7) 46.4 / 48.4.  Halves of 64-row units cost more of theirs: only where
// the last round is at most half full (1536 x 768 336 + 336 (2.6) 31.0 / 31.8; 2048 x 1024 352 + 352 (2.75) 37.8 / 40.6).  Nor with less than one
// round, where nothing waits: 1280 x 512, 1 to 3 tokens, 1 to 3 us lost.
// Halves keep their unit's walk over K, so no result depends on the split.  Not for more rounds or more tokens, and not in the second
// product, where the workgroups end 7 to 26 us apart: the last units in halves or quarters cost more than the even end gave (64 tokens
// 241 -> 247 us, 256 tokens 2028 -> 2046).
template <typename C>
__device__ __forceinline__ int whole_units(int grid, int first, int second) {  // positions below are whole units, above there are two for each
  if (!C::SPLIT || first <= grid || first >= 3 * grid) return first;
  const int over = first < 2 * grid ? first - grid : first - 2 * grid;
  int last = first + second;  // (of the remainder: few rounds, where a division is a long chain)
  while (last >= grid) last -= grid;
  const int room = C::PN == 2 ? grid / 2 : grid - over;
  return 2 * over <= grid && last > 0 && last <= room ? first - over : first;
}
// What a stored unit of the first product adds to its chunk's completion counter, which ends at kDone G.
constexpr int kDone = 2;
__device__ __forceinline__ int done_by(const FfnUnit& u) { return u.how ? 1 : kDone; }

// The scheduling wave.  Position v of a product's units belongs to list v % 8.
struct Sched {
  int w;                 // claim in flight: position in list `list` of product `mode`
  int mode, list, home;
  int chunk, g, how;
  i32x4 en;
  int pairs;             // src are pairs, not rows yet
  int stored;            // what its chunk's completion counter holds
  uint32_t src[3];       // the source rows lane, lane + 64, ... of the chunk
};

__device__ __forceinline__ int32_t* sched_counter(const FfnArgs& a, int mode, int list) {
  return a.plan + kDecCtr + (mode * 8 + list) * kDecCtrStride;
}
__device__ __forceinline__ void sched_claim(const FfnArgs& a, Sched& s) {
  if ((threadIdx.x & 63) == 0 && s.mode <= a.last_mode) s.w = claim_next(sched_counter(a, s.mode, s.list));
}
// own: the plan in LDS of a call that routes itself.
template <typename C, bool ROUTED>
__device__ __forceinline__ void sched_entry(const FfnArgs& a, const SchedDims& d, const RoutePlan* own, int n_chunks, int whole, Sched& s) {
  const int lane = threadIdx.x & 63;
  for (;;) {
    if (s.mode > a.last_mode) {
      s.chunk = -1;
      return;
    }
    const int G = s.mode ? d.units1 : d.units0, units = n_chunks * G, n = C::SPLIT && !s.mode ? 2 * units - whole : units;
    const int v = __builtin_amdgcn_readfirstlane(s.w) * 8 + s.list;
    if (v < n) {
      int u = v;
      s.how = 0;
      if (C::SPLIT && !s.mode && v >= whole) {
        u = whole + ((v - whole) >> 1);
        s.how = 1 + ((v - whole) & 1);
      }
      // u / G, without an integer division's chain of instructions in front of the first loads: off by one at most
      s.chunk = (int)(((float)u + 0.5f) * __builtin_amdgcn_rcpf((float)G));
      s.g = u - s.chunk * G;
      if (s.g < 0) {
        --s.chunk;
        s.g += G;
      } else if (s.g >= G) {
        ++s.chunk;
        s.g -= G;
      }
      if constexpr (ROUTED) {
        const uint2 en = own->entry[s.chunk];
        s.en = (i32x4){(int)(en.x & 0xFFFFu), (int)(en.x >> 16), (int)en.y, 0};
      } else {
        s.en = *reinterpret_cast<const i32x4*>(a.plan + kDecEnt + 4 * s.chunk);
      }
      return;
    }
    // this list is empty: the next one that is not, or the next product
    const int x = (s.home + lane) & 7;
    const bool left = lane < 8 && __hip_atomic_load(sched_counter(a, s.mode, x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) * 8 + x < n;
    const unsigned long long m = __ballot(left);
    if (m) {
      s.list = (s.home + __ffsll((long long)m) - 1) & 7;
    } else {
      s.list = s.home;
      ++s.mode;
      if (s.mode > a.last_mode) continue;
    }
    sched_claim(a, s);
  }
}
template <int QI, bool ROUTED>
__device__ __forceinline__ void sched_rows(const FfnArgs& a, const RoutePlan* own, Sched& s) {
  if (s.chunk < 0) return;
  const int slot = s.en[0], rows = s.en[1], off = s.en[2];
  const bool shared = slot >= a.P;
  s.pairs = !ROUTED && s.mode == 0 && !shared;
  const int first = s.mode == 0 && shared ? off - a.rows_routed - (slot - a.P) * a.sh_rows : off;
#pragma unroll
  for (int h = 0; h < QI / 64; ++h) {
    const int r = min((int)(threadIdx.x & 63) + 64 * h, rows - 1);
    s.src[h] = first + r;
    if (ROUTED) {
      if (s.mode == 0 && !shared) s.src[h] = own->token[off + r];
    } else if (s.pairs && a.por) {
      s.src[h] = a.por[off + r];
    }
  }
}
// Asked for as late as it still comes back in time: a unit whose rows are stored by then costs its token waves no look of their own.
__device__ __forceinline__ void sched_stored(const FfnArgs& a, Sched& s) {
  if (s.chunk >= 0 && s.mode) s.stored = __hip_atomic_load(a.done + s.chunk * kDecDoneStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <int QI>
__device__ __forceinline__ void sched_publish(const FfnArgs& a, const SchedDims& d, const Sched& s, int32_t* q) {
  const int lane = threadIdx.x & 63;
  if (s.chunk < 0) {
    if (lane == 0) q[0] = -1;
  } else {
    const uint32_t pitch = (uint32_t)(s.mode ? d.pitch1 : d.pitch0);
#pragma unroll
    for (int h = 0; h < QI / 64; ++h) q[8 + 64 * h + lane] = (int32_t)((s.pairs ? s.src[h] / (uint32_t)a.k : s.src[h]) * pitch);
    if (lane == 0) {
      q[0] = s.en[0]; q[1] = s.en[2]; q[2] = s.en[1]; q[3] = s.g; q[4] = s.mode; q[5] = s.chunk; q[7] = s.how;
      q[6] = s.mode == 0 || s.stored >= kDone * d.units0;
    }
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// ROLE 0: weight wave, 1: token wave, 2: scheduler, 3: multiplying wave.  All roles execute the same number of barriers.
template <int NTF, int MR, int ROLE, bool ROUTED>
__device__ __forceinline__ void dec_body(const FfnArgs& a, const Routed<DecCfg<NTF, MR>>& rt, unsigned char* s_lds) {
  using C = DecCfg<NTF, MR>;
  [[maybe_unused]] const RoutePlan* own = ROUTED ? &Routed<C>::plan(s_lds) : nullptr;
  constexpr int kShift = MR == 64 ? 7 : 6;                                    // log2 of a slab's contraction elements
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lw = ROLE == 0 ? wave : wave - C::NW;                             // index among the waves of this role
  constexpr bool LOADS = ROLE <= 1;
  const int depth = ROLE == 0 ? a.depth_w : a.depth_t;
  int32_t* queue = reinterpret_cast<int32_t*>(s_lds + C::Q_OFF);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)s_lds;
  const uint32_t q0 = lds0 + C::Q_OFF;

  [[maybe_unused]] Sched sc{};
  [[maybe_unused]] const SchedDims sd = ROLE == 2 ? sched_dims(a) : SchedDims{};
  [[maybe_unused]] int n_chunks = 0, whole = 0;  // whole: units of the first product that are not split
  [[maybe_unused]] bool both = false;            // the first two units are looked up together
  [[maybe_unused]] int pending = -1, pending_by = 0;  // scheduler: chunk of the previous unit, counted inside the slab loop of the present one
  if constexpr (ROLE == 2) {
    // The first two units, three round trips each, the second one's a step behind: its last one alone competes with the bulk
    // loads that the first unit starts.  One after the other the second unit was known 5.8 us into the launch, and
    // nothing can be multiplied before.  With fewer units than workgroups the second claim comes after the first unit's loads:
    // at once, the workgroups that start first would take two and the others none (1 token, 4 experts of 1024 x 896: 20.6 / 22.6 us;
    // 2 tokens, 5 of 1280 x 512: 18.5 / 20.1).  With the plan in LDS only the second claim itself is a round trip, and the first
    // unit's loads do not wait for it.
    n_chunks = ROUTED ? rt.n_chunks : a.plan[0];
    whole = whole_units<C>(a.grid, n_chunks * a.m[0].G, n_chunks * a.m[1].G);
    both = n_chunks * (a.first_mode ? a.m[1].G : a.m[0].G) >= a.grid;
    Sched s0{};
    s0.home = s0.list = (int)(blockIdx.x & 7);
    s0.mode = a.first_mode;
    if constexpr (ROUTED) s0.w = rt.claim;
    else sched_claim(a, s0);
    sched_entry<C, ROUTED>(a, sd, own, n_chunks, whole, s0);
    sc = s0;
    if (both) sched_claim(a, sc);
    sched_rows<C::QI, ROUTED>(a, own, s0);
    if (both && !ROUTED) sched_entry<C, ROUTED>(a, sd, own, n_chunks, whole, sc);
    sched_stored(a, s0);
    sched_publish<C::QI>(a, sd, s0, queue);
  }
  __builtin_amdgcn_s_barrier();
  FfnUnit cur = read_unit(q0);
  if (cur.slot < 0) return;
  FfnUnit nxt{-1, 0, 0, 0, 0, 0, 0, 0};

  // ---- the loading side: position in the stream of slabs
  // Instruction i of a loading wave covers LDS rows (i * waves + lw) * RPI + lane / (64 / RPI).  pm: that row of a 16-row
  // fragment (token waves with two instructions per fragment: of the first one; the second is 8 rows and half a row of
  // pieces further on); piece: the 16 bytes that belong at the lane's position.
  [[maybe_unused]] const int pm = MR == 64 ? lw * 4 + (lane >> 4) : (lw & 1) * 8 + (lane >> 3);
  [[maybe_unused]] const uint32_t piece = (uint32_t)(MR == 64 ? (lane & 15) ^ pm : (lane & 7) ^ (pm >> 1)) << 4;
  [[maybe_unused]] const unsigned char* p_base = nullptr;                     // the loading unit's source
  [[maybe_unused]] uint32_t p_off[C::NTI * NTF] = {};                         // token waves: byte offset of the lane's row per fragment
  [[maybe_unused]] uint32_t p_w = 0, p_ws = 0;                                // weight waves: lane offset, stride between fragments
  // Cache policy of the activation rows' loads.  Where a unit of the first product writes whole 128-byte lines, plain loads do:
  // a line has one writer, nothing reads it before its chunk is complete, and no cache keeps lines of earlier launches; the
  // units of an XCD then share the rows in its L2 (2000 tokens: 265 -> 257 us).  Half lines (units of 64 rows, halves of units of
  // 128) are read past the L2.
  constexpr bool kHalfLines = MR == 64 || C::SPLIT;
  int p_k = 0, p_nk = 1, p_rot = 0, p_n = 0, p_mode = 0;
  [[maybe_unused]] bool p_half = false;
  int p_slot = 0;                                                             // ring slot of the next slab
  bool p_next = false;                                                        // the loading unit is `nxt`
  // Token waves: instructions per slab.  Rows that the chunk does not have are not loaded, down to a whole instruction: their places
  // hold what was there, which reaches only sums that are not stored.  (A chunk has five rows on average at 64 tokens, and a
  // token wave waits for the weights in flight with every instruction.)
  [[maybe_unused]] auto token_loads = [&](const FfnUnit& u) {
    const int n = (u.rows - lw * C::RPI + C::NT * C::RPI - 1) / (C::NT * C::RPI);
    return n > 0 ? n : 0;
  };
  auto aim = [&](const FfnUnit& u, [[maybe_unused]] int qi) {
    const FfnProd& m = u.mode ? a.m[1] : a.m[0];
    p_k = 0;
    p_nk = m.K >> kShift;
    p_rot = first_slab(u, p_nk);
    p_mode = u.mode;
    p_half = C::SPLIT && u.how;
    if constexpr (ROLE == 0) {
      p_base = reinterpret_cast<const unsigned char*>(u.slot < a.P ? m.w + (size_t)u.slot * m.slot_stride
                                                                   : m.w_sh + (size_t)(u.slot - a.P) * m.slot_stride);
      const int f0 = (MR == 128 ? lw >> 1 : 0) + (C::SPLIT && u.how == 2 ? C::PN / 2 : 0);  // pair of instruction 0
      const uint32_t row = u.mode == 0 ? (uint32_t)((pm & 2 ? m.NOUT : 0) + u.g * (MR / 2) + f0 * 16 + 4 * (pm >> 2) + (pm & 1))
                                       : (uint32_t)(u.g * MR + f0 * 32 + 8 * (pm >> 2) + (pm & 3));
      p_w = row * (uint32_t)(m.K * 2) + piece;
      p_ws = (uint32_t)((u.mode + 1) * m.K * 2);
    } else if constexpr (ROLE == 1) {
      p_base = reinterpret_cast<const unsigned char*>(m.x);
      p_n = token_loads(u);
      // the source rows' byte offsets, as the scheduler left them
      constexpr int N = C::NTI * NTF;
      const uint32_t at = q0 + (uint32_t)(qi * C::QI + 8 + pm) * 4u;
      uint32_t r[N];
      read_lds_ints<N, 16 / C::NTI * 4>(at, r);
#pragma unroll
      for (int i = 0; i < N; ++i) p_off[i] = r[i] + (piece ^ (C::NTI == 2 && (i & 1) ? C::RB / 2u : 0u));
    }
  };
  auto issue = [&]() {
    int kk = p_k + p_rot;
    if (kk >= p_nk) kk -= p_nk;
    const unsigned char* src = p_base + (size_t)kk * C::RB;
    if constexpr (ROLE == 0) {
      const uint32_t dst = lds0 + p_slot * C::WSLAB + lw * 1024;
      auto load = [&](auto half) {
#pragma unroll
        for (int i = 0; i < C::NWI; ++i) {
          const int pair = i * C::FPI % C::PN;
          const uint32_t rows = 16 * pair + 2 * (i * C::FPI / C::PN);         // see the fragment layout at the top
          if (!decltype(half)::value || pair < C::PN / 2) load_to_lds<2>(src + rows * p_ws, p_w, dst + i * C::NW * 1024);
        }
      };
      if (C::SPLIT && p_half) load(std::true_type{});
      else load(std::false_type{});
    } else if constexpr (ROLE == 1) {
      const uint32_t dst = lds0 + C::DW * C::WSLAB + p_slot * C::TSLAB + lw * 1024;
#pragma unroll
      for (int i = 0; i < C::NTI * NTF; ++i)
        if (i < p_n) {
          // second product: rows written by other workgroups of this launch, read at the point of coherence
          if (kHalfLines && p_mode) load_to_lds<16>(src, p_off[i], dst + i * C::NT * 1024);
          else load_to_lds<0>(src, p_off[i], dst + i * C::NT * 1024);
        }
    }
    ++p_k;
    p_slot = p_slot + 1 == depth ? 0 : p_slot + 1;
  };
  [[maybe_unused]] int polls = a.wait_polls;
  auto wait_done = [&](const FfnUnit& u, int qi) {  // token waves: the unit's activation rows are stored
    if (u.mode == 0 || u.ready) return;
    wait_stored(a.done + u.chunk * kDecDoneStride, kDone * a.m[0].G, polls, queue + qi * C::QI);
  };

  // ---- the multiplying side
  // wave cw: weight fragments pair and pair + PN, token fragments nh, nh + FSTEP, ...
  constexpr int FSTEP = 8 / C::PN, NF = (NTF + FSTEP - 1) / FSTEP, MFW = 2;
  [[maybe_unused]] const int cw = wave - (C::NW + C::NT + 1), pair = cw / FSTEP, nh = cw % FSTEP;
  [[maybe_unused]] const int n16 = lane & 15, q = lane >> 4;
  [[maybe_unused]] const uint32_t rd = (uint32_t)(n16 * C::RB + ((q ^ (MR == 64 ? n16 : n16 >> 1)) << 4));
  [[maybe_unused]] const uint32_t rd_w = lds0 + pair * C::FRAG + rd, rd_t = lds0 + C::DW * C::WSLAB + nh * C::FRAG + rd;
  [[maybe_unused]] int c_w = 0, c_t = 0;                                                       // ring slots of the slab being multiplied
  int seq = 0;                                                                // units done

  if constexpr (LOADS) {
    if (ROLE == 1) wait_done(cur, 0);
    aim(cur, 0);
    for (int i = 0; i < depth - 1; ++i) issue();
  } else if constexpr (ROLE == 2) {
    if (!both) sched_claim(a, sc);
    if (!both || ROUTED) sched_entry<C, ROUTED>(a, sd, own, n_chunks, whole, sc);
    sched_rows<C::QI, ROUTED>(a, own, sc);
    sched_stored(a, sc);
    sched_publish<C::QI>(a, sd, sc, queue + C::QI);
  }
  __builtin_amdgcn_s_barrier();
  nxt = read_unit(q0 + C::QI * 4);

  for (;;) {
    const FfnProd& m = cur.mode ? a.m[1] : a.m[0];
    const int nk = m.K >> kShift;
    const bool change = nxt.slot >= 0 && nxt.mode != cur.mode;
    [[maybe_unused]] const int nld = (cur.rows + 15) >> 4;                    // live token fragments
    [[maybe_unused]] const int t_n = ROLE == 1 ? token_loads(cur) : 0;
    [[maybe_unused]] const bool half = C::SPLIT && cur.how;
    [[maybe_unused]] const int live = half ? C::PN / 2 : C::PN;               // pairs of weight fragments that the unit has
    if constexpr (ROLE == 3) {
      const int at_pair = C::SPLIT && cur.how == 2 ? live + pair : pair;      // inside the whole unit
      // one loop per number of live token fragments (above four: eight or ten, the rest multiplied for nothing), so that the
      // accumulators stay where they are
      auto unit = [&](auto nb_tag) {
        constexpr int NB = decltype(nb_tag)::value, KS = C::SK / 32;
        f32x4 acc[MFW][NB > 0 ? NB : 1] = {};
        for (int kt = 0; kt < nk; ++kt) {
          if (kt == a.depth_w - 1) __builtin_amdgcn_s_waitcnt(0x0F70);        // the previous unit's stores are acknowledged
          __builtin_amdgcn_s_barrier();
          if constexpr (NB > 0) mul_slab<MFW, NB, KS, C::PN * C::FRAG, FSTEP * C::FRAG>(rd_w + c_w * C::WSLAB, rd_t + c_t * C::TSLAB, acc);
          c_w = c_w + 1 == a.depth_w ? 0 : c_w + 1;
          c_t = c_t + 1 == a.depth_t ? 0 : c_t + 1;
        }
#pragma unroll
        for (int f = 0; f < NB; ++f) {
          const int tr = (nh + FSTEP * f) * 16 + n16;
          if (tr < cur.rows) {
            uint16_t* row = m.out + (size_t)(cur.off + tr) * m.NOUT;
            const f32x4 v = acc[0][f], w = acc[1][f];
            if (cur.mode == 0) {
              ushort4 o;
              o.x = f32_to_bf16(silu_f32(v[0]) * v[2]); o.y = f32_to_bf16(silu_f32(v[1]) * v[3]);
              o.z = f32_to_bf16(silu_f32(w[0]) * w[2]); o.w = f32_to_bf16(silu_f32(w[1]) * w[3]);
              // agent scope: written through to the point of coherence of the GPU's XCDs
              unsigned long long bits;
              __builtin_memcpy(&bits, &o, 8);
              __hip_atomic_store(reinterpret_cast<unsigned long long*>(row + cur.g * (MR / 2) + at_pair * 16 + 4 * q), bits, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
            } else {
              union { uint16_t h[8]; uint4 u; } o;
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                o.h[r] = f32_to_bf16(v[r]);
                o.h[4 + r] = f32_to_bf16(w[r]);
              }
              *reinterpret_cast<uint4*>(row + cur.g * MR + pair * 32 + 8 * q) = o.u;
            }
          }
        }
      };
      const int nf = !C::SPLIT || pair < live ? (nld - nh + FSTEP - 1) / FSTEP : 0;  // this wave's live token fragments
      if (NF >= 10 && nf > 8) unit(std::integral_constant<int, NF >= 10 ? 10 : 0>{});
      else if (NF >= 8 && nf > 4) unit(std::integral_constant<int, NF >= 8 ? 8 : 0>{});
      else if (NF >= 4 && nf == 4) unit(std::integral_constant<int, NF >= 4 ? 4 : 0>{});
      else if (NF >= 3 && nf == 3) unit(std::integral_constant<int, NF >= 3 ? 3 : 0>{});
      else if (NF >= 2 && nf == 2) unit(std::integral_constant<int, NF >= 2 ? 2 : 0>{});
      else if (nf >= 1) unit(std::integral_constant<int, 1>{});
      else unit(std::integral_constant<int, 0>{});
      if (wait_expired(cur, q0 + (uint32_t)((seq & 3) * C::QI) * 4u)) {       // over what this wave has just stored (second product: a whole unit)
        __builtin_amdgcn_s_waitcnt(0x0F70);
#pragma unroll 1
        for (int tr = nh * 16 + n16; tr < cur.rows; tr += FSTEP * 16)
          store_nan(m.out + (size_t)(cur.off + tr) * m.NOUT + cur.g * MR + pair * 32 + 8 * q);
      }
    } else
    for (int kt = 0; kt < nk; ++kt) {
      if constexpr (LOADS) {
        // this wave's part of slab kt has landed once only later slabs' loads are outstanding
        const int ahead_next = p_next ? p_k : 0;                              // slabs of nxt in flight
        const int ahead = (p_next ? nk : p_k) - (kt + 1);                     // later slabs of cur
        wait_vm_upto(ROLE == 0 ? (half ? C::NWI / 2 : C::NWI) * ahead + (C::SPLIT && p_half ? C::NWI / 2 : C::NWI) * ahead_next : t_n * ahead + p_n * ahead_next);
      }
      __builtin_amdgcn_s_barrier();                                           // everyone's part is there, slab kt-1 has been read
      if constexpr (ROLE == 2) {
        if (kt == a.depth_w - 1 && pending >= 0) {
          // every multiplying wave has waited for its stores of the previous unit
          if (lane == 0) __hip_atomic_fetch_add(a.done + pending * kDecDoneStride, pending_by, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          pending = -1;
        }
        // the unit after the next: one round trip at a time, each used slabs after it was started where the unit has enough of them, from about
        // eight on (a wait here is a wait for everyone at the barrier)
        const SchedSteps at = steps_spread(nk);
        if (kt == at.claim) sched_claim(a, sc);
        if (kt == at.entry) sched_entry<C, ROUTED>(a, sd, own, n_chunks, whole, sc);
        if (kt == at.rows) sched_rows<C::QI, ROUTED>(a, own, sc);
        if (kt == at.stored) sched_stored(a, sc);
        if (kt == at.publish) sched_publish<C::QI>(a, sd, sc, queue + ((seq + 2) & 3) * C::QI);
      } else if constexpr (LOADS) {
        if (!p_next && p_k == nk && nxt.slot >= 0 && !(ROLE == 1 && change)) {
          if (ROLE == 1) wait_done(nxt, (seq + 1) & 3);
          aim(nxt, (seq + 1) & 3);
          p_next = true;
        }
        if (p_next || p_k < nk) issue();
      }
    }
    if (nxt.slot < 0 || change) {
      // the stores are acknowledged (and nothing is in flight at the end of the kernel): count the unit at once
      if constexpr (ROLE != 2) __builtin_amdgcn_s_waitcnt(0x0F70);
      __builtin_amdgcn_s_barrier();
      if constexpr (ROLE == 2) {
        if (cur.mode == 0 && lane == 0) __hip_atomic_fetch_add(a.done + cur.chunk * kDecDoneStride, done_by(cur), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if (nxt.slot < 0) return;
    } else if constexpr (ROLE == 2) {
      pending = cur.mode == 0 ? cur.chunk : -1;
      pending_by = done_by(cur);
    }
    ++seq;
    cur = nxt;
    nxt = read_unit(q0 + (uint32_t)(((seq + 1) & 3) * C::QI) * 4u);
    if constexpr (LOADS) {
      if (!p_next) {  // nothing of this unit is in flight yet (token waves, from the first product to the second)
        if (ROLE == 1) wait_done(cur, seq & 3);
        aim(cur, seq & 3);
        for (int i = 0; i < depth - 1; ++i) issue();
      }
      p_next = false;
    }
  }
}

template <int NTF, int MR, bool ROUTED>
__device__ __forceinline__ void dec_roles(const FfnArgs& a, const Routed<DecCfg<NTF, MR>>& rt, unsigned char* s_lds) {
  using C = DecCfg<NTF, MR>;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (wave < C::NW) dec_body<NTF, MR, 0, ROUTED>(a, rt, s_lds);
  else if (wave < C::NW + C::NT) dec_body<NTF, MR, 1, ROUTED>(a, rt, s_lds);
  else if (wave == C::NW + C::NT) dec_body<NTF, MR, 2, ROUTED>(a, rt, s_lds);
  else dec_body<NTF, MR, 3, ROUTED>(a, rt, s_lds);
}

template <int NTF, int MR>
__global__ __launch_bounds__((DecCfg<NTF, MR>::THREADS)) void k_ffn_dec(FfnArgs a) {
  __shared__ __align__(1024) unsigned char s_lds[DecCfg<NTF, MR>::LDS];
  if (a.pick && picked(a) != a.pick) return;  // the counts chose the other kernel
  dec_roles<NTF, MR, false>(a, {}, s_lds);
}

// The same for a call that routes itself, with one wave more: it selects as the others do, in the first workgroup it then writes what
// the call hands out, and ends.
template <int NTF, int MR>
__global__ __launch_bounds__((DecCfg<NTF, MR>::THREADS + 64)) void k_ffn_dec_routed(FfnArgs a, FfnRoute r) {
  using C = DecCfg<NTF, MR>;
  constexpr int kSched = C::NW + C::NT, kWriter = C::THREADS / 64;
  __shared__ __align__(1024) unsigned char s_lds[Routed<C>::LDS];
  RouteScratch* sc = reinterpret_cast<RouteScratch*>(s_lds);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Routed<C> rt;
  // (the first claim is made by every workgroup whatever the plan, and comes back while the experts are selected)
  if (wave == kSched && (threadIdx.x & 63) == 0)
    rt.claim = claim_next(sched_counter(a, 0, (int)(blockIdx.x & 7)));
  if (wave == kSched) {
    // Each of the arguments' cache lines (of 64 bytes) would be a round trip where it is first read, in the chain up to the first loads: this
    // wave, which mostly has no token to select for, brings them in meanwhile.
    const auto* args = (const __attribute__((address_space(4))) uint32_t*)__builtin_amdgcn_kernarg_segment_ptr();
    uint32_t any = 0;
#pragma unroll
    for (unsigned i = 0; i < (sizeof(FfnArgs) + sizeof(FfnRoute)) / 4; i += 16) any |= args[i];
    asm volatile("" ::"s"(any));
  }
  const bool writes = blockIdx.x == 0;
  route_select<kWriter + 1, kSched + 1>(r, a.P, sc, writes ? 2 : 1);
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  if (wave == kSched) rt.n_chunks = route_rank<false>(r, a.P, 16 * NTF, sc[0], Routed<C>::plan(s_lds));
  if (wave == kWriter) {
    if (writes) route_rank<true>(r, a.P, 16 * NTF, sc[1], Routed<C>::plan(s_lds));
    // the first unit is published behind this barrier, and only then is anything loaded into the rings that the scratch lies in
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    return;
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  dec_roles<NTF, MR, true>(a, rt, s_lds);
}

template <int NTF, int MR>
int launch(FfnArgs a, const FfnPlanShape& sh, int n_cu, hipStream_t st, [[maybe_unused]] const FfnRoute* route = nullptr) {
  using C = DecCfg<NTF, MR>;
  a.m[0].G = a.m[0].NOUT / (MR / 2);
  a.m[1].G = a.m[1].NOUT / MR;
  const int nk = (a.m[0].K < a.m[1].K ? a.m[0].K : a.m[1].K) / C::SK;  // >= 2
  a.depth_w = C::DW < nk ? C::DW : nk;
  a.depth_t = C::DT < nk ? C::DT : nk;
  const bool merged = sh.merged != 0;
  for (int mode = 0; mode < (merged ? 1 : 2); ++mode) {
    a.first_mode = mode;
    a.last_mode = merged ? 1 : mode;
    const long long units = (long long)sh.dec_cap * (merged ? a.m[0].G + a.m[1].G : a.m[mode].G);
    a.grid = units < n_cu ? (int)units : n_cu;
    const dim3 grid(a.grid);
    if constexpr (NTF <= 4) {
      if (route) {
        hipLaunchKernelGGL((k_ffn_dec_routed<NTF, MR>), grid, dim3(C::THREADS + 64), 0, st, a, *route);
        EW_LAUNCH_CHECK("k_ffn_dec_routed");
        continue;
      }
    }
    hipLaunchKernelGGL((k_ffn_dec<NTF, MR>), grid, dim3(C::THREADS), 0, st, a);
    EW_LAUNCH_CHECK("k_ffn_dec");
  }
  return EW_OK;
}

}  // namespace

bool ffn_routes(const FfnPlanShape& sh, int T, int E, int k, int P, int S) {
  return sh.dec >= 1 && sh.dec <= 4 && !sh.big && sh.merged && T <= kRouteTokens && T * k <= kRoutePairs && k <= 16 && k <= E && E <= 256 &&
         P <= kPlanMaxP && S * dec_chunks(T, 16 * sh.dec) <= kRouteShared;
}

int launch_ffn_dec(FfnArgs a, const FfnPlanShape& sh, int n_cu, hipStream_t st, const FfnRoute* route) {
  const int H = a.m[0].K, I = a.m[1].K;
  // Units of 128 weight rows read every token row half as often as units of 64: C1-shaped calls 261 -> 247 us, 48 tokens on
  // 84 small experts 111 -> 101 us.  Only where even 64-row units leave a compute unit no more than two of the first
  // product (one token: 8 experts) does the finer split win: 44 -> 42 us.  (Its slabs are 128 contraction elements, of
  // which a unit must have two.)
  const bool fine = sh.dec == 1 && H >= 256 && I >= 256 && (long long)sh.dec_cap * (I / 32) <= 2 * n_cu;
  switch (sh.dec) {
    case 1: return fine ? launch<1, 64>(a, sh, n_cu, st, route) : launch<1, 128>(a, sh, n_cu, st, route);
    case 2: return launch<2, 128>(a, sh, n_cu, st, route);
    case 4: return launch<4, 128>(a, sh, n_cu, st, route);
    case 10: return launch<10, 256>(a, sh, n_cu, st);
    default: return H % 256 == 0 ? launch<8, 256>(a, sh, n_cu, st) : launch<8, 128>(a, sh, n_cu, st);
  }
}

}  // namespace ew
