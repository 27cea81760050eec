// Grouped SwiGLU expert FFN for calls with many rows per slot on gfx950: 256 weight rows x up to 256 token rows per unit.
//
// What bounds it is not known: loads and MFMAs together, more than either.  8192 tokens, this kernel alone, base-only / 20 adapters: complete
// 989 / 1218 us, 1.70 / 2.24 M cycles at 1.72 / 1.84 GHz (MFMA busy 64 / 51 %, TD 78 / 88 %); with nothing multiplied 801 / 1111 us, 1.91 / 2.60 M
// cycles at 2.38 / 2.34 GHz (TD 92 / 94 %).  So the loads alone take 0.81 / 0.91 of the time, and the power limit lowers the clock once there are
// MFMAs beside them.  But a walk that makes the loads alone 11 / 7 % shorter makes the pass 0.6 to 1.3 % shorter (sched_rows), so they do not hold it by
// themselves; what the MFMAs' idle cycles wait for is not measured.  One token slab and up to three weight halves are in flight while a slab is
// multiplied.
#include "ffn_roles.h"

namespace ew {

namespace {

// LDS rows: 64 contraction elements, 128 bytes, eight 16-byte pieces, the piece index XOR-ed with swz(row).
constexpr int kHalf = 128 * 128;           // bytes of half a weight slab (128 rows), the unit of the weight ring
constexpr int kWRing = 5;                  // halves in the weight ring
constexpr int kTSlab = 256 * 128;          // bytes of a token slab
constexpr int kTRing = 2;
constexpr int kQI = 8 + 256;               // ints of a queue entry
constexpr int kTOff = kWRing * kHalf, kQOff = kTOff + kTRing * kTSlab, kLds = kQOff + 4 * kQI * 4;
static_assert(kLds <= 160 * 1024, "LDS budget of a CU");
constexpr int kAlone = 1;                  // FfnUnit::how: no other chunk reads this unit's weights
constexpr int kThreads = 768;              // waves 0-1 load weights, 2 token rows, 3 schedules, 4-11 multiply

__device__ __forceinline__ int swz(int r) { return ((r >> 1) ^ ((r & 1) << 2)) & 7; }

// ------------------------------------------------------------------------------------------
// The scheduling wave: lane i < 8 knows list (home + i) % 8 of the plan (ffn_plan.h).
struct Sched {
  int w, mode, t, home;      // claim in flight: list (home + t) % 8
  int n_ent, chunks;         // lane i: entries and chunks of list (home + i) % 8
  int ent[6];                // lane e: entry e of the claimed list
  int ok, slot, rows, off, g, chunk, how;
  int pairs;                 // src are pairs, not rows yet
  int stored;                // first-product units of the chunk that are stored
  uint32_t src[4];
};

__device__ __forceinline__ int32_t* counter(const FfnArgs& a, int mode, int list) { return a.plan + kPlanCtr + (mode * 8 + list) * kPlanCtrStride; }

__device__ __forceinline__ void sched_claim(const FfnArgs& a, Sched& s) {
  if ((threadIdx.x & 63) == 0 && s.mode <= a.last_mode)
    s.w = claim_next(counter(a, s.mode, (s.home + s.t) & 7));
}
__device__ __forceinline__ void load_entry(const FfnArgs& a, Sched& s, int e) {  // of a list that has entries; lanes past its last take that one
  const int x = (s.home + s.t) & 7, n = __shfl(s.n_ent, s.t, 64);
  const int32_t* en = a.plan + kPlanHdr + kEnt * (x * a.cap + min(e, n - 1));
#pragma unroll
  for (int i = 0; i < kEnt; ++i) s.ent[i] = en[i];
}
__device__ __forceinline__ void sched_entry(const FfnArgs& a, const SchedDims& d, Sched& s) {
  const int lane = threadIdx.x & 63;
  for (;;) {
    s.ok = s.mode <= a.last_mode;
    if (!s.ok) return;
    const int G = s.mode ? d.units1 : d.units0;
    s.w = __builtin_amdgcn_readfirstlane(s.w);
    if (s.w < __shfl(s.chunks, s.t, 64) * G) {
      load_entry(a, s, lane);
      return;
    }
    // this list is empty: the next one that is not, or the next product
    const bool left = lane < 8 && __hip_atomic_load(counter(a, s.mode, (s.home + lane) & 7), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < s.chunks * G;
    const unsigned long long m = __ballot(left);
    s.t = m ? __ffsll((long long)m) - 1 : 0;
    if (!m && ++s.mode > a.last_mode) continue;
    sched_claim(a, s);
  }
}
__device__ __forceinline__ void sched_rows(const FfnArgs& a, const SchedDims& d, Sched& s) {
  if (!s.ok) return;
  const int lane = threadIdx.x & 63, G = s.mode ? d.units1 : d.units0;
  unsigned long long m;
  for (int e0 = 0;; e0 += 64) {  // every claimed unit lies in exactly one entry
    if (e0) load_entry(a, s, e0 + lane);
    m = __ballot(s.w >= s.ent[2] * G && s.w < (s.ent[2] + s.ent[1]) * G);
    if (m || e0 > kPlanMaxEnt) break;
  }
  const int e = __ffsll((long long)m) - 1;  // (the first of equal ones)
  const int nch = __shfl(s.ent[1], e, 64), base = __shfl(s.ent[2], e, 64), bts = __shfl(s.ent[3], e, 64), c = __shfl(s.ent[4], e, 64);
  const int i = s.w - base * G, j = i % nch;
  s.slot = __builtin_amdgcn_readfirstlane(__shfl(s.ent[0], e, 64));
  s.g = i / nch;
  // Every unit walks over K from slab 0 on, so that a row's result does not depend on the chunk it falls into, that is on what else
  // is in the batch.  Half of the units walking over each pair of slabs in the opposite order, by the parity of chunk and feature
  // group, would shorten the loads alone (us: 819 -> 726 base-only, 1121 -> 1037 with 20 adapters) and the whole pass by 0.6 %.
  s.how = nch == 1 ? kAlone : 0;
  s.rows = min(bts, c - j * bts);
  s.off = __shfl(s.ent[5], e, 64) + j * bts;
  s.chunk = ((s.home + s.t) & 7) * a.list_chunks + base + j;
  const bool shared = s.slot >= a.P;
  s.pairs = s.mode == 0 && !shared;
  const int first = s.mode == 0 && shared ? s.off - a.rows_routed - (s.slot - a.P) * a.sh_rows : s.off;
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    const int r = min(lane + 64 * h, s.rows - 1);
    s.src[h] = s.pairs && a.por ? a.por[s.off + r] : first + r;
  }
}
// Asked for as late as it still comes back in time: a unit whose rows are stored by then costs its token wave no look of its own.
__device__ __forceinline__ void sched_stored(const FfnArgs& a, Sched& s) {
  if (s.ok && s.mode) s.stored = __hip_atomic_load(a.done + s.chunk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void sched_publish(const FfnArgs& a, const SchedDims& d, const Sched& s, int32_t* q) {
  const int lane = threadIdx.x & 63;
  if (!s.ok) {
    if (lane == 0) q[0] = -1;
  } else {
    const uint32_t pitch = (uint32_t)(s.mode ? d.pitch1 : d.pitch0);
#pragma unroll
    for (int h = 0; h < 4; ++h) q[8 + 64 * h + lane] = (int32_t)((s.pairs ? s.src[h] / (uint32_t)a.k : s.src[h]) * pitch);
    if (lane == 0) {
      q[0] = s.slot; q[1] = s.off; q[2] = s.rows; q[3] = s.g; q[4] = s.mode; q[5] = s.chunk; q[7] = s.how;
      q[6] = s.mode == 0 || s.stored >= d.units0;
    }
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// ------------------------------------------------------------------------------------------
// An operand read of a k-step, issued without waiting: 16 bytes per lane at a constant distance.
template <int OFF>
__device__ __forceinline__ void read_op(uint32_t at, u32x4& v) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(v) : "v"(at), "n"(OFF));
}
constexpr int kWFrag = 4096, kTFrag = 8192;   // between a wave's weight fragments, its token fragments
template <int N>
__device__ __forceinline__ void wait_lds() {
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void use(u32x4& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ f32x16 mfma(const u32x4& a, const u32x4& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// One unit's K loop of a multiplying wave with NB live token fragments.  step(kt) is called before slab kt is read: it
// meets the other waves at the barrier and moves wa / tb to the slab.
template <int NB, typename Step>
__device__ __forceinline__ void multiply(int nk, uint32_t& wa, uint32_t& tb, f32x16 (&acc)[2][NB > 0 ? NB : 1], Step step) {
  if constexpr (NB == 0) {
    for (int kt = 0; kt < nk; ++kt) step(kt);
  } else if constexpr (NB < 3) {
    // both operand sets double: the reads run a k-step ahead of the MFMAs, across slabs too
    u32x4 a[2][2], b[2][NB];
    auto read = [&](int c, uint32_t x) {
      read_op<0>(wa ^ x, a[c][0]);
      read_op<kWFrag>(wa ^ x, a[c][1]);
      read_op<0>(tb ^ x, b[c][0]);
      if constexpr (NB > 1) read_op<kTFrag>(tb ^ x, b[c][1]);
    };
    auto landed = [&](int c) {
      wait_lds<0>();
      use(a[c][0]); use(a[c][1]);
#pragma unroll
      for (int f = 0; f < NB; ++f) use(b[c][f]);
    };
    auto mul = [&](int c) {
#pragma unroll
      for (int f = 0; f < NB; ++f)
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i][f] = mfma(a[c][i], b[c][f], acc[i][f]);
    };
    for (int kt = 0; kt < nk; ++kt) {
      step(kt);
      read(0, 0u);
      if (kt) mul(1);
      landed(0);
      read(1, 16u); mul(0); landed(1);
      read(0, 32u); mul(1); landed(0);
      read(1, 48u); mul(0); landed(1);
    }
    mul(1);
  } else {
    // 96 or 128 accumulators leave room for one set of operands.  A k-step multiplies weight fragment 0 with the token
    // fragments in one order and weight fragment 1 with them in the opposite one, and the next k-step starts where this one
    // ended: a register set is read into again as soon as its last MFMA is issued, and needed again at least NB - 1 MFMAs
    // later.  REV: the token fragments' first order is descending.
    u32x4 a[2], b[NB];
    auto read_b = [&](uint32_t at, auto f_tag) { read_op<kTFrag * decltype(f_tag)::value>(at, b[decltype(f_tag)::value]); };
    auto kstep = [&](auto rev_tag, bool more, auto next) {  // next(): moves wa / tb to the following k-step, returns its XOR
      constexpr bool REV = decltype(rev_tag)::value;
      auto first = [&](auto i_tag) {
        constexpr int i = decltype(i_tag)::value, f = REV ? NB - 1 - i : i;
        wait_lds<NB - i>();  // later reads: the NB - 1 - i fragments behind this one, and weight fragment 1
        if (i == 0) use(a[0]);
        use(b[f]);
        acc[0][f] = mfma(a[0], b[f], acc[0][f]);
        __builtin_amdgcn_sched_barrier(0);
      };
      first(std::integral_constant<int, 0>{});
      first(std::integral_constant<int, 1>{});
      first(std::integral_constant<int, 2>{});
      if constexpr (NB > 3) first(std::integral_constant<int, 3>{});
      wait_lds<0>();
      use(a[1]);
      uint32_t x = 0;
      if (more) {
        x = next();
        read_op<0>(wa ^ x, a[0]);
      }
      auto second = [&](auto i_tag) {
        constexpr int i = decltype(i_tag)::value, f = REV ? i : NB - 1 - i;
        acc[1][f] = mfma(a[1], b[f], acc[1][f]);
        __builtin_amdgcn_sched_barrier(0);
        if (more) read_b(tb ^ x, std::integral_constant<int, f>{});
        __builtin_amdgcn_sched_barrier(0);
      };
      second(std::integral_constant<int, 0>{});
      second(std::integral_constant<int, 1>{});
      second(std::integral_constant<int, 2>{});
      if constexpr (NB > 3) second(std::integral_constant<int, 3>{});
      if (more) read_op<kWFrag>(wa ^ x, a[1]);
      __builtin_amdgcn_sched_barrier(0);
    };
    step(0);
    read_op<0>(wa, a[0]);
    read_b(tb, std::integral_constant<int, 0>{});
    read_b(tb, std::integral_constant<int, 1>{});
    read_b(tb, std::integral_constant<int, 2>{});
    if constexpr (NB > 3) read_b(tb, std::integral_constant<int, 3>{});
    read_op<kWFrag>(wa, a[1]);
    const std::false_type fwd{};
    const std::true_type rev{};
    // The loop's place in the instruction stream is pinned: left to chance, a change anywhere before it moves passes of 8192
    // tokens by up to 1 % (4 bytes behind a 128-byte line 1129 us, on one 1134, other distances 1131 .. 1137; unpinned 1127 or 1140).
    asm volatile(".p2align 7\n\ts_nop 0");
    for (int kt = 0; kt < nk; ++kt) {
      kstep(fwd, true, [] { return 16u; });
      kstep(rev, true, [] { return 32u; });
      kstep(fwd, true, [] { return 48u; });
      kstep(rev, kt + 1 < nk, [&] { step(kt + 1); return 0u; });
    }
  }
}

// ROLE 0: weight wave, 1: token wave, 2: scheduler, 3: multiplying wave.  All roles execute the same number of barriers.
template <int ROLE>
__device__ __forceinline__ void big_body(const FfnArgs& a, unsigned char* s_lds) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int32_t* queue = reinterpret_cast<int32_t*>(s_lds + kQOff);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)s_lds;
  const uint32_t q0 = lds0 + kQOff;

  [[maybe_unused]] Sched sc{};
  [[maybe_unused]] const SchedDims sd = ROLE == 2 ? sched_dims(a) : SchedDims{};
  [[maybe_unused]] int pending = -1;  // scheduler: chunk of the previous unit, counted in the last slab of the present one
  if constexpr (ROLE == 2) {
    sc.home = (int)(blockIdx.x & 7);
    sc.mode = a.first_mode;
    if (lane < 8) {
      const int x = (sc.home + lane) & 7;
      sc.n_ent = a.plan[x];
      sc.chunks = a.plan[8 + x];
    }
    sched_claim(a, sc);
    sched_entry(a, sd, sc);
    sched_rows(a, sd, sc);
    sched_stored(a, sc);
    sched_publish(a, sd, sc, queue);
  }
  __builtin_amdgcn_s_barrier();
  FfnUnit cur = read_unit(q0);
  if (cur.slot < 0) return;
  FfnUnit nxt{-1, 0, 0, 0, 0, 0, 0, 0};

  // ---- the loading side: position in the stream of weight halves / token slabs
  [[maybe_unused]] const int lw = wave & 1;
  // weight waves: instruction n of a half covers LDS rows 128 half + 16 n + 8 lw + lane / 8; token wave: rows 8 n + lane / 8
  [[maybe_unused]] const int prow = ROLE == 0 ? 8 * lw + (lane >> 3) : lane >> 3;
  [[maybe_unused]] const uint32_t piece = (uint32_t)((lane & 7) ^ swz(prow)) << 4;
  [[maybe_unused]] const unsigned char* p_base = nullptr;
  [[maybe_unused]] uint32_t p_w = 0, p_up = 0, p_i = 0, p_wr = 0;
  [[maybe_unused]] bool p_alone = false;                                      // no other chunk reads this unit's weights
  [[maybe_unused]] bool p_part = false;                                       // the unit's second half of weight rows does not exist
  [[maybe_unused]] uint32_t p_off[ROLE == 1 ? 32 : 1] = {};
  int p_h = 0, p_n = 1, p_nfl = 0, p_slot = 0;                                // next piece of the loading unit, their number
  bool p_next = false;
  auto aim = [&](const FfnUnit& u, [[maybe_unused]] int qi) {
    const FfnProd& m = u.mode ? a.m[1] : a.m[0];
    p_h = 0;
    if constexpr (ROLE == 0) {
      p_n = m.K >> 5;
      const uint32_t k2 = (uint32_t)(m.K * 2);
      p_base = reinterpret_cast<const unsigned char*>(u.slot < a.P ? m.w + (size_t)u.slot * m.slot_stride
                                                                   : m.w_sh + (size_t)(u.slot - a.P) * m.slot_stride);
      const uint32_t row = u.mode == 0 ? (uint32_t)(u.g * 128 + 16 * (lane >> 5) + 8 * lw + ((lane >> 3) & 3))
                                       : (uint32_t)(u.g * 256 + 32 * (lane >> 5) + 8 * lw + ((lane >> 3) & 3));
      p_w = row * k2 + piece;
      p_up = (u.mode == 0 ? (uint32_t)m.NOUT : 16u) * k2;
      p_i = 4u * k2;
      p_wr = (u.mode == 0 ? 32u : 64u) * k2;
      p_alone = u.how & kAlone;
      p_part = u.mode == 1 && u.g * 256 + 128 >= m.NOUT;
    } else if constexpr (ROLE == 1) {
      p_n = m.K >> 6;
      p_base = reinterpret_cast<const unsigned char*>(m.x);
      p_nfl = (u.rows + 31) >> 5;
      read_lds_ints<32, 32>(q0 + (uint32_t)(qi * kQI + 8 + prow) * 4u, p_off);
#pragma unroll
      for (int n = 0; n < 32; ++n) p_off[n] += piece ^ (n & 1 ? 64u : 0u);
    }
  };
  auto issue = [&]() {
    if constexpr (ROLE == 0) {
      const int half = p_h & 1;
      const unsigned char* src = p_base + (size_t)(p_h >> 1) * 128 + (half && !p_part ? 2 * p_wr : 0u);
      const uint32_t dst = lds0 + p_slot * kHalf + lw * 1024;
      auto load = [&](auto aux) {
#pragma unroll
        for (int n = 0; n < 8; ++n)
          load_to_lds<decltype(aux)::value>(src + ((n & 1) * p_up + ((n >> 1) & 1) * p_i + (n >> 2) * p_wr), p_w, dst + n * 2048);
      };
      // Cache policy: weights that one chunk alone reads stream past the caches (nt), others are kept for the chunks beside
      // it (sc1).
      if (p_alone) load(std::integral_constant<int, 2>{});
      else load(std::integral_constant<int, 16>{});
      p_slot = p_slot + 1 == kWRing ? 0 : p_slot + 1;
    } else if constexpr (ROLE == 1) {
      const unsigned char* src = p_base + (size_t)p_h * 128;
      const uint32_t dst = lds0 + kTOff + p_slot * kTSlab;
#pragma unroll
      for (int f = 0; f < 8; ++f)
        if (f < p_nfl) {
#pragma unroll
          for (int n = 4 * f; n < 4 * f + 4; ++n)
            load_to_lds<0>(src, p_off[n], dst + n * 1024);
        }
      p_slot ^= 1;
    }
    ++p_h;
  };
  [[maybe_unused]] int polls = a.wait_polls;
  auto wait_done = [&](const FfnUnit& u, int qi) {
    if (u.mode == 0 || u.ready) return;
    wait_stored(a.done + u.chunk, a.m[0].G, polls, queue + qi * kQI);
  };

  // ---- the multiplying side: wave (wr, p) owns 64 weight rows and token fragments p, p + 2, ...
  [[maybe_unused]] const int cw = wave - 4, wr = cw >> 1, p = cw & 1;
  [[maybe_unused]] const int r32 = lane & 31, h = lane >> 5;
  [[maybe_unused]] const uint32_t lane_off = (uint32_t)(r32 * 128 + (((4 * h) ^ swz(r32)) << 4));
  [[maybe_unused]] int c_w = 0, c_t = 0;
  int seq = 0;

  if constexpr (ROLE == 0) {
    aim(cur, 0);
    for (int i = 0; i < 3; ++i) issue();
  } else if constexpr (ROLE == 1) {
    wait_done(cur, 0);
    aim(cur, 0);
    issue();
  } else if constexpr (ROLE == 2) {
    sched_claim(a, sc);
    sched_entry(a, sd, sc);
    sched_rows(a, sd, sc);
    sched_stored(a, sc);
    sched_publish(a, sd, sc, queue + kQI);
  }
  __builtin_amdgcn_s_barrier();
  nxt = read_unit(q0 + kQI * 4);

  for (;;) {
    const FfnProd& m = cur.mode ? a.m[1] : a.m[0];
    const int nk = m.K >> 6;
    const bool change = nxt.slot >= 0 && nxt.mode != cur.mode;
    if constexpr (ROLE == 3) {
      const int nfl = (cur.rows + 31) >> 5, nb = (nfl - p + 1) >> 1;
      uint32_t wa = 0, tb = 0;
      auto step = [&](int kt) {
        if (kt == nk - 1) __builtin_amdgcn_s_waitcnt(0x0F70);                 // the previous unit's stores are acknowledged
        __builtin_amdgcn_s_barrier();
        int half = c_w + (wr >> 1);
        half = half >= kWRing ? half - kWRing : half;
        wa = lds0 + half * kHalf + (wr & 1) * 8192 + lane_off;
        tb = lds0 + kTOff + c_t * kTSlab + p * 4096 + lane_off;
        c_w = c_w + 2 >= kWRing ? c_w + 2 - kWRing : c_w + 2;
        c_t ^= 1;
      };
      auto unit = [&](auto nb_tag) {
        constexpr int NB = decltype(nb_tag)::value;
        f32x16 acc[2][NB > 0 ? NB : 1];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int f = 0; f < (NB > 0 ? NB : 1); ++f)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][f][e] = 0.f;
        multiply<NB>(nk, wa, tb, acc, step);
        // Every wave is done with the unit's last slab, whose ring slots (two weight halves, one token slab: 64 KB) are not
        // loaded into before the next unit's first barrier.  Each wave turns its output there, 8 KB at a time, so that whole
        // rows of it leave in one piece: accumulator element e = 4 b + j of fragment i is weight row 8 b + 4 h + j of the
        // fragment and token r32, a lane would store 16 bytes here and there.
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if constexpr (NB > 0) {
          // (lane numbers the compiler cannot see through: it would compute every address below once, outside the unit loop,
          // have no registers for them and reload them from scratch memory between the stores, each time waiting for the
          // stores before: 200 of 1100 us)
          int el = lane;
          asm volatile("" : "+v"(el));
          const int t32 = el & 31, hh = el >> 5;
          const int hw = c_w + 3 + (cw >> 1), half = hw >= kWRing ? hw - kWRing : hw;   // the two halves before c_w
          unsigned char* tile = cw < 4 ? s_lds + half * kHalf + (cw & 1) * 8192 : s_lds + kTOff + (c_t ^ 1) * kTSlab + (cw - 4) * 8192;
          if (cur.mode == 0) {
            // 32 features = 64 bytes per token row, up to 128 rows
            unsigned char* put = tile + t32 * 64;
            const int sw = (t32 >> 2) & 3;
#pragma unroll
            for (int f = 0; f < NB; ++f)
#pragma unroll
              for (int b = 0; b < 2; ++b) {
                union { uint16_t h16[8]; u32x4 v; } o;
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                  for (int j = 0; j < 4; ++j) o.h16[4 * i + j] = f32_to_bf16(silu_f32(acc[i][f][4 * b + j]) * acc[i][f][8 + 4 * b + j]);
                *reinterpret_cast<u32x4*>(put + f * 2048 + (((2 * hh + b) ^ sw) << 4)) = o.v;
              }
            // 16 rows per instruction; the piece's place does not depend on n
            const int t0 = el >> 2, pc = el & 3;
            const unsigned char* get = tile + t0 * 64 + ((pc ^ ((t0 >> 2) & 3)) << 4);
            const size_t pitch = (size_t)m.NOUT;
            uint16_t* dst = m.out + (size_t)(cur.off + p * 32 + t0) * pitch + cur.g * 128 + wr * 32 + pc * 8;
            int tr = p * 32 + t0;
#pragma unroll
            for (int n = 0; n < 2 * NB; ++n) {
              const u32x4 v = *reinterpret_cast<const u32x4*>(get + n * 1024);
              if (tr < cur.rows) store_agent_16(dst, v);
              const int step = n & 1 ? 48 : 16;                               // on to token fragment p + 2 (n + 1) / 2
              tr += step;
              dst += step * pitch;
            }
          } else if (cur.g * 256 + wr * 64 < m.NOUT) {
            // 64 features = 128 bytes per token row, two fragments at a time
            unsigned char* put = tile + t32 * 128;
            const int sw = t32 & 7;
            const int t0 = el >> 3, pc = el & 7;
            const unsigned char* get = tile + t0 * 128 + ((pc ^ t0) << 4);
            const size_t pitch = (size_t)m.NOUT;
            uint16_t* dst = m.out + (size_t)(cur.off + p * 32 + t0) * pitch + cur.g * 256 + wr * 64 + pc * 8;
            int tr = p * 32 + t0;
#pragma unroll
            for (int f0 = 0; f0 < NB; f0 += 2) {
#pragma unroll
              for (int f = f0; f < f0 + 2 && f < NB; ++f)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                  union { uint16_t h16[8]; u32x4 v; } o;
#pragma unroll
                  for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) o.h16[4 * i + j] = f32_to_bf16(acc[i][f][4 * b + j]);
                  *reinterpret_cast<u32x4*>(put + (f - f0) * 4096 + (((4 * hh + b) ^ sw) << 4)) = o.v;
                }
#pragma unroll
              for (int n = 0; n < (NB - f0 > 1 ? 8 : 4); ++n) {
                const u32x4 v = *reinterpret_cast<const u32x4*>(get + n * 1024);
                if (tr < cur.rows) *reinterpret_cast<u32x4*>(dst) = v;
                const int step = (n & 3) == 3 ? 40 : 8;                       // on to the next token fragment of this wave
                tr += step;
                dst += step * pitch;
              }
            }
          }
        }
        asm volatile("" ::: "memory");
      };
      switch (nb) {
        case 4: unit(std::integral_constant<int, 4>{}); break;
        case 3: unit(std::integral_constant<int, 3>{}); break;
        case 2: unit(std::integral_constant<int, 2>{}); break;
        case 1: unit(std::integral_constant<int, 1>{}); break;
        default: unit(std::integral_constant<int, 0>{}); break;
      }
      if (wait_expired(cur, q0 + (uint32_t)((seq & 3) * kQI) * 4u)) {         // over what this wave has just stored
        __builtin_amdgcn_s_waitcnt(0x0F70);
        if (cur.g * 256 + wr * 64 < m.NOUT)
#pragma unroll 1
          for (int tr = p * 32 + (lane >> 3); tr < cur.rows; tr += (tr & 31) < 24 ? 8 : 40)
            store_nan(m.out + (size_t)(cur.off + tr) * m.NOUT + cur.g * 256 + wr * 64 + (lane & 7) * 8);
      }
    } else {
      for (int kt = 0; kt < nk; ++kt) {
        if constexpr (ROLE == 0) {
          // slab kt (halves 2 kt, 2 kt + 1) has landed once only later halves are outstanding
          const int later = (p_next ? 2 * nk + p_h : p_h) - (2 * kt + 2);
          wait_vm_upto(8 * later);
        } else if constexpr (ROLE == 1) {
          __builtin_amdgcn_s_waitcnt(0x0F70);
        }
        __builtin_amdgcn_s_barrier();                                         // everyone's part is there, slab kt-1 has been read
        if constexpr (ROLE == 2) {
          if (kt == nk - 1 && pending >= 0) {
            // every multiplying wave has waited for its stores of the previous unit
            if (lane == 0) __hip_atomic_fetch_add(a.done + pending, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            pending = -1;
          }
          // One round trip at a time, each used slabs after it was started where the unit has eight or more of them: a wait here is a wait for
          // everyone at the barrier.  Claimed as late as that allows: a workgroup that is behind otherwise still takes two more units at the end.
          // Claims in slab 0 / now, passes, us: 1700 tokens on 107 slots of 1280 x 512 151 / 136, 2200 156 / 146; 1700 on 80 of 2048 x 1408 344 / 342.
          const SchedSteps at = steps_late(nk);
          if (kt == at.claim) sched_claim(a, sc);
          if (kt == at.entry) sched_entry(a, sd, sc);
          if (kt == at.rows) sched_rows(a, sd, sc);
          if (kt == at.stored) sched_stored(a, sc);
          if (kt == at.publish) sched_publish(a, sd, sc, queue + ((seq + 2) & 3) * kQI);
        } else {
#pragma unroll
          for (int i = 0; i < (ROLE == 0 ? 2 : 1); ++i) {
            if (!p_next && p_h == p_n && nxt.slot >= 0 && !(ROLE == 1 && change)) {
              if (ROLE == 1) wait_done(nxt, (seq + 1) & 3);
              aim(nxt, (seq + 1) & 3);
              p_next = true;
            }
            if (p_next || p_h < p_n) issue();
          }
        }
      }
      __builtin_amdgcn_s_barrier();                                           // the multiplying waves have read the last slab
    }
    if (nxt.slot < 0 || change) {
      // the stores are acknowledged (and nothing is in flight at the end of the kernel): count the unit at once
      if constexpr (ROLE != 2) __builtin_amdgcn_s_waitcnt(0x0F70);
      __builtin_amdgcn_s_barrier();
      if constexpr (ROLE == 2) {
        if (cur.mode == 0 && lane == 0) __hip_atomic_fetch_add(a.done + cur.chunk, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if (nxt.slot < 0) return;
    } else if constexpr (ROLE == 2) {
      pending = cur.mode == 0 ? cur.chunk : -1;
    }
    ++seq;
    cur = nxt;
    nxt = read_unit(q0 + (uint32_t)(((seq + 1) & 3) * kQI) * 4u);
    if constexpr (ROLE <= 1) {
      if (!p_next) {  // the token wave, from the first product to the second: nothing of this unit is in flight yet
        if (ROLE == 1) wait_done(cur, seq & 3);
        aim(cur, seq & 3);
        for (int i = 0; i < (ROLE == 0 ? 3 : 1); ++i) issue();
      }
      p_next = false;
    }
  }
}

__global__ __launch_bounds__(kThreads) void k_ffn_big(FfnArgs a) {
  __shared__ __align__(1024) unsigned char s_lds[kLds];
  if (a.pick && picked(a) != a.pick) return;  // the counts chose the other kernel
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (wave < 2) big_body<0>(a, s_lds);
  else if (wave < 3) big_body<1>(a, s_lds);
  else if (wave < 4) big_body<2>(a, s_lds);
  else big_body<3>(a, s_lds);
}

}  // namespace

int launch_ffn_big(FfnArgs a, const FfnPlanShape& sh, int max_chunks, int n_cu, hipStream_t st) {
  a.m[0].G = a.m[0].NOUT / 128;
  a.m[1].G = ceil_div(a.m[1].NOUT, 256);
  const bool merged = sh.merged != 0;
  for (int mode = 0; mode < (merged ? 1 : 2); ++mode) {
    a.first_mode = mode;
    a.last_mode = merged ? 1 : mode;
    const long long units = (long long)max_chunks * (merged ? a.m[0].G + a.m[1].G : a.m[mode].G);
    hipLaunchKernelGGL(k_ffn_big, dim3(units < n_cu ? (int)((units + 7) / 8 * 8) : n_cu), dim3(kThreads), 0, st, a);
    EW_LAUNCH_CHECK("k_ffn_big");
  }
  return EW_OK;
}

}  // namespace ew
