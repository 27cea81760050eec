// Pieces shared by the grouped-FFN kernels whose loading, scheduling and multiplying are different waves (ffn_dec.hip,
// ffn_big.hip): argument structs, LDS accesses and waits placed by hand.
#pragma once
#include "ew_internal.h"
#include "ffn_steps.h"

#include <type_traits>

namespace ew {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

struct FfnProd {
  const uint16_t* x;   // first product: tokens [*, K]; second: activations [rows, K]
  const uint16_t* w;   // slots 0 .. P-1
  const uint16_t* w_sh;
  uint16_t* out;       // [rows, NOUT]
  size_t slot_stride;  // elements per slot
  int K, NOUT, G;      // G: units per chunk
};

struct FfnArgs {
  FfnProd m[2];
  const int32_t* por;   // row map of the first product; may be NULL
  int32_t* plan;
  int32_t* done;        // per chunk: first-product units stored
  int P, rows_routed, sh_rows, k;
  int first_mode, last_mode;  // the launch's products
  int depth_w, depth_t;       // k_ffn_dec: slabs in its rings
  int cap, list_chunks;       // k_ffn_big: entries and chunks per list of the plan at most
  int pick;                   // 0, or this kernel's number in plan[kPlanPick]
  int wait_polls;             // looks at a completion counter before a wait for it is given up
  int grid;                   // k_ffn_dec: workgroups of the launch
};

// The kernel that the counts chose (wave-uniform, as the branch on it has to be).
__device__ __forceinline__ int picked(const FfnArgs& a) { return __builtin_amdgcn_readfirstlane(a.plan[kPlanPick]); }

__device__ __forceinline__ uint16_t f32_to_bf16(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ float silu_f32(float g) { return g * __builtin_amdgcn_rcpf(1.f + __expf(-g)); }

struct FfnUnit {
  int slot, off, rows, g, mode, chunk;  // slot < 0: no unit left
  int ready;                            // 1: nothing to wait for; kExpired: the wait was given up
  int how;                              // k_ffn_big: kAlone; k_ffn_dec: 0 a whole unit, 1 / 2 the first / second half of one
};

// LDS-direct load: 16 bytes per lane from base + off (base: wave-uniform) to lds + 16 * lane.  AUX: 0 plain, 2 nt, 16 sc1.
// Written out for its scalar base: given 64-bit lane addresses (which the compiler likes to compute ahead of a loop) the
// same loads cost the 256-row kernel 5 %.  The loads are not seen by the compiler's own counting of outstanding ones.
template <int AUX>
__device__ __forceinline__ void load_to_lds(const unsigned char* base, uint32_t off, uint32_t lds) {
  if constexpr (AUX == 2)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(off), "s"(base), "s"(lds) : "memory");
  else if constexpr (AUX == 16)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 sc1" ::"v"(off), "s"(base), "s"(lds) : "memory");
  else
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds) : "memory");
}

// 16 bytes written through to the point of coherence of the GPU's XCDs (an agent-scope store; the language's go to 8 bytes).
__device__ __forceinline__ void store_agent_16(void* p, u32x4 v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");  // (nop: the data registers may be written next)
}

// LDS reads the compiler must not see (it would wait for every LDS-direct load in flight before them).
__device__ __forceinline__ FfnUnit read_unit(uint32_t addr) {
  i32x4 lo, hi;
  asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %2 offset:16\n\ts_waitcnt lgkmcnt(0)" : "=&v"(lo), "=&v"(hi) : "v"(addr) : "memory");
  FfnUnit u;
  u.slot = __builtin_amdgcn_readfirstlane(lo[0]);
  u.off = __builtin_amdgcn_readfirstlane(lo[1]);
  u.rows = __builtin_amdgcn_readfirstlane(lo[2]);
  u.g = __builtin_amdgcn_readfirstlane(lo[3]);
  u.mode = __builtin_amdgcn_readfirstlane(hi[0]);
  u.chunk = __builtin_amdgcn_readfirstlane(hi[1]);
  u.ready = __builtin_amdgcn_readfirstlane(hi[2]);
  u.how = __builtin_amdgcn_readfirstlane(hi[3]);
  return u;
}
// Adds 1 to a claim counter; the value before comes back while the wave goes on (it is waited for where it is used).  The address is
// a vector one on purpose: given a uniform one the compiler combines the lanes' additions and waits for the result at once, a round
// trip in which the scheduling wave is missing at the slabs' barriers.
__device__ __forceinline__ int32_t claim_next(int32_t* counter) {
  uint32_t at = 0;
  asm volatile("" : "+v"(at));
  return __hip_atomic_fetch_add(reinterpret_cast<int32_t*>(reinterpret_cast<char*>(counter) + at), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// What a scheduling wave needs of the two products, in registers: selected by product out of the arguments it would be a load each
// time, from memory and waited for.
struct SchedDims {
  int units0, units1;  // per chunk
  int pitch0, pitch1;  // bytes of a source row
};
__device__ __forceinline__ int in_sgpr(int v) {
  asm volatile("" : "+s"(v));
  return v;
}
__device__ __forceinline__ SchedDims sched_dims(const FfnArgs& a) {
  return {in_sgpr(a.m[0].G), in_sgpr(a.m[1].G), in_sgpr(2 * a.m[0].K), in_sgpr(2 * a.m[1].K)};
}
// N ints STEP bytes apart (N: 1, 2 or a multiple of 4).
template <int N, int STEP>
__device__ __forceinline__ void read_lds_ints(uint32_t addr, uint32_t* r) {
  if constexpr (N == 1)
    asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(r[0]) : "v"(addr) : "memory");
  else if constexpr (N == 2)
    asm volatile("ds_read_b32 %0, %2\n\tds_read_b32 %1, %2 offset:%3\n\ts_waitcnt lgkmcnt(0)" : "=&v"(r[0]), "=&v"(r[1]) : "v"(addr), "n"(STEP) : "memory");
  else {
    asm volatile("ds_read_b32 %0, %4\n\tds_read_b32 %1, %4 offset:%5\n\tds_read_b32 %2, %4 offset:%6\n\tds_read_b32 %3, %4 offset:%7\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]) : "v"(addr), "n"(STEP), "n"(2 * STEP), "n"(3 * STEP) : "memory");
    if constexpr (N > 4) read_lds_ints<N - 4, STEP>(addr + 4 * STEP, r + 4);
  }
}

// A token wave's wait for the first-product units of its unit's chunk, `target` of them.  It always ends by itself (the
// argument is in ffn_dec.hip); should that ever fail it is given up after a number of looks, which only count while the wave
// runs, and the unit's entry in the LDS queue says so: its output is then written as NaN, never made from rows that may not be
// stored.  The waits after one that was given up look once.
constexpr int kExpired = -1, kReadyWord = 6;  // the word of a queue entry
__device__ __forceinline__ void wait_stored(const int32_t* flag, int target, int& polls, int32_t* entry) {
  for (int looks = 1; __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target; ++looks) {
    if (looks >= polls) {
      polls = 1;
      if ((threadIdx.x & 63) == 0) entry[kReadyWord] = kExpired;
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      break;
    }
    __builtin_amdgcn_s_sleep(1);
  }
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void store_nan(uint16_t* p) { *reinterpret_cast<u32x4*>(p) = (u32x4)0x7FC07FC0u; }
// Multiplying waves, behind a unit: whether its token waves gave up.  entry: LDS address of the unit's queue entry.
__device__ __forceinline__ bool wait_expired(const FfnUnit& u, uint32_t entry) {
  if (u.mode == 0) return false;
  uint32_t r;
  read_lds_ints<1, 4>(entry + 4 * kReadyWord, &r);
  return (int)__builtin_amdgcn_readfirstlane(r) == kExpired;
}

// ffn_dec.hip: calls with few rows per slot.  route: the launch routes too (ffn_routes), no plan is there.
int launch_ffn_dec(FfnArgs a, const FfnPlanShape& sh, int n_cu, hipStream_t st, const FfnRoute* route = nullptr);
// ffn_big.hip: the calls with many rows per slot; max_chunks: row chunks of the plan at most.
int launch_ffn_big(FfnArgs a, const FfnPlanShape& sh, int max_chunks, int n_cu, hipStream_t st);

// At most n vector-memory operations of this wave still outstanding (n is wave-uniform; waiting for fewer is safe).
__device__ __forceinline__ void wait_vm_upto(int n) {
#define EW_VM(N) __builtin_amdgcn_s_waitcnt(0x0F70 | ((N) & 15) | (((N) >> 4) << 14))
  if (n >= 32) {
    if (n >= 40) EW_VM(40); else if (n >= 36) EW_VM(36); else EW_VM(32);
  } else if (n >= 16) {
    if (n >= 24) EW_VM(24); else if (n >= 20) EW_VM(20); else EW_VM(16);
  } else if (n >= 8) {
    if (n >= 12) EW_VM(12); else if (n >= 10) EW_VM(10); else EW_VM(8);
  } else if (n >= 4) {
    if (n >= 6) EW_VM(6); else if (n >= 5) EW_VM(5); else EW_VM(4);
  } else {
    if (n >= 3) EW_VM(3); else if (n >= 2) EW_VM(2); else if (n >= 1) EW_VM(1); else EW_VM(0);
  }
#undef EW_VM
}

}  // namespace ew
