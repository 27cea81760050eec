// Work plans of the grouped-FFN kernels (k_ffn_dec, k_ffn_big): layouts and the device routines that build them.
// Shared by the FFN's own plan kernel and by the decode-sized permutation kernel, which can append the plan of the FFN
// call that follows it to its own launch.
#pragma once
#include <cstdint>
#include <hip/hip_runtime.h>

namespace ew {

// Work plan of one moe_grouped_ffn call, built on the device (the host never reads the counts).
//   plan[kPlanPick]        calls for which the counts decide which kernel runs: 1 = k_ffn_dec, 2 = k_ffn_big
constexpr int kPlanPick = 31;

// Plan of k_ffn_big.
//  * A slot with more than bt rows is cut into equal chunks (rounded up to whole 32-row fragments),
//    so all work items of a slot take the same time.
//  * A slot with more than `ch` chunks is cut further into entries of at most `ch` chunks each.  An
//    entry's items (chunk x feature group) are enumerated group-major, so the 32 workgroups of an XCD
//    that work through one entry hold about 32 / ch feature groups of ch chunks at any time: every
//    weight row they fetch serves ch of them and every token row 32 / ch of them out of the XCD's L2.
//    (A whole slot of 32 chunks per list made 32 workgroups share one feature group and nothing else:
//    every token row came from the fabric once per feature group.)
//  * Entries are ordered by chunk size, largest first (slot id, then position in the slot, break
//    ties), and dealt round-robin to 8 lists, one per XCD (workgroup b runs on XCD b % 8).  The
//    workgroups that share an entry's weights (different chunks) or its token rows (different feature
//    groups) thus run on the same XCD and meet in that XCD's L2; equal durations inside an entry and similar
//    ones between neighbours in the list keep them together.
//  * Up to kTurnRows rows per active slot on average, list x begins x eighths into its order and wraps around, so that at any time
//    some XCDs work on slots of many rows (matrix cores) and some on slots of few (weights from HBM).  All of them in step from large
//    to small: 8192 tokens with 20 adapters (260 rows per slot) 1381 us, now 1347; odd lists in the opposite order 1367.  Beyond, hardly
//    a slot has few rows, and XCDs in step share more of what they fetch: 8192 tokens base-only (990 rows per slot) 1093.1 us and 3.34
//    GB read turned, 1089.6 and 3.0 to 3.2 in step.  At 500 rows (8192 tokens on 130 slots, 16384 on 256) turning gives 1 to 2 %.
//   plan[x]        x < 8   entries of list x
//   plan[8 + x]            row chunks of list x
//   plan[kPlanCtr + kPlanCtrStride i]   claim counters, one cache line each (zeroed here, every call)
//   plan[kPlanHdr + 6 (x cap + e)] ...  entry e of list x: slot, chunks, chunks of the list before it,
//                                 rows per chunk, rows of the entry, first row of the entry
//   plan[done_off + c]     first-product units of chunk c that are stored (zeroed here, every call)
constexpr int kPlanCtr = 32, kPlanCtrStride = 32;  // product 0's lists, then product 1's
constexpr int kPlanHdr = kPlanCtr + 16 * kPlanCtrStride;
constexpr int kEnt = 6;
constexpr int kPlanMaxP = 2048;    // slots a plan can sort
constexpr int kPlanMaxEnt = 4096;  // entries a plan can hold (the host picks ch accordingly)

// Inclusive scan over the wave's 64 lanes (all active): inside rows of 16, then row totals to the rows behind.  DPP moves cost a
// few cycles each, shuffles through LDS over a hundred.
__device__ __forceinline__ uint32_t wave_incl_scan_u32(uint32_t v) {
#define EW_DPP_ADD(ctrl, rows) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rows, 0xf, false)
  EW_DPP_ADD(0x111, 0xf);  // row_shr:1
  EW_DPP_ADD(0x112, 0xf);  // row_shr:2
  EW_DPP_ADD(0x114, 0xf);  // row_shr:4
  EW_DPP_ADD(0x118, 0xf);  // row_shr:8
  EW_DPP_ADD(0x142, 0xa);  // row_bcast:15 into rows 1 and 3
  EW_DPP_ADD(0x143, 0xc);  // row_bcast:31 into rows 2 and 3
#undef EW_DPP_ADD
  return v;
}

// chunks and rows per chunk of a slot with c > 0 rows
__device__ __forceinline__ void chunking(int c, int bt, int& nch, int& bts) {
  nch = (c + bt - 1) / bt;
  bts = ((c + nch - 1) / nch + 31) & ~31;
}

// Shape of the plan and of the kernels that consume it, chosen on the host from the call's dimensions.  A call may name
// both kernels: the counts decide then (ffn_plan_build).
struct FfnPlanShape {
  int dec;           // > 0: k_ffn_dec is a candidate, with chunks of 16 * dec rows
  int dec_cap;       // its chunks at most
  int dec_round;     // its chunks whose units of both products fit one round of workgroups (chunks of more than kDecCut rows only)
  int big;           // k_ffn_big is a candidate
  int bt;            // its rows per chunk at most
  int ch;            // its chunks per entry at most
  int cap;           // its entries per list at most
  int n_done;        // its completion counters
  int done_off;      // where the completion counters start, in ints from the start of the plan
  int merged;        // the two products share a launch
  int wait_polls;    // looks at a completion counter before a wait is given up
};

// Both candidates: k_ffn_big runs where an active slot has more rows on average than k_ffn_dec takes at once with certainty (beyond that
// it reads weights of more and more slots twice).  The line lies below the place where the two cross for hidden sizes that 256 divides, whose chunks
// reach 160 rows (call with plan, us, k_ffn_dec / k_ffn_big, at rows per active slot, 96 such slots): 2048 x 1408 112: 322 / 334, 128: 326 / 337, 136: 333 / 339,
// 144: 347 / 345, 152: 397 / 352; 1536 x 640 128: 129 / 135, 136: 133 / 139, 144: 150 / 142; 1024 x 896 128: 125 / 134, 144: 130 / 140, 152: 145 / 140; 1280 x 512
// 128: 99 / 101, 144: 104 / 105, 152: 111 / 108; 32 slots of 2048 x 1408 152: 143 / 164, 160: 172 / 168.  For other hidden sizes, with chunks of at
// most 128 rows, it lies above it with many slots (96 slots: 1152 x 640 100: 115 / 99, 128: 145 / 104; 640 x 896 100: 97 / 86, 128: 121 / 93) and at it with
// fewer (32: 1152 x 640 128: 63 / 65, 144: 68 / 68; 640 x 896 128: 57 / 64).  The kernel that is not chosen costs a launch (3 to 5 us); both bodies in
// one kernel did not fit the registers.
constexpr int kPickRows = 128;

constexpr int kTurnRows = 640;

struct BigPlanLds {
  uint32_t sorted[kPlanMaxEnt];  // entries in processing order: slot | part << 16
  uint32_t wtot[8][8];           // per size class and wave: entries (and slots << 16), then those before
  int n_total, n_slots;          // entries, active slots
  int32_t cnt[kPlanMaxP], off[kPlanMaxP];
};

// Builds the plan of k_ffn_big.  rows / first: rows and first row of slots 4 tid .. 4 tid + 3 of every thread tid < 512
// (thread order is slot order); rows_all: all rows of the call.  Called by every thread of a block of at least 512 threads (it contains barriers).
__device__ __forceinline__ void big_plan_build(const int (&rows)[4], const int (&first)[4], long long rows_all, const FfnPlanShape& sh, int32_t* __restrict__ plan,
                                               BigPlanLds& L) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const bool worker = tid < 512;
  const int bt = sh.bt, ch = sh.ch, cap = sh.cap;
  for (int i = tid; i < sh.n_done; i += blockDim.x) plan[sh.done_off + i] = 0;
  // size class of a slot: 8 - (32-row fragments per chunk), i.e. 0 = largest chunks.  mine, wtot: entries, in the upper half slots.
  int cls[4], nent[4];
  uint32_t mine[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
  if (worker) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int sl = 4 * tid + i, c = rows[i];
      L.cnt[sl] = c;
      L.off[sl] = first[i];
      cls[i] = -1;
      nent[i] = 0;
      if (c > 0) {
        int nch, bts;
        chunking(c, bt, nch, bts);
        cls[i] = 8 - (bts >> 5);
        nent[i] = (nch + ch - 1) / ch;
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (cls[i] == k) mine[k] += (uint32_t)nent[i] | 1u << 16;
      }
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint32_t inc = wave_incl_scan_u32(mine[k]);
      mine[k] = inc - mine[k];  // entries of the class in the wave's threads before this one
      if (lane == 63) L.wtot[k][wave] = inc;
    }
  }
  __syncthreads();
  if (tid < 64) {  // (class, wave) pairs in order: one wave scans them all
    const uint32_t v = (&L.wtot[0][0])[tid], inc = wave_incl_scan_u32(v);
    (&L.wtot[0][0])[tid] = inc - v;
    if (tid == 63) {
      L.n_total = (int)(inc & 0xFFFFu);
      L.n_slots = (int)(inc >> 16);
    }
  }
  __syncthreads();
  if (worker) {
#pragma unroll
    for (int k = 0; k < 8; ++k) mine[k] = (mine[k] + L.wtot[k][wave]) & 0xFFFFu;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (cls[i] < 0) continue;
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (cls[i] == k) {
          for (int part = 0; part < nent[i]; ++part) L.sorted[mine[k]++] = (uint32_t)(4 * tid + i) | ((uint32_t)part << 16);
        }
    }
  }
  __syncthreads();
  if (!worker) return;
  // wave x builds list x from positions x, x + 8, ...
  const int n_total = L.n_total;
  const int x = wave;
  int32_t* list = plan + kPlanHdr + kEnt * x * cap;
  int n_chunks = 0, n_entries = 0;
  const int n_list = (n_total - x + 7) / 8, turn = rows_all <= (long long)kTurnRows * L.n_slots ? x * n_list / 8 : 0;
  for (int e0 = 0; e0 < n_list; e0 += 64) {
    const int e = e0 + lane;
    const bool ok = e < n_list;
    const int pos = 8 * (e + turn < n_list ? e + turn : e + turn - n_list) + x;
    int sl = 0, c = 0, nch = 0, bts = 0, at = 0;
    if (ok) {
      const uint32_t v = L.sorted[pos];
      sl = (int)(v & 0xFFFFu);
      int all;
      chunking(L.cnt[sl], bt, all, bts);
      at = (int)(v >> 16) * ch;                      // first chunk of this entry inside its slot
      nch = min(ch, all - at);
      c = min(L.cnt[sl] - at * bts, nch * bts);   // rows of this entry
    }
    const int incl = (int)wave_incl_scan_u32((uint32_t)nch);
    if (ok) {
      int32_t* en = list + kEnt * e;
      en[0] = sl;
      en[1] = nch;
      en[2] = n_chunks + incl - nch;
      en[3] = bts;
      en[4] = c;
      en[5] = L.off[sl] + at * bts;
    }
    n_chunks += __shfl(incl, 63, 64);
    n_entries += __popcll(__ballot(ok));
  }
  if (lane == 0) {
    plan[x] = n_entries;
    plan[8 + x] = n_chunks;
    plan[kPlanCtr + x * kPlanCtrStride] = 0;
    plan[kPlanCtr + (8 + x) * kPlanCtrStride] = 0;
  }
}

// Plan of the decode kernel (k_ffn_dec): a flat list of row chunks, the shared experts' first (theirs are the ones with
// more than one chunk), then the active routed slots in slot order.  Units are (chunk, group of weight rows), numbered by
// chunk, so nothing else has to be written down.
//   plan[0]                chunks
//   plan[kDecCtr + kDecCtrStride i]       claim counters, one cache line each (zeroed here, every call)
//   plan[kDecEnt + 4 c]                   slot, rows, first sorted row, unused
//   plan[done_off + kDecDoneStride c]     first-product units of chunk c that are stored (zeroed here)
constexpr int kDecCtr = 32, kDecCtrStride = 32;
constexpr int kDecEnt = kDecCtr + 16 * kDecCtrStride;
constexpr int kDecDoneStride = 16;

// Zeroes them, n_done completion counters: thread tid of n threads' share.
__device__ __forceinline__ void dec_zero_counters(int32_t* __restrict__ plan, int done_off, int n_done, int tid, int n) {
  for (int i = tid; i < n_done; i += n) plan[done_off + kDecDoneStride * i] = 0;
  if (tid < 16) plan[kDecCtr + kDecCtrStride * tid] = 0;
}

// Chunks of a slot with c rows.  Chunks of up to bt = 160 rows are there for slots of 129 to 160, whose weights are then read once;
// larger ones are cut at 128 all the same, and so are the shared experts' (shared_bt).  Passes, us, at most 128 / 160: 1999 tokens, 128
// experts of 1536 x 640, k = 8 (32 of 194 slots in between) 305.7 / 281.1; 1500 tokens, 64 experts of 2048 x 1408 615 / 534.  Cutting
// the larger ones at 160 too: 160 tokens and two shared experts of 1280 x 512 92.0 / 95.4, 768 tokens 112.6 / 114.3.
// Calls whose units, cut at 128, all have a workgroup of their own (dec_round) keep that cut: their time is that of one unit of each
// product, which a chunk of half the rows shortens, and workgroups would stay idle.  Calls with plan, us, at most 128 / 160, slots of 144 rows (units cut
// at 128): 2048 x 1408 1 slot (38) 55.8 / 65.3, 4 (152) 60.8 to 65.8 / 68.5, 6 (228) 68.6 / 77.2, 7 (266) 82.5 / 72.5; 1024 x 896 4 (88) 40.3 / 45.3, 10 (220)
// 44.9 / 48.1, 13 (286) 58.6 / 51.3; 1280 x 512 8 (144) 41.9 / 45.7, 15 (270) 52.3 / 50.0; 1536 x 768 10 (240) 52.5 / 54.8, 11 (264) 62.6 / 55.0.
constexpr int kDecCut = 128;
__host__ __device__ inline int shared_bt(int bt) { return bt < kDecCut ? bt : kDecCut; }
__host__ __device__ inline int dec_chunks(int c, int bt) { return c <= bt ? (c > 0 ? 1 : 0) : (c + shared_bt(bt) - 1) / shared_bt(bt); }

struct DecPlanLds {
  uint32_t wtot[8];
};

// Builds the plan of k_ffn_dec; rows / first as for big_plan_build, without the shared experts' slots: S of them follow the
// P routed ones, sh_rows rows each, from row sh_first on.
__device__ __forceinline__ void dec_plan_build(const int (&rows)[4], const int (&first)[4], int P, int S, int sh_rows, int sh_first,
                                               const FfnPlanShape& sh, int32_t* __restrict__ plan, DecPlanLds& L) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  int bt = 16 * sh.dec, round = sh.dec_round;
  asm volatile("" : "+s"(round));  // (loaded here, with the others, and not as a round trip of its own where it is needed)
  const int sh_chunks = dec_chunks(sh_rows, shared_bt(bt));
  // Sums are chunks and, where chunks may be longer than kDecCut, above bit 16 the slots that kDecCut would cut (there are fewer than
  // 2^16 chunks then: at most kPickRows rows per slot, and kPlanMaxP slots).
  const bool longer = bt > kDecCut;
  uint32_t mine = 0, before = 0, total = 0;
  if (tid < 512) {
#pragma unroll
    for (int i = 0; i < 4; ++i) mine += (uint32_t)dec_chunks(rows[i], bt) + (longer && rows[i] > kDecCut && rows[i] <= bt ? 1u << 16 : 0u);
    const uint32_t inc = wave_incl_scan_u32(mine);
    if (lane == 63) L.wtot[wave] = inc;
    mine = inc - mine;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 8; ++w) {
    const uint32_t t = L.wtot[w];
    if (w < wave) before += t;
    total += t;
  }
  before += mine;
  if (longer) {
    const uint32_t more = total >> 16;
    total &= 0xFFFFu;
    const bool cut = S * sh_chunks + (int)(total + more) <= round;
    before = (before & 0xFFFFu) + (cut ? before >> 16 : 0u);
    if (cut) {
      total += more;
      bt = kDecCut;
    }
  }
  const int chunks = S * sh_chunks + (int)total;
  auto put = [&](int at, int slot, int c, int first_row, int n) {
    const int bts = ((c + n - 1) / n + 15) & ~15;
    for (int j = 0; j < n; ++j) {
      int32_t* en = plan + kDecEnt + 4 * (at + j);
      en[0] = slot;
      en[1] = min(bts, c - j * bts);
      en[2] = first_row + j * bts;
    }
  };
  if (tid < 512) {
    int at = S * sh_chunks + (int)before;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (rows[i] > 0) {
        const int n = dec_chunks(rows[i], bt);
        put(at, 4 * tid + i, rows[i], first[i], n);
        at += n;
      }
    if (tid >= 512 - 64)  // the last wave: it has no routed slot below 1792 of them
      for (int s = tid - (512 - 64); s < S; s += 64) put(s * sh_chunks, P + s, sh_rows, sh_first + s * sh_rows, sh_chunks);
  }
  dec_zero_counters(plan, sh.done_off, chunks, tid, (int)blockDim.x);
  if (tid == 0) plan[0] = chunks;
}

union FfnPlanLds {
  BigPlanLds big;
  DecPlanLds dec;
};

// Builds a call's plan from the rows and first row of the routed slots 4 tid .. 4 tid + 3 of every thread tid < 512 (0 from
// slot P on).  Slots P .. P+S-1 are the shared experts of the call, if any: each holds every token (sh_rows of them), and
// their rows follow the routed ones (first at sh_first).  Called by every thread of a block of at least 512 threads.
__device__ __forceinline__ void ffn_plan_build(int (&rows)[4], int (&first)[4], int P, int S, int sh_rows, int sh_first, const FfnPlanShape& sh,
                                               int32_t* __restrict__ plan, FfnPlanLds& L) {
  const int tid = threadIdx.x;
  const long long rows_all = sh_first + (long long)S * sh_rows;
  bool big = sh.big;
  if (sh.dec && sh.big) {
    int active = S;
#pragma unroll
    for (int i = 0; i < 4; ++i) active += __syncthreads_count(tid < 512 && rows[i] > 0);
    big = rows_all > (long long)kPickRows * active;
    if (tid == 0) plan[kPlanPick] = big ? 2 : 1;
  }
  if (!big) {
    dec_plan_build(rows, first, P, S, sh_rows, sh_first, sh, plan, L.dec);
    return;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int s = 4 * tid + i - P;
    if (s >= 0 && s < S) {
      rows[i] = sh_rows;
      first[i] = sh_first + s * sh_rows;
    }
  }
  big_plan_build(rows, first, rows_all, sh, plan, L.big);
}

}  // namespace ew
