// Grouped SwiGLU expert FFN in bf16: the choice between the two kernels that stream both operands into LDS, their work
// plans and the call itself.
//   k_ffn_dec (ffn_dec.hip)  few rows per slot: a stream of weights, chunks of at most 160 rows
//   k_ffn_big (ffn_big.hip)  many rows per slot: matrix-core bound, chunks of at most 256 rows
// Any counts are correct with either: larger slots are cut into chunks.
#include "ffn_roles.h"

#include <atomic>

namespace ew {

namespace {

// Thread t reads the slots 4 t .. 4 t + 3.
__global__ __launch_bounds__(512) void k_ffn_plan(const int32_t* __restrict__ counts, const int32_t* __restrict__ offsets, int P, int S,
                                                  int sh_rows, int sh_first, FfnPlanShape sh, int32_t* __restrict__ plan) {
  __shared__ FfnPlanLds lds;
  int rows[4], first[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int sl = 4 * (int)threadIdx.x + i;
    rows[i] = sl < P ? counts[sl] : 0;
    first[i] = sl < P ? offsets[sl] : 0;
  }
  ffn_plan_build(rows, first, P, S, sh_rows, sh_first, sh, plan, lds);
}

// k_ffn_big: chunks per plan entry at most: 8 (a quarter of an XCD's workgroups per feature group), doubled until the
// entries of the worst case -- every possible slot active plus one more entry per ch * bt rows -- fit a plan.
int entry_chunks(int rows, int P, int bt) {
  const int max_active = P < rows ? P : rows;
  int ch = 8;
  while ((long long)max_active + rows / ((long long)ch * bt) > kPlanMaxEnt) ch *= 2;
  return ch;
}

// Entries per list at most.  A slot of c rows makes at most 1 + c / (ch * bt) entries, so a call makes at most
// max_active + rows / (ch * bt) of them: never more than kPlanMaxEnt (choice of ch), nor than the figure for the
// smallest chunk the tuning cap can ask for (bt = 32, ch = 8).
int list_cap(int rows, int P) {
  const int max_active = P < rows ? P : rows;
  const long long worst = (long long)max_active + rows / 256;
  return ceil_div((int)(worst < kPlanMaxEnt ? worst : kPlanMaxEnt), 8) + 1;
}

constexpr int kCus = 256;  // of an MI355X, a workgroup of k_ffn_dec on each

// A look takes well over half a microsecond: seconds, where a wait lasts as long as two units at most.
constexpr int kWaitPolls = 1 << 22;

// k_ffn_dec: chunks of a plan at most: one per active slot and one more per bt rows (kDecCut, where that is less).
int dec_chunk_cap(int rows, int P, int bt) { return (P < rows ? P : rows) + rows / shared_bt(bt) + 1; }

}  // namespace

// Never less for more tokens (a workspace made for a largest batch serves the smaller ones): k_ffn_dec's chunks are 16 rows up
// to 16 tokens and more above, so the first 16 tokens alone can take more chunks than the whole batch.
size_t ffn_plan_ints(int T, int rows, int P) {
  const int cap = list_cap(rows, P);
  const size_t big = (size_t)kPlanHdr + (size_t)8 * kEnt * cap, big_done = (size_t)8 * entry_chunks(rows, P, 32) * cap;
  const int first = dec_chunk_cap(rows / T * (T < 16 ? T : 16), P, 16), all = T > 16 ? dec_chunk_cap(rows, P, 32) : 0;
  const size_t chunks = first > all ? first : all, dec = kDecEnt + 4 * chunks, dec_done = kDecDoneStride * chunks;
  return (big > dec ? big : dec) + (big_done > dec_done ? big_done : dec_done);
}

// The host knows totals only: no slot has more rows than the call has tokens, and rows / slots is the least that an active
// slot has on average.  Above kPickRows rows per slot k_ffn_big runs; at or below it k_ffn_dec does up to 512 tokens, and above
// 512 the counts decide.  Measured up to 512 tokens in a pool whose other slots are idle (call with plan, us, k_ffn_dec / k_ffn_big; 2048 x
// 1408 experts, rows per active slot x slots): 128 x 4: 68 / 70; 200 x 4: 67 / 82; 128 x 8: 80 / 77; 144 x 8: 74 / 78; 160 x 8: 77 / 84; 176 x 8:
// 91 / 82; 200 x 8: 92 / 86; 128 x 32: 131 / 154; 152 x 32: 143 / 164; 160 x 32: 172 / 168; 176 x 32: 198 / 178.  (1024 x 896: 200 x 8: 47 / 57;
// 160 x 32: 77 / 76; 200 x 32: 81 / 87.)  So k_ffn_big wins in a corner only, eight or more slots of more than 160 rows while the pool's other slots keep
// the average low; to let the counts find it would cost every call up to 512 tokens a second launch (3 to 5 us).
FfnPlanShape ffn_plan_shape(int T, int rows, int slots, int H, int I, int frags, int chunk_frags, bool merge, int wait_polls) {
  FfnPlanShape sh{};
  sh.merged = merge;
  sh.wait_polls = wait_polls > 0 ? wait_polls : kWaitPolls;
  const int per_slot = rows / (slots < rows ? slots : rows);
  const bool forced = frags > 0 || chunk_frags > 0;
  if (forced ? frags == 8 || frags == 0 : T > 512 || per_slot > kPickRows) {
    sh.big = 1;
    sh.bt = 32 * (chunk_frags >= 1 && chunk_frags <= 8 ? chunk_frags : 8);
    sh.ch = entry_chunks(rows, slots, sh.bt);
    sh.cap = list_cap(rows, slots);
    sh.n_done = 8 * sh.ch * sh.cap;
  }
  if (forced ? frags > 0 && frags < 8 : per_slot <= kPickRows) {
    if (forced) {
      const int most = chunk_frags >= 1 && chunk_frags < frags ? chunk_frags : frags;
      sh.dec = most >= 4 ? 8 : most >= 2 ? 4 : 2;
    } else {
      sh.dec = T <= 16 ? 1 : T <= 32 ? 2 : T <= 64 ? 4 : T <= 128 || H % 256 ? 8 : 10;
    }
    sh.dec_cap = dec_chunk_cap(rows, slots, 16 * sh.dec);
    if (16 * sh.dec > kDecCut) sh.dec_round = kCus / (I / 128 + H / 256);
  }
  const int big_end = kPlanHdr + 8 * kEnt * sh.cap, dec_end = kDecEnt + 4 * sh.dec_cap;  // (of a kernel that is no candidate: headers alone)
  sh.done_off = big_end > dec_end ? big_end : dec_end;
  return sh;
}

int launch_ffn_plan(const int32_t* counts, const int32_t* offsets, int P, int S, int T, int rows_routed, const FfnPlanShape& sh,
                    int32_t* plan, hipStream_t st) {
  hipLaunchKernelGGL(k_ffn_plan, dim3(1), dim3(512), 0, st, counts, offsets, P, S, T, rows_routed, sh, plan);
  EW_LAUNCH_CHECK("k_ffn_plan");
  return EW_OK;
}

int launch_ffn_bf16(const void* x, int rows_routed, int k, int H, int I, int P, int S, const FfnPlanShape& sh, bool plan_ready,
                    const int32_t* counts, const int32_t* offsets, const int32_t* por, const void* w13, const void* w2, const void* w13_sh,
                    const void* w2_sh, void* act, void* y, int32_t* plan, hipStream_t st, const FfnRoute* route) {
  const int T = rows_routed / k;              // tokens = rows of each shared expert
  const int rows = rows_routed + S * T, slots = P + S;
  // persistent grids: one workgroup per CU, a multiple of the 8 XCDs; the count is kept per device
  // (relaxed atomics: two threads racing on the first call store the same value)
  constexpr int kMaxDev = 64;
  static std::atomic<int> cu_of_dev[kMaxDev];
  int dev = 0;
  EW_HIP(hipGetDevice(&dev));
  int n_cu = dev >= 0 && dev < kMaxDev ? cu_of_dev[dev].load(std::memory_order_relaxed) : 0;
  if (n_cu == 0) {
    int v = 0;
    EW_HIP(hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev));
    n_cu = v < 8 ? 8 : v / 8 * 8;
    if (dev >= 0 && dev < kMaxDev) cu_of_dev[dev].store(n_cu, std::memory_order_relaxed);
  }
  if (!plan_ready && !route) {
    const int rc = launch_ffn_plan(counts, offsets, P, S, T, rows_routed, sh, plan, st);
    if (rc != EW_OK) return rc;
  }
  FfnArgs a{};
  a.m[0] = FfnProd{(const uint16_t*)x, (const uint16_t*)w13, (const uint16_t*)w13_sh, (uint16_t*)act, (size_t)2 * I * H, H, I, 0};
  a.m[1] = FfnProd{(const uint16_t*)act, (const uint16_t*)w2, (const uint16_t*)w2_sh, (uint16_t*)y, (size_t)H * I, I, H, 0};
  a.por = por; a.plan = plan; a.done = plan + sh.done_off;
  a.P = P; a.rows_routed = rows_routed; a.sh_rows = T > 0 ? T : 1; a.k = k;
  a.cap = sh.cap; a.list_chunks = sh.ch * sh.cap;
  a.wait_polls = sh.wait_polls;
  if (route) return launch_ffn_dec(a, sh, n_cu, st, route);
  const bool both = sh.dec && sh.big;
  if (sh.dec) {
    a.pick = both ? 1 : 0;
    const int rc = launch_ffn_dec(a, sh, n_cu, st);
    if (rc != EW_OK) return rc;
  }
  if (sh.big) {
    a.pick = both ? 2 : 0;
    return launch_ffn_big(a, sh, rows / sh.bt + (slots < rows ? slots : rows), n_cu, st);
  }
  return EW_OK;
}

}  // namespace ew
