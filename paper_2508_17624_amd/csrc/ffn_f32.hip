// Grouped SwiGLU expert FFN in fp32 (test-sized layers, and checks of a port against a reference), on the fp32 matrix
// instruction v_mfma_f32_16x16x4_f32: plain fp32 products and sums, no reduced-precision format anywhere.
//
// At the sizes this type is used for (configuration 0: 64 tokens, hidden 256) nothing but latency counts, so the split is
// made for short chains: a workgroup computes 16 features x 32 rows of one slot and its four waves split the contraction
// (each a quarter of the 16-element steps), their partial tiles meet in LDS.  A wave then has all its loads of a step
// batch in flight at once and at K = 256 makes four steps.  The kernels this replaced ran one thread per output element,
// a serial chain of K loads each: 111 + 26 us for the two products at configuration 0, now 6 + 5 us.
// Inside a 16-element step lane quarter q holds elements 4q .. 4q+3 of both operands (16-byte loads), one MFMA per
// element: the contraction index may be permuted as long as both sides agree.
// Slots without rows are never dereferenced.
#include "ew_internal.h"

namespace ew {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

struct F32Args {
  const float* x;       // GATED: tokens [*, K]; otherwise activations [rows, K]
  const int32_t* counts;
  const int32_t* offsets;
  const int32_t* por;   // GATED only; NULL: row r is pair r
  const float* w;       // weights of slots 0 .. P-1, and of the shared experts' slots P .. P+S-1
  const float* w_sh;
  float* out;           // [rows, NOUT]
  size_t slot_stride;   // elements per slot
  int P, S, k, K, NOUT, rows_routed, tokens;
};

// Elements kk .. kk+3 of a row of K: zero past its end.
template <bool VEC>
__device__ __forceinline__ f32x4 load4(const float* __restrict__ row, int kk, int K) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if constexpr (VEC) {
    if (kk < K) v = *reinterpret_cast<const f32x4*>(row + kk);  // K % 4 == 0
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (kk + j < K) v[j] = row[kk + j];
  }
  return v;
}

// GATED: out = silu(x.Wg^T) * (x.Wu^T), Wg rows [0,NOUT), Wu rows [NOUT,2NOUT) of the slot; otherwise out = x.W^T.
template <bool GATED, bool VEC>
__global__ __launch_bounds__(256) void k_ffn_f32(F32Args a) {
  constexpr int NW = GATED ? 2 : 1;
  __shared__ f32x4 s_part[4][NW][2][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m = lane & 15, q = lane >> 4;
  const int f0 = blockIdx.x * 16, K = a.K, NOUT = a.NOUT;
  const int feat = min(f0 + m, NOUT - 1);
  for (int s = blockIdx.y; s < a.P + a.S; s += gridDim.y) {
    const bool shared = s >= a.P;
    const int c = shared ? a.tokens : a.counts[s];
    if (c <= (int)blockIdx.z * 32) continue;
    const int off = shared ? a.rows_routed + (s - a.P) * a.tokens : a.offsets[s];
    const float* w0 = (shared ? a.w_sh + (size_t)(s - a.P) * a.slot_stride : a.w + (size_t)s * a.slot_stride) + (size_t)feat * K;
    const float* w1 = w0 + (size_t)NOUT * K;
    for (int r0 = blockIdx.z * 32; r0 < c; r0 += gridDim.z * 32) {
      const bool two = c - r0 > 16;  // the second 16-row tile has rows
      const float* xr[2];
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
        const int r = min(r0 + rt * 16 + m, c - 1);
        int src = off + r;
        if (GATED) src = shared ? r : (a.por ? a.por[off + r] : off + r) / a.k;
        xr[rt] = a.x + (size_t)src * K;
      }
      f32x4 acc[NW][2];
#pragma unroll
      for (int g = 0; g < NW; ++g)
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) acc[g][rt] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
      for (int k0 = wave * 16; k0 < K; k0 += 64) {
        const int kk = k0 + 4 * q;
        f32x4 wv[NW], xv[2];
        wv[0] = load4<VEC>(w0, kk, K);
        if (GATED) wv[NW - 1] = load4<VEC>(w1, kk, K);
        xv[0] = load4<VEC>(xr[0], kk, K);
        if (two) xv[1] = load4<VEC>(xr[1], kk, K);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int g = 0; g < NW; ++g) {
            acc[g][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[g][j], xv[0][j], acc[g][0], 0, 0, 0);
            if (two) acc[g][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[g][j], xv[1][j], acc[g][1], 0, 0, 0);
          }
      }
#pragma unroll
      for (int g = 0; g < NW; ++g)
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) s_part[wave][g][rt][lane] = acc[g][rt];
      __syncthreads();
      // lane l of a tile: row l % 16, features 4 (l / 16) .. + 3
      const int rt = wave, row = r0 + rt * 16 + m, fo = f0 + 4 * q;
      if (rt < 2 && row < c) {
        f32x4 v[NW];
#pragma unroll
        for (int g = 0; g < NW; ++g) v[g] = s_part[0][g][rt][lane] + s_part[1][g][rt][lane] + s_part[2][g][rt][lane] + s_part[3][g][rt][lane];
        f32x4 o = v[0];
        if (GATED) {
#pragma unroll
          for (int j = 0; j < 4; ++j) o[j] = v[0][j] / (1.f + expf(-v[0][j])) * v[NW - 1][j];
        }
        float* dst = a.out + (size_t)(off + row) * NOUT + fo;
        if (VEC && fo + 4 <= NOUT) {
          *reinterpret_cast<f32x4*>(dst) = o;
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (fo + j < NOUT) dst[j] = o[j];
        }
      }
      __syncthreads();  // the partial tiles are read
    }
  }
}

template <bool GATED>
int launch(const F32Args& a, bool vec, int rows_per_slot, hipStream_t st) {
  const int gx = ceil_div(a.NOUT, 16), slots = a.P + a.S, gy = slots < 65535 ? slots : 65535;
  // row splits: enough for the largest slot there can be, unless features and slots alone make a full grid
  int gz = ceil_div(rows_per_slot, 32);
  const long long xy = (long long)gx * gy;
  const int most = xy >= 16384 ? 1 : (int)(16384 / xy);
  gz = gz < most ? gz : most;
  if (vec) hipLaunchKernelGGL((k_ffn_f32<GATED, true>), dim3(gx, gy, gz), dim3(256), 0, st, a);
  else hipLaunchKernelGGL((k_ffn_f32<GATED, false>), dim3(gx, gy, gz), dim3(256), 0, st, a);
  EW_LAUNCH_CHECK("k_ffn_f32");
  return EW_OK;
}

inline bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace

// Both products.  S > 0: slots P .. P+S-1 are shared experts that each of the T tokens visits; their rows follow the T*k
// routed ones in act and y.
int launch_ffn_f32(const void* x, int T, int k, int H, int I, int P, int S, const int32_t* counts, const int32_t* offsets,
                   const int32_t* por, const void* w13, const void* w2, const void* w13_sh, const void* w2_sh, void* act, void* y,
                   hipStream_t st) {
  F32Args a{};
  a.counts = counts; a.offsets = offsets; a.por = por; a.P = P; a.S = S; a.k = k; a.rows_routed = T * k; a.tokens = T;
  // 16-byte accesses need rows and buffers that keep that alignment; anything else goes element by element
  const bool al = H % 4 == 0 && I % 4 == 0 && aligned16(x) && aligned16(w13) && aligned16(w2) && aligned16(act) && aligned16(y) &&
                  (S == 0 || (aligned16(w13_sh) && aligned16(w2_sh)));
  a.x = (const float*)x; a.w = (const float*)w13; a.w_sh = (const float*)w13_sh; a.out = (float*)act;
  a.slot_stride = (size_t)2 * I * H; a.K = H; a.NOUT = I;
  const int rc = launch<true>(a, al, T, st);
  if (rc != EW_OK) return rc;
  a.x = (const float*)act; a.w = (const float*)w2; a.w_sh = (const float*)w2_sh; a.out = (float*)y;
  a.slot_stride = (size_t)H * I; a.K = I; a.NOUT = H;
  return launch<false>(a, al, T, st);
}

}  // namespace ew
