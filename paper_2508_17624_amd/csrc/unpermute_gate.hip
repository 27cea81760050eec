// Weighted un-permute (+ shared experts) and router scores.
//
// Paper Sec. 2.1: expert outputs are weighted with the router's weights and put back into the
// original token order; the router computes g(x) over all experts.
// Both kernels are bandwidth bound: 16-byte accesses, fp32 accumulation, one pass.
#include "ew_internal.h"

#include <type_traits>

namespace {

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {  // round to nearest even (finite inputs)
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

struct alignas(16) U16x8 { uint16_t v[8]; };

// Sum over a block of 256 threads, in the order k_rmsnorm uses (lanes by butterfly, then the four waves in order).
__device__ __forceinline__ float block_sum_256(float v, float* s_part) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = v;
  __syncthreads();
  return s_part[0] + s_part[1] + s_part[2] + s_part[3];
}

// out[t][h] = sum_j w[t][j] * y[rop[t*k+j]][h] + sum_s shared[s][t][h] (+ residual[t][h]); one block per token.
// normed != nullptr: also normed[t] = out[t] / sqrt(mean_h out[t][h]^2 + eps), from the rounded out[t] and in
// k_rmsnorm's order of operations, so the pair equals moe_unpermute followed by moe_rmsnorm bit for bit.
__global__ __launch_bounds__(256) void k_unpermute_bf16(const uint16_t* __restrict__ y, const int32_t* __restrict__ rop,
                                                        const float* __restrict__ w, const uint16_t* __restrict__ shared,
                                                        const uint16_t* __restrict__ residual, int S, int T, int k, int H,
                                                        uint16_t* __restrict__ out, float eps, uint16_t* __restrict__ normed) {
  const int t = blockIdx.x;
  __shared__ int32_t s_row[64];
  __shared__ float s_w[64];
  __shared__ float s_part[4];
  float ss = 0.f;
  if (threadIdx.x < k) {
    s_row[threadIdx.x] = rop[(size_t)t * k + threadIdx.x];
    s_w[threadIdx.x] = w[(size_t)t * k + threadIdx.x];
  }
  __syncthreads();
  for (int h = threadIdx.x * 8; h < H; h += blockDim.x * 8) {
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int j = 0; j < k; ++j) {
      const U16x8 v = *reinterpret_cast<const U16x8*>(y + (size_t)s_row[j] * H + h);
      const float wj = s_w[j];
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] += wj * bf16_to_f32(v.v[i]);
    }
    for (int sh = 0; sh < S; ++sh) {
      const U16x8 v = *reinterpret_cast<const U16x8*>(shared + ((size_t)sh * T + t) * H + h);
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] += bf16_to_f32(v.v[i]);
    }
    if (residual) {
      const U16x8 v = *reinterpret_cast<const U16x8*>(residual + (size_t)t * H + h);
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] += bf16_to_f32(v.v[i]);
    }
    U16x8 o;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      o.v[i] = f32_to_bf16(acc[i]);
      const float f = bf16_to_f32(o.v[i]);
      ss = fmaf(f, f, ss);
    }
    *reinterpret_cast<U16x8*>(out + (size_t)t * H + h) = o;
  }
  if (normed) {
    const float scale = 1.f / sqrtf(block_sum_256(ss, s_part) / (float)H + eps);
    for (int h = threadIdx.x * 8; h < H; h += blockDim.x * 8) {
      const U16x8 v = *reinterpret_cast<const U16x8*>(out + (size_t)t * H + h);  // this thread's own stores
      U16x8 o;
#pragma unroll
      for (int i = 0; i < 8; ++i) o.v[i] = f32_to_bf16(bf16_to_f32(v.v[i]) * scale);
      *reinterpret_cast<U16x8*>(normed + (size_t)t * H + h) = o;
    }
  }
}

__global__ __launch_bounds__(256) void k_unpermute_f32(const float* __restrict__ y, const int32_t* __restrict__ rop,
                                                       const float* __restrict__ w, const float* __restrict__ shared,
                                                       const float* __restrict__ residual, int S, int T, int k, int H,
                                                       float* __restrict__ out, float eps, float* __restrict__ normed) {
  const int t = blockIdx.x;
  __shared__ int32_t s_row[64];
  __shared__ float s_w[64];
  __shared__ float s_part[4];
  float ss = 0.f;
  if (threadIdx.x < k) {
    s_row[threadIdx.x] = rop[(size_t)t * k + threadIdx.x];
    s_w[threadIdx.x] = w[(size_t)t * k + threadIdx.x];
  }
  __syncthreads();
  for (int h = threadIdx.x * 4; h < H; h += blockDim.x * 4) {
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int j = 0; j < k; ++j) {
      const float4 v = *reinterpret_cast<const float4*>(y + (size_t)s_row[j] * H + h);
      const float wj = s_w[j];
      acc.x += wj * v.x; acc.y += wj * v.y; acc.z += wj * v.z; acc.w += wj * v.w;
    }
    for (int sh = 0; sh < S; ++sh) {
      const float4 v = *reinterpret_cast<const float4*>(shared + ((size_t)sh * T + t) * H + h);
      acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    }
    if (residual) {
      const float4 v = *reinterpret_cast<const float4*>(residual + (size_t)t * H + h);
      acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    }
    *reinterpret_cast<float4*>(out + (size_t)t * H + h) = acc;
    ss = fmaf(acc.x, acc.x, fmaf(acc.y, acc.y, fmaf(acc.z, acc.z, fmaf(acc.w, acc.w, ss))));
  }
  if (normed) {
    const float scale = 1.f / sqrtf(block_sum_256(ss, s_part) / (float)H + eps);
    for (int h = threadIdx.x * 4; h < H; h += blockDim.x * 4) {
      float4 v = *reinterpret_cast<const float4*>(out + (size_t)t * H + h);  // this thread's own stores
      v.x *= scale; v.y *= scale; v.z *= scale; v.w *= scale;
      *reinterpret_cast<float4*>(normed + (size_t)t * H + h) = v;
    }
  }
}

// 16 bytes of a row, kept as the words that a load brings: taken apart where they are used, so that no load is waited
// for at the end of the branch that issues it.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <bool BF16>
struct Elem;
template <>
struct Elem<true> {
  using T = uint16_t;
  static constexpr int N = 8;
  u32x4 r;
  __device__ __forceinline__ float get(int i) const { return __uint_as_float(i & 1 ? r[i / 2] & 0xFFFF0000u : r[i / 2] << 16); }
  __device__ __forceinline__ void set(const float (&f)[N]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = (uint32_t)f32_to_bf16(f[2 * i]) | ((uint32_t)f32_to_bf16(f[2 * i + 1]) << 16);
  }
};
template <>
struct Elem<false> {
  using T = float;
  static constexpr int N = 4;
  u32x4 r;
  __device__ __forceinline__ float get(int i) const { return __uint_as_float(r[i]); }
  __device__ __forceinline__ void set(const float (&f)[N]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = __float_as_uint(f[i]);
  }
};

// The same for few tokens and k = K <= 8, where the time is memory latency (a block or less per CU): a token's row numbers and
// weights come in scalar loads (they are the same for the whole block) and its K rows, the first shared rows and the
// residual are all in flight before the first is added.  Same sums in the same order.
template <bool BF16, int K>
__global__ __launch_bounds__(256) void k_unpermute_few(const typename Elem<BF16>::T* __restrict__ y, const int32_t* __restrict__ rop,
                                                   const float* __restrict__ w, const typename Elem<BF16>::T* __restrict__ shared,
                                                   const typename Elem<BF16>::T* __restrict__ residual, int S, int T, int H,
                                                   typename Elem<BF16>::T* __restrict__ out, float eps,
                                                   typename Elem<BF16>::T* __restrict__ normed) {
  using E = Elem<BF16>;
  constexpr int N = E::N, kStep = 256 * N, kAhead = 2;
  const int t = blockIdx.x;
  __shared__ float s_part[4];
  float ss = 0.f;
  const int32_t* __restrict__ rows = rop + (size_t)t * K;
  const float* __restrict__ ws = w + (size_t)t * K;
  E o;
  auto row16 = [](const typename E::T* p) {
    E v;
    v.r = *reinterpret_cast<const u32x4*>(p);
    return v;
  };
  for (int h = threadIdx.x * N; h < H; h += kStep) {
    float acc[N] = {};
    E sh_v[kAhead], res;
    E v[K];
#pragma unroll
    for (int j = 0; j < K; ++j) v[j] = row16(y + (size_t)rows[j] * H + h);
#pragma unroll
    for (int s = 0; s < kAhead; ++s)
      if (s < S) sh_v[s] = row16(shared + ((size_t)s * T + t) * H + h);
    if (residual) res = row16(residual + (size_t)t * H + h);
#pragma unroll
    for (int j = 0; j < K; ++j)
#pragma unroll
      for (int i = 0; i < N; ++i) acc[i] += ws[j] * v[j].get(i);
#pragma unroll
    for (int s = 0; s < kAhead; ++s)
      if (s < S) {
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] += sh_v[s].get(i);
      }
    for (int s = kAhead; s < S; ++s) {
      const E v = row16(shared + ((size_t)s * T + t) * H + h);
#pragma unroll
      for (int i = 0; i < N; ++i) acc[i] += v.get(i);
    }
    if (residual) {
#pragma unroll
      for (int i = 0; i < N; ++i) acc[i] += res.get(i);
    }
    o.set(acc);
    if constexpr (BF16) {
#pragma unroll
      for (int i = 0; i < N; ++i) ss = fmaf(o.get(i), o.get(i), ss);
    } else {
      ss = fmaf(acc[0], acc[0], fmaf(acc[1], acc[1], fmaf(acc[2], acc[2], fmaf(acc[3], acc[3], ss))));
    }
    *reinterpret_cast<u32x4*>(out + (size_t)t * H + h) = o.r;
  }
  if (normed) {
    const float scale = 1.f / sqrtf(block_sum_256(ss, s_part) / (float)H + eps);
    for (int h = threadIdx.x * N; h < H; h += kStep) {
      if (H > kStep) o = row16(out + (size_t)t * H + h);  // this thread's own stores; a single step is still in registers
      float f[N];
#pragma unroll
      for (int i = 0; i < N; ++i) f[i] = o.get(i) * scale;
      o.set(f);
      *reinterpret_cast<u32x4*>(normed + (size_t)t * H + h) = o.r;
    }
  }
}

// out[t] = x[t] / sqrt(mean_h x[t][h]^2 + eps): unit-gain RMS normalisation, one block per token.
// A stacking aid (pre-norm residual chains), not a step of the paper's method.
template <bool BF16>
__global__ __launch_bounds__(256) void k_rmsnorm(const void* __restrict__ x_, int H, float eps, void* __restrict__ out_) {
  __shared__ float s_part[4];
  const int t = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float ss = 0.f;
  if constexpr (BF16) {
    const uint16_t* x = reinterpret_cast<const uint16_t*>(x_) + (size_t)t * H;
    for (int h = threadIdx.x * 8; h < H; h += 256 * 8) {
      const U16x8 v = *reinterpret_cast<const U16x8*>(x + h);
#pragma unroll
      for (int i = 0; i < 8; ++i) { const float f = bf16_to_f32(v.v[i]); ss = fmaf(f, f, ss); }
    }
  } else {
    const float* x = reinterpret_cast<const float*>(x_) + (size_t)t * H;
    for (int h = threadIdx.x * 4; h < H; h += 256 * 4) {
      const float4 v = *reinterpret_cast<const float4*>(x + h);
      ss = fmaf(v.x, v.x, fmaf(v.y, v.y, fmaf(v.z, v.z, fmaf(v.w, v.w, ss))));
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
  if (lane == 0) s_part[wave] = ss;
  __syncthreads();
  const float scale = 1.f / sqrtf((s_part[0] + s_part[1] + s_part[2] + s_part[3]) / (float)H + eps);
  if constexpr (BF16) {
    const uint16_t* x = reinterpret_cast<const uint16_t*>(x_) + (size_t)t * H;
    uint16_t* out = reinterpret_cast<uint16_t*>(out_) + (size_t)t * H;
    for (int h = threadIdx.x * 8; h < H; h += 256 * 8) {
      const U16x8 v = *reinterpret_cast<const U16x8*>(x + h);
      U16x8 o;
#pragma unroll
      for (int i = 0; i < 8; ++i) o.v[i] = f32_to_bf16(bf16_to_f32(v.v[i]) * scale);
      *reinterpret_cast<U16x8*>(out + h) = o;
    }
  } else {
    const float* x = reinterpret_cast<const float*>(x_) + (size_t)t * H;
    float* out = reinterpret_cast<float*>(out_) + (size_t)t * H;
    for (int h = threadIdx.x * 4; h < H; h += 256 * 4) {
      float4 v = *reinterpret_cast<const float4*>(x + h);
      v.x *= scale; v.y *= scale; v.z *= scale; v.w *= scale;
      *reinterpret_cast<float4*>(out + h) = v;
    }
  }
}

// Router scores without the matrix cores (fp32 tokens, odd widths): one wave per token and eight experts (blockIdx.y), whose gate
// rows are read coalesced, so that eight reductions run side by side: in the first three steps a lane gives half of its sums away
// and keeps the other half.  What bounds it is the chain of loads and shuffles of a wave; one expert after the other, each with
// six dependent shuffles, 64 tokens of 8 experts of 256 in fp32 took 4.9 us, now 3.6.
template <bool BF16>
__global__ __launch_bounds__(256) void k_gate_logits(const void* __restrict__ x_, const float* __restrict__ Wg, int T, int H,
                                                     int E, const int32_t* __restrict__ aid, const float* __restrict__ bias,
                                                     float* __restrict__ logits) {
  const int wave = threadIdx.x / 64, lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + wave;
  if (t >= T) return;
  for (int e0 = 8 * blockIdx.y; e0 < E; e0 += 8 * gridDim.y) {
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int h = lane * 4; h < H; h += 256) {
      float4 xv;
      if constexpr (BF16) {
        const ushort4 v = *reinterpret_cast<const ushort4*>(reinterpret_cast<const uint16_t*>(x_) + (size_t)t * H + h);
        xv = make_float4(bf16_to_f32(v.x), bf16_to_f32(v.y), bf16_to_f32(v.z), bf16_to_f32(v.w));
      } else {
        xv = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(x_) + (size_t)t * H + h);
      }
      float4 wv[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) wv[j] = *reinterpret_cast<const float4*>(Wg + (size_t)min(e0 + j, E - 1) * H + h);
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[j] += xv.x * wv[j].x + xv.y * wv[j].y + xv.z * wv[j].z + xv.w * wv[j].w;
    }
    // lane l ends with expert e0 + (l >> 3): bits 5, 4, 3 of the lane are bits 2, 1, 0 of the expert
#pragma unroll
    for (int n = 4; n > 0; n >>= 1) {
      const bool up = lane & (8 * n);
#pragma unroll
      for (int j = 0; j < n; ++j) {
        const float keep = up ? acc[j + n] : acc[j], give = up ? acc[j] : acc[j + n];
        acc[j] = keep + __shfl_xor(give, 8 * n, 64);
      }
    }
#pragma unroll
    for (int o = 4; o > 0; o >>= 1) acc[0] += __shfl_xor(acc[0], o, 64);
    const int e = e0 + (lane >> 3);
    if ((lane & 7) == 0 && e < E) logits[(size_t)t * E + e] = acc[0] + (bias ? bias[(size_t)aid[t] * E + e] : 0.f);
  }
}

// Router scores on the matrix cores (bf16 tokens): A operand = token rows straight from global
// memory (16 bytes per lane), B operand = gate rows
// read as fp32 and split in registers into a bf16 head and a bf16 tail (w = hi + lo to 2^-17),
// so two bf16 MFMAs per tile reproduce the fp32 product to fp32-accumulation accuracy.
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void split_bf16(const float4& lo4, const float4& hi4, bf16x8_t* head, bf16x8_t* tail) {
  const float f[8] = {lo4.x, lo4.y, lo4.z, lo4.w, hi4.x, hi4.y, hi4.z, hi4.w};
  bf16x8_t h, t;
  // float -> bf16 casts: the hardware's packed round-to-nearest-even conversion (a fifth of the integer sequence; the
  // split is what bounds this kernel at prefill sizes, every workgroup splits its experts' whole gate rows)
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    h[i] = (__bf16)f[i];
    t[i] = (__bf16)(f[i] - (float)h[i]);
  }
  *head = h;
  *tail = t;
}

// A workgroup owns 16*TT tokens and EW experts (blockIdx.y picks them); its NW waves split the contraction (K/NW each) and their
// partial sums meet in LDS, added in wave order: for a given NW the sums do not depend on TT or EW.
// What bounds it is the workgroup's own reads (its token rows and fp32 gate rows, mostly from L2) at what one CU takes in,
// so the tile is the smallest one that still gives every CU at most one workgroup (gate_tile below).  In a pass, us, before (tiles
// by the token count alone) / now: 1 token 5.0 / 3.8, 64 tokens 7.1 / 4.7, 512 9.5 / 6.7, 1999 (128 experts of 1536) 19.3 / 11.0,
// 8192 22.8 / 22.0.
template <int NW, int TT, int EW>
__global__ __launch_bounds__(64 * NW) void k_gate_logits_mfma(const uint16_t* __restrict__ x, const float* __restrict__ Wg, int T,
                                                          int H, int E, const int32_t* __restrict__ aid,
                                                          const float* __restrict__ bias, float* __restrict__ logits, ew::FfnCounters zero) {
  constexpr int J = (EW + 15) / 16;  // 16-expert tiles; of a narrower one the last row repeats
  __shared__ float s_red[NW][16 * TT][16 * J + 4];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int m = lane & 15, q = lane >> 4;
  const int t0 = blockIdx.x * 16 * TT, e0 = blockIdx.y * EW;
  const int Kw = H / NW, k_lo = wave * Kw;  // H % (32 NW) == 0
  if (zero.plan && blockIdx.x == 0 && blockIdx.y == 0) ew::dec_zero_counters(zero.plan, zero.done_off, zero.n_done, threadIdx.x, 64 * NW);
  const uint16_t* xr[TT];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) xr[tt] = x + (size_t)min(t0 + tt * 16 + m, T - 1) * H + k_lo + q * 8;
  const float* wr[J];
#pragma unroll
  for (int j = 0; j < J; ++j) wr[j] = Wg + (size_t)min(e0 + min(j * 16 + m, EW - 1), E - 1) * H + k_lo + q * 8;
  f32x4_t acc[TT][J];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt)
#pragma unroll
    for (int j = 0; j < J; ++j) acc[tt][j] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int k0 = 0; k0 < Kw; k0 += 32) {
    bf16x8_t a[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) a[tt] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(xr[tt] + k0));
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const float4 w0 = *reinterpret_cast<const float4*>(wr[j] + k0);
      const float4 w1 = *reinterpret_cast<const float4*>(wr[j] + k0 + 4);
      bf16x8_t head, tail;
      split_bf16(w0, w1, &head, &tail);
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) {
        acc[tt][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[tt], head, acc[tt][j], 0, 0, 0);
        acc[tt][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[tt], tail, acc[tt][j], 0, 0, 0);
      }
    }
  }
  // lane holds expert e0 + 16j + m of tokens t0 + 16tt + 4q + r
#pragma unroll
  for (int tt = 0; tt < TT; ++tt)
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) s_red[wave][tt * 16 + q * 4 + r][j * 16 + m] = acc[tt][j][r];
  __syncthreads();
  for (int idx = threadIdx.x; idx < 16 * TT * EW; idx += 64 * NW) {
    const int tr = idx / EW, ee = idx % EW;
    const int t = t0 + tr, e = e0 + ee;
    if (t < T && e < E) {
      float sum = s_red[0][tr][ee];
#pragma unroll
      for (int wv = 1; wv < NW; ++wv) sum += s_red[wv][tr][ee];
      logits[(size_t)t * E + e] = sum + (bias ? bias[(size_t)aid[t] * E + e] : 0.f);
    }
  }
}

// f(TT, EW): the first of these tiles, ordered by what a workgroup reads, whose grid is at most one workgroup per CU; the last
// beyond that.  Kernel alone, us, 64 experts of 2048: 64 tokens with 2 / 4 / 8 / 16 experts 4.7 / 5.1 / 5.7 / 7.0; 512 tokens with 8 /
// 16 experts 5.8 / 7.1; 1024 tokens as 1 / 2 / 4 token tiles of 16 experts 7.2 / 8.9 / 12.6; 4096 tokens as 4 token tiles of 16 / 32
// experts 13.3 / 17.6; 8192 tokens as 1 / 4 token tiles of 16 / 32 experts 43.7 / 17.3.
template <typename F>
void gate_tile(int T, int E, F f) {
  constexpr int kCus = 256;  // of the whole gfx950; on a partition the tile is one size too small, no more
  auto one = [&](auto TT, auto EW) { return (long long)ew::ceil_div(T, 16 * decltype(TT)::value) * ew::ceil_div(E, decltype(EW)::value) <= kCus; };
  using std::integral_constant;
  const integral_constant<int, 1> n1{};
  const integral_constant<int, 2> n2{};
  const integral_constant<int, 4> n4{};
  const integral_constant<int, 8> n8{};
  const integral_constant<int, 16> n16{};
  const integral_constant<int, 32> n32{};
  if (one(n1, n2)) f(n1, n2);
  else if (one(n1, n4)) f(n1, n4);
  else if (one(n1, n8)) f(n1, n8);
  else if (one(n1, n16)) f(n1, n16);
  else if (one(n2, n16)) f(n2, n16);
  else if (one(n4, n16)) f(n4, n16);
  else f(n4, n32);
}

}  // namespace

namespace {

int unpermute(const char* who, const void* y_sorted, const int32_t* row_of_pair, const float* topk_w, const void* shared_out,
              int num_shared, const void* residual, int T, int k, int H, int dtype, void* out, float eps, void* normed,
              void* stream) {
  using ew::fail;
  if (T < 0 || k < 1 || H < 1 || num_shared < 0) return fail(EW_ERR_INVALID_ARG, "%s: need T>=0, k>=1, H>=1, num_shared>=0", who);
  if (num_shared > 0 && !shared_out) return fail(EW_ERR_INVALID_ARG, "%s: shared_out is NULL but num_shared=%d", who, num_shared);
  const int S = shared_out ? num_shared : 0;
  if (dtype != EW_F32 && dtype != EW_BF16) return fail(EW_ERR_INVALID_ARG, "%s: unknown dtype %d", who, dtype);
  if (k > 64) return fail(EW_ERR_UNSUPPORTED, "%s: k=%d above the supported 64", who, k);
  if (H % (dtype == EW_BF16 ? 8 : 4)) return fail(EW_ERR_UNSUPPORTED, "%s: H=%d must be a multiple of %d", who, H, dtype == EW_BF16 ? 8 : 4);
  if (T == 0) return EW_OK;
  if (!y_sorted || !row_of_pair || !topk_w || !out) return fail(EW_ERR_INVALID_ARG, "%s: NULL device pointer", who);
  hipStream_t st = (hipStream_t)stream;
  auto few = [&](auto K) {
    if (dtype == EW_BF16)
      hipLaunchKernelGGL((k_unpermute_few<true, decltype(K)::value>), dim3(T), dim3(256), 0, st, (const uint16_t*)y_sorted, row_of_pair,
                         topk_w, (const uint16_t*)shared_out, (const uint16_t*)residual, S, T, H, (uint16_t*)out, eps, (uint16_t*)normed);
    else
      hipLaunchKernelGGL((k_unpermute_few<false, decltype(K)::value>), dim3(T), dim3(256), 0, st, (const float*)y_sorted, row_of_pair,
                         topk_w, (const float*)shared_out, (const float*)residual, S, T, H, (float*)out, eps, (float*)normed);
  };
  // k_unpermute_few up to a token per CU.  The kernel alone (replayed in a graph), us, without / with it, bf16: 1 token, k = 6, H =
  // 2048, two shared rows 2.8 / 2.2, 64 tokens 3.1 / 2.5, 256 tokens 3.2 / 2.7; k = 1, H = 256 2.3 / 2.2.  fp32: 3.4 / 2.5, 3.6 / 2.7,
  // 3.9 / 3.1, 2.2 / 2.2.  Whole passes: 1 token 58.0 / 56.7, 64 tokens 239.8 / 238.6; 1999 tokens 319 / 321, where its registers
  // cost occupancy.
  switch (T <= 256 ? k : 0) {
    case 1: few(std::integral_constant<int, 1>{}); break;
    case 2: few(std::integral_constant<int, 2>{}); break;
    case 3: few(std::integral_constant<int, 3>{}); break;
    case 4: few(std::integral_constant<int, 4>{}); break;
    case 5: few(std::integral_constant<int, 5>{}); break;
    case 6: few(std::integral_constant<int, 6>{}); break;
    case 7: few(std::integral_constant<int, 7>{}); break;
    case 8: few(std::integral_constant<int, 8>{}); break;
    default:
      if (dtype == EW_BF16)
        hipLaunchKernelGGL(k_unpermute_bf16, dim3(T), dim3(256), 0, st, (const uint16_t*)y_sorted, row_of_pair, topk_w,
                           (const uint16_t*)shared_out, (const uint16_t*)residual, S, T, k, H, (uint16_t*)out, eps, (uint16_t*)normed);
      else
        hipLaunchKernelGGL(k_unpermute_f32, dim3(T), dim3(256), 0, st, (const float*)y_sorted, row_of_pair, topk_w,
                           (const float*)shared_out, (const float*)residual, S, T, k, H, (float*)out, eps, (float*)normed);
  }
  EW_LAUNCH_CHECK("k_unpermute");
  return EW_OK;
}

}  // namespace

extern "C" int moe_unpermute(const void* y_sorted, const int32_t* row_of_pair, const float* topk_w, const void* shared_out,
                             int num_shared, const void* residual, int T, int k, int H, int dtype, void* out, void* stream) {
  return unpermute("moe_unpermute", y_sorted, row_of_pair, topk_w, shared_out, num_shared, residual, T, k, H, dtype, out, 0.f,
                   nullptr, stream);
}

extern "C" int moe_unpermute_rmsnorm(const void* y_sorted, const int32_t* row_of_pair, const float* topk_w, const void* shared_out,
                                     int num_shared, const void* residual, int T, int k, int H, int dtype, void* out, float eps,
                                     void* normed_out, void* stream) {
  if (!(eps >= 0.f)) return ew::fail(EW_ERR_INVALID_ARG, "moe_unpermute_rmsnorm: need eps>=0");
  if (T > 0 && !normed_out) return ew::fail(EW_ERR_INVALID_ARG, "moe_unpermute_rmsnorm: normed_out is NULL");
  if (T > 0 && normed_out == out) return ew::fail(EW_ERR_INVALID_ARG, "moe_unpermute_rmsnorm: normed_out must not be out");
  return unpermute("moe_unpermute_rmsnorm", y_sorted, row_of_pair, topk_w, shared_out, num_shared, residual, T, k, H, dtype, out,
                   eps, normed_out, stream);
}

int ew::gate_logits(const void* x, int dtype, const float* Wg, int T, int H, int E, const int32_t* adapter_id, const float* bias, float* logits,
                    const FfnCounters& zero, hipStream_t st) {
  if (T < 0 || H < 1 || E < 1) return fail(EW_ERR_INVALID_ARG, "moe_gate_logits: need T>=0, H>=1, E>=1");
  if (dtype != EW_F32 && dtype != EW_BF16) return fail(EW_ERR_INVALID_ARG, "moe_gate_logits: unknown dtype %d", dtype);
  if ((adapter_id == nullptr) != (bias == nullptr)) return fail(EW_ERR_INVALID_ARG, "moe_gate_logits: adapter_id and bias go together");
  if (H % 4) return fail(EW_ERR_UNSUPPORTED, "moe_gate_logits: H=%d must be a multiple of 4", H);
  if (T == 0) return EW_OK;
  if (!x || !Wg || !logits) return fail(EW_ERR_INVALID_ARG, "moe_gate_logits: NULL device pointer");
  if (dtype == EW_BF16 && H % 128 == 0) {
    gate_tile(T, E, [&](auto tt, auto ew_tag) {
      constexpr int TT = decltype(tt)::value, EW = decltype(ew_tag)::value;
      const dim3 grid(ew::ceil_div(T, 16 * TT), ew::ceil_div(E, EW));
      // 16 waves where they divide the contraction: a wave then has its whole part in flight at once
      if (H % 512 == 0)
        hipLaunchKernelGGL((k_gate_logits_mfma<16, TT, EW>), grid, dim3(1024), 0, st, (const uint16_t*)x, Wg, T, H, E, adapter_id, bias, logits, zero);
      else
        hipLaunchKernelGGL((k_gate_logits_mfma<4, TT, EW>), grid, dim3(256), 0, st, (const uint16_t*)x, Wg, T, H, E, adapter_id, bias, logits, zero);
    });
    EW_LAUNCH_CHECK("k_gate_logits");
    return EW_OK;
  }
  const dim3 grid(ew::ceil_div(T, 4), ew::ceil_div(E, 8) < 65535 ? ew::ceil_div(E, 8) : 65535);
  if (dtype == EW_BF16)
    hipLaunchKernelGGL((k_gate_logits<true>), grid, dim3(256), 0, st, x, Wg, T, H, E, adapter_id, bias, logits);
  else
    hipLaunchKernelGGL((k_gate_logits<false>), grid, dim3(256), 0, st, x, Wg, T, H, E, adapter_id, bias, logits);
  EW_LAUNCH_CHECK("k_gate_logits");
  return EW_OK;
}

extern "C" int moe_gate_logits(const void* x, int dtype, const float* Wg, int T, int H, int E, const int32_t* adapter_id,
                               const float* bias, float* logits, void* stream) {
  return ew::gate_logits(x, dtype, Wg, T, H, E, adapter_id, bias, logits, ew::FfnCounters{}, (hipStream_t)stream);
}

extern "C" int moe_rmsnorm(const void* x, int dtype, int T, int H, float eps, void* out, void* stream) {
  using ew::fail;
  if (T < 0 || H < 1 || !(eps >= 0.f)) return fail(EW_ERR_INVALID_ARG, "moe_rmsnorm: need T>=0, H>=1, eps>=0");
  if (dtype != EW_F32 && dtype != EW_BF16) return fail(EW_ERR_INVALID_ARG, "moe_rmsnorm: unknown dtype %d", dtype);
  if (H % (dtype == EW_BF16 ? 8 : 4)) return fail(EW_ERR_UNSUPPORTED, "moe_rmsnorm: H=%d must be a multiple of %d", H, dtype == EW_BF16 ? 8 : 4);
  if (T == 0) return EW_OK;
  if (!x || !out) return fail(EW_ERR_INVALID_ARG, "moe_rmsnorm: NULL device pointer");
  hipStream_t st = (hipStream_t)stream;
  if (dtype == EW_BF16) hipLaunchKernelGGL((k_rmsnorm<true>), dim3(T), dim3(256), 0, st, x, H, eps, out);
  else hipLaunchKernelGGL((k_rmsnorm<false>), dim3(T), dim3(256), 0, st, x, H, eps, out);
  EW_LAUNCH_CHECK("k_rmsnorm");
  return EW_OK;
}
