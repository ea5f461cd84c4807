// Router gate: the affinities the router of Sections 3.1 and 3.2 turns into
// scores, logits = x W_r^T, with x bfloat16 [n x H], W_r float32 [E x H] and
// logits float32 [n x E].  Products and sums are float32 and every logit is
// accumulated in an order fixed by (n <= kGateFewTokens, H), so a forward is
// deterministic.
//
// Few tokens (decode): one workgroup per expert.  Thread t owns the float4
// columns t, t + 256, ... of the expert's row, keeps one partial sum per
// token, and the 256 partials are reduced by a fixed tree (DPP within a
// wave, then the four waves in order).  The row of W_r is streamed once.
//
// Many tokens: the matrix cores.  W_r is split in registers into three
// bfloat16 parts that add up to it exactly (8 + 8 + 8 significant bits), so
// every product with the bfloat16 x is exact in float32 and the sums are
// float32 sums (relative error 1.7e-7 at H = 7168 against 1.5e-6 of one fused
// multiply-add chain per logit).  The hidden index is cut into 32 runs
// whatever n is: 8 over the grid, so that 16 tokens already fill 64
// compute units and 1000 tokens two workgroups on each, and 4 over a
// workgroup's waves.  The four waves' sums meet in LDS and the eight
// workgroups' in a second kernel, always in the same order, so a token's
// logits do not depend on n.
#include "internal.h"
#include "layout.h"

namespace moeq {

namespace {

__device__ __forceinline__ float wave_sum(float v) {
  v += __shfl_xor(v, 1, 64);
  v += __shfl_xor(v, 2, 64);
  v += __shfl_xor(v, 4, 64);
  v += __shfl_xor(v, 8, 64);
  v += __shfl_xor(v, 16, 64);
  v += __shfl_xor(v, 32, 64);
  return v;
}

// grid = E workgroups of 256 threads; H a multiple of 128, n <= kGateFewTokens
__global__ __launch_bounds__(256) void gate_few_kernel(const uint16_t* x, const float* w, int n, int H, int E,
                                                      float* logits) {
  __shared__ float part[4][kGateFewTokens];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int e = blockIdx.x;
  const int C = H / 4;  // float4 columns
  const MOEQ_GLOBAL f32x4* wr = gptr(reinterpret_cast<const f32x4*>(w + (size_t)e * H));
  const MOEQ_GLOBAL u32x2* xg = gptr(reinterpret_cast<const u32x2*>(x));
  float acc[kGateFewTokens];
#pragma unroll
  for (int t = 0; t < kGateFewTokens; ++t) acc[t] = 0.0f;
  // H <= 8192 gives at most 8 columns per thread: load them all, then use them
  constexpr int kMaxCols = 8;
  f32x4 wv[kMaxCols];
#pragma unroll
  for (int i = 0; i < kMaxCols; ++i) {
    const int c = tid + 256 * i;
    wv[i] = c < C ? __builtin_nontemporal_load(wr + c) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
#pragma unroll
  for (int t = 0; t < kGateFewTokens; ++t) {
    if (t < n) {
      float a = 0.0f;
#pragma unroll
      for (int i = 0; i < kMaxCols; ++i) {
        const int c = tid + 256 * i;
        if (c < C) {
          const u32x2 p = xg[(size_t)t * C + c];
          a = fmaf(bf16_lo(p.x), wv[i].x, a);
          a = fmaf(bf16_hi(p.x), wv[i].y, a);
          a = fmaf(bf16_lo(p.y), wv[i].z, a);
          a = fmaf(bf16_hi(p.y), wv[i].w, a);
        }
      }
      acc[t] = a;
    }
  }
#pragma unroll
  for (int t = 0; t < kGateFewTokens; ++t) {
    if (t < n) {
      const float v = wave_sum(acc[t]);
      if (lane == 0) part[wave][t] = v;
    }
  }
  __syncthreads();
  if (tid < n) logits[(size_t)tid * E + e] = ((part[0][tid] + part[1][tid]) + part[2][tid]) + part[3][tid];
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// upper 16 bits of two dwords: (bf16 truncation of a, of b) with a in the low half
__device__ __forceinline__ uint32_t pack_hi16(float a, float b) {
  return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
}
__device__ __forceinline__ float hi16(float v) { return __uint_as_float(__float_as_uint(v) & 0xFFFF0000u); }

// Partial logits of one run of the hidden index: workgroup (z, expert tile,
// token tile), wave w takes run 4 z + w of 32.  Operands of
// v_mfma_f32_32x32x16_bf16: lane (r, h) = (lane % 32, lane / 32) holds, of a
// group of 32 hidden values, values 16 h + 8 s .. + 7 of expert row r (first
// operand) and token r (second) in step s = 0, 1: contiguous loads, and any
// order of k serves as long as both agree.
//
// Bound by latency for few tokens (16 tokens, 256 experts, H = 7168: 64
// workgroups, 10 us) and by the reads of x and W_r from L2 beyond (1000
// tokens: 26 us; z is the fastest grid index, so an XCD holds one eighth of
// both).  A kernel with 64 x 64 tiles in LDS and one fused multiply-add chain
// per logit took 686 us at 16 tokens (4 workgroups) and 649 us at 1000.
// grid = (kGateSplit, ceil(E / 32), ceil(n / (32 NT))), 256 threads
template <int NT>
__global__ __launch_bounds__(256, 2) void gate_mfma_kernel(const uint16_t* x, const float* w, int n, int H, int E,
                                                          float* part) {
  __shared__ f32x4 red[4][NT * 4 * 64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, h = lane >> 5;
  const int e0 = blockIdx.y * 32, t0 = blockIdx.z * 32 * NT;
  const int G = H / 32, run = blockIdx.x * 4 + wave;
  const int g0 = run * G / (4 * kGateSplit), g1 = (run + 1) * G / (4 * kGateSplit);
  const MOEQ_GLOBAL f32x4* wr = gptr(reinterpret_cast<const f32x4*>(w + (size_t)min(e0 + r, E - 1) * H)) + 4 * h;
  const MOEQ_GLOBAL u32x4* xr[NT];
#pragma unroll
  for (int T = 0; T < NT; ++T)
    xr[T] = gptr(reinterpret_cast<const u32x4*>(x + (size_t)min(t0 + 32 * T + r, n - 1) * H)) + 2 * h;
  f32x16 acc[NT];
#pragma unroll
  for (int T = 0; T < NT; ++T)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[T][v] = 0.0f;
  f32x4 wn[4];
  u32x4 xn[NT][2];
  auto load = [&](int g) {
#pragma unroll
    for (int i = 0; i < 4; ++i) wn[i] = wr[8 * g + i];
#pragma unroll
    for (int T = 0; T < NT; ++T) {
      xn[T][0] = xr[T][4 * g];
      xn[T][1] = xr[T][4 * g + 1];
    }
  };
  if (g0 < g1) load(g0);
  for (int g = g0; g < g1; ++g) {
    f32x4 wv[4];
    u32x4 xv[NT][2];
#pragma unroll
    for (int i = 0; i < 4; ++i) wv[i] = wn[i];
#pragma unroll
    for (int T = 0; T < NT; ++T) {
      xv[T][0] = xn[T][0];
      xv[T][1] = xn[T][1];
    }
    load(min(g + 1, g1 - 1));
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const float f[8] = {wv[2 * s].x, wv[2 * s].y, wv[2 * s].z, wv[2 * s].w,
                          wv[2 * s + 1].x, wv[2 * s + 1].y, wv[2 * s + 1].z, wv[2 * s + 1].w};
      u32x4 hi, md, lo;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float a = f[2 * i], b = f[2 * i + 1];
        const float a1 = a - hi16(a), b1 = b - hi16(b);      // exact
        const float a2 = a1 - hi16(a1), b2 = b1 - hi16(b1);  // exact, at most 8 bits
        hi[i] = pack_hi16(a, b);
        md[i] = pack_hi16(a1, b1);
        lo[i] = pack_hi16(a2, b2);
      }
#pragma unroll
      for (int T = 0; T < NT; ++T) {
        const bf16x8 xb = __builtin_bit_cast(bf16x8, xv[T][s]);
        acc[T] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, lo), xb, acc[T], 0, 0, 0);
        acc[T] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, md), xb, acc[T], 0, 0, 0);
        acc[T] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, hi), xb, acc[T], 0, 0, 0);
      }
    }
  }
  // element v of lane (c, h): expert 8 (v / 4) + 4 h + v % 4, token c
#pragma unroll
  for (int T = 0; T < NT; ++T)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      red[wave][(T * 4 + q) * 64 + lane] = f32x4{acc[T][4 * q], acc[T][4 * q + 1], acc[T][4 * q + 2], acc[T][4 * q + 3]};
  __syncthreads();
  const int Ep = gate_pitch(E);
  for (int i = tid; i < NT * 4 * 64; i += 256) {
    const f32x4 s = ((red[0][i] + red[1][i]) + red[2][i]) + red[3][i];
    const int l = i & 63, q = (i >> 6) & 3, T = i >> 8;
    const int t = t0 + 32 * T + (l & 31), e = e0 + 8 * q + 4 * (l >> 5);
    if (t < n) *reinterpret_cast<f32x4*>(part + ((size_t)blockIdx.x * n + t) * Ep + e) = s;
  }
}

// logits = the eight partial sums in order.  A value that is not finite (an
// infinite or NaN x, or an overflow) is summed again as one fused
// multiply-add chain: the split of W_r turns an infinite x into NaN.
__global__ __launch_bounds__(256) void gate_sum_kernel(const float* part, const uint16_t* x, const float* w, int n,
                                                       int H, int E, float* logits) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n * E) return;
  const int t = i / E, e = i % E, Ep = gate_pitch(E);
  float v[kGateSplit];
#pragma unroll
  for (int z = 0; z < kGateSplit; ++z) v[z] = part[((size_t)z * n + t) * Ep + e];
  float s = v[0];
#pragma unroll
  for (int z = 1; z < kGateSplit; ++z) s += v[z];
  if (!(fabsf(s) < INFINITY)) {
    s = 0.0f;
    for (int k = 0; k < H; ++k) s = fmaf(__uint_as_float((uint32_t)x[(size_t)t * H + k] << 16), w[(size_t)e * H + k], s);
  }
  logits[i] = s;
}

}  // namespace

namespace {
template <int NT>
hipError_t launch_gate_mfma(const uint16_t* x, const float* w, int n, int H, int E, float* part, float* logits,
                            hipStream_t s) {
  const dim3 grid(kGateSplit, (E + 31) / 32, (n + 32 * NT - 1) / (32 * NT));
  gate_mfma_kernel<NT><<<grid, 256, 0, s>>>(x, w, n, H, E, part);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  gate_sum_kernel<<<(n * E + 255) / 256, 256, 0, s>>>(part, x, w, n, H, E, logits);
  return hipGetLastError();
}
}  // namespace

// n <= kGateFewTokens: the streaming kernel reads W_r once with a workgroup
// per expert and needs no second launch (4.8 us at one token).  Beyond, the
// tokens per workgroup grow with n: 32 up to 64 tokens (more workgroups), 128
// above (fewer reads of W_r).
hipError_t launch_router_gate(const uint16_t* x, const float* w, int n, int H, int E, float* part, float* logits,
                              hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (n <= kGateFewTokens) {
    gate_few_kernel<<<E, 256, 0, s>>>(x, w, n, H, E, logits);
    return hipGetLastError();
  }
  for (int t = 0; t < n; t += kGateChunk) {
    const int m = n - t < kGateChunk ? n - t : kGateChunk;
    const uint16_t* xt = x + (size_t)t * H;
    float* lt = logits + (size_t)t * E;
    const hipError_t e = n <= 64 ? launch_gate_mfma<1>(xt, w, m, H, E, part, lt, s)
                                 : launch_gate_mfma<4>(xt, w, m, H, E, part, lt, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace moeq
