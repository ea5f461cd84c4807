// Weight-format kernels: canonical packing -> device layout (repack), device
// layout -> float32 through each decoder the products use (diagnostics), and
// float32 -> canonical packing (quantize).
//
// The format is the symmetric block format standing in for the paper's
// per-tensor low-bit formats (Section 3.3): weight = d * (c - 2^(b-1)), one
// binary16 scale d per 32 weights, b-bit codes packed least significant bit
// first within each block.
#include "internal.h"
#include "layout.h"

namespace moeq {

namespace {

// codes of one block (32 values < 2^b) -> its b device dwords
template <int B>
__device__ __forceinline__ void encode_block(const uint8_t* c, uint32_t* w) {
#pragma unroll
  for (int d = 0; d < B; ++d) w[d] = 0u;
  if constexpr (B == 8) {
    uint8_t lo[32], hi[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) {
      lo[i] = c[i] & 15;
      hi[i] = c[i] >> 4;
    }
    encode_block<4>(lo, w);
    encode_block<4>(hi, w + 4);
  } else if constexpr (B == 6) {
#pragma unroll
    for (int d = 0; d < 6; ++d)
#pragma unroll
      for (int f = 0; f < 2; ++f)
        w[d] |= (uint32_t)c[4 * d + 2 * f] << (6 * f) | (uint32_t)c[4 * d + 2 * f + 1] << (16 + 6 * f);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const uint32_t c0 = c[24 + 2 * m], c1 = c[25 + 2 * m];
      w[m] |= (c0 & 15u) << 12 | (c1 & 15u) << 28;
      const int sh = 12 + 2 * (m & 1);
      w[4 + m / 2] |= (c0 >> 4) << sh | (c1 >> 4) << (16 + sh);
    }
  } else if constexpr (B == 5) {
#pragma unroll
    for (int d = 0; d < 5; ++d)
#pragma unroll
      for (int f = 0; f < 3; ++f)
        w[d] |= (uint32_t)c[6 * d + 2 * f] << (5 * f) | (uint32_t)c[6 * d + 2 * f + 1] << (16 + 5 * f);
#pragma unroll
    for (int q = 0; q < 5; ++q)
      w[q] |= ((uint32_t)(c[30] >> q) & 1u) << 15 | ((uint32_t)(c[31] >> q) & 1u) << 31;
  } else if constexpr (B == 4) {
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
      for (int s = 0; s < 4; ++s)
        w[d] |= (uint32_t)c[8 * d + 2 * s] << (4 * s) | (uint32_t)c[8 * d + 2 * s + 1] << (16 + 4 * s);
  } else if constexpr (B == 2) {
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int s = 0; s < 8; ++s)
        w[d] |= (uint32_t)c[16 * d + 2 * s] << (2 * s) |
                (uint32_t)c[16 * d + 2 * s + 1] << (16 + 2 * s);
  } else {
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int f = 0; f < 5; ++f)
        w[d] |= (uint32_t)c[10 * d + 2 * f] << (3 * f) |
                (uint32_t)c[10 * d + 2 * f + 1] << (16 + 3 * f);
#pragma unroll
    for (int q = 0; q < 3; ++q)
      w[q] |= ((uint32_t)(c[30] >> q) & 1u) << 15 | ((uint32_t)(c[31] >> q) & 1u) << 31;
  }
}

// One thread per (row, unit), lanes along the 64 rows of a tile so that the
// chunks leave in whole lines: 4 canonical blocks (16 * B bytes) in, b chunks
// out, the codes moved between registers with shifts known at compile time.
// WORDS: the canonical codes are 4-byte aligned (else bytes).
template <int B, bool WORDS>
__global__ __launch_bounds__(256) void repack_kernel(const uint8_t* canon, int rows, int K, uint32_t* dev) {
  const int U = K / kUnit;
  const long long gid = (long long)blockIdx.x * 256 + threadIdx.x;
  if (gid >= (long long)rows * U) return;
  const long long tu = gid / kRowTile;
  const int r = (int)(tu / U) * kRowTile + (int)(gid % kRowTile), u = (int)(tu % U);
  const uint8_t* src = canon + ((size_t)r * U + u) * 16 * B;
  uint32_t cw[4 * B];
#pragma unroll
  for (int i = 0; i < 4 * B; ++i) {
    if constexpr (WORDS)
      cw[i] = reinterpret_cast<const uint32_t*>(src)[i];
    else
      cw[i] = (uint32_t)src[4 * i] | (uint32_t)src[4 * i + 1] << 8 | (uint32_t)src[4 * i + 2] << 16 |
              (uint32_t)src[4 * i + 3] << 24;
  }
  uint32_t w[4 * B];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    uint8_t c[kBlock];
#pragma unroll
    for (int i = 0; i < kBlock; ++i) {
      const int bit = i * B, d = q * B + (bit >> 5), s = bit & 31;
      uint32_t v = cw[d] >> s;
      if (s + B > 32) v |= cw[d + 1] << (32 - s);
      c[i] = (uint8_t)(v & ((1u << B) - 1u));
    }
    encode_block<B>(c, w + q * B);
  }
  u32x4* out = reinterpret_cast<u32x4*>(dev) + (size_t)tu * B * kRowTile + gid % kRowTile;
#pragma unroll
  for (int j = 0; j < B; ++j) out[j * kRowTile] = u32x4{w[4 * j], w[4 * j + 1], w[4 * j + 2], w[4 * j + 3]};
}

__device__ __forceinline__ uint32_t scale_key(uint32_t v) {
  const uint32_t mag = v & 0x7FFFu;
  return (v & 0x8000u) || mag == 0 || mag >= 0x7C00u ? 0xFFFFu : mag;
}

// one thread per (row, pair of units): 8 scales (4 and zeros past an odd row)
__global__ __launch_bounds__(256) void repack_scales_kernel(const uint16_t* canon, int rows, int K, uint16_t* dev,
                                                            uint32_t* key) {
  __shared__ uint32_t wmax[4];
  const int U = K / kUnit, P = (U + 1) / 2;
  const long long gid = (long long)blockIdx.x * 256 + threadIdx.x;
  uint32_t m = 0;
  if (gid < (long long)rows * P) {
    const long long tp = gid / kRowTile;
    const int r = (int)(tp / P) * kRowTile + (int)(gid % kRowTile), p = (int)(tp % P);
    const uint16_t* src = canon + (size_t)r * (K / kBlock) + 8 * p;
    const int ns = 2 * p + 1 < U ? 8 : 4;
    uint32_t v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      v[i] = i < ns ? src[i] : 0u;
      if (i < ns) m = max(m, scale_key(v[i]));
    }
    reinterpret_cast<u32x4*>(dev)[gid] =
        u32x4{v[0] | v[1] << 16, v[2] | v[3] << 16, v[4] | v[5] << 16, v[6] | v[7] << 16};
  }
  for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, 64));
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    m = max(max(wmax[0], wmax[1]), max(wmax[2], wmax[3]));
    if (m) atomicMax(key, m);
  }
}

// one thread per (row, unit): the bfloat16-form unpacking of block_pairs
// (the 5/6/8-bit matrix-vector kernels), then
// d * (c - 2^(b-1)) exactly
template <int B>
__global__ __launch_bounds__(256) void dequant_kernel(TensorDev t, float* out) {
  const int U = t.K / kUnit;
  const long long gid = (long long)blockIdx.x * 256 + threadIdx.x;
  if (gid >= (long long)t.rows * U) return;
  const int r = (int)(gid / U), u = (int)(gid % U);
  uint32_t w[4 * B];
  load_unit<B>(row_chunks(t.codes, B, U, r), u, w);
  const u32x2 sc = row_scales(t.scales, U, r)[scale_step(u)];
  const float z = (float)(1 << (B - 1)), unit = (float)(1 << (B <= 7 ? 7 - B : 0));
  float* o = out + (size_t)r * t.K + kUnit * u;
  const PairConsts pk = pair_consts();
  for (int q = 0; q < 4; ++q) {
    const float d = half_to_float(((q < 2 ? sc.x : sc.y) >> (16 * (q & 1))) & 0xFFFFu);
    if constexpr (B == 8) {
      uint32_t pl[16], ph[16];
      block_pairs<4>(w + 8 * q, pk, pl);
      block_pairs<4>(w + 8 * q + 4, pk, ph);
      for (int P = 0; P < 16; ++P) {
        const float c0 = (bf16_lo(ph[P]) - 128.0f) * 2.0f + (bf16_lo(pl[P]) - 128.0f) / 8.0f;
        const float c1 = (bf16_hi(ph[P]) - 128.0f) * 2.0f + (bf16_hi(pl[P]) - 128.0f) / 8.0f;
        o[32 * q + 2 * P] = d * (c0 - z);
        o[32 * q + 2 * P + 1] = d * (c1 - z);
      }
    } else {
      uint32_t p[16];
      block_pairs<B>(w + q * B, pk, p);
      for (int P = 0; P < 16; ++P) {
        const float c0 = (bf16_lo(p[P]) - 128.0f) / unit, c1 = (bf16_hi(p[P]) - 128.0f) / unit;
        o[32 * q + 2 * P] = d * (c0 - z);
        o[32 * q + 2 * P + 1] = d * (c1 - z);
      }
    }
  }
}

// one thread per (row, unit): the binary16-subnormal code pairs of
// block_pairs_sub (the one-token gate/up and the 2-4-bit down matrix-vector
// kernels).  Pair P's two halves are c * 2^(k-24) with k = sub_shift<B>(P);
// c is rebuilt exactly as that value times 2^(24-k), then d * (c - 2^(b-1)).
template <int B>
__global__ __launch_bounds__(256) void dequant_sub_kernel(TensorDev t, float* out) {
  const int U = t.K / kUnit;
  const long long gid = (long long)blockIdx.x * 256 + threadIdx.x;
  if (gid >= (long long)t.rows * U) return;
  const int r = (int)(gid / U), u = (int)(gid % U);
  uint32_t w[4 * B];
  load_unit<B>(row_chunks(t.codes, B, U, r), u, w);
  const u32x2 sc = row_scales(t.scales, U, r)[scale_step(u)];
  const float z = (float)(1 << (B - 1));
  float* o = out + (size_t)r * t.K + kUnit * u;
  for (int q = 0; q < 4; ++q) {
    const float d = half_to_float(((q < 2 ? sc.x : sc.y) >> (16 * (q & 1))) & 0xFFFFu);
    uint32_t p[16];
    block_pairs_sub<B>(w + q * B, p);
#pragma unroll
    for (int P = 0; P < 16; ++P) {
      const float up = __builtin_amdgcn_ldexpf(1.0f, 24 - sub_shift<B>(P));
      const float c0 = half_to_float(p[P] & 0xFFFFu) * up, c1 = half_to_float(p[P] >> 16) * up;
      o[32 * q + 2 * P] = d * (c0 - z);
      o[32 * q + 2 * P + 1] = d * (c1 - z);
    }
  }
}

// binary16 of amax / qm, rounded once to nearest even from the exact quotient:
// the float32 quotient is made odd when it is inexact (truncated, last bit
// set), so that the second rounding sees which side of a tie the exact value
// lies on.
__device__ __forceinline__ uint16_t half_rne_quotient(float amax, float qm) {
  const float q = amax / qm;  // correctly rounded
  const float r = fmaf(-q, qm, amax);
  uint32_t u = __float_as_uint(q);
  if (r != 0.0f && q < 65536.0f) {
    if (r < 0.0f) --u;
    u |= 1u;
  }
  return __builtin_bit_cast(uint16_t, (_Float16)__uint_as_float(u));
}

// clamp(rint(w / d), -qm, qm), ties to even from the exact quotient; d > 0 or
// infinite (then 0), inv = 1 / d.  w * inv is within 2^-22 of the quotient
// relatively, so the rounded product k is off by at most one and only next to
// a tie; the remainder w - k d is exact (one fused multiply-add) and decides.
__device__ __forceinline__ int quantize_code(float w, float d, float inv, float qm) {
  float k = rintf(fminf(fmaxf(w * inv, -256.0f), 256.0f));
  const float r2 = 2.0f * fmaf(-k, d, w), a = fabsf(r2);
  const bool odd = (int)k & 1;
  if (a > d || (a == d && odd)) k += r2 > 0.0f ? 1.0f : -1.0f;
  return (int)fminf(fmaxf(k, -qm), qm);
}

// Eight values per lane, four lanes per block of 32, kQuantSteps wave-wide
// pieces of 512 values per wave with all their loads in flight; the lanes'
// packed bits meet in LDS and leave as dwords.  Memory-bound: 4 bytes read
// and bits / 8 written per value (16 us for 2048 x 7168 at 3 bits, 4 TB/s).  One thread per block (128-byte strides
// between lanes, a byte store per code byte, double-precision quotients) took
// 233 us.
// ALIGNED: w on 16 bytes and codes on 4 (else element loads, byte stores).
constexpr int kQuantSteps = 2;
template <int B, bool ALIGNED>
__global__ __launch_bounds__(256) void quantize_kernel(const float* w, long long n, uint8_t* codes,
                                                       uint16_t* scales) {
  __shared__ uint32_t bits_l[4][kQuantSteps][16 * B];  // 64 * B bytes per wave piece
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long base = ((long long)blockIdx.x * 4 + wave) * (512 * kQuantSteps);  // the wave's first value
  constexpr int z = 1 << (B - 1);
  constexpr float qm = (float)(z - 1);
  float f[kQuantSteps][8];
#pragma unroll
  for (int s = 0; s < kQuantSteps; ++s) {
    const long long i = base + 512 * s + 8 * lane;
    // (n is a multiple of 32: a block's four lanes are all in or all out)
    if (i < n) {
      if constexpr (ALIGNED) {
        const MOEQ_GLOBAL f32x4* src = gptr(reinterpret_cast<const f32x4*>(w + i));
        const f32x4 v0 = src[0], v1 = src[1];
        f[s][0] = v0.x; f[s][1] = v0.y; f[s][2] = v0.z; f[s][3] = v0.w;
        f[s][4] = v1.x; f[s][5] = v1.y; f[s][6] = v1.z; f[s][7] = v1.w;
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) f[s][j] = w[i + j];
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) f[s][j] = 0.0f;
    }
  }
#pragma unroll
  for (int s = 0; s < kQuantSteps; ++s) {
    float am = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) am = fmaxf(am, fabsf(f[s][j]));
    am = fmaxf(am, __shfl_xor(am, 1, 64));
    am = fmaxf(am, __shfl_xor(am, 2, 64));
    const uint16_t hb = half_rne_quotient(am, qm);
    const float d = half_to_float(hb);
    const float inv = 1.0f / d;
    uint64_t acc = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int q = d > 0.0f ? quantize_code(f[s][j], d, inv, qm) : 0;
      acc |= (uint64_t)(uint32_t)(q + z) << (B * j);
    }
    const long long i = base + 512 * s + 8 * lane;
    if (i < n && (lane & 3) == 0) scales[i / kBlock] = hb;
    uint8_t* dst = reinterpret_cast<uint8_t*>(bits_l[wave][s]) + lane * B;
#pragma unroll
    for (int j = 0; j < B; ++j) dst[j] = (uint8_t)(acc >> (8 * j));
  }
  __syncthreads();
#pragma unroll
  for (int s = 0; s < kQuantSteps; ++s) {
    const long long i = base + 512 * s;
    const int nb = (int)(min(512ll, max(0ll, n - i)) * B / 8);  // bytes of this piece, a multiple of 4 B
    uint8_t* dst = codes + i * B / 8;
    if constexpr (ALIGNED) {
      for (int j = lane; j < nb / 4; j += 64) reinterpret_cast<uint32_t*>(dst)[j] = bits_l[wave][s][j];
    } else {
      const uint8_t* src = reinterpret_cast<const uint8_t*>(bits_l[wave][s]);
      for (int j = lane; j < nb; j += 64) dst[j] = src[j];
    }
  }
}

}  // namespace

hipError_t launch_repack(const uint8_t* canon, int rows, int K, int bits, uint32_t* dev,
                         hipStream_t s) {
  const long long n = (long long)rows * (K / kUnit);
  const int grid = (int)((n + 255) / 256);
#define REPACK(B)                                             \
  case B:                                                     \
    if (((uintptr_t)canon & 3) == 0)                          \
      repack_kernel<B, true><<<grid, 256, 0, s>>>(canon, rows, K, dev);  \
    else                                                      \
      repack_kernel<B, false><<<grid, 256, 0, s>>>(canon, rows, K, dev); \
    break
  switch (bits) {
    REPACK(2);
    REPACK(3);
    REPACK(4);
    REPACK(5);
    REPACK(6);
    REPACK(8);
    default: return hipErrorInvalidValue;
  }
#undef REPACK
  return hipGetLastError();
}

hipError_t launch_repack_scales(const uint16_t* canon, int rows, int K, uint16_t* dev, uint32_t* key, hipStream_t s) {
  const long long n = (long long)rows * ((K / kUnit + 1) / 2);
  repack_scales_kernel<<<(int)((n + 255) / 256), 256, 0, s>>>(canon, rows, K, dev, key);
  return hipGetLastError();
}

hipError_t launch_dequant_sub(const TensorDev& t, float* out, hipStream_t s) {
  const long long n = (long long)t.rows * (t.K / kUnit);
  const int grid = (int)((n + 255) / 256);
  switch (t.bits) {
    case 2: dequant_sub_kernel<2><<<grid, 256, 0, s>>>(t, out); break;
    case 3: dequant_sub_kernel<3><<<grid, 256, 0, s>>>(t, out); break;
    case 4: dequant_sub_kernel<4><<<grid, 256, 0, s>>>(t, out); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_dequant(const TensorDev& t, float* out, hipStream_t s) {
  const long long n = (long long)t.rows * (t.K / kUnit);
  const int grid = (int)((n + 255) / 256);
  switch (t.bits) {
    case 2: dequant_kernel<2><<<grid, 256, 0, s>>>(t, out); break;
    case 3: dequant_kernel<3><<<grid, 256, 0, s>>>(t, out); break;
    case 4: dequant_kernel<4><<<grid, 256, 0, s>>>(t, out); break;
    case 5: dequant_kernel<5><<<grid, 256, 0, s>>>(t, out); break;
    case 6: dequant_kernel<6><<<grid, 256, 0, s>>>(t, out); break;
    case 8: dequant_kernel<8><<<grid, 256, 0, s>>>(t, out); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

namespace {
template <int B>
void quantize_launch(const float* w, long long n, uint8_t* codes, uint16_t* scales, hipStream_t s) {
  const int grid = (int)((n + 2048 * kQuantSteps - 1) / (2048 * kQuantSteps));
  if (((uintptr_t)w & 15) == 0 && ((uintptr_t)codes & 3) == 0)
    quantize_kernel<B, true><<<grid, 256, 0, s>>>(w, n, codes, scales);
  else
    quantize_kernel<B, false><<<grid, 256, 0, s>>>(w, n, codes, scales);
}
}  // namespace

hipError_t launch_quantize(const float* w, int rows, int K, int bits, uint8_t* codes,
                           uint16_t* scales, hipStream_t s) {
  const long long n = (long long)rows * K;
  switch (bits) {
    case 2: quantize_launch<2>(w, n, codes, scales, s); break;
    case 3: quantize_launch<3>(w, n, codes, scales, s); break;
    case 4: quantize_launch<4>(w, n, codes, scales, s); break;
    case 5: quantize_launch<5>(w, n, codes, scales, s); break;
    case 6: quantize_launch<6>(w, n, codes, scales, s); break;
    case 8: quantize_launch<8>(w, n, codes, scales, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace moeq
