// Decode path: fused dequantize x matrix-vector products for small batches.
//
// Per token the layer (Fig. 1, middle, of arXiv 2509.25689) evaluates the k
// routed experts it chose and the shared expert(s), each a SwiGLU network
// h = silu(W_gate x) * (W_up x), o = W_down h, and sums the outputs with the
// routing weights.  The work per token is about 2 * sum_i k_i P_i FLOPs
// (Section 3.2), but at batch sizes of a few tokens every weight byte is used
// once, so the path is bound by streaming the packed weights from HBM.
//
// Work decomposition.  A workgroup handles one (expert slot, row tile) pair:
// the slot is a shared expert or one entry of the device-built list of active
// experts (no host synchronization: slots beyond the active count exit at
// once).  Lanes hold neighbouring rows (R of them) at 64 / R neighbouring
// 128-weight units, so a load of 16-byte chunks takes runs of 16 R bytes
// (layout.h) and reads the staged activations of only 64 / R units; the lanes
// and waves that share a row meet at the end in a fixed order, so results are
// deterministic.  The dot products accumulate in float32; the per-block scale
// and zero point are applied once per block.
//
// gate/up kernel: writes h (float32) for every assignment in bucket order.
// Arithmetic of the 2-4-bit kernels: the activations (x, exactly, and h) are
// staged in binary16 after a power-of-two prescale per block of 32 (11
// significant bits at any magnitude), the code pairs masked out of the packed
// dwords as binary16 subnormals (layout.h), the dot products run on
// v_dot2_f32_f16.  The 5/6/8-bit kernels stage bfloat16 and unpack to it.
// down kernel: the result, times the token's routing weight, is written as
// one partial row per (token, slot).
// combine kernel: y_t = sum_j partial(t, j) (j in slot order) + shared.
#include "internal.h"
#include "layout.h"
#include "route_wave.h"

namespace moeq {

namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

constexpr int kXStride = 68;  // dwords per staged unit: 64 + 4 padding against LDS bank conflicts

__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a),
                                         __builtin_bit_cast(bf16x2, b), c, false);
}
__device__ __forceinline__ float dot2h(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, a), __builtin_bit_cast(f16x2, b), c, false);
}

// Which expert and tokens a slot covers.
struct Slot {
  int desc;     // descriptor row (expert id, or E + s for shared expert s)
  int M;        // tokens in the bucket
  int base;     // first activation row (h) of the bucket
  int shared;   // shared expert index, or -1
};

// The slot's bucket; M = -1 for a slot beyond the active count.
__device__ __forceinline__ Slot slot_info(const DecodeArgs& a, int slot) {
  Slot s;
  if (slot < a.S) {
    s.desc = a.E + slot;
    s.M = a.n;
    s.base = a.n * a.k + slot * a.n;
    s.shared = slot;
    return s;
  }
  const int i = slot - a.S;
  s.shared = -1;
  if (i >= a.active[0]) {
    s.desc = 0;
    s.M = -1;
    s.base = 0;
    return s;
  }
  const int e = a.active[1 + i];
  s.desc = e;
  s.base = a.offsets[e];
  s.M = a.offsets[e + 1] - s.base;
  return s;
}

// One block's contribution for one token: d * sum_i (c_i - z) x_i, from the
// block's code pairs p, the token's 16 activation dwords at xl (and their lo
// parts at xl + lo_offset when NX = 2) and the block sum X.
template <int NX>
__device__ __forceinline__ float block_dot(const uint32_t (&p)[16], const uint32_t* xl, int lo_offset,
                                           float ds, float X, float acc_out) {
  float acc = 0.0f;
  const u32x4* x4 = reinterpret_cast<const u32x4*>(xl);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const u32x4 xv = x4[c];
    acc = dot2(p[4 * c + 0], xv.x, acc);
    acc = dot2(p[4 * c + 1], xv.y, acc);
    acc = dot2(p[4 * c + 2], xv.z, acc);
    acc = dot2(p[4 * c + 3], xv.w, acc);
  }
  if constexpr (NX == 2) {
    const u32x4* l4 = reinterpret_cast<const u32x4*>(xl + lo_offset);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const u32x4 xv = l4[c];
      acc = dot2(p[4 * c + 0], xv.x, acc);
      acc = dot2(p[4 * c + 1], xv.y, acc);
      acc = dot2(p[4 * c + 2], xv.z, acc);
      acc = dot2(p[4 * c + 3], xv.w, acc);
    }
  }
  return fmaf(ds, fmaf(-192.0f, X, acc), acc_out);
}

// block q's scale (binary16, 4 per unit in sc) times 2^24, for subnormal pairs
__device__ __forceinline__ float block_scale_sub(u32x2 sc, int q) {
  const uint32_t s16 = ((q < 2 ? sc.x : sc.y) >> (16 * (q & 1))) & 0xFFFFu;
  return half_to_float(s16) * 16777216.0f;
}

// One block's contribution for one token from its subnormal code pairs p
// (pair P = c * 2^(k_P - 24)), the token's 16 binary16 activation dwords at xl
// (prescaled by 2^-e) and xf = (X, 2^e), X the sum of the staged values:
//   d 2^e (2^24 sum_k 2^-k dot_k - z X) = (d 2^24) 2^e (dot - z 2^-24 X).
template <int B>
__device__ __forceinline__ float block_dot_sub(const uint32_t (&p)[16], const uint32_t* xl, float ds, float2 xf,
                                               float acc_out) {
  constexpr int NC = sub_classes<B>(), ST = sub_step<B>();
  float acc[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) acc[c] = 0.0f;
  const u32x4* x4 = reinterpret_cast<const u32x4*>(xl);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const u32x4 xv = x4[c];
    acc[sub_shift<B>(4 * c + 0) / ST] = dot2h(p[4 * c + 0], xv.x, acc[sub_shift<B>(4 * c + 0) / ST]);
    acc[sub_shift<B>(4 * c + 1) / ST] = dot2h(p[4 * c + 1], xv.y, acc[sub_shift<B>(4 * c + 1) / ST]);
    acc[sub_shift<B>(4 * c + 2) / ST] = dot2h(p[4 * c + 2], xv.z, acc[sub_shift<B>(4 * c + 2) / ST]);
    acc[sub_shift<B>(4 * c + 3) / ST] = dot2h(p[4 * c + 3], xv.w, acc[sub_shift<B>(4 * c + 3) / ST]);
  }
  float dot = acc[NC - 1];
#pragma unroll
  for (int c = NC - 2; c >= 0; --c) dot = fmaf(dot, 1.0f / (float)(1 << ST), acc[c]);
  constexpr float zs = (float)(1 << (B - 1)) * 0x1p-24f;
  return fmaf(ds * xf.y, fmaf(-zs, xf.x, dot), acc_out);
}

// A block's prescale exponent from its largest magnitude am: am * 2^-e lies in
// [2^14, 2^15); e >= -100 keeps 2^-e finite for an all-zero block.
__device__ __forceinline__ int block_exp(float am) {
  return max((int)((__float_as_uint(am) >> 23) & 0xFFu) - 141, -100);
}

// One thread's 16-byte piece (8 values) of a block of 32, whose four pieces
// are held by four consecutive threads of one wave (all active): binary16
// after the block's power-of-two prescale 2^-e (no overflow, 11 significant
// bits at any scale).
// The piece goes to dst; the block's first thread (first) writes
// (X, 2^e) to *xf, X the sum of the staged values.
__device__ __forceinline__ void stage_piece(const float (&f)[8], uint32_t* dst, float2* xf, bool first) {
  float am = 0.0f;
#pragma unroll
  for (int i = 0; i < 8; ++i) am = fmaxf(am, fabsf(f[i]));
  am = fmaxf(am, __shfl_xor(am, 1, 64));
  am = fmaxf(am, __shfl_xor(am, 2, 64));
  const int e = block_exp(am);
  const float sc = __builtin_amdgcn_ldexpf(1.0f, -e);
  uint32_t hv[4];
  float sum = 0.0f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const _Float16 h0 = (_Float16)(f[2 * i] * sc), h1 = (_Float16)(f[2 * i + 1] * sc);
    hv[i] = (uint32_t)__builtin_bit_cast(uint16_t, h0) | (uint32_t)__builtin_bit_cast(uint16_t, h1) << 16;
    sum += (float)h0 + (float)h1;
  }
  sum += __shfl_xor(sum, 1, 64);
  sum += __shfl_xor(sum, 2, 64);
  *reinterpret_cast<u32x4*>(dst) = u32x4{hv[0], hv[1], hv[2], hv[3]};
  if (first) *xf = make_float2(sum, __builtin_amdgcn_ldexpf(1.0f, e));
}

// the 8 bfloat16 values of a 16-byte piece as float
__device__ __forceinline__ void bf16x8_to_f32(const u32x4 v, float (&f)[8]) {
  f[0] = bf16_lo(v.x); f[1] = bf16_hi(v.x); f[2] = bf16_lo(v.y); f[3] = bf16_hi(v.y);
  f[4] = bf16_lo(v.z); f[5] = bf16_hi(v.z); f[6] = bf16_lo(v.w); f[7] = bf16_hi(v.w);
}

template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xF, false));
}

// sum over 8 lanes (half a DPP row); every lane holds it
__device__ __forceinline__ float half_sum8(float v) {
  v += dpp_f<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_f<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_f<0x141>(v);  // row_half_mirror: the other quad of the half row
  return v;
}

// v of lane l plus v of lane l ^ 16 (l ^ 32) in one vector instruction each
// (a shuffle through LDS at the end of every workgroup: 0.1 us per step of one token)
__device__ __forceinline__ float swap_sum16(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap_sum32(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Sum over the lanes l % R of a wave (R = 8, 16, 32 or 64), in a fixed order;
// every lane holds its row's total.
template <int R>
__device__ __forceinline__ float row_sum(float v) {
  if constexpr (R <= 8) v += dpp_f<0x128>(v);  // row_ror:8
  if constexpr (R <= 16) v = swap_sum16(v);
  if constexpr (R <= 32) v = swap_sum32(v);
  return v;
}

__device__ __forceinline__ float silu(float g) { return g / (1.0f + expf(-g)); }

// One unit of a row: its chunks and scales.
template <int B>
struct UnitBuf {
  uint32_t w[4 * B];
  u32x2 s;
};

// A row's chunks and scales (lanes of a wave hold different rows).
struct RowPtr {
  const MOEQ_GLOBAL u32x4* c;
  const MOEQ_GLOBAL u32x2* s;
};
__device__ __forceinline__ RowPtr row_ptr(const TensorDev& t, int bits, int U, int row) {
  return RowPtr{row_chunks(t.codes, bits, U, row), row_scales(t.scales, U, row)};
}

template <int B>
__device__ __forceinline__ void load_unit_buf(UnitBuf<B>& b, const RowPtr& r, int u) {
  load_unit<B>(r.c, u, b.w);
  b.s = r.s[scale_step(u)];
}

// acc[m] += d * sum (c - z) x_m over one 128-weight unit, for the mc <= TM
// tokens staged at xu / su4 (strides xts, sts)
template <int B, int TM>
__device__ __forceinline__ void unit_dots(const uint32_t* w, u32x2 sc, const uint32_t* xu, const float2* su4, int xts,
                                          int sts, int mc, float (&acc)[TM]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    uint32_t p[16];
    block_pairs_sub<B>(w + q * B, p);
    const float ds = block_scale_sub(sc, q);
    if constexpr (TM == 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < TM; ++m)
      if (TM == 1 || m < mc) acc[m] = block_dot_sub<B>(p, xu + m * xts + 16 * q, ds, su4[m * sts + q], acc[m]);
  }
}

// This lane's share of a row against the staged tokens: units u0, u0 + step,
// ... < U, the next one in flight while one is reduced; `first` holds unit
// min(u0, U - 1).
// One token: no branch in the loop.  A lane past the row computes on its last
// unit and drops the result, and an odd unit comes after the loop; scheduling
// barriers keep the next unit's requests before this one's products.  With a
// branch around the products the compiler no longer knows which loads are
// outstanding and waited for a unit's chunks before it requested the next
// (one token of the benchmark's layer, 7 slots 36.9 -> 35.9 us, 9 slots 44.1
// -> 42.8).  Several tokens keep the branches: without them the products of
// both units are scheduled together and spill.
template <int B, int TM>
__device__ __forceinline__ void row_dots(const RowPtr& r, int U, int u0, int step, const uint32_t* xl,
                                         const float2* xs, int xts, int sts, int mc, const UnitBuf<B>& first,
                                         float (&acc)[TM]) {
  UnitBuf<B> buf[2];
  buf[0] = first;
#pragma unroll
  for (int m = 0; m < TM; ++m) acc[m] = 0.0f;
  const int n = (U + step - 1) / step;  // the same for every lane
  // (requests past the row repeat its last unit)
  auto load = [&](UnitBuf<B>& b, int i) { load_unit_buf<B>(b, r, min(u0 + step * min(i, n - 1), U - 1)); };
  if constexpr (TM == 1) {
    auto dots = [&](const UnitBuf<B>& b, int i) {
      const int u = u0 + step * i, uc = min(u, U - 1);
      float v[1] = {acc[0]};
      unit_dots<B, 1>(b.w, b.s, xl + uc * kXStride, xs + uc * 4, xts, sts, mc, v);
      acc[0] = u < U ? v[0] : acc[0];
    };
#pragma unroll 1
    for (int i = 0; i + 2 <= n; i += 2) {
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        load(buf[1 - b], i + b + 1);
        __builtin_amdgcn_sched_barrier(0);
        dots(buf[b], i + b);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (n & 1) dots(buf[0], n - 1);
  } else {
#pragma unroll 1
    for (int i0 = 0; i0 < n; i0 += 2) {
      asm volatile("" ::: "memory");
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int i = i0 + b;
        if (i < n) {
          load(buf[1 - b], i + 1);
          const int u = u0 + step * i;
          if (u < U) unit_dots<B, TM>(buf[b].w, buf[b].s, xl + u * kXStride, xs + u * 4, xts, sts, mc, acc);
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Down x routing weight, one partial row per (token, slot).  A workgroup owns
// 4 R rows of one slot, a wave R of them with 64 / R units per step; TM tokens
// are staged per pass.
template <int B, int TM, int R>
__device__ __forceinline__ void down_body(const DecodeArgs& a, const Slot sl, const TensorDev& td, uint32_t* smem) {
  const int H = a.H, I = a.I, U = I / kUnit;
  const int xts = U * kXStride, sts = U * 4;  // per-token LDS strides (dwords, float2)
  uint32_t* xl = smem;
  float2* xs = reinterpret_cast<float2*>(smem + TM * xts);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int row = blockIdx.x * (4 * R) + wave * R + lane % R;  // (H is a multiple of 128)
  const RowPtr rp = row_ptr(td, B, U, row);
  for (int m0 = 0; m0 < sl.M; m0 += TM) {
    const int mc = min(TM, sl.M - m0);
    // the first unit is requested before h is staged
    UnitBuf<B> first;
    load_unit_buf<B>(first, rp, min(lane / R, U - 1));
    if (m0 > 0) __syncthreads();
    // stage h rows in binary16 with per-block prescales
    for (int m = 0; m < mc; ++m) {
      const MOEQ_GLOBAL f32x4* src = gptr(reinterpret_cast<const f32x4*>(a.h + (size_t)(sl.base + m0 + m) * I));
      for (int q = threadIdx.x; q < I / 8; q += 256) {
        const f32x4 v0 = src[2 * q], v1 = src[2 * q + 1];
        const float f[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
        const int uu = q >> 4, cq = q & 15;
        stage_piece(f, xl + m * xts + uu * kXStride + cq * 4, xs + m * sts + uu * 4 + (cq >> 2), (cq & 3) == 0);
      }
    }
    __syncthreads();
    float o[TM];
    row_dots<B, TM>(rp, U, lane / R, 64 / R, xl, xs, xts, sts, mc, first, o);
#pragma unroll
    for (int m = 0; m < TM; ++m) {
      if (m < mc) {
        const float os = row_sum<R>(o[m]);
        if (lane < R) {
          int prow;
          float wv;
          if (sl.shared >= 0) {
            prow = a.n * a.k + sl.shared * a.n + m0 + m;
            wv = 1.0f;
          } else {
            prow = a.perm[sl.base + m0 + m];
            wv = a.w[prow];
          }
          a.partial[(size_t)prow * H + row] = wv * os;
        }
      }
    }
  }
}

// grid = (H / (4 R), S + max_active), 256 threads
template <int TM, int R>
__global__ __launch_bounds__(256, TM <= 4 ? 4 : 2) void down_kernel(DecodeArgs a) {
  extern __shared__ uint32_t smem[];
  const Slot sl = slot_info(a, blockIdx.y);
  if (sl.M < 0 || sl.M > a.gemm_above) return;  // (large buckets: the grouped GEMMs)
  const TensorDev td = a.desc[sl.desc * 3 + 2];
  if (!td.codes) return;
  switch (td.bits) {
    case 2: down_body<2, TM, R>(a, sl, td, smem); break;
    case 3: down_body<3, TM, R>(a, sl, td, smem); break;
    case 4: down_body<4, TM, R>(a, sl, td, smem); break;
    default: break;
  }
}

// ---------------------------------------------------------------------------
// One token: down x routing weight and the combine in one pass, for layers
// whose down tensors are 2-4 bits wide with at most 16 units per row: one
// width BD, or (BD = 0) widths that differ between tensors, where every
// unit is fetched as four chunk loads, those past the slot's width from 16
// zero bytes that stay in the vector cache, and the slot's width picks the
// decoder.  A workgroup of 512 threads owns 32 rows of y across every slot
// (the token's k choices in choice order, then the shared experts): lane l of
// wave w holds row l % 32 and unit 2 w + l / 32 of it in every slot, with D
// slots' codes in flight.  A wave stages its own two units of every h row
// (binary16 with per-block prescales, as in the down kernel), so no barrier
// parts the staging from the products.  The lane accumulates w_j * (its partial
// dot of slot j) in slot order and the 16 lanes of a row are summed in a fixed
// order: no partial rows, no combine launch.
struct DownSlot {
  const uint32_t* codes;
  const uint16_t* scales;
  float w;
  int hrow;
  int bits;
};

// w_j-free partial dot of one slot's unit
template <int B>
__device__ __forceinline__ float down1_unit_dot(const uint32_t* w, u32x2 sc, const uint32_t* xu, const float2* su4) {
  float o[1] = {0.0f};
  unit_dots<B, 1>(w, sc, xu, su4, 0, 0, 1, o);
  return o[0];
}

// slots whose h a wave requests together, of those present (requests for absent
// ones, repeating the last, cost 0.5 us at 7 slots: 37.5 -> 37.0 us per step)
constexpr int kDown1Batch = 12;

template <int BD, int D>
__global__ __launch_bounds__(512) void down1_kernel(DecodeArgs a) {
  extern __shared__ uint32_t smem[];
  __shared__ DownSlot slots[kMaxTopK + kMaxShared];
  constexpr int R = 32, NW = 8;
  __shared__ float red[NW][R];
  const int H = a.H, I = a.I, U = I / kUnit, k = a.k, NS = a.k + a.S;
  if ((int)threadIdx.x < NS) {
    const int j = threadIdx.x;
    DownSlot v;
    if (j < k) {
      // choice j of the token: its bucket of one holds h row offsets[e]
      const int e = a.idx[j];
      const TensorDev t = a.desc[e * 3 + 2];
      v.codes = t.codes;
      v.scales = t.scales;
      v.w = a.w[j];
      v.hrow = a.offsets[e];
      v.bits = t.bits;
    } else {
      const TensorDev t = a.desc[(a.E + (j - k)) * 3 + 2];
      v.codes = t.codes;
      v.scales = t.scales;
      v.w = 1.0f;
      v.hrow = k + (j - k);
      v.bits = t.bits;
    }
    slots[j] = v;
  }
  __syncthreads();

  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int u = 2 * wave + lane / R;
  const int row = blockIdx.x * R + lane % R;  // (H is a multiple of 128)
  const int uc = min(u, U - 1);
  constexpr int BL = BD == 0 ? 4 : BD;  // chunks loaded per unit
  // (one width: the unit's place is the same in every slot)
  const size_t c_at = chunk_index(BL, U, row) + uc * BL * kRowTile, s_at = scale_index(U, row) + scale_step(uc);
  auto load_slot = [&](UnitBuf<BL>& b, int j) {
    const DownSlot& sl = slots[min(j, NS - 1)];
    if constexpr (BD == 0) {
      const int bits = sl.bits;
      const MOEQ_GLOBAL u32x4* r4 = row_chunks(sl.codes, bits, U, row) + uc * bits * kRowTile;
      const MOEQ_GLOBAL u32x4* z4 = gptr(reinterpret_cast<const u32x4*>(a.zeros));
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const u32x4 v = __builtin_nontemporal_load(c < bits ? r4 + c * kRowTile : z4);
        b.w[4 * c + 0] = v.x;
        b.w[4 * c + 1] = v.y;
        b.w[4 * c + 2] = v.z;
        b.w[4 * c + 3] = v.w;
      }
    } else {
      load_unit<BD>(gptr(reinterpret_cast<const u32x4*>(sl.codes)) + c_at, 0, b.w);
    }
    b.s = gptr(reinterpret_cast<const u32x2*>(sl.scales))[s_at];
  };
  UnitBuf<BL> buf[D];
#pragma unroll
  for (int i = 0; i < D - 1; ++i) load_slot(buf[i], i);

  // This wave's two units of every slot's h row: lane l converts values 4 l ..
  // of them, a block of 32 in 8 lanes.  (a unit past the row repeats the last
  // one; waves past the row stage nothing and add zeros)
  constexpr int kHs = 2 * kXStride;  // dwords per slot and wave
  const int nw = (U + 1) / 2;        // waves with units
  uint32_t* xl = smem + wave * NS * kHs;
  float2* xs = reinterpret_cast<float2*>(smem + nw * NS * kHs) + wave * NS * 8;
  if (wave < nw) {
    const int hu = lane >> 5, at = min(2 * wave + hu, U - 1) * kUnit + 4 * (lane & 31);
    for (int j0 = 0; j0 < NS; j0 += kDown1Batch) {
      f32x4 v[kDown1Batch];
#pragma unroll
      for (int i = 0; i < kDown1Batch; ++i)
        if (j0 + i < NS) v[i] = *gptr(reinterpret_cast<const f32x4*>(a.h + (size_t)slots[j0 + i].hrow * I + at));
#pragma unroll
      for (int i = 0; i < kDown1Batch; ++i) {
        if (j0 + i < NS) {
          float am = fmaxf(fmaxf(fabsf(v[i].x), fabsf(v[i].y)), fmaxf(fabsf(v[i].z), fabsf(v[i].w)));
          am = fmaxf(am, dpp_f<0xB1>(am));   // quad_perm [1,0,3,2]
          am = fmaxf(am, dpp_f<0x4E>(am));   // quad_perm [2,3,0,1]
          am = fmaxf(am, dpp_f<0x141>(am));  // row_half_mirror: the other quad of the 8 lanes
          const int e = block_exp(am);
          const float sc = __builtin_amdgcn_ldexpf(1.0f, -e);
          const _Float16 h0 = (_Float16)(v[i].x * sc), h1 = (_Float16)(v[i].y * sc), h2 = (_Float16)(v[i].z * sc),
                         h3 = (_Float16)(v[i].w * sc);
          const float sum = half_sum8(((float)h0 + (float)h1) + ((float)h2 + (float)h3));
          *reinterpret_cast<u32x2*>(xl + (j0 + i) * kHs + hu * kXStride + (lane & 31) * 2) =
              u32x2{(uint32_t)__builtin_bit_cast(uint16_t, h0) | (uint32_t)__builtin_bit_cast(uint16_t, h1) << 16,
                    (uint32_t)__builtin_bit_cast(uint16_t, h2) | (uint32_t)__builtin_bit_cast(uint16_t, h3) << 16};
          if ((lane & 7) == 0) xs[(j0 + i) * 8 + (lane >> 3)] = make_float2(sum, __builtin_amdgcn_ldexpf(1.0f, e));
        }
      }
    }
  }
  wave_sync();  // (the wave reads only what it wrote)

  const uint32_t* xu = xl + (lane / R) * kXStride;
  const float2* su4 = xs + (lane / R) * 4;
  float acc = 0.0f;
#pragma unroll 1
  for (int j0 = 0; j0 < (wave < nw ? NS : 0); j0 += D) {
    asm volatile("" ::: "memory");
#pragma unroll
    for (int b = 0; b < D; ++b) {
      const int j = j0 + b;
      if (j < NS) {
        // slot j + D - 1 goes out before slot j is reduced
        load_slot(buf[(b + D - 1) % D], j + D - 1);
        float o;
        if constexpr (BD == 0) {
          switch (__builtin_amdgcn_readfirstlane(slots[j].bits)) {
            case 2: o = down1_unit_dot<2>(buf[b].w, buf[b].s, xu + j * kHs, su4 + j * 8); break;
            case 3: o = down1_unit_dot<3>(buf[b].w, buf[b].s, xu + j * kHs, su4 + j * 8); break;
            default: o = down1_unit_dot<4>(buf[b].w, buf[b].s, xu + j * kHs, su4 + j * 8); break;
          }
        } else {
          o = down1_unit_dot<BD>(buf[b].w, buf[b].s, xu + j * kHs, su4 + j * 8);
        }
        acc = fmaf(slots[j].w, u < U ? o : 0.0f, acc);
      }
    }
  }
  acc = row_sum<R>(acc);
  if (lane < R) red[wave][lane] = acc;
  __syncthreads();
  if ((int)threadIdx.x < R) {
    float ys = red[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < NW; ++w) ys += red[w][threadIdx.x];
    a.y[row] = ys;
  }
}

// ---------------------------------------------------------------------------
// y_t = sum_j partial(t*k + j) + sum_s partial(n*k + s*n + t), fixed order;
// the loads of eight partial rows are issued together.
__global__ __launch_bounds__(256) void combine_kernel(DecodeArgs a) {
  const int H4 = a.H / 4;
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= (long long)a.n * H4) return;
  const int t = (int)(i / H4), c = (int)(i % H4);
  const float4* p = reinterpret_cast<const float4*>(a.partial);
  const int rows = a.k + a.S;
  float4 acc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  for (int j0 = 0; j0 < rows; j0 += 8) {
    float4 v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int j = j0 + q;
      if (j < rows) {
        const size_t r = j < a.k ? (size_t)t * a.k + j : (size_t)a.n * a.k + (size_t)(j - a.k) * a.n + t;
        v[q] = p[r * H4 + c];
      }
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (j0 + q < rows) {
        acc.x += v[q].x; acc.y += v[q].y; acc.z += v[q].z; acc.w += v[q].w;
      }
    }
  }
  reinterpret_cast<float4*>(a.y)[i] = acc;
}

// ---------------------------------------------------------------------------
// Gate/up + SwiGLU.  A workgroup of four waves owns R features of one slot: two
// waves take their gate rows, two their up rows (a wave decodes one width),
// each wave R rows at 64 / R units per step, the units of a row dealt to the
// two waves of its tensor.  The partial sums meet in LDS in wave order.
// One token: R = 16, so that the nine slots of the benchmark's layer make 1152
// workgroups, all resident at once (R = 32: 56.7 instead of 53.9 us per step,
// regrouped).  More tokens: R = 32, which halves the staging of x per weight (16
// tokens: 297 -> 270 us beside the one-token buckets).  Workgroups in launch order:
// renumbered so that the four of a 64-row tile share an XCD, or so that an XCD
// sees every quarter of its tiles, a step of one token takes 0.5 to 0.8 us more;
// with three units in flight instead of two 1.5 us more at 7 slots.
constexpr int kGuWaves = 4, kGuThreads = 64 * kGuWaves, kGuHalf = kGuWaves / 2;
constexpr int kGuRows1 = 16, kGuRowsN = 32;

template <int TM>
struct GateUpShared {
  float red[kGuWaves][TM][32];
};

// this lane's share of its row (of the tensor its wave takes); the first
// unit is requested before `stage` brings the tokens into LDS
template <int B, int TM, int R, typename F>
__device__ __forceinline__ void gateup_dots(const TensorDev& t, int row, int U, int u0, const uint32_t* xl,
                                            const float2* xs, int xts, int sts, int mc, F stage, float (&acc)[TM]) {
  const RowPtr rp = row_ptr(t, B, U, row);
  UnitBuf<B> first;
  load_unit_buf<B>(first, rp, min(u0, U - 1));
  stage();
  row_dots<B, TM>(rp, U, u0, kGuHalf * (64 / R), xl, xs, xts, sts, mc, first, acc);
}

// features [f0, f0 + R) of one slot for mc <= TM tokens, which `stage`
// brings into LDS (with a barrier at its end); h rows hrow .. hrow + mc - 1
template <int TM, int R, typename F>
__device__ __forceinline__ void gateup_rows(const DecodeArgs& a, const TensorDev& tg, const TensorDev& tu, int f0,
                                            int hrow, int mc, const uint32_t* xl, const float2* xs, int xts, int sts,
                                            GateUpShared<TM>& sh, F stage) {
  static_assert(128 % R == 0 && R <= 32, "whole workgroups, and their sums fit");
  const int H = a.H, I = a.I, U = H / kUnit;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const TensorDev& t = wave < kGuHalf ? tg : tu;
  const int row = f0 + lane % R, u0 = (wave % kGuHalf) * (64 / R) + lane / R;
  float acc[TM];
  switch (__builtin_amdgcn_readfirstlane(t.bits)) {
    case 2: gateup_dots<2, TM, R>(t, row, U, u0, xl, xs, xts, sts, mc, stage, acc); break;
    case 3: gateup_dots<3, TM, R>(t, row, U, u0, xl, xs, xts, sts, mc, stage, acc); break;
    default: gateup_dots<4, TM, R>(t, row, U, u0, xl, xs, xts, sts, mc, stage, acc); break;
  }
#pragma unroll
  for (int m = 0; m < TM; ++m) {
    const float v = row_sum<R>(acc[m]);
    if (lane < R) sh.red[wave][m][lane] = v;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < R * mc; i += kGuThreads) {
    const int m = i / R, r = i % R;
    float g = sh.red[0][m][r], u = sh.red[kGuHalf][m][r];
#pragma unroll
    for (int w = 1; w < kGuHalf; ++w) {
      g += sh.red[w][m][r];
      u += sh.red[kGuHalf + w][m][r];
    }
    a.h[(size_t)(hrow + m) * I + f0 + r] = silu(g) * u;
  }
}

// token t's x into LDS at xl / xs (binary16 with per-block prescales)
__device__ __forceinline__ void stage_x_token(const DecodeArgs& a, int t, uint32_t* xl, float2* xs) {
  const int H = a.H;
  const MOEQ_GLOBAL u32x4* src = gptr(reinterpret_cast<const u32x4*>(a.x + (size_t)t * H));
  for (int q = threadIdx.x; q < H / 8; q += kGuThreads) {
    float f[8];
    bf16x8_to_f32(src[q], f);
    const int uu = q >> 4, cq = q & 15;
    stage_piece(f, xl + uu * kXStride + cq * 4, xs + uu * 4 + (cq >> 2), (cq & 3) == 0);
  }
}

// token 0's x staged by threads [t0, t0 + nt) of the workgroup (nt a multiple
// of 64, t0 of 64: the four pieces of a block stay in four lanes of a wave)
__device__ __forceinline__ void stage_x1_token0(const DecodeArgs& a, int t0, int nt, uint32_t* xl, float2* xs) {
  const int H = a.H;
  const MOEQ_GLOBAL u32x4* src = gptr(reinterpret_cast<const u32x4*>(a.x));
  for (int q = (int)threadIdx.x - t0; q < H / 8; q += nt) {
    float f[8];
    bf16x8_to_f32(src[q], f);
    const int uu = q >> 4, cq = q & 15;
    stage_piece(f, xl + uu * kXStride + cq * 4, xs + uu * 4 + (cq >> 2), (cq & 3) == 0);
  }
}

// 2-4-bit gate and up tensors (the others: the wide kernels)
__device__ __forceinline__ bool narrow_gateup(const TensorDev& tg, const TensorDev& tu) {
  return tg.codes && tu.codes && tg.bits <= 4 && tu.bits <= 4;
}

// one workgroup's share of the gate/up of a bucket of one token (staged: x is
// in LDS already; one instance for both, uniform over the workgroup)
template <int R>
__device__ __forceinline__ void gateup1_slot(const DecodeArgs& a, const Slot& sl, uint32_t* smem, GateUpShared<1>& sh,
                                             bool staged) {
  const TensorDev tg = a.desc[sl.desc * 3 + 0], tu = a.desc[sl.desc * 3 + 1];
  if (!narrow_gateup(tg, tu)) return;
  uint32_t* xl = smem;
  float2* xs = reinterpret_cast<float2*>(smem + a.H / kUnit * kXStride);
  gateup_rows<1, R>(a, tg, tu, blockIdx.x * R, sl.base, 1, xl, xs, 0, 0, sh, [&] {
    if (!staged) {
      // (one token: token 0, without reading the bucket permutation, which the
      // routing workgroup of gateup1_route_kernel may still be writing)
      stage_x_token(a, sl.shared >= 0 || a.n == 1 ? 0 : a.perm[sl.base] / a.k, xl, xs);
      __syncthreads();
    }
  });
}

// The same for a forward of one token that needs no routing launch: wave 0
// of every workgroup of a routed slot routes the token itself (the routing
// kernels' selection, deterministic, so every workgroup finds the same
// experts; the other waves stage x meanwhile) while the shared experts'
// workgroups start at once.  Routed slot
// i is the i-th chosen expert in ascending id order, as the bucketing lists
// them.  Workgroup (0, S) also writes what the routing launch would have:
// idx and w in choice order, offsets, the active list and the permutation,
// which the down kernel and any 5/6/8-bit gate/up kernel read after this
// launch.  grid = (I / kGuRows1, S + k), kGuThreads threads.
template <int EPL>
__global__ __launch_bounds__(kGuThreads, 5) void gateup1_route_kernel(DecodeArgs a, RouterParams rp,
                                                                                Workspace ws) {
  extern __shared__ uint32_t smem[];
  __shared__ GateUpShared<1> sh;
  __shared__ float gs_l[64];
  __shared__ int32_t chosen[kMaxTopK];
  rp.kept_ids = nullptr;  // (gateup1_routes)
  Slot sl;
  if ((int)blockIdx.y < a.S) {
    sl = slot_info(a, blockIdx.y);
  } else {
    if (threadIdx.x < 64) {
      // (slots past the choices, which the creation checks rule out, read
      // expert 0's descriptor: in range, skipped if it holds no tensor)
      if (threadIdx.x < kMaxTopK) chosen[threadIdx.x] = 0;
      const bool out = blockIdx.x == 0 && (int)blockIdx.y == a.S;
      const LaneChoice<EPL> ch =
          route_token_wave<EPL>(rp, 0, gs_l, out ? ws.idx : nullptr, out ? ws.w : nullptr, nullptr);
      const int lane = threadIdx.x, E = rp.E_row;
      const int cnt = __popc(ch.bits);
      const int below = wave_incl_sum(cnt) - cnt;  // chosen ids of the lanes below
#pragma unroll
      for (int i = 0; i < EPL; ++i) {
        const int e = lane * EPL + i;
        const int r = below + __popc(ch.bits & ((1u << i) - 1u));
        const bool c = (ch.bits >> i) & 1u;
        if (c) chosen[r] = e;
        if (out) {
          if (e < E) ws.offsets[e] = r;
          if (c) {
            ws.active[1 + r] = e;
            ws.perm[r] = ch.order[i];
          }
        }
      }
      if (out && lane == 0) {
        ws.offsets[E] = rp.k;
        ws.active[0] = rp.k;
      }
    } else {
      // the other waves stage the token's x meanwhile
      const int U = a.H / kUnit;
      stage_x1_token0(a, 64, kGuThreads - 64, smem, reinterpret_cast<float2*>(smem + U * kXStride));
    }
    __syncthreads();
    const int i = blockIdx.y - a.S;
    sl.desc = __builtin_amdgcn_readfirstlane(chosen[i]);
    sl.base = i;
    sl.M = 1;
    sl.shared = -1;
  }
  gateup1_slot<kGuRows1>(a, sl, smem, sh, (int)blockIdx.y >= a.S);
}

// A forward of one token whose routing is a launch of its own (regrouped
// experts, or more than 256): the same 16 rows per workgroup (32 in
// gateupn_kernel: 56.7 instead of 53.9 us per step of the benchmark's layer).
// grid = (I / kGuRows1, S + max_active), kGuThreads threads
__global__ __launch_bounds__(kGuThreads, 5) void gateup1_kernel(DecodeArgs a) {
  extern __shared__ uint32_t smem[];
  __shared__ GateUpShared<1> sh;
  const Slot sl = slot_info(a, blockIdx.y);
  if (sl.M == 1) gateup1_slot<kGuRows1>(a, sl, smem, sh, false);
}

// ---------------------------------------------------------------------------
// The buckets of 1 .. gemm_above tokens, TM tokens staged per pass: each unit's
// code pairs are unpacked once and multiplied with every staged token.  One
// launch: two, the larger buckets' on a second stream, cost as much at 16
// tokens (the streams' events take about 20 us each way) and more below.
// TM = 2, or 8 for small layers (fits_8_tokens); W workgroups per compute unit
// at least.
// grid = (I / kGuRowsN, S + max_active), kGuThreads threads
template <int TM, int W>
__global__ __launch_bounds__(kGuThreads, W) void gateupn_kernel(DecodeArgs a) {
  extern __shared__ uint32_t smem[];
  __shared__ GateUpShared<TM> sh;
  const Slot sl = slot_info(a, blockIdx.y);
  if (sl.M < 1 || sl.M > a.gemm_above) return;
  if (sl.M == 1) {
    gateup1_slot<kGuRowsN>(a, sl, smem, reinterpret_cast<GateUpShared<1>&>(sh), false);
    return;
  }
  const TensorDev tg = a.desc[sl.desc * 3 + 0], tu = a.desc[sl.desc * 3 + 1];
  if (!narrow_gateup(tg, tu)) return;
  const int U = a.H / kUnit, xts = U * kXStride, sts = U * 4;  // per-token LDS strides (dwords, float2)
  uint32_t* xl = smem;
  float2* xs = reinterpret_cast<float2*>(smem + TM * xts);
  for (int m0 = 0; m0 < sl.M; m0 += TM) {
    const int mc = min(TM, sl.M - m0);
    // (the previous pass's last barrier came after its reads of x; its sums
    // are read before the barrier that ends the staging)
    gateup_rows<TM, kGuRowsN>(a, tg, tu, blockIdx.x * kGuRowsN, sl.base + m0, mc, xl, xs, xts, sts, sh, [&] {
      for (int m = 0; m < mc; ++m) {
        const int t = sl.shared >= 0 ? m0 + m : a.perm[sl.base + m0 + m] / a.k;
        stage_x_token(a, t, xl + m * xts, xs + m * sts);
      }
      __syncthreads();
    });
  }
}

// ---------------------------------------------------------------------------
// Wide tensors (5, 6 and 8 bits).  The kernels above skip a slot whose gate or
// up (down) tensor is wide; these take exactly those slots.  A workgroup of
// NW waves owns R rows of the tensor, a wave 64 / R units of each per step,
// the units of a row dealt to the waves, for up to TM tokens per pass (1 for a
// single token, else 4).  Gate, up and down are reduced one tensor at a time,
// so a wave decodes one width at a time.  Few slots (shared experts only)
// take 16 rows and, in gate/up, eight waves, so that the grid still covers the
// chip; many take 32 rows, which halves the staging.
__device__ __forceinline__ bool wide_bits(int b) { return b > 4; }

// acc[m] += d * sum (c - z) x_m over one unit, for the mc staged tokens
template <int B, int NX, int TM>
__device__ __forceinline__ void wide_unit_dot(const UnitBuf<B>& b, const uint32_t* xu, int xts, int lo,
                                              const float* su4, int sts, int mc, float (&acc)[TM]) {
  const PairConsts pk = pair_consts();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float d = half_to_float(((q < 2 ? b.s.x : b.s.y) >> (16 * (q & 1))) & 0xFFFFu);
    if constexpr (B == 8) {
      // two 4-bit planes: d (c - 128) = 16 d (hi - 8) + d (lo - 8) + 8 d
      uint32_t p[16];
      block_pairs<4>(b.w + 8 * q + 4, pk, p);
#pragma unroll
      for (int m = 0; m < TM; ++m)
        if (m < mc) acc[m] = block_dot<NX>(p, xu + m * xts + 16 * q, lo, 2.0f * d, su4[m * sts + q], acc[m]);
      block_pairs<4>(b.w + 8 * q, pk, p);
#pragma unroll
      for (int m = 0; m < TM; ++m) {
        if (m < mc) {
          const float X = su4[m * sts + q];
          acc[m] = fmaf(8.0f * d, X, block_dot<NX>(p, xu + m * xts + 16 * q, lo, 0.125f * d, X, acc[m]));
        }
      }
    } else {
      uint32_t p[16];
      block_pairs<B>(b.w + q * B, pk, p);
      const float ds = d * (1.0f / (float)(1 << (7 - B)));
#pragma unroll
      for (int m = 0; m < TM; ++m)
        if (m < mc) acc[m] = block_dot<NX>(p, xu + m * xts + 16 * q, lo, ds, su4[m * sts + q], acc[m]);
    }
  }
}

template <int TM>
struct WideAcc {
  float v[TM];
};

// The staged tokens live in the kernel's dynamic LDS; naming it here (not
// through a pointer argument) keeps the accesses LDS instructions.
extern __shared__ uint32_t wide_lds[];

// This lane's share (units j, j + step, ...) of row `row` against the staged
// tokens.  Not inlined: one function per width keeps each width's registers
// to itself (inlined together, the allocator merges all six).
template <int B, int NX, int TM>
__device__ __noinline__ WideAcc<TM> wide_row_dot(const TensorDev t, int row, int U, int j, int step, int xts, int lo,
                                                 int sts, int mc) {
  const uint32_t* xl = wide_lds;
  const float* xs = reinterpret_cast<const float*>(wide_lds + TM * xts);
  WideAcc<TM> r;
#pragma unroll
  for (int m = 0; m < TM; ++m) r.v[m] = 0.0f;
  const int UPL = (U + step - 1) / step;
  const RowPtr rp = row_ptr(t, B, U, row);
  UnitBuf<B> buf[2];
  load_unit_buf<B>(buf[0], rp, min(j, U - 1));
  auto load = [&](UnitBuf<B>& b, int i) { load_unit_buf<B>(b, rp, min(j + step * min(i, UPL - 1), U - 1)); };
  if constexpr (TM == 1) {
    // (no branch in the loop, as in row_dots: one token of the benchmark's layer
    // with an 8-bit shared expert 62.3 -> 60.3 us, every width mixed 81.5 -> 78.7)
    auto dots = [&](const UnitBuf<B>& b, int i) {
      const int u = j + step * i, uc = min(u, U - 1);
      float v[1] = {r.v[0]};
      wide_unit_dot<B, NX, 1>(b, xl + uc * kXStride, xts, lo, xs + uc * 4, sts, 1, v);
      r.v[0] = u < U ? v[0] : r.v[0];
    };
#pragma unroll 1
    for (int i = 0; i + 2 <= UPL; i += 2) {
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        load(buf[1 - b], i + b + 1);
        __builtin_amdgcn_sched_barrier(0);
        dots(buf[b], i + b);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (UPL & 1) dots(buf[0], UPL - 1);
  } else {
#pragma unroll 1
    for (int i0 = 0; i0 < UPL; i0 += 2) {
      asm volatile("" ::: "memory");
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int i = i0 + b;
        if (i < UPL) {
          // the next unit (clamped to the last valid one) goes out before this one is reduced
          load(buf[1 - b], i + 1);
          const int u = j + step * i;
          if (u < U) wide_unit_dot<B, NX, TM>(buf[b], xl + u * kXStride, xts, lo, xs + u * 4, sts, mc, r.v);
        }
      }
    }
  }
  return r;
}

template <int NX, int TM>
__device__ __forceinline__ WideAcc<TM> wide_row_dot_any(const TensorDev& t, int row, int U, int j, int step, int xts,
                                                        int lo, int sts, int mc) {
  switch (__builtin_amdgcn_readfirstlane(t.bits)) {
    case 2: return wide_row_dot<2, NX, TM>(t, row, U, j, step, xts, lo, sts, mc);
    case 3: return wide_row_dot<3, NX, TM>(t, row, U, j, step, xts, lo, sts, mc);
    case 4: return wide_row_dot<4, NX, TM>(t, row, U, j, step, xts, lo, sts, mc);
    case 5: return wide_row_dot<5, NX, TM>(t, row, U, j, step, xts, lo, sts, mc);
    case 6: return wide_row_dot<6, NX, TM>(t, row, U, j, step, xts, lo, sts, mc);
    default: return wide_row_dot<8, NX, TM>(t, row, U, j, step, xts, lo, sts, mc);
  }
}

// The row totals of a workgroup's waves: red[tensor][wave][token][row], summed
// over the waves in order by the threads that store them.
template <int TM, int R>
__device__ __forceinline__ void wide_put(const WideAcc<TM>& v, float (*red)[TM][R], int wave, int lane) {
#pragma unroll
  for (int m = 0; m < TM; ++m) {
    const float s = row_sum<R>(v.v[m]);
    if (lane < R) red[wave][m][lane] = s;
  }
}
template <int TM, int NW, int R>
__device__ __forceinline__ float wide_total(float (*red)[TM][R], int m, int r) {
  float s = red[0][m][r];
#pragma unroll
  for (int w = 1; w < NW; ++w) s += red[w][m][r];
  return s;
}

// grid = (I / R, slots), 64 * NW threads
template <int TM, int NW, int R>
__global__ __launch_bounds__(64 * NW) void wide_gateup_kernel(DecodeArgs a) {
  const Slot sl = slot_info(a, blockIdx.y);
  if (sl.M < 0 || sl.M > a.gemm_above) return;  // (large buckets: the grouped GEMMs)
  const TensorDev tg = a.desc[sl.desc * 3 + 0], tu = a.desc[sl.desc * 3 + 1];
  if (!tg.codes || !tu.codes) return;
  if (!wide_bits(tg.bits) && !wide_bits(tu.bits)) return;
  const int H = a.H, I = a.I, U = H / kUnit;
  const int xts = U * kXStride, sts = U * 4;
  uint32_t* xl = wide_lds;
  float* xs = reinterpret_cast<float*>(wide_lds + TM * xts);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  constexpr int ULANES = 64 / R;  // units of a row per wave and step
  __shared__ float red[2][NW][TM][R];
  const int row = blockIdx.x * R + lane % R, j = wave * ULANES + lane / R;
  for (int m0 = 0; m0 < sl.M; m0 += TM) {
    const int mc = min(TM, sl.M - m0);
    __syncthreads();
    for (int m = 0; m < mc; ++m) {
      const int t = sl.shared >= 0 ? m0 + m : a.perm[sl.base + m0 + m] / a.k;
      const MOEQ_GLOBAL u32x4* src = gptr(reinterpret_cast<const u32x4*>(a.x + (size_t)t * H));
      for (int q = threadIdx.x; q < H / 8; q += 64 * NW) {
        const u32x4 v = src[q];
        float s = 0.0f;
        s += bf16_lo(v.x); s += bf16_hi(v.x); s += bf16_lo(v.y); s += bf16_hi(v.y);
        s += bf16_lo(v.z); s += bf16_hi(v.z); s += bf16_lo(v.w); s += bf16_hi(v.w);
        s += __shfl_xor(s, 1, 64);
        s += __shfl_xor(s, 2, 64);
        const int uu = q >> 4, cq = q & 15;
        *reinterpret_cast<u32x4*>(xl + m * xts + uu * kXStride + cq * 4) = v;
        if ((cq & 3) == 0) xs[m * sts + uu * 4 + (cq >> 2)] = s;
      }
    }
    __syncthreads();
    wide_put<TM, R>(wide_row_dot_any<1, TM>(tg, row, U, j, NW * ULANES, xts, 0, sts, mc), red[0], wave, lane);
    wide_put<TM, R>(wide_row_dot_any<1, TM>(tu, row, U, j, NW * ULANES, xts, 0, sts, mc), red[1], wave, lane);
    __syncthreads();
    for (int i = threadIdx.x; i < R * mc; i += 64 * NW) {
      const int m = i / R, r = i % R;
      a.h[(size_t)(sl.base + m0 + m) * I + blockIdx.x * R + r] =
          silu(wide_total<TM, NW, R>(red[0], m, r)) * wide_total<TM, NW, R>(red[1], m, r);
    }
  }
}

// One token and one shared expert, whose down tensor alone is wide: the kernel
// adds the routed experts' partial rows (written by the launch before it) in
// slot order and writes y, which saves the combine launch.
__host__ __device__ __forceinline__ bool wide_down_combines(const DecodeArgs& a) {
  return a.n == 1 && a.wide_down == 1 && a.S == 1;
}

// grid = (H / R, slots), 64 * NW threads
template <int TM, int NW, int R>
__global__ __launch_bounds__(64 * NW) void wide_down_kernel(DecodeArgs a) {
  const Slot sl = slot_info(a, blockIdx.y);
  if (sl.M < 0 || sl.M > a.gemm_above) return;  // (large buckets: the grouped GEMMs)
  const TensorDev td = a.desc[sl.desc * 3 + 2];
  if (!td.codes || !wide_bits(td.bits)) return;
  const int H = a.H, I = a.I, U = I / kUnit;
  const int xts = 2 * U * kXStride, sts = U * 4, lo = U * kXStride;
  uint32_t* xl = wide_lds;
  float* xs = reinterpret_cast<float*>(wide_lds + TM * xts);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  constexpr int ULANES = 64 / R;  // units of a row per wave and step
  __shared__ float red[NW][TM][R];
  const int row0 = blockIdx.x * R, row = row0 + lane % R, j = wave * ULANES + lane / R;
  // (one token, the only shared expert wide: this launch ends the forward)
  const bool combine = TM == 1 && wide_down_combines(a);
  float others = 0.0f;
  if (combine && (int)threadIdx.x < R)
    for (int j = 0; j < a.k; ++j) others += a.partial[(size_t)j * H + row0 + threadIdx.x];
  for (int m0 = 0; m0 < sl.M; m0 += TM) {
    const int mc = min(TM, sl.M - m0);
    __syncthreads();
    // h rows as bfloat16 hi + lo pairs; block sums of hi + lo
    for (int m = 0; m < mc; ++m) {
      const MOEQ_GLOBAL f32x4* src = gptr(reinterpret_cast<const f32x4*>(a.h + (size_t)(sl.base + m0 + m) * I));
      for (int q = threadIdx.x; q < I / 8; q += 64 * NW) {
        const f32x4 v0 = src[2 * q], v1 = src[2 * q + 1];
        const float f[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
        uint32_t hi[4], lw[4];
        float s = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t h0 = bf16_rne(f[2 * i]), h1 = bf16_rne(f[2 * i + 1]);
          const uint32_t l0 = bf16_rne(f[2 * i] - __uint_as_float(h0 << 16));
          const uint32_t l1 = bf16_rne(f[2 * i + 1] - __uint_as_float(h1 << 16));
          hi[i] = h0 | h1 << 16;
          lw[i] = l0 | l1 << 16;
          s += __uint_as_float(h0 << 16) + __uint_as_float(l0 << 16);
          s += __uint_as_float(h1 << 16) + __uint_as_float(l1 << 16);
        }
        s += __shfl_xor(s, 1, 64);
        s += __shfl_xor(s, 2, 64);
        const int uu = q >> 4, cq = q & 15;
        uint32_t* dst = xl + m * xts + uu * kXStride + cq * 4;
        *reinterpret_cast<u32x4*>(dst) = u32x4{hi[0], hi[1], hi[2], hi[3]};
        *reinterpret_cast<u32x4*>(dst + lo) = u32x4{lw[0], lw[1], lw[2], lw[3]};
        if ((cq & 3) == 0) xs[m * sts + uu * 4 + (cq >> 2)] = s;
      }
    }
    __syncthreads();
    wide_put<TM, R>(wide_row_dot_any<2, TM>(td, row, U, j, NW * ULANES, xts, lo, sts, mc), red, wave, lane);
    __syncthreads();
    for (int i = threadIdx.x; i < R * mc; i += 64 * NW) {
      const int m = i / R, r = i % R;
      int prow;
      float wv;
      if (sl.shared >= 0) {
        prow = a.n * a.k + sl.shared * a.n + m0 + m;
        wv = 1.0f;
      } else {
        prow = a.perm[sl.base + m0 + m];
        wv = a.w[prow];
      }
      const float v = wv * wide_total<TM, NW, R>(red, m, r);
      if (combine)
        a.y[row0 + r] = others + v;
      else
        a.partial[(size_t)prow * H + row0 + r] = v;
    }
  }
}

// launches a kernel whose dynamic LDS may exceed the 64 KiB default: the
// largest is the wide down kernel's, 4 tokens of intermediate 8192
constexpr size_t kMostLds = 4 * (2 * 64 * kXStride + 64 * 4) * 4;
template <auto Kernel>
hipError_t launch_lds(dim3 grid, size_t lds, hipStream_t s, const DecodeArgs& a, int threads = 256) {
  if (lds > 65536) {
    static std::atomic<uint64_t> done{0};
    const hipError_t e = raise_lds_limit((const void*)Kernel, done, kMostLds);
    if (e != hipSuccess) return e;
  }
  Kernel<<<grid, threads, lds, s>>>(a);
  return hipGetLastError();
}

template <int TM, int NW, int R>
hipError_t launch_wide_gateup_tm(const DecodeArgs& a, hipStream_t s) {
  const int U = a.H / kUnit;
  const size_t lds = (size_t)TM * (U * kXStride + U * 4) * 4;
  dim3 grid(a.I / R, a.wide_gateup == 1 ? a.S : a.S + a.max_active);
  return launch_lds<wide_gateup_kernel<TM, NW, R>>(grid, lds, s, a, 64 * NW);
}

template <int TM, int NW, int R>
hipError_t launch_wide_down_tm(const DecodeArgs& a, hipStream_t s) {
  const int U = a.I / kUnit;
  const size_t lds = (size_t)TM * (2 * U * kXStride + U * 4) * 4;
  dim3 grid(a.H / R, a.wide_down == 1 ? a.S : a.S + a.max_active);
  return launch_lds<wide_down_kernel<TM, NW, R>>(grid, lds, s, a, 64 * NW);
}

}  // namespace

hipError_t launch_wide_gateup(const DecodeArgs& a, hipStream_t s) {
  if (!a.wide_gateup) return hipSuccess;
  const bool few = a.wide_gateup == 1;  // shared experts only
  // shared experts only: 8 rows per workgroup unless 16 still make one per compute
  // unit (us per step, 6 bits, 8 -> 16 rows: one shared expert of the benchmark's
  // layer 57.2 -> 58.9, two 68.6 -> 66.6, four 91.4 -> 84.1)
  if (a.n == 1 && few)
    return a.S * (a.I / 16) >= 256 ? launch_wide_gateup_tm<1, 4, 16>(a, s) : launch_wide_gateup_tm<1, 4, 8>(a, s);
  if (a.n == 1) return launch_wide_gateup_tm<1, 4, 32>(a, s);
  return few ? launch_wide_gateup_tm<4, 8, 16>(a, s) : launch_wide_gateup_tm<4, 4, 32>(a, s);
}

hipError_t launch_wide_down(const DecodeArgs& a, hipStream_t s) {
  if (!a.wide_down) return hipSuccess;
  const bool few = a.wide_down == 1;
  if (a.n == 1) return few ? launch_wide_down_tm<1, 8, 32>(a, s) : launch_wide_down_tm<1, 4, 32>(a, s);
  return few ? launch_wide_down_tm<4, 4, 16>(a, s) : launch_wide_down_tm<4, 4, 32>(a, s);
}

// A gate/up launch of more than 8 workgroups per compute unit.
static bool many_gateup_groups(const DecodeArgs& a) {
  return (long long)(a.I / kGuRowsN) * (a.S + a.max_active) > 2048;
}

// Layers so small that a pass over a bucket is its latency (loading, staging,
// two barriers) stage 8 tokens per pass instead of 2 (gate/up) or 4 (down), at
// most 13 units of 128 weights (32 KB of LDS).  With the grouped GEMMs taking
// the buckets of more than 2 tokens, 2 suffice.  Above 13 units per down row and
// in a long launch the buckets of one token decide, which the larger kernel
// serves no faster: 8 tokens then only for buckets of 2 and more on average.
// us per step, 2 / 4 tokens per pass -> 8 (4 bits; units per gate/up, down row;
// kept experts, top-k): 4, 2 (48, 6): 8 tokens 31.0 -> 29.0, 23: 69.5 -> 62.2; 8, 8:
// 43.3 -> 40.4, 98.0 -> 86.2; 13, 13: 62.9 -> 61.6, 145 -> 126; 13, 13 (192, 8): 74.3 ->
// 76.9, 192 -> 167; 13, 32 (12, 2): 74.3 -> 71.0; 13, 32 (48, 6): 108 -> 111 (not
// taken), 16 tokens 183 -> 176.
static bool fits_8_tokens(const DecodeArgs& a, int K) {
  return a.n > 4 && a.gemm_above > 4 && K / kUnit <= 13 &&
         (a.I / kUnit <= 13 || !many_gateup_groups(a) || (long long)a.n * a.k >= 2ll * a.max_active);
}

hipError_t launch_gateup_decode(const DecodeArgs& a, hipStream_t s) {
  const int U = a.H / kUnit;
  const size_t token_lds = (size_t)(U * kXStride + U * 8) * 4;
  if (a.n == 1)
    return launch_lds<gateup1_kernel>(dim3(a.I / kGuRows1, a.S + a.max_active), token_lds, s, a, kGuThreads);
  const bool small = fits_8_tokens(a, a.H);
  const size_t lds = (small ? 8 : 2) * token_lds;
  dim3 grid(a.I / kGuRowsN, a.S + a.max_active);
  if (!small) return launch_lds<gateupn_kernel<2, 4>>(grid, lds, s, a, kGuThreads);
  // four workgroups per compute unit cost a few spilled registers (9, 9 units,
  // 12 kept, 8 tokens 41.0 -> 41.5 us; 8, 8 units, 192 kept, 23 tokens 101 -> 104) and
  // pay where many buckets of one token wait on their weights (4, 13 units, 192
  // kept, 8 tokens 56.7 -> 53.3; 13, 13: 74.9 -> 73.3)
  return a.I / kUnit > 8 && many_gateup_groups(a) ? launch_lds<gateupn_kernel<8, 4>>(grid, lds, s, a, kGuThreads)
                                                  : launch_lds<gateupn_kernel<8, 2>>(grid, lds, s, a, kGuThreads);
}

bool gateup1_routes(const RouterParams& rp) { return !rp.kept_ids && rp.E_row <= 256 && rp.k <= kMaxTopK; }

hipError_t launch_gateup_decode_routing(const DecodeArgs& a, const RouterParams& rp, const Workspace& ws,
                                        hipStream_t s) {
  const int U = a.H / kUnit;
  const size_t lds = (size_t)(U * kXStride + U * 8) * 4;
  dim3 grid(a.I / kGuRows1, a.S + rp.k);
  if (rp.E_row <= 64)
    gateup1_route_kernel<1><<<grid, kGuThreads, lds, s>>>(a, rp, ws);
  else if (rp.E_row <= 128)
    gateup1_route_kernel<2><<<grid, kGuThreads, lds, s>>>(a, rp, ws);
  else
    gateup1_route_kernel<4><<<grid, kGuThreads, lds, s>>>(a, rp, ws);
  return hipGetLastError();
}

namespace {
size_t down1_lds(const DecodeArgs& a) {
  const size_t units = (a.I / kUnit + 1) / 2 * 2, NS = a.k + a.S;
  return NS * units * (kXStride * 4 + 4 * sizeof(float2));
}

// three slots in flight per lane (two: the same; four: 1.2 us slower)
template <int BD>
hipError_t launch_down1_b(const DecodeArgs& a, hipStream_t s) {
  down1_kernel<BD, 3><<<a.H / 32, 512, down1_lds(a), s>>>(a);
  return hipGetLastError();
}
}  // namespace

static bool down1_serves(const DecodeArgs& a) {
  return a.n == 1 && a.wide_down == 0 && a.down_bits <= 4 && a.I / kUnit <= 16 &&
         down1_lds(a) <= 65536;
}

bool down_combines(const DecodeArgs& a) { return down1_serves(a) || wide_down_combines(a); }

hipError_t launch_down_decode(const DecodeArgs& a, hipStream_t s) {
  if (down1_serves(a)) {
    switch (a.down_bits) {
      case 0: return launch_down1_b<0>(a, s);  // widths differ between tensors
      case 2: return launch_down1_b<2>(a, s);
      case 3: return launch_down1_b<3>(a, s);
      default: return launch_down1_b<4>(a, s);
    }
  }
  // R = 32 halves the staging of h per weight; few slots take R = 16, whose
  // twice as many workgroups cover the chip (2 tokens of the benchmark's layer,
  // 17 slots: 99.9 us per step against 101.4; 16 tokens: 431 against 426)
  const size_t lds1 = (size_t)(a.I / kUnit) * (kXStride + 8) * 4;  // per staged token
  const int slots = a.S + a.max_active;
  hipError_t e;
  if (a.n == 1)
    e = launch_lds<down_kernel<1, 16>>(dim3(a.H / 64, slots), lds1, s, a);
  else if (fits_8_tokens(a, a.I) && fits_8_tokens(a, a.H))
    e = launch_lds<down_kernel<8, 16>>(dim3(a.H / 64, slots), 8 * lds1, s, a);
  else if (a.H / 128 * slots < 2048)
    e = launch_lds<down_kernel<4, 16>>(dim3(a.H / 64, slots), 4 * lds1, s, a);
  else
    e = launch_lds<down_kernel<4, 32>>(dim3(a.H / 128, slots), 4 * lds1, s, a);
  return e;
}

hipError_t launch_combine(const DecodeArgs& a, hipStream_t s) {
  const long long items = (long long)a.n * (a.H / 4);
  combine_kernel<<<(int)((items + 255) / 256), 256, 0, s>>>(a);
  return hipGetLastError();
}

}  // namespace moeq
