// Internal declarations shared by the host runtime (api.cpp) and the HIP
// kernel files.  Not part of the public interface (include/moeq.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdint.h>

#include <atomic>

#include "moeq.h"

namespace moeq {

// Records the calling thread's error text (moeq_last_error) and returns st.
moeq_status vset_error(moeq_status st, const char* fmt, va_list ap);

// Weights per device unit: four blocks of 32.  A lane of a GEMV wave owns one
// unit of a row at a time; hidden and inter must be multiples of this.
constexpr int kUnit = 128;
constexpr int kBlock = 32;
constexpr int kMaxExperts = 1024;
constexpr int kMaxTopK = 32;
constexpr int kMaxShared = 4;
constexpr int kChunk = 64;          // tokens per bucketing chunk (one bit per token in a 64-bit mask)
constexpr int kDecodeMaxTokens = 64;
constexpr int kDefaultDecodeMax = 64;
constexpr int kMaxDevices = 64;

// One stored tensor in the device layout.
//   codes:  tiles of 64 rows (rows are a multiple of 128), each U = K/128 units
//           of `bits` chunks of 64 x 16 bytes: row r's 16-byte chunk j of unit u
//           is the (((r/64 * U + u) * bits + j) * 64 + r%64)-th.  A wave whose
//           lanes hold neighbouring rows reads runs of 16 bytes per row, in
//           full lines.  Inside a unit, block q (q = 0..3) is the dwords
//           [q*bits, q*bits + bits) of the unit's 4*bits dwords, encoded as in
//           encode_block() (weights.hip).
//   scales: the same tiles by pairs of units: the four binary16 scales of row
//           r's unit u are the ((r/64 * ceil(U/2) + u/2) * 128 + r%64 * 2 +
//           u%2)-th 8 bytes.  With U odd the last pair's second unit is zero
//           (a weight decoded with it is zero).
// With rows kept whole (a chunk plane of consecutive units, row after row) a
// GEMM wave's load of 32 rows touched 32 separate half lines.
struct TensorDev {
  const uint32_t* codes;
  const uint16_t* scales;
  int32_t bits;
  int32_t rows;
  int32_t K;
  int32_t flags;  // kTensor* bits
};

// TensorDev.flags: the grouped GEMMs' register-decoded kernels cannot take
// the tensor, because some block scale is not a positive finite binary16 at
// most rd_scale_limit(bits) (they form d * (c - z) from d * 2^(14 + b)); its
// tiles go to the LDS-decoded kernels instead.
constexpr int32_t kTensorOffRegisterDecoder = 1;
// Largest binary16 bit pattern of a scale d with d * 2^(14 + b) finite.
constexpr uint32_t rd_scale_limit(int b) { return 0x7BFFu - ((uint32_t)(14 + b) << 10); }

struct RouterParams {
  const float* logits;    // [n x E_row]
  const uint8_t* mask;    // [E_row] device copy
  const float* bias;      // [E_row] device copy (zeros when none was given)
  // router experts: E_row (original ids) or, when kept_ids is set, the E
  // kept experts in ascending id order (groups formed over them alone)
  const int32_t* kept_ids;
  int32_t E_row;
  int32_t E, G, TG, k, topn, norm;
  float scale;
};

// Workspace views (device pointers) for one forward.
struct Workspace {
  int32_t* idx;        // [T*k]   chosen experts, token-major
  float* w;            // [T*k]   combine weights
  int32_t* offsets;    // [E+1]
  int32_t* perm;       // [T*k]   bucket order -> t*k + j
  int32_t* active;     // [1+E]   count, then active expert ids ascending
  int32_t* chunk_cnt;  // [C*E]   per-chunk counts, then per-chunk bucket bases
  int32_t* rank;       // [T*k]   rank of an assignment inside its chunk and expert
  float* h;            // [(T*k + T*S) x I] SwiGLU activations, bucket order then shared
  float* partial;      // [(T*k + T*S) x H] per-assignment expert outputs, t*k + j then shared
  int32_t* xexp;       // [T]     per-token exponent e: x * 2^-e fits binary16
  uint32_t* rowmax;    // [T*k + T*S] max |h| of each activation row (float bits)
  int32_t* tiles_all;  // [1 + 2*max_mtiles] count, then (slot, first row) of every bucket's
                       // tiles of up to 128 rows, slot order
  int32_t* tiles_rd;   // [1 + 2*max_rtiles] the same for tiles of up to rd_tile rows, dealt to the XCDs
  uint16_t* x16;       // [T x H]  binary16 x * 2^-xexp (many-token path)
  uint16_t* h16;       // [(T*k + T*S) x I] binary16 h * 2^-(row exponent) (many-token path)
  uint32_t* zeros;     // [64]    zeroed at create, never written again
};

// Raises a kernel's dynamic LDS limit to the most it is ever launched with,
// once per device and kernel (`done`): set per call to the call's own need, a
// thread could lower it between another's setting and launch.
inline hipError_t raise_lds_limit(const void* kernel, std::atomic<uint64_t>& done, size_t most) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev < kMaxDevices ? 1ull << dev : 0ull;
  if (!bit || !(done.load(std::memory_order_acquire) & bit)) {
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
    if (e != hipSuccess) return e;
    done.fetch_or(bit, std::memory_order_release);
  }
  return hipSuccess;
}

// ---- launchers (return hipSuccess or the launch error) ----
// route.hip
hipError_t launch_route_bucket_small(const RouterParams& rp, const int32_t* idx_in, int n,
                                     const Workspace& ws, hipStream_t s);
// (with x, bf16 [n x H], also ws.xexp and ws.x16)
hipError_t launch_route_tokens(const RouterParams& rp, int n, int32_t* idx, float* w, const uint16_t* x, int H,
                               const Workspace& ws, hipStream_t s);
hipError_t launch_bucket_chunked(const int32_t* idx, int n, int k, int E, const Workspace& ws,
                                 hipStream_t s);
// weights.hip
hipError_t launch_repack(const uint8_t* canon_codes, int rows, int K, int bits,
                         uint32_t* dev_codes, hipStream_t s);
// canonical scales [rows x K/32] -> device layout; *key = max over them of
// their key: the magnitude bits of a positive finite scale, 0xFFFF for a
// zero, negative or non-finite one (atomic maximum: *key must start at 0)
hipError_t launch_repack_scales(const uint16_t* canon, int rows, int K, uint16_t* dev, uint32_t* key,
                                hipStream_t s);
hipError_t launch_dequant(const TensorDev& t, float* out, hipStream_t s);
// widths 2-4: the binary16-subnormal pair decoder rebuilt to float32
hipError_t launch_dequant_sub(const TensorDev& t, float* out, hipStream_t s);
hipError_t launch_quantize(const float* w, int rows, int K, int bits, uint8_t* codes,
                           uint16_t* scales, hipStream_t s);
// decode.hip
struct DecodeArgs {
  const TensorDev* desc;  // [(E + S) * 3]
  const uint16_t* x;      // bf16 [n x H]
  const int32_t* active;
  const int32_t* offsets;
  const int32_t* perm;
  const float* w;
  float* h;
  float* partial;
  float* y;
  int32_t n, H, I, E, S, k;
  int32_t max_active;     // routed slots launched: min(n*k, kept experts)
  // many-token path
  int32_t* xexp;
  uint32_t* rowmax;
  int32_t max_mtiles;
  int32_t* tiles_all;
  int32_t max_rtiles;
  int32_t rd_tile;        // tokens per register-decoded tile (prefill_rd_tile)
  int32_t* tiles_rd;
  uint16_t* x16;
  uint16_t* h16;
  const uint32_t* zeros;  // 256 zero bytes
  const int32_t* idx;     // [n*k] chosen experts, token-major
  // width shared by every kept routed and shared down tensor (2-4), else 0
  int32_t down_bits;
  // slots with a 5/6/8-bit gate or up (down) tensor: 0 none, 1 shared
  // experts only, 2 routed experts too
  int32_t wide_gateup, wide_down;
  // many-token path: some kept or shared gate/up (down) tensor is off the
  // register decoder, so the LDS-decoded GEMM runs too
  int32_t lds_gateup, lds_down;
  // buckets of more rows take the grouped GEMMs (prefill path: 0, every
  // bucket; decode path: the large buckets of a skewed routing), the others
  // the dequant-GEMV kernels
  int32_t gemm_above;
};
// gate/up of the buckets of 1 .. gemm_above tokens with 2-4-bit tensors, and
// (if any) of those with a 5/6/8-bit one
hipError_t launch_gateup_decode(const DecodeArgs& a, hipStream_t s);
hipError_t launch_wide_gateup(const DecodeArgs& a, hipStream_t s);
// One token without a routing launch: the gate/up workgroups route the
// token themselves and one of them writes the routing and bucket outputs
// (gateup1_routes: the mask-based router with at most 256 experts)
bool gateup1_routes(const RouterParams& rp);
hipError_t launch_gateup_decode_routing(const DecodeArgs& a, const RouterParams& rp, const Workspace& ws,
                                        hipStream_t s);
// down x routing weight; for one token (down_combines) with 2-4-bit down tensors,
// or with one shared expert whose down tensor alone is wider, the last of the
// two launches also sums the slots into y, and the combine is not launched
hipError_t launch_down_decode(const DecodeArgs& a, hipStream_t s);
hipError_t launch_wide_down(const DecodeArgs& a, hipStream_t s);
bool down_combines(const DecodeArgs& a);
hipError_t launch_combine(const DecodeArgs& a, hipStream_t s);
// gate.hip: logits = x W_r^T (bf16 x [n x H], float32 W_r [E x H]); up to
// kGateFewTokens tokens take the streaming kernel, more the matrix cores, at
// most kGateChunk at a time with partial sums in `part` (gate_part_floats)
constexpr int kGateFewTokens = 8;
constexpr int kGateSplit = 8;     // runs of the hidden index over the grid
constexpr int kGateChunk = 4096;  // tokens whose partial sums are held at a time
__host__ __device__ constexpr int gate_pitch(int E) { return (E + 31) / 32 * 32; }
constexpr size_t gate_part_floats(int max_tokens, int E) {
  return max_tokens <= kGateFewTokens
             ? 0
             : (size_t)kGateSplit * (max_tokens < kGateChunk ? max_tokens : kGateChunk) * gate_pitch(E);
}
hipError_t launch_router_gate(const uint16_t* x, const float* w, int n, int H, int E, float* part, float* logits,
                              hipStream_t s);
// prune.hip
hipError_t launch_fill_u8(uint8_t* p, int n, uint8_t v, hipStream_t s);
// dst[0..n) = src[0..n) (HOST floats, NULL = zeros), passed by value in the
// kernel arguments: src may be reused as soon as this returns
hipError_t launch_store_host_floats(float* dst, const float* src, int n, hipStream_t s);
hipError_t launch_expert_importance(const int32_t* offsets, const int32_t* perm, const float* w, int E, int n,
                                    double alpha, int keep, double* importance, uint8_t* mask, int32_t* counts,
                                    hipStream_t s);
// prefill.hip
constexpr int kGemmBM = 128;  // tokens per m-tile of the LDS-decoded GEMMs
constexpr int kRdTile = 128;  // tokens per tile of the register-decoded GEMMs, at most
int prefill_max_mtiles(int n, int k, int S, int n_kept);
int prefill_rd_tile(int n, int k, int S, int n_kept, int I);
int prefill_max_rtiles(int n, int k, int S, int n_kept, int rd_tile);
// the tile list (and cleared h row maxima) and, with a.x, the binary16 copy of
// x; then the gate/up GEMMs, then h in binary16 and the down GEMMs.  With ws the
// launch also buckets a.idx (bucket_fits)
bool bucket_fits(int n, int k, int E);
hipError_t launch_prefill_tiles(const DecodeArgs& a, const Workspace* ws, hipStream_t s);
hipError_t launch_gateup_prefill(const DecodeArgs& a, hipStream_t s);
hipError_t launch_down_prefill(const DecodeArgs& a, hipStream_t s);
// the grouped GEMMs' weight decoder: binary16 d * (c - 2^(b-1)) bit patterns
hipError_t launch_dequant_gemm(const TensorDev& t, uint16_t* out, hipStream_t s);

}  // namespace moeq
