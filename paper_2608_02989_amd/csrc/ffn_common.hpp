// Shared pieces of the expert FFN passes: the routing row, the two element
// types and the weight loads.
#pragma once

#include "common.hpp"
#include "launch.hpp"

namespace amoe {

// A node's routing row, loaded once: experts e[j] and a bit per slot that
// takes part in the dispatch.  A slot is skipped when its index lies outside
// [0, E) or repeats the expert of an earlier slot of the same node (a repeated
// expert is used once, at its first slot).
template <int KMAX>
__device__ __forceinline__ uint32_t load_route_row(const int32_t* __restrict__ row, int k, int E,
                                                   int (&e)[KMAX]) {
#pragma unroll
  for (int j = 0; j < KMAX; ++j) e[j] = j < k ? row[j] : -1;
  uint32_t valid = 0u;
#pragma unroll
  for (int j = 0; j < KMAX; ++j) {
    bool ok = (e[j] >= 0) & (e[j] < E);
#pragma unroll
    for (int j2 = 0; j2 < j; ++j2) ok = ok & (e[j2] != e[j]);
    valid |= ok ? (1u << j) : 0u;
  }
  return valid;
}

// ---------------------------------------------------------------------------
// element-type traits for the two MFMA paths
// ---------------------------------------------------------------------------
struct Bf16Path {
  static constexpr int kElemBytes = 2;
  static constexpr int kKF = 32;  // K elements per 64-byte fragment row chunk
  // one 16x16x32 MFMA per fragment
  static __device__ __forceinline__ floatx4 mma(const uint4& a, const uint4& b, floatx4 c) {
    return mfma_bf16_16x16x32(a, b, c);
  }
};

struct F32Path {
  static constexpr int kElemBytes = 4;
  static constexpr int kKF = 16;
  // four 16x16x4 MFMAs per fragment; component j of lane (r, g) is K index 4g + j
  static __device__ __forceinline__ floatx4 mma(const uint4& a, const uint4& b, floatx4 c) {
    c = mfma_f32_16x16x4(__uint_as_float(a.x), __uint_as_float(b.x), c);
    c = mfma_f32_16x16x4(__uint_as_float(a.y), __uint_as_float(b.y), c);
    c = mfma_f32_16x16x4(__uint_as_float(a.z), __uint_as_float(b.z), c);
    c = mfma_f32_16x16x4(__uint_as_float(a.w), __uint_as_float(b.w), c);
    return c;
  }
};

__device__ __forceinline__ float silu_mul(float g, float u) { return g / (1.0f + __expf(-g)) * u; }

// Weight streams.  Weights go through buffer loads whose cache policy is chosen
// per pass.  The column path reads every fragment once per 16 to 64 tokens of an
// expert: its gate/up stream is non-temporal, its down stream takes the default
// policy where a workgroup has two column tiles (H >= 4096: 68.6 us against 75.6 us
// non-temporal, H = 4096, I = 1536) and is non-temporal otherwise (at H = 2048 the
// default policy saves 0.8 us of the down pass but lets its weights evict the next
// layer's router planes from the Infinity Cache: the 48-layer pass ran 5027
// against 4941 us per block).  The grouped GEMMs stream non-temporal in one M group
// (gate/up 478 against 530 us, 8 trees x 64 nodes, H = 4096, I = 1536) and take the
// default policy in two, which read the same fragments (229 -> 215 us at 32 x 60
// nodes, H = 2048, I = 768).  A weight run is addressed by a wave-uniform base and
// its length in bytes: a load past the run returns zero instead of reading other
// memory.
constexpr int kPolicyStream = 2;  // "nt": non-temporal
constexpr int kPolicyPlain = 0;   // default cache policy
constexpr int kBufferWord3 = 0x00020000;  // raw (untyped) buffer resource, 32-bit data format

// a pointer the whole wave holds, moved to scalar registers
__device__ __forceinline__ const uint4* uniform_ptr(const uint4* p) {
  const uint64_t u = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(u));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(u >> 32));
  return reinterpret_cast<const uint4*>((static_cast<uint64_t>(hi) << 32) | lo);
}

// 16-byte piece `piece` (lane included) of the run [base, base + bytes)
template <int kPolicy>
__device__ __forceinline__ uint4 load_weight(const uint4* base, int bytes, int piece) {
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  __amdgpu_buffer_rsrc_t r =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4*>(base), static_cast<short>(0), bytes, kBufferWord3);
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, piece * 16, 0, kPolicy);
  return make_uint4(v.x, v.y, v.z, v.w);
}

}  // namespace amoe
