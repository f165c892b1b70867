// What the two decode attention kernels (bf16: k4_attn.hip, fp32: k4_attn_f32.hip) share.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ckv_internal.h"

namespace ckv {

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kAttnMaxSplits = 1024;   // slices per sequence: the merge keeps one weight per slice and head in LDS
constexpr int kAttnMaxTable = 2048;    // blocks a slice of a paged cache may span: its table entries sit in LDS

struct AttnCall {
  const void *q, *K, *V;
  TensorView kv;
  int n_b, kv_heads, seq;
  const int32_t *lens, *deg;
  float scale;
  void* o;
  int o_dtype;
  void* workspace;
  int32_t* counters;      // arrival counters kept outside the workspace, or NULL
  PagedView paged;
  AttnCut cut;
  hipStream_t st;
};

// workspace: arrival counters (one per (batch, KV head), zero between calls) | partial outputs | (max, sum)
// pairs; with counters kept elsewhere the partial outputs start the workspace
inline void attn_carve(const AttnCall& c, int n_splits, int out_floats, int32_t** arrived, float** o_part, float** ml_part) {
  *arrived = c.counters ? c.counters : static_cast<int32_t*>(c.workspace);
  *o_part = reinterpret_cast<float*>(static_cast<unsigned char*>(c.workspace) +
                                     (c.counters ? 0 : attn_counter_bytes(c.n_b, c.kv_heads)));
  *ml_part = *o_part + (size_t)c.n_b * c.kv_heads * n_splits * out_floats;
}

__device__ inline uint16_t f32_to_bf16_rne(float f) {
  const uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);  // NaN stays NaN
  return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

// 2^x as the bare hardware instruction (1 ulp; results below 2^-126 come out as zero).  The library
// routine wraps it in a range fix-up for denormal results, five more instructions per call, which buys
// nothing for a softmax weight.
__device__ __forceinline__ float exp2_raw(float x) { return __builtin_amdgcn_exp2f(x); }

hipError_t launch_attn_f32(int G, int dim, const AttnCall& c);

}  // namespace ckv
