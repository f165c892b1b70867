// What the two decode attention kernels (bf16: k4_attn.hip, fp32: k4_attn_f32.hip) share.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

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
// nothing for a token's softmax weight.  The weights of row groups, waves and slices, worked out once each, take exp2f:
// a factor that came out as zero there would make a NaN of an infinite sum.
__device__ __forceinline__ float exp2_raw(float x) { return __builtin_amdgcn_exp2f(x); }

namespace {

// Partial results travel between workgroups that may sit on different XCDs (each with its own L2)
// inside one launch.  They are written and read with device-scope relaxed atomic accesses (8 bytes
// each), which go through to the level all XCDs share, instead of plain accesses bracketed by
// device-scope fences: such a fence writes back / invalidates a whole L2, and one per workgroup cost
// this kernel a factor of three.
struct __attribute__((aligned(8))) F2 { float x, y; };
__device__ __forceinline__ void store_shared(float* p, float x, float y) {
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p), __builtin_bit_cast(uint64_t, F2{x, y}), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ F2 load_shared(const float* p) {
  return __builtin_bit_cast(F2, __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT));
}

// op over the lanes of a wave whose numbers differ in the bits of MASK, the result in every one of them.  Inside the vector
// unit: the same through LDS (shuffles) took 0.1 us a step where a workgroup waits for it.
template <int MASK, class Op>
__device__ __forceinline__ float across_lanes(float x, Op&& op) {
  static_assert((MASK & 7) == 0 || (MASK & 7) == 7, "eight neighbouring lanes together or none");
  auto dpp = [&](auto ctrl) {
    return op(x, __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), decltype(ctrl)::value, 0xF, 0xF, true)));
  };
  if constexpr (MASK & 7) {
    x = dpp(std::integral_constant<int, 0xB1>{});    // lane ^ 1
    x = dpp(std::integral_constant<int, 0x4E>{});    // lane ^ 2
    x = dpp(std::integral_constant<int, 0x141>{});   // mirrored within 8
  }
  if constexpr (MASK & 8) x = dpp(std::integral_constant<int, 0x128>{});   // lane ^ 8: turned by 8 within 16
  if constexpr (MASK & 16) {             // (the rows of the first result are 0 0 2 2, those of the second 1 1 3 3)
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  if constexpr (MASK & 32) {             // (0 1 0 1 and 2 3 2 3)
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = op(__uint_as_float(r[0]), __uint_as_float(r[1]));
  }
  return x;
}

// two neighbouring outputs: sums over the tokens divided by the sum of the weights (0 for an empty cache)
__device__ __forceinline__ void put_out(void* __restrict__ o, int o_dtype, int64_t at, float x, float y, float den) {
  const float rx = den > 0.f ? x / den : 0.f, ry = den > 0.f ? y / den : 0.f;
  if (o_dtype == CKV_BF16) {
    uint16_t* op = reinterpret_cast<uint16_t*>(o) + at;
    op[0] = f32_to_bf16_rne(rx);
    op[1] = f32_to_bf16_rne(ry);
  } else {
    float* op = reinterpret_cast<float*>(o) + at;
    op[0] = rx;
    op[1] = ry;
  }
}

// The waves' sums of one slice, added up: as the slice's partial result, or as the output where it is the only one.
// s_o: wave w's [G][D] sums at w * part floats; s_m, s_l: [W][G] its softmax references and sums of weights.  The waves leave
// their sums unweighed and whoever adds them up works out the weights for itself: one barrier.  (Weighed by the waves, behind a
// barrier of their own, and the sum of the weights worked out by G threads at the end, one sequence of 515 tokens of 8 heads of 4,
// bf16, took 8.5 us a launch, now 7.3; 32768 tokens 28.4, now 27.0, the merge by whole blocks with it.)
template <int D, int G, int W>
__device__ __forceinline__ void put_waves(const float* s_o, int part, const float* s_m, const float* s_l, bool only,
                                          float* __restrict__ o_part, float* __restrict__ ml_part, int64_t pbase,
                                          void* __restrict__ o, int o_dtype, int64_t o_base) {
  for (int c = 2 * threadIdx.x; c < G * D; c += 2 * W * 64) {
    const int g = c / D;
    float f[W], M = -INFINITY, L = 0.f, x = 0.f, y = 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w) f[w] = s_m[w * G + g];
#pragma unroll
    for (int w = 0; w < W; ++w) M = fmaxf(M, f[w]);
#pragma unroll
    for (int w = 0; w < W; ++w) {
      f[w] = (f[w] == -INFINITY) ? 0.f : exp2f(f[w] - M);
      const float2 v = *reinterpret_cast<const float2*>(s_o + w * part + c);
      x = fmaf(v.x, f[w], x);
      y = fmaf(v.y, f[w], y);
      L = fmaf(s_l[w * G + g], f[w], L);
    }
    if (only) put_out(o, o_dtype, o_base + c, x, y, L);
    else {
      store_shared(&o_part[pbase * D + c], x, y);
      if (c % D == 0) store_shared(&ml_part[(pbase + g) * 2], M, L);
    }
  }
}

// The weights of a (batch, KV head)'s slices in the merge, per query head (a wave takes a head): s_w [G][kAttnMaxSplits], and in
// s_den the sums that they divide by.  A lane's first M slices are read once, before request() asks for what comes next: loads
// come back in order.  M = 1 (bf16): of a wave's first head; M > 1 (fp32): of all its heads.
template <int G, int W, int M, class F>
__device__ __forceinline__ void weigh_slices(const float* __restrict__ ml_part, int64_t sbase, int n_slices, float* s_w,
                                             float* s_den, F&& request) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  auto pair = [&](int g, int sp) { return load_shared(&ml_part[((sbase + sp) * G + g) * 2]); };
  auto weigh = [&](int g, const F2 (&mine)[M]) __attribute__((always_inline)) {
    float mloc = mine[0].x;
#pragma unroll
    for (int i = 1; i < M; ++i) mloc = fmaxf(mloc, mine[i].x);
    for (int sp = lane + 64 * M; sp < n_slices; sp += 64) mloc = fmaxf(mloc, pair(g, sp).x);
    mloc = across_lanes<0x3f>(mloc, [](float a, float b) { return fmaxf(a, b); });
    float dloc = 0.f;
    auto count = [&](const F2& ml, int sp) {
      const float f = (ml.x == -INFINITY) ? 0.f : exp2f(ml.x - mloc);
      s_w[g * kAttnMaxSplits + sp] = f;
      dloc += f * ml.y;
    };
#pragma unroll
    for (int i = 0; i < M; ++i)
      if (lane + 64 * i < n_slices) count(mine[i], lane + 64 * i);
    for (int sp = lane + 64 * M; sp < n_slices; sp += 64) count(pair(g, sp), sp);
    dloc = across_lanes<0x3f>(dloc, [](float a, float b) { return a + b; });
    if (lane == 0) s_den[g] = dloc;
  };
  auto first = [&](int g, F2 (&mine)[M]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < M; ++i) mine[i] = (g < G && lane + 64 * i < n_slices) ? pair(g, lane + 64 * i) : F2{-INFINITY, 0.f};
  };
  if constexpr (M == 1) {
    F2 mine[1];
    first(wave, mine);
    request();
    for (int g = wave; g < G; g += W) {
      if (g != wave) first(g, mine);
      weigh(g, mine);
    }
  } else {
    constexpr int H = (G + W - 1) / W;
    F2 mine[H][M];
#pragma unroll
    for (int h = 0; h < H; ++h) first(wave + h * W, mine[h]);
    request();
#pragma unroll
    for (int h = 0; h < H; ++h)
      if (wave + h * W < G) weigh(wave + h * W, mine[h]);
  }
}

// The slices of one (batch, KV head), merged by the workgroup that arrived last: weights of the slices
// per query head (a wave takes a head), and the slices' sums: every thread owns NC pairs of neighbouring
// channels and adds them up over the slices; with fewer pairs than threads, groups of threads take every
// SG-th slice and their sums are added in group order.  The first N slices of a thread (all of them for
// up to N * SG slices) are requested before the weights are worked out, so that one memory latency covers both.
//
// TWO: the next block is asked for before one is added up (bf16).  Without (fp32), a whole block is requested and added up as it
// arrives, in one piece of code: the longer merges of fp32 are bound by what one CU takes in, and a wait that is decided behind a
// branch is one for the whole block.  us a layer, with TWO / without: fp32, 2 pairs of 60000 tokens, 2 heads 32.0 / 30.8, 1 head
// 29.5 / 28.4; bf16, 4 heads, 1 pair of 100000 21.5 / 22.3, 8 of 32769 24.5 / 24.7.
// s_w: [G][kAttnMaxSplits] floats, s_red: two per thread.
template <int D, int G, int W, bool TWO>
__device__ __forceinline__ void merge_slices(const float* __restrict__ o_part, const float* __restrict__ ml_part,
                                             int64_t sbase, int n_slices, float* s_w, float* s_den, float* s_red,
                                             void* __restrict__ o, int o_dtype, int64_t o_base) {
  const int tid = threadIdx.x;
  constexpr int kThreads = W * 64, PAIRS = G * D / 2;
  constexpr int SG = (PAIRS < kThreads) ? kThreads / PAIRS : 1, NC = (PAIRS + kThreads - 1) / kThreads;
  static_assert(PAIRS * SG == kThreads * NC, "whole pairs per thread");
  constexpr int N = (SG * NC >= 4) ? 8 : 32 / (SG * NC);
  const int sg = tid / (kThreads / SG);
  float nx[NC], ny[NC];
  const float* col[NC];
  const float* wcol[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const int c = 2 * ((tid % (kThreads / SG)) + k * kThreads);
    nx[k] = ny[k] = 0.f;
    col[k] = o_part + (sbase * G + c / D) * D + c % D;
    wcol[k] = s_w + (c / D) * kAttnMaxSplits;
  }
  constexpr int64_t pitch = (int64_t)G * D;
  F2 xa[NC][N], xb[TWO ? NC : 1][TWO ? N : 1];
  // A whole block of N slices a thread without a question asked: where it is clamped and masked, a slice costs a dozen vector
  // instructions (one pair of 20000 tokens, 2 heads of 4, bf16, 79 slices 13.4 -> 12.5 us; fp32, 8 pairs of 32769 tokens, 64
  // slices, 4 heads 59.5 -> 58.2).  In
  // the last one four slices per branch, those past the last loaded as the last one and counted as zero: with a branch
  // around each of them every weight read from LDS is waited for by itself (one pair of dim 128, 4 heads: 313
  // slices 37.3 -> 32.1 us, 256 slices 35.7 -> 23.9; 8 heads, 313 slices 59.3 -> 46.5).
  auto whole = [&](int s0) { return s0 - sg + SG * N <= n_slices; };
  auto request_whole = [&](F2 (&x)[NC][N], int s0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int k = 0; k < NC; ++k) x[k][i] = load_shared(col[k] + s0 * pitch + i * (SG * pitch));
  };
  auto request = [&](F2 (&x)[NC][N], int s0) __attribute__((always_inline)) {
    if (whole(s0)) {
      request_whole(x, s0);
    } else {
#pragma unroll
      for (int i0 = 0; i0 < N; i0 += 4)
        if (s0 + i0 * SG < n_slices) {
#pragma unroll
          for (int i = i0; i < i0 + 4; ++i)
#pragma unroll
            for (int k = 0; k < NC; ++k) x[k][i] = load_shared(col[k] + min(s0 + i * SG, n_slices - 1) * pitch);
        }
    }
  };
  weigh_slices<G, W, TWO ? 1 : 2>(ml_part, sbase, n_slices, s_w, s_den, [&] { request(xa, sg); });
  __syncthreads();
  auto add_whole = [&](const F2 (&x)[NC][N], int s0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        const float w = wcol[k][s0 + i * SG];
        nx[k] = fmaf(x[k][i].x, w, nx[k]);
        ny[k] = fmaf(x[k][i].y, w, ny[k]);
      }
  };
  auto add = [&](const F2 (&x)[NC][N], int s0) __attribute__((always_inline)) {
    if (whole(s0)) {
      add_whole(x, s0);
    } else {
#pragma unroll
      for (int i0 = 0; i0 < N; i0 += 4)
        if (s0 + i0 * SG < n_slices) {
          float w[NC][4];
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int k = 0; k < NC; ++k) w[k][i] = wcol[k][min(s0 + (i0 + i) * SG, n_slices - 1)];
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int k = 0; k < NC; ++k) {
              const bool in = s0 + (i0 + i) * SG < n_slices;
              nx[k] = fmaf(in ? x[k][i0 + i].x : 0.f, in ? w[k][i] : 0.f, nx[k]);
              ny[k] = fmaf(in ? x[k][i0 + i].y : 0.f, in ? w[k][i] : 0.f, ny[k]);
            }
        }
    }
  };
  if constexpr (TWO) {
    for (int s0 = sg;;) {                // (the next block asked for before one is added up)
      const int s1 = s0 + SG * N, s2 = s1 + SG * N;
      if (s1 < n_slices) request(xb, s1);
      add(xa, s0);
      if (s1 >= n_slices) break;
      if (s2 < n_slices) request(xa, s2);
      add(xb, s1);
      if (s2 >= n_slices) break;
      s0 = s2;
    }
  } else {
    int s0 = sg;
    add(xa, s0);
    for (s0 += SG * N; whole(s0); s0 += SG * N) {
      request_whole(xa, s0);
      add_whole(xa, s0);
    }
    if (s0 < n_slices) {
      request(xa, s0);
      add(xa, s0);
    }
  }
  if constexpr (SG > 1) {
    s_red[2 * tid] = nx[0];
    s_red[2 * tid + 1] = ny[0];
    __syncthreads();
    if (sg > 0) return;
#pragma unroll
    for (int i = 1; i < SG; ++i) {
      nx[0] += s_red[2 * (tid + i * PAIRS)];
      ny[0] += s_red[2 * (tid + i * PAIRS) + 1];
    }
  }
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const int c = 2 * ((tid % (kThreads / SG)) + k * kThreads);
    put_out(o, o_dtype, o_base + c, nx[k], ny[k], s_den[c / D]);
  }
}

// The same where fp32 caches leave many slices and two channels a thread or more: every thread owns NC channels, consecutive
// threads consecutive ones, and adds them up in slice order (the same bits), in blocks of 32 slices.  By pairs of channels two
// merges at a time take in a tenth less.  us a layer, before fp32 shared merge_slices / with it / this: 8 heads of dim 128, 2 pairs
// of 60000 tokens, 235 slices 56.4 / 58.4 / 51.4, over pages 57.6 / 63.0 / 56.4, 4 pairs 71.4 / 72.7 / 69.6, 1 pair of 120000 67.7 /
// 67.7 / 61.6; dim 64, 2 pairs of 60000 36.1 / 37.3 / 32.2; 4 heads of dim 128 35.8 / 36.8 / 33.3.
template <int D, int G, int W>
__device__ __forceinline__ void merge_many_slices(const float* __restrict__ o_part, const float* __restrict__ ml_part,
                                                  int64_t sbase, int n_slices, float* s_w, float* s_den,
                                                  void* __restrict__ o, int o_dtype, int64_t o_base) {
  constexpr int kThreads = W * 64, NC = G * D / kThreads, N = 32;
  static_assert(NC >= 2 && G * D % kThreads == 0, "whole channels per thread");
  const int tid = threadIdx.x;
  const float* col = o_part + sbase * G * D + tid;
  constexpr int64_t pitch = (int64_t)G * D;
  float num[NC] = {}, x[NC][N];
  auto load = [&](int k, int sp) { return __hip_atomic_load(col + sp * pitch + k * kThreads, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  auto weight = [&](int k, int sp) { return s_w[(tid + k * kThreads) / D * kAttnMaxSplits + sp]; };
  auto request = [&](int s0, auto n_c) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < decltype(n_c)::value; ++i)
#pragma unroll
      for (int k = 0; k < NC; ++k) x[k][i] = load(k, s0 + i);
  };
  auto add = [&](int s0, auto n_c) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < decltype(n_c)::value; ++i)
#pragma unroll
      for (int k = 0; k < NC; ++k) num[k] = fmaf(x[k][i], weight(k, s0 + i), num[k]);
  };
  constexpr std::integral_constant<int, N> whole{};
  constexpr std::integral_constant<int, 8> eight{};
  constexpr std::integral_constant<int, 1> one{};
  weigh_slices<G, W, 4>(ml_part, sbase, n_slices, s_w, s_den, [] {});
  __syncthreads();
  int s0 = 0;
  for (; s0 + N <= n_slices; s0 += N) { request(s0, whole); add(s0, whole); }
  for (; s0 + 8 <= n_slices; s0 += 8) { request(s0, eight); add(s0, eight); }
  for (; s0 < n_slices; ++s0) { request(s0, one); add(s0, one); }
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const int c = tid + k * kThreads;
    const float den = s_den[c / D], res = den > 0.f ? num[k] / den : 0.f;
    if (o_dtype == CKV_BF16) reinterpret_cast<uint16_t*>(o)[o_base + c] = f32_to_bf16_rne(res);
    else reinterpret_cast<float*>(o)[o_base + c] = res;
  }
}

}  // namespace

hipError_t launch_attn_f32(int G, int dim, const AttnCall& c);

}  // namespace ckv
