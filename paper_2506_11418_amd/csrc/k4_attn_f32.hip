// Decode attention over an fp32 KV cache: see k4_attn.hip for the split along the sequence, the merge by
// the workgroup that arrives last and the bf16 kernel.  Here both contractions are vector arithmetic: one
// row per row_bytes/16 lanes, G query heads from registers.  (The bf16 kernel's scheme with fp32 operands
// was measured and is slower, 68.7 against 46.5 us at 8 pairs of 32768 x 128 tokens: q.k then takes depth-4
// products too.)
#include <type_traits>

#include "ckv_internal.h"
#include "ckv_device.h"
#include "k4_attn.h"

namespace ckv {
namespace {

constexpr int kThreads = 256;

// A lane holds 4 consecutive channels of a row.
__device__ __forceinline__ float dot4(const float4& a, const float4& b) {
  return fmaf(a.w, b.w, fmaf(a.z, b.z, fmaf(a.y, b.y, a.x * b.x)));
}

// Sum over the LANES consecutive lanes (aligned) that share a cache row; every lane gets the sum.
// Quad steps and the mirrored half-row / row are DPP adds; 32 lanes add one cross-row exchange.
template <int LANES>
__device__ __forceinline__ float row_sum(float x) {
  auto dpp = [](float v, auto ctrl) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), decltype(ctrl)::value,
                                                                 0xF, 0xF, true));
  };
  x += dpp(x, std::integral_constant<int, 0xB1>{});                    // lane ^ 1
  x += dpp(x, std::integral_constant<int, 0x4E>{});                    // lane ^ 2
  if (LANES >= 8) x += dpp(x, std::integral_constant<int, 0x141>{});   // mirrored within 8
  if (LANES >= 16) x += dpp(x, std::integral_constant<int, 0x140>{});  // mirrored within 16
  if (LANES >= 32) x += __shfl_xor(x, 16);
  return x;
}

// partial layout: o_part[((b*Hkv + kvh)*S + split)*G + g][D], ml_part[...][2] = (max, sum)
//
// Thread mapping: LPR = row_bytes/16 lanes share one cache row ("row group"); a wave holds 64/LPR
// row groups, so one wave-wide 16-byte load covers 64/LPR consecutive rows = 1 KiB contiguous.
// Every row group takes kUnroll tokens per iteration: their K and V loads are all issued before
// the first use (bytes in flight hide HBM latency), the logits of the kUnroll tokens share one
// running-max update, so the accumulators are rescaled once per kUnroll tokens.
constexpr int kUnroll = 4;

// PAGED: K, V are a block pool [n_blocks, heads, block_size, dim] (kv.stride_s = dim, kv.stride_h =
// block_size*dim: the tokens of one head are contiguous inside a block), token t of sequence b
// lives in block table[b][t / block_size] at offset t % block_size, degrees in a pool
// [n_blocks, heads, block_size].  A table entry outside the pool masks its tokens.
template <int D, int G, bool PAGED>
__global__ __launch_bounds__(kThreads, G <= 4 ? 3 : 2) void attn_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ K, const float* __restrict__ V, TensorView kv, int kv_heads,
    int seq, const int32_t* __restrict__ lens, const int32_t* __restrict__ deg, float scale_log2e,
    int n_splits, int span, float* __restrict__ o_part, float* __restrict__ ml_part,
    int32_t* __restrict__ arrived, void* __restrict__ o, int o_dtype, PagedView paged) {
  constexpr int E = 4;
  constexpr int LPR = D / E;
  constexpr int NRG = kThreads / LPR;
  constexpr int U = kUnroll;
  constexpr int W = kThreads / 64;
  __shared__ float s_m[W][G], s_l[W][G];
  __shared__ float s_red[2 * kThreads];
  // the waves' sums; later the slice weights [G][kAttnMaxSplits] of the merge
  constexpr int kStageFloats = W * G * D, kWeightFloats = G * kAttnMaxSplits;
  __shared__ __attribute__((aligned(16))) float s_raw[kStageFloats > kWeightFloats ? kStageFloats : kWeightFloats];

  const int split = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, rg = tid / LPR, piece = tid % LPR;
  const int len = lens ? min(lens[b], seq) : seq;
  const int t0 = split * span, t1 = min(t0 + span, len);
  const int64_t base = PAGED ? piece * E : (int64_t)b * kv.stride_b + (int64_t)kvh * kv.stride_h + piece * E;
  const float* Kp = K + base;
  const float* Vp = V + base;
  const int32_t* dseq = !deg ? nullptr : PAGED ? deg : deg + ((int64_t)b * kv_heads + kvh) * kv.deg_stride;
  const int32_t* tbl = PAGED ? paged.table + (int64_t)b * paged.max_blocks : nullptr;
  const int bs_mask = (1 << paged.shift) - 1;
  // the slice's blocks go to LDS first, each as the pool row ((block, head) pair times block size)
  // its first token of this head sits in, or -1 for an entry outside the pool: a row's address then
  // needs no second trip to memory and one add (the host sizes the slices so that their table
  // entries fit, and refuses pools of 2^31 rows or more)
  __shared__ int32_t s_tbl[PAGED ? kAttnMaxTable : 1];
  const int blk0 = t0 >> paged.shift;
  if (PAGED && t0 < t1) {
    const int n_ent = min(((t1 - 1) >> paged.shift) - blk0 + 1, kAttnMaxTable);
    for (int i = tid; i < n_ent; i += kThreads) {
      const int blk = tbl[blk0 + i];
      s_tbl[i] = ((unsigned)blk < (unsigned)paged.n_blocks) ? ((blk * kv_heads + kvh) << paged.shift) : -1;
    }
    __syncthreads();
  }

  float4 qv[G];
#pragma unroll
  for (int g = 0; g < G; ++g)
    qv[g] = *reinterpret_cast<const float4*>(q + ((int64_t)b * kv_heads * G + kvh * G + g) * D + piece * E);
  float m[G], l[G], acc[G][E];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    m[g] = -INFINITY;
    l[g] = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) acc[g][e] = 0.f;
  }

  // token of (iteration, slot u) for this row group: tb + u*NRG + rg.  The loads of iteration
  // i+1 are issued before iteration i is consumed (two register sets, software pipeline).
  struct Stage {
    float4 kr[U], vr[U];
    int dg[U];
  };
  auto issue = [&](Stage& st, int tb) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int tc = min(tb + u * NRG + rg, t1 - 1);   // clamp: always a valid row, masked at use
      if (PAGED) {
        const int row0 = s_tbl[min((tc >> paged.shift) - blk0, kAttnMaxTable - 1)];
        const bool in_pool = row0 >= 0;
        // row 0 when outside the pool: always a valid address, masked through the degree
        const int row = in_pool ? row0 + (tc & bs_mask) : 0;
        st.kr[u] = *reinterpret_cast<const float4*>(Kp + (int64_t)row * kv.stride_s);
        st.vr[u] = *reinterpret_cast<const float4*>(Vp + (int64_t)row * kv.stride_s);
        const int d = dseq ? dseq[row] : 1;
        st.dg[u] = in_pool ? d : 0;
      } else {
        st.kr[u] = *reinterpret_cast<const float4*>(Kp + (int64_t)tc * kv.stride_s);
        st.vr[u] = *reinterpret_cast<const float4*>(Vp + (int64_t)tc * kv.stride_s);
        st.dg[u] = dseq ? dseq[tc] : 1;
      }
    }
  };
  auto consume = [&](const Stage& st, int tb) {
    float z[U][G];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int g = 0; g < G; ++g) z[u][g] = row_sum<LPR>(dot4(qv[g], st.kr[u]));
      const float lb = dseq ? __log2f((float)st.dg[u]) : 0.f;
      const bool ok = (tb + u * NRG + rg) < t1 && (!PAGED || st.dg[u] > 0);
#pragma unroll
      for (int g = 0; g < G; ++g) z[u][g] = ok ? fmaf(z[u][g], scale_log2e, lb) : -INFINITY;
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float mn = m[g];
#pragma unroll
      for (int u = 0; u < U; ++u) mn = fmaxf(mn, z[u][g]);
      // a row group that has seen no valid token yet keeps mn = -inf: subtract 0 instead, so that
      // exp2(-inf) = 0 comes out rather than NaN
      const float ref = (mn == -INFINITY) ? 0.f : mn;
      const float alpha = exp2_raw(m[g] - ref);
      m[g] = mn;
      l[g] *= alpha;
#pragma unroll
      for (int e = 0; e < E; ++e) acc[g][e] *= alpha;
#pragma unroll
      for (int u = 0; u < U; ++u) z[u][g] = exp2_raw(z[u][g] - ref);   // now the weight p
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float vx[E] = {st.vr[u].x, st.vr[u].y, st.vr[u].z, st.vr[u].w};
#pragma unroll
      for (int g = 0; g < G; ++g) {
        l[g] += z[u][g];
#pragma unroll
        for (int e = 0; e < E; ++e) acc[g][e] = fmaf(z[u][g], vx[e], acc[g][e]);
      }
    }
  };
  constexpr int STEP = NRG * U;
  if (t0 < t1) {
    Stage sa, sb;
    issue(sa, t0);
    for (int tb = t0; tb < t1; tb += 2 * STEP) {
      if (tb + STEP < t1) issue(sb, tb + STEP);
      consume(sa, tb);
      if (tb + STEP < t1) {
        if (tb + 2 * STEP < t1) issue(sa, tb + 2 * STEP);
        consume(sb, tb + STEP);
      }
    }
  }

  // ---- merge the row groups of every wave, then the waves of this workgroup --------------------
  const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    constexpr int ROWS = 64 - LPR;        // the bits of a lane's number that say which row group it belongs to
    const float mw = across_lanes<ROWS>(m[g], [](float a, float b2) { return fmaxf(a, b2); });
    const float f = (m[g] == -INFINITY) ? 0.f : exp2f(m[g] - mw);
    auto sum = [&](float x) { return across_lanes<ROWS>(x * f, [](float a, float b2) { return a + b2; }); };
    float4 x;
    x.x = sum(acc[g][0]); x.y = sum(acc[g][1]); x.z = sum(acc[g][2]); x.w = sum(acc[g][3]);
    const float lw = sum(l[g]);
    if (lane < LPR) *reinterpret_cast<float4*>(s_raw + (wave * G + g) * D + lane * E) = x;
    if (lane == 0) { s_m[wave][g] = mw; s_l[wave][g] = lw; }
  }
  __syncthreads();
  const int64_t sbase = ((int64_t)b * kv_heads + kvh) * n_splits, o_base = ((int64_t)b * kv_heads + kvh) * G * D;
  put_waves<D, G, W>(s_raw, G * D, &s_m[0][0], &s_l[0][0], n_splits == 1, o_part, ml_part, (sbase + split) * G, o, o_dtype, o_base);
  if (n_splits == 1) return;

  // ---- the last slice of this (batch, KV head) to arrive merges them all ----------------------
  // Every thread waits until its own partial stores have been acknowledged, the workgroup meets,
  // and one thread counts the workgroup in; the workgroup that finds all others counted takes the
  // merge.  The counter is only ever touched with device-scope atomics.
  __shared__ int s_is_last;
  __builtin_amdgcn_s_waitcnt(0);          // vmcnt = lgkmcnt = expcnt = 0: the stores above are complete
  __syncthreads();
  int32_t* my_count = arrived + (b * kv_heads + kvh);
  if (tid == 0) s_is_last = (atomicAdd(my_count, 1) == n_splits - 1);
  __syncthreads();
  if (!s_is_last) return;
  if (tid == 0) atomicExch(my_count, 0);  // all have arrived: the workspace is ready for the next call
  // (from where many slices pay, two blocks of merge_slices, us in pairs / many: 4 heads of dim 128, 2 pairs, 63 slices 19.9 / 20.6,
  // 118 24.0 / 23.5; 8 heads of dim 64, 4 pairs, 63 20.7 / 21.4; 8 of 128, 2 pairs, 36 26.4 / 26.4, 8 pairs, 64 50.1 / 48.8)
  if constexpr (G * D >= 2 * kThreads) {
    if (n_splits > 128 * kThreads / (G * D)) {
      merge_many_slices<D, G, W>(o_part, ml_part, sbase, n_splits, s_raw, &s_l[0][0], o, o_dtype, o_base);
      return;
    }
  }
  merge_slices<D, G, W, false>(o_part, ml_part, sbase, n_splits, s_raw, &s_l[0][0], s_red, o, o_dtype, o_base);
}

template <int D, int G>
hipError_t launch_f32_t(const AttnCall& c) {
  const int n_splits = c.cut.slices;
  const int span = div_up(c.seq, n_splits);
  if (c.paged.table && span > (kAttnMaxTable << c.paged.shift)) return hipErrorInvalidValue;
  float *o_part, *ml_part;
  int32_t* arrived;
  attn_carve(c, n_splits, G * D, &arrived, &o_part, &ml_part);
  ScopedTimer t(c.paged.table ? "attn_paged_f32" : "attn_f32", c.st);
#define CKV_ATTN_LAUNCH(PG)                                                                                          \
  hipLaunchKernelGGL((attn_f32_kernel<D, G, PG>), dim3(n_splits, c.kv_heads, c.n_b), dim3(kThreads), 0, c.st,        \
                     static_cast<const float*>(c.q), static_cast<const float*>(c.K), static_cast<const float*>(c.V), \
                     c.kv, c.kv_heads, c.seq, c.lens, c.deg, c.scale * kLog2e, n_splits, span, o_part, ml_part,      \
                     arrived, c.o, c.o_dtype, c.paged)
  if (c.paged.table) CKV_ATTN_LAUNCH(true);
  else CKV_ATTN_LAUNCH(false);
#undef CKV_ATTN_LAUNCH
  return hipGetLastError();
}

template <int D>
hipError_t launch_f32_g(int G, const AttnCall& c) {
  switch (G) {
    case 1: return launch_f32_t<D, 1>(c);
    case 2: return launch_f32_t<D, 2>(c);
    case 4: return launch_f32_t<D, 4>(c);
    case 8: return launch_f32_t<D, 8>(c);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_attn_f32(int G, int dim, const AttnCall& c) {
  if (dim == 128) return launch_f32_g<128>(G, c);
  if (dim == 64) return launch_f32_g<64>(G, c);
  if (dim == 32) return launch_f32_g<32>(G, c);
  return hipErrorInvalidValue;
}

}  // namespace ckv
