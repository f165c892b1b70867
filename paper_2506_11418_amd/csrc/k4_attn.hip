// Decode attention over a (compressed) KV cache (Eq. 3; Algorithm 1, decode line):
//   o_h = softmax(q_h K^T * scale + ln N) V,   one query token, G query heads per KV head.
// Split along the sequence: every workgroup streams a contiguous slice of K and V once, serves all G
// query heads of its KV head, keeps an online softmax in the exp2 domain, and writes (max, sum, o)
// partials.  The slice that finishes last for a (batch, KV head) - found with one counter word per pair
// in the workspace, which that workgroup puts back to zero - merges the partials of all slices with the
// usual log-sum-exp rescaling, in an order fixed by the slice numbers, so the result does not depend on
// which one that is.  One launch per call; nothing in it is a memset.
#include <type_traits>

#include "ckv_internal.h"
#include "ckv_device.h"
#include "k4_attn.h"

namespace ckv {
namespace {

constexpr int kTableSlots = kAttnMaxTable + 64;   // block table of a slice in LDS: slices start and end on whole tiles

// How a lane sees a cache row of D bf16 channels.  K rows arrive whole (16-byte pieces, consecutive lanes
// consecutive pieces) and turn into MFMA operands through LDS.  Of a V row lane n of a 16-lane group
// takes the EV = D/16 channels EV*n .. EV*n + EV - 1: at dim 128 a 16-byte piece straight from memory, at
// dim 64 half a piece, for which V rows go the way of the K rows (16 pairs of 15000 .. 30000 tokens, 4
// heads each: 25.2 us, with 8-byte loads of V 26.6).
// A wave takes 8 KiB at a time: one tile of 16 tokens (the token side of a 16x16 MFMA) of dim 128, two of
// dim 64.
template <int D>
struct RowOf {
  static constexpr int RB = D * 2;                       // bytes of a row
  static constexpr int PIECES = RB / 16;                 // 16-byte pieces of a row
  static constexpr int KROWS = 64 / PIECES;              // rows per wave-wide K load
  static constexpr int KL = 16 / KROWS;                  // K loads per tile
  static constexpr int KSTEPS = PIECES / 4;              // a contraction step takes four pieces of every row
  static constexpr int EV = D / 16;
  static constexpr int TILES = 128 / D;
  static constexpr bool VLDS = D == 64;
  static constexpr int VL = VLDS ? KL : 4;               // V loads per tile, 16 bytes each
  static constexpr int LDS = (VLDS ? 2 : 1) * 16 * RB;   // staging of a wave's tile
  static constexpr int TOKENS = 16 * TILES;              // tokens per step of a wave
  // byte offset of a 16-byte piece of a tile's row in LDS: the XOR spreads the 16 rows of one piece
  // column over all banks
  __device__ static int lds(int token, int piece) {
    const int key = (PIECES == 8) ? (token >> 1) & 7 : token & 15;
    return token * RB + ((piece ^ key) << 4);
  }
};

typedef __attribute__((ext_vector_type(4))) short s16x4;

// Four fp32 weights, all of the sign that `smallest` has, as sums of three bf16 numbers each, largest parts first, exactly but
// for 2^-125.  smallest: two bf16 of +-2^-126.  No part of a weight that is not zero is smaller: a zero part would make a
// NaN of an infinite value.  (Of equal signs, the larger bits are the larger magnitude.)
__device__ __forceinline__ void split_weights(const float (&z)[4], uint32_t smallest, s16x4 (&part)[3]) {
  uint32_t u[3][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    u[0][i] = __float_as_uint(z[i]);
    const float r = z[i] - __uint_as_float(u[0][i] & 0xffff0000u);
    u[1][i] = __float_as_uint(r);
    u[2][i] = __float_as_uint(r - __uint_as_float(u[1][i] & 0xffff0000u));
  }
  struct Words { uint32_t w[2]; } out[3];
#pragma unroll
  for (int i = 0; i < 2; ++i) {    // the upper halves of two words side by side
    u16x2 v[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) v[p] = __builtin_bit_cast(u16x2, __builtin_amdgcn_perm(u[p][2 * i + 1], u[p][2 * i], 0x07060302u));
    const u16x2 least = __builtin_elementwise_min(v[0], __builtin_bit_cast(u16x2, smallest));   // (zero for a weight of zero)
    out[0].w[i] = __builtin_bit_cast(uint32_t, v[0]);
#pragma unroll
    for (int p = 1; p < 3; ++p) out[p].w[i] = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(v[p], least));
  }
#pragma unroll
  for (int p = 0; p < 3; ++p) part[p] = __builtin_bit_cast(s16x4, out[p]);
}

// The lower (0) or upper (1) bf16 of four words.
template <int HI>
__device__ __forceinline__ s16x4 column(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  constexpr uint32_t sel = HI ? 0x07060302u : 0x05040100u;
  return __builtin_bit_cast(s16x4, make_uint2(__builtin_amdgcn_perm(b, a, sel), __builtin_amdgcn_perm(d, c, sel)));
}

// K piece . q piece for 16 tokens x 16 heads: one MFMA of depth 32, or two of depth 16 where a row has only
// two steps (products exact, fp32 accumulation).  Every MFMA starts from zero and the results are added
// up in pairs: one chain through all channels doubled the error of large logits.
template <bool SPLIT>
__device__ __forceinline__ f32x4 qk_step(const uint4& k, const uint4& qv) {
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  if constexpr (SPLIT) {
    struct Halves { s16x4 h[2]; };
    const Halves a = __builtin_bit_cast(Halves, k), b = __builtin_bit_cast(Halves, qv);
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a.h[0], b.h[0], zero, 0, 0, 0) +
           __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a.h[1], b.h[1], zero, 0, 0, 0);
  } else {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k), __builtin_bit_cast(bf16x8, qv), zero, 0, 0, 0);
  }
}

// A wave takes tiles of 16 tokens, both contractions on the matrix cores.  The 16 columns of a tile are
// the G query heads (repeated to fill 16), lane = 16 q + column:
//   S[token, head]: K rows are the A operand (through a 4 KiB region of LDS per wave and back, no
//     barrier: a wave's LDS accesses are in order), q the B operand.  MFMA row 4q + i is token 4i + q of
//     the tile, so that a lane's four results belong to tokens q, 4 + q, 8 + q, 12 + q;
//   O[head, channel]: those four weights, each an exact sum of three bf16 numbers, ARE the A operand of three bf16
//     MFMAs of depth 16 (contraction index 4q + i = token 4i + q), and the V rows a lane group loads are their B
//     operand: wave-wide load i covers the four consecutive rows 4i .. 4i + 3.
// Weights, sums and products stay fp32 (the parts add up to the fp32 weight, products are exact, sums accumulate in
// fp32).  The matrix unit rounds its sums downwards: over a long cache of values around zero that bias added up
// (32768 tokens: 4.4e-7 of the result, fp32 MFMAs of depth 4 2.35e-7), so every other tile, and every other wave's, sums
// up the negated weights and is subtracted: 2.24e-7.  The softmax reference of a head
// moves only when a logit exceeds it by more than 8 (in log2): weights stay below 2^8, which costs no
// precision, and after the first tiles the rescaling of the accumulators is rare.
//
// What bounds it: HBM reads (a kernel that does nothing but read reaches 6.2 TB/s on 134 MB, 6.7 on 403
// MB), and for short caches the chain of a tile.  Against four fp32 MFMAs of depth 4 per channel, three bf16 ones of depth 16
// keep the matrix units busy 0.41 of the cycles (counted over the 134 MB launch; vector instructions 2105 a wave against 2108,
// what widened V now splits the weights).  Per layer, fp32 / bf16 parts, either in turn on one GPU (us, 4 heads per KV head, dim
// 128): one sequence of 515 tokens 8.64 / 8.21, of 32768 (134 MB) 29.8 / 27.8; 16 sequences of 1000 17.6 / 15.9, of 8000 91.1 /
// 87.6; 32 of 1000 28.4 / 23.8; 4 of 32768, 8 heads 95.0 / 90.8; dim 64, 8 of 5000, 2 heads 22.7 / 20.0.
// Time line of the 134 MB launch with fp32 MFMAs, from clock readings in the kernel: the streaming loops end between 17 and
// 24 us (3 us between the waves of a workgroup), the reduction after its slowest wave took 1.8 us, partials were
// acknowledged and counted in 1.1 us, the merge by the last arriver took 2.4 us.  Since then the reduction has one barrier and the
// merge whole blocks of slices (28.4 us a launch -> 27.0).
//
// PAGED: K, V are a block pool [n_blocks, heads, block_size, dim] (kv.stride_s = dim, kv.stride_h =
// block_size*dim: the tokens of one head are contiguous inside a block), token t of sequence b
// lives in block table[b][t / block_size] at offset t % block_size, degrees in a pool
// [n_blocks, heads, block_size].  A table entry outside the pool masks its tokens.
//
// partial layout: o_part[((b*Hkv + kvh)*S + split)*G + g][D], ml_part[...][2] = (max, sum)
//
// Registers: three waves per SIMD (168) wherever the compiler gets there without scratch, for which the wave's number, and with
// it the loop over the tiles, is scalar; the other paged variants, with a row's address to work out for every load, stay at two.
// With 172 and two waves (us, two waves / three): 40 sequences of 8 heads, 4000 tokens, one query head each 123.1 / 106.1, eight on
// pages of 16 125.2 / 115.9; 80 of 6000, one 338.6 / 304.1; 256 of 300, one 51.2 / 48.0.
template <int D, int G, int W, bool PAGED>   // W: waves per workgroup
__global__ __launch_bounds__(W * 64, !PAGED || (D == 128 && G == 8) ? 3 : 2) void attn_mfma_kernel(
    const __bf16* __restrict__ q, const __bf16* __restrict__ K, const __bf16* __restrict__ V, TensorView kv, int kv_heads,
    int seq, const int32_t* __restrict__ lens, const int32_t* __restrict__ deg, float scale_log2e,
    int n_splits, float* __restrict__ o_part, float* __restrict__ ml_part,
    int32_t* __restrict__ arrived, void* __restrict__ o, int o_dtype, PagedView paged) {
  typedef RowOf<D> R;
  constexpr int kThreads = W * 64;
  constexpr int kStageBytes = W * R::LDS;                 // the waves' K tiles (and V tiles at dim 64)
  constexpr int kWeightBytes = G * kAttnMaxSplits * 4;
  constexpr int kRawBytes = kStageBytes > kWeightBytes ? kStageBytes : kWeightBytes;
  __shared__ __attribute__((aligned(16))) unsigned char s_raw[kRawBytes];   // one after the other
  __shared__ float s_m[W][G], s_l[W][G];
  __shared__ float s_red[2 * kThreads];
  __shared__ int s_is_last;
  __shared__ int32_t s_tbl[PAGED ? kTableSlots : 1];

  const int split = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qd = lane >> 4, n = lane & 15;
  const int len = lens ? max(min(lens[b], seq), 0) : seq;
  // whole tiles, split evenly over as many slices as give every wave one (a sequence far below the
  // capacity takes fewer slices than the launch holds)
  const int n_tiles = div_up(len, R::TOKENS);
  const int n_slices = max(min(n_splits, div_up(n_tiles, W)), 1);
  if (split >= n_slices) return;
  const int tile0 = (int)((int64_t)split * n_tiles / n_slices), tile1 = (int)((int64_t)(split + 1) * n_tiles / n_slices);
  const int t0 = tile0 * R::TOKENS, t1 = min(tile1 * R::TOKENS, len);
  const int64_t seq_base = PAGED ? 0 : (int64_t)b * kv.stride_b + (int64_t)kvh * kv.stride_h;
  const int32_t* dseq = !deg ? nullptr : PAGED ? deg : deg + ((int64_t)b * kv_heads + kvh) * kv.deg_stride;
  // the slice's blocks go to LDS first, each as the pool row ((block, head) pair times block size)
  // its first token of this head sits in, or -1 for an entry outside the pool: a row's address then
  // needs no second trip to memory and one add (the host sizes the slices so that their table
  // entries fit, and refuses pools of 2^31 rows or more)
  const int bs_mask = (1 << paged.shift) - 1;
  const int blk0 = t0 >> paged.shift;
  if (PAGED && t0 < t1) {
    const int32_t* tbl = paged.table + (int64_t)b * paged.max_blocks;
    const int n_ent = min(((t1 - 1) >> paged.shift) - blk0 + 1, kTableSlots);
    for (int i = tid; i < n_ent; i += kThreads) {
      const int blk = tbl[blk0 + i];
      s_tbl[i] = ((unsigned)blk < (unsigned)paged.n_blocks) ? ((blk * kv_heads + kvh) << paged.shift) : -1;
    }
    __syncthreads();
  }

  const __bf16* Kp = K + seq_base + (lane % R::PIECES) * 8;
  const __bf16* Vp = V + seq_base + (R::VLDS ? lane % R::PIECES : n) * 8;
  unsigned char* ktile = s_raw + wave * R::LDS;
  uint4 qv[R::KSTEPS];
  {
    const __bf16* qp = q + ((int64_t)b * kv_heads * G + kvh * G + n % G) * D;
#pragma unroll
    for (int s = 0; s < R::KSTEPS; ++s) qv[s] = *reinterpret_cast<const uint4*>(qp + (4 * s + qd) * 8);
  }

  struct Tile {
    uint4 k[R::KL];
    uint4 v[R::VL];
    int dg[4], out[4];
  };
  struct Stage { Tile tile[R::TILES]; };
  // every load of a tile, its rows clamped to the slice (always valid rows, masked at use)
  auto issue_tile = [&](Tile& st, int t) {
    auto row_of = [&](int tok, int& out) -> int {    // out: -1 for a token whose block is outside the pool, else 0
      if (!PAGED) return tok;
      const int row0 = s_tbl[min((tok >> paged.shift) - blk0, kTableSlots - 1)];
      out = row0 >> 31;
      return max(row0, 0) + (tok & bs_mask & ~out);  // outside the pool: row 0, masked through the degree
    };
    // elements from a row's first to its piece: pools are contiguous, rows of a head dim elements apart
    auto at = [&](int row) -> int64_t { return PAGED ? (int64_t)((uint64_t)(uint32_t)row * D) : (int64_t)row * kv.stride_s; };
    int out = 0;
    if (dseq) {            // (the same for every workgroup of the launch)
#pragma unroll
      for (int i = 0; i < 4; ++i) st.dg[i] = dseq[row_of(min(t + 4 * i + qd, t1 - 1), out)];
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) st.dg[i] = 1;
    }
#pragma unroll
    for (int i = 0; i < R::KL; ++i) {
      const int64_t x = at(row_of(min(t + R::KROWS * i + lane / R::PIECES, t1 - 1), out));
      st.k[i] = ldg16_stream(Kp + x);
      if (R::VLDS) st.v[i] = ldg16_stream(Vp + x);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = row_of(min(t + 4 * i + qd, t1 - 1), out);
      if (!R::VLDS) st.v[i % R::VL] = ldg16_stream(Vp + at(row));
      if (PAGED) st.out[i] = out;
    }
  };
  auto issue = [&](Stage& st, int t) {
#pragma unroll
    for (int u = 0; u < R::TILES; ++u) issue_tile(st.tile[u], t + 16 * u);
  };

  f32x4 acc[R::EV];
#pragma unroll
  for (int j = 0; j < R::EV; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  float ref = -INFINITY, ref_used = 0.f, l = 0.f;   // of this lane's head; ref_used: 0 until a token counted
  auto consume_tile = [&](const Tile& st, int t, float sign) {
#pragma unroll
    for (int i = 0; i < R::KL; ++i) {
      const int at = R::lds(R::KROWS * i + lane / R::PIECES, lane % R::PIECES);
      *reinterpret_cast<uint4*>(ktile + at) = st.k[i];
      if (R::VLDS) *reinterpret_cast<uint4*>(ktile + 16 * R::RB + at) = st.v[i];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // other lanes' pieces are read next: keep the order
    const int tk = 4 * (n & 3) + (n >> 2);
    f32x4 s[R::KSTEPS];
#pragma unroll
    for (int k = 0; k < R::KSTEPS; ++k)
      s[k] = qk_step<R::KSTEPS == 2>(*reinterpret_cast<const uint4*>(ktile + R::lds(tk, 4 * k + qd)), qv[k]);
#pragma unroll
    for (int w = 1; w < R::KSTEPS; w *= 2)
#pragma unroll
      for (int k = 0; k + w < R::KSTEPS; k += 2 * w) s[k] += s[k + w];
    struct { uint32_t w[R::EV / 2]; } v[4];        // this lane's channels of tokens 4i + qd
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (R::VLDS) {
        const uint2 x = *reinterpret_cast<const uint2*>(ktile + 16 * R::RB + R::lds(4 * i + qd, n >> 1) + (n & 1) * 8);
        v[i].w[0] = x.x; v[i].w[1] = x.y;
      } else {
        const uint4 x = st.v[i];
        v[i].w[0] = x.x; v[i].w[1] = x.y; v[i].w[2] = x.z; v[i].w[3] = x.w;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    float z[4], zmax;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float lb = dseq ? __log2f((float)st.dg[i]) : 0.f;
      const bool ok = (t + 4 * i + qd) < t1 && (!PAGED || (st.out[i] == 0 && st.dg[i] > 0));
      z[i] = ok ? fmaf(s[0][i], scale_log2e, lb) : -INFINITY;
    }
    zmax = fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3]));
    if (__any(zmax > ref + 8.f)) {     // some head's reference moves: rescale what has been summed
      zmax = fmaxf(zmax, __shfl_xor(zmax, 16));
      zmax = fmaxf(zmax, __shfl_xor(zmax, 32));
      const float moved = fmaxf(ref, zmax);
      ref_used = (moved == -INFINITY) ? 0.f : moved;
      const float alpha = exp2_raw(ref - ref_used);
      ref = moved;
      l *= alpha;
#pragma unroll
      for (int i = 0; i < 4; ++i) {    // accumulator row 4*qd + i is that column's head
        const float a = __shfl(alpha, 4 * qd + i);
#pragma unroll
        for (int j = 0; j < R::EV; ++j) acc[j][i] *= a;
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) z[i] = exp2_raw(z[i] - ref_used);
    l += (z[0] + z[1]) + (z[2] + z[3]);
    // the tile's own sum from zero, then one addition into the running sums: a quarter of the roundings there.
    // The weights as three bf16 parts (8 + 8 + 8 bits: exactly the 24 of an fp32), the smallest first, all of a tile
    // with one sign
    s16x4 part[3];
#pragma unroll
    for (int i = 0; i < 4; ++i) z[i] *= sign;
    split_weights(z, sign < 0.f ? 0x80808080u : 0x00800080u, part);
#pragma unroll
    for (int j = 0; j < R::EV; j += 2) {
      const s16x4 v0 = column<0>(v[0].w[j / 2], v[1].w[j / 2], v[2].w[j / 2], v[3].w[j / 2]);
      const s16x4 v1 = column<1>(v[0].w[j / 2], v[1].w[j / 2], v[2].w[j / 2], v[3].w[j / 2]);
      f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
      for (int p = 2; p >= 0; --p) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(part[p], v0, s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(part[p], v1, s1, 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        acc[j][i] = fmaf(s0[i], sign, acc[j][i]);
        acc[j + 1][i] = fmaf(s1[i], sign, acc[j + 1][i]);
      }
    }
  };
  auto consume = [&](const Stage& st, int t, float sign) {
#pragma unroll
    for (int u = 0; u < R::TILES; ++u) consume_tile(st.tile[u], t + 16 * u, u % 2 ? -sign : sign);
  };
  // the loads of a wave's next step are issued before this one is consumed (two register sets)
  constexpr int STEP = W * R::TOKENS;
  const int tw = t0 + wave * R::TOKENS;
  if (tw < t1) {
    Stage sa, sb;
    const float sign = (wave & 1) ? -1.f : 1.f;
    issue(sa, tw);
    for (int t = tw; t < t1; t += 2 * STEP) {
      issue(sb, t + STEP);
      consume(sa, t, sign);
      if (t + STEP >= t1) break;
      issue(sa, t + 2 * STEP);
      consume(sb, t + STEP, -sign);
    }
  }

  // ---- merge the waves of this workgroup: every wave leaves its sums as they are, in its own part of the staging area ------
  l = across_lanes<0x30>(l, [](float a, float b) { return a + b; });
  if (lane < G) { s_m[wave][lane] = ref; s_l[wave][lane] = l; }   // (lane = column = head)
  static_assert(G * D * 4 <= R::LDS, "a wave's sums in its own part");
  float* s_o = reinterpret_cast<float*>(s_raw);
  constexpr int kPart = R::LDS / 4;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int g = 4 * qd + i;
    if (g < G) {
      float* at = s_o + wave * kPart + g * D + R::EV * n;
#pragma unroll
      for (int j = 0; j < R::EV; j += 4) *reinterpret_cast<f32x4*>(at + j) = f32x4{acc[j][i], acc[j + 1][i], acc[j + 2][i], acc[j + 3][i]};
    }
  }
  __syncthreads();
  const int64_t sbase = ((int64_t)b * kv_heads + kvh) * n_splits;
  const int64_t pbase = (sbase + split) * G, o_base = ((int64_t)b * kv_heads + kvh) * G * D;
  put_waves<D, G, W>(s_o, kPart, &s_m[0][0], &s_l[0][0], n_slices == 1, o_part, ml_part, pbase, o, o_dtype, o_base);
  if (n_slices == 1) return;

  // ---- the last slice of this (batch, KV head) to arrive merges them all ----------------------
  // Every thread waits until its own partial stores have been acknowledged, the workgroup meets,
  // and one thread counts the workgroup in; the workgroup that finds all others counted takes the
  // merge.  The counter is only ever touched with device-scope atomics.
  __builtin_amdgcn_s_waitcnt(0);          // vmcnt = lgkmcnt = expcnt = 0: the stores above are complete
  __syncthreads();
  int32_t* my_count = arrived + (b * kv_heads + kvh);
  if (tid == 0) s_is_last = (atomicAdd(my_count, 1) == n_slices - 1);
  __syncthreads();
  if (!s_is_last) return;
  if (tid == 0) atomicExch(my_count, 0);  // all have arrived: the workspace is ready for the next call
  merge_slices<D, G, W, true>(o_part, ml_part, sbase, n_slices, reinterpret_cast<float*>(s_raw), &s_l[0][0], s_red, o, o_dtype,
                        o_base);
}

template <int D, int G, int W>
hipError_t launch_mfma_w(const AttnCall& c) {
  const int n_splits = c.cut.slices;
  if (c.paged.table && div_up(c.seq, n_splits) > (kAttnMaxTable << c.paged.shift)) return hipErrorInvalidValue;
  float *o_part, *ml_part;
  int32_t* arrived;
  attn_carve(c, n_splits, G * D, &arrived, &o_part, &ml_part);
  ScopedTimer t(c.paged.table ? "attn_paged_bf16" : "attn_bf16", c.st);
#define CKV_ATTN_LAUNCH(PG)                                                                                             \
  hipLaunchKernelGGL((attn_mfma_kernel<D, G, W, PG>), dim3(n_splits, c.kv_heads, c.n_b), dim3(W * 64), 0, c.st,         \
                     static_cast<const __bf16*>(c.q), static_cast<const __bf16*>(c.K), static_cast<const __bf16*>(c.V), \
                     c.kv, c.kv_heads, c.seq, c.lens, c.deg, c.scale * kLog2e, n_splits, o_part, ml_part, arrived, c.o, \
                     c.o_dtype, c.paged)
  if (c.paged.table) CKV_ATTN_LAUNCH(true);
  else CKV_ATTN_LAUNCH(false);
#undef CKV_ATTN_LAUNCH
  return hipGetLastError();
}

template <int D, int G>
hipError_t launch_mfma_t(const AttnCall& c) {
  return c.cut.waves == 8 ? launch_mfma_w<D, G, 8>(c) : launch_mfma_w<D, G, 4>(c);
}

template <int D>
hipError_t launch_mfma_g(int G, const AttnCall& c) {
  switch (G) {
    case 1: return launch_mfma_t<D, 1>(c);
    case 2: return launch_mfma_t<D, 2>(c);
    case 4: return launch_mfma_t<D, 4>(c);
    case 8: return launch_mfma_t<D, 8>(c);
  }
  return hipErrorInvalidValue;
}

}  // namespace

// Waves per workgroup (bf16).  With few (batch, KV head) pairs a long cache is cut into many slices, and
// the merge of the slices by one workgroup counts: workgroups of eight waves halve their number (8 pairs of
// 33000 tokens: 28.7 us with 32 slices of eight waves, 34.1 with 64 of four).  With more pairs, two smaller
// workgroups per CU even out sequences of different lengths (16 pairs of 16500 and 33000 tokens, 4 heads:
// 40.9 against 46.2 us; of 4096 and 8192 tokens 20.3 against 18.0; 128 pairs of 4112 .. 8223 tokens 74 against
// 81), and a cache that gives the four waves of 512 workgroups no second tile has nothing to merge that would
// be worth the longer reduction (8 pairs of 515 tokens: 9.6 against 11.0 us).  One or two pairs of dim 128 leave most of
// the chip idle, and the longest chain of tiles decides: from 8192 tokens on, where 64 slices hold a tile for each of eight
// waves, up to 24576, they are cut so (four waves in 32 to 96 slices -> eight in 64; 1 pair, 2 heads: 8192 tokens 12.0 -> 10.9 us,
// 16384 13.6 -> 12.9, 24001 15.5 -> 15.0; 4 heads: 13.4 -> 12.6, 15.9 -> 14.7, 18.6 -> 16.7; 8 heads, 24001: 24.0 -> 19.7; 2 pairs,
// 4 heads: 13.6 -> 13.4, 16.4 -> 15.6, 18.3 -> 17.4, 8 heads: 16.3 -> 16.6, 20.4 -> 18.6, 22.3 -> 20.4).  Longer ones want more
// slices (one head, 32768: 15.1 -> 15.4); three and four pairs gain at some lengths and lose at others.
//
// Slices.  Eight waves per CU stream fastest (two workgroups of four or one of eight), and as many workgroups
// as run at once are cut, not one more: a CU that gets another one ends last (24 pairs of 70000 tokens, one head:
// 112 us with 504 workgroups, 134 with 528).  Each workgroup has a fixed merge/write cost, so slices have at least
// 256 tokens; a short bf16 cache, bound by the latency of its longest slice, is cut finer, down to one step of
// every wave, but into no more than 16 slices (few pairs: 32 or, with one or two heads, 64), since one workgroup merges
// all slices of a pair: one pair of 20001 tokens, 4 heads: 17.1 us in 79 slices, 27.3 in 313; 8 pairs of 4096 tokens: 14.0
// in 16, 18.5 in 64; 8 pairs of 1030: 10.4 in 16, 12.5 in 5; 1 of 4096: 10.3 in 32, 12.8 in 16.  One head: 1 pair of 8192
// 9.7 in 64, 11.3 in 32; 4 pairs of 4097 11.3 in 64, 9.3 in 32; dim 64, 4 pairs of 5500 9.5 in 64, 10.4 in 32.
//
// One slice.  Partials and their merge cost as much as two to three steps of a wave: a cache of up to two steps of four
// waves is not cut (4 heads, us, two slices / one: 8 pairs of 128 tokens 7.9 / 6.7, of 130 7.7 / 7.8; dim 64, 8 pairs of 256
// 8.1 / 7.2, of 260 8.0 / 8.7).  Nor are up to 1536 tokens of 192 to 256 pairs, a workgroup per pair and CU: four waves up to
// 128 tokens (4 heads, eight waves / four: 256 pairs of 64 tokens 5.74 / 5.47, of 128 7.71 / 6.68, 192 pairs of 128 7.19 /
// 6.37; 8 heads, 256 pairs of 64 5.80 / 5.84, of 128 7.73 / 6.90; dim 64, 4 heads, 256 pairs of 128 5.81 / 5.60, of 160 6.87 / 7.20), then
// eight (half to all of n tokens, two slices of four waves / one of eight: 256 pairs, n = 200 11.3 / 9.9,
// 700 19.5 / 18.2, 2000 40.4 / 40.6, 4000 76.0 / 75.2; 192 pairs 11.1 / 9.8, 18.5 / 17.3, 37.7 / 37.6, 66.5 / 68.3; 160 pairs,
// 700 15.4 / 17.1).
//
// The counts above are those of 256 CUs whatever the device: the cut also sizes the workspace, which is asked for without one.
AttnCut attn_cut(int dtype, int n_b, int kv_heads, int q_heads, int dim, int seq, int span_limit) {
  const bool bf16 = dtype == CKV_BF16;
  const int group = q_heads / kv_heads;
  const int64_t bh = (int64_t)n_b * kv_heads;
  AttnCut cut{};
  if (bf16 && dim == 128 && bh <= 2 && seq >= 64 * 8 * 16 && seq <= 24576) {
    cut.waves = 8;
    cut.slices = 64;      // (at most 384 tokens: a paged slice's table entries always fit)
    return cut;
  }
  if (bf16 && (seq <= 2 * 4 * (dim == 64 ? 32 : 16) || (bh >= 192 && bh <= 256 && seq <= 1536))) {
    cut.waves = bh >= 192 && bh <= 256 && seq > 128 ? 8 : 4;
    cut.slices = 1;       // (at most 1536 tokens: a paged slice's table entries always fit)
    return cut;
  }
  cut.waves = bf16 && bh * seq > 512 * 4 * 16 && (bh <= 8 || (bh <= 16 && seq <= 24576)) ? 8 : 4;
  const int64_t groups = 2048 / cut.waves;
  auto most = [&](int64_t want, int tokens) { const int cap = (seq + tokens - 1) / tokens; return want < cap ? (int)want : cap; };
  int want = most(bf16 && 2 * bh <= groups ? groups / bh : (groups + bh - 1) / bh, 256);
  if (bf16) {
    const bool light = group == 1 ? bh <= (dim == 64 ? 4 : 2) : dim == 64 && group == 2 && bh <= 2;   // little to merge
    const int finest = light ? 64 : bh <= (dim == 64 ? 8 : 4) ? 32 : 16;
    const int fine = most(groups / bh < finest ? groups / bh : finest, cut.waves * (dim == 64 ? 32 : 16));
    if (fine > want) want = fine;
  }
  if (want > kAttnMaxSplits) want = kAttnMaxSplits;
  if (want < 1) want = 1;
  // paged caches: a slice's block-table entries must fit the kernel's LDS table
  if (span_limit > 0 && (seq + want - 1) / want > span_limit) want = (seq + span_limit - 1) / span_limit;
  if (want > kAttnMaxSplits) want = kAttnMaxSplits;
  cut.slices = want;
  return cut;
}

size_t attn_counter_bytes(int n_b, int kv_heads) { return ((size_t)n_b * kv_heads * sizeof(int32_t) + 255) / 256 * 256; }

int attn_paged_span_limit(int block_size) { return kAttnMaxTable * block_size; }

size_t attn_workspace_bytes(int dtype, int n_b, int kv_heads, int q_heads, int dim, int seq, int span_limit) {
  // one arrival counter per (batch, KV head), then partial outputs and (max, sum) pairs per
  // (batch, query head, slice)
  const size_t rows = (size_t)n_b * q_heads * attn_cut(dtype, n_b, kv_heads, q_heads, dim, seq, span_limit).slices;
  return attn_counter_bytes(n_b, kv_heads) + rows * (dim + 2) * sizeof(float);
}

// The slices of attn_cut go down as well as up with the length (they halve where eight waves are taken) and
// with the batch.  All pairs together have at most this many, whatever the lengths up to seq and the number
// of pairs up to n_b * kv_heads: ceil(512 / pairs) each, or one per 256 tokens (bf16: per 64 or more) of a
// shorter cache.
size_t attn_reserve_bytes(int dtype, int n_b, int kv_heads, int q_heads, int dim, int seq, int span_limit) {
  const int64_t bh = (int64_t)n_b * kv_heads;
  int64_t slices = bh * ((seq + 255) / 256) * (dtype == CKV_BF16 ? 4 : 1);
  if (slices > bh + 511) slices = bh + 511;
  const int64_t spans = span_limit > 0 ? bh * ((seq + span_limit - 1) / span_limit) : 0;
  if (slices < spans) slices = spans;
  return attn_counter_bytes(n_b, kv_heads) + (size_t)slices * (q_heads / kv_heads) * (dim + 2) * sizeof(float);
}

hipError_t launch_decode_attn(const void* q, int q_heads, const void* K, const void* V, int dtype, int dim,
                              TensorView kv, int n_b, int kv_heads, int seq, const int32_t* lens,
                              const int32_t* deg, float scale, void* o, int o_dtype, void* workspace,
                              PagedView paged, hipStream_t st, int32_t* counters) {
  const int G = q_heads / kv_heads;
  const AttnCut cut = attn_cut(dtype, n_b, kv_heads, q_heads, dim, seq, paged.table ? (kAttnMaxTable << paged.shift) : 0);
  const AttnCall c{q, K, V, kv, n_b, kv_heads, seq, lens, deg, scale, o, o_dtype, workspace, counters, paged, cut, st};
  if (dtype != CKV_BF16) return launch_attn_f32(G, dim, c);
  if (dim == 128) return launch_mfma_g<128>(G, c);
  if (dim == 64) return launch_mfma_g<64>(G, c);
  return hipErrorInvalidValue;
}

}  // namespace ckv
