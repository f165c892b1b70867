// One clustering round in one launch, for chunks whose rows fit the LDS: similarity, matching, top-r, merge and
// compaction (Sec. 5.2 - 5.3).  bf16: 256 consecutive tokens per workgroup for chunks of 64, 128 or 256, one chunk of 512
// tokens or, at dim 64, of 1024.
//
// The block's keys and values are read once, in order, and written once, in order: the key rows are parked
// in LDS, where the similarity tiles, the merge and the compaction read them; the value rows are requested
// together with them, wait in registers while the matching runs, and take the keys' place in LDS once these
// have been emitted.  A launch pair of a match kernel and merge_kernel reads the keys twice, gathers
// the rows of both tensors from memory behind LDS lookups and passes the matching through memory.
// Same operand order, norms, fold, member order and rounding as those two: same bits.
//
// What bounds it: large launches the HBM stream (64 sequences of 50003 tokens, chunk 256, seven rounds: 9.3 GB, by the
// counters as by the sizes, in 1603 us = 5.8 TB/s, nine tenths of the chip's copy rate, the vector ALU busy 59 % of the
// first; two launches a round took 2283), small ones the
// chain of one workgroup: request 1.0 us, keys 1.8, similarity 2.2, ranking and lists 2.8, keys out 2.9, values
// in and out 2.8 (8 x 8448 tokens, 21.6 us a call; two launches 35.4).  Two workgroups per CU: 64 KiB of rows
// each, and 128 registers, 32 of them the waiting values.  Whole chunks (us a call, two launches a round / one): dim 128,
// chunk 512: 8 x 8448 tokens, r = 0.8 40.0 / 25.2, 64 x 50003, annealed 2176 / 2011 (one workgroup per CU: 128 KiB of
// rows); dim 64: chunk 512, 64 x 32768, two rounds 355 / 269, chunk 1024, 8 x 40000 88.4 / 64.9.  Chunks of 1024 at dim
// 128 do not fit; holding the B rows in registers instead and each tensor's halves in turn was slower than two launches
// (256 x 131072, two rounds 10.2 ms against 9.7): one workgroup per CU ends up in a chain of 54 us a chunk.
#include <type_traits>

#include "ckv_internal.h"
#include "ckv_device.h"

namespace ckv {
namespace {

constexpr int kTok = 256;        // tokens of a workgroup that takes chunks of up to as many
constexpr uint32_t kPlace = 0x1ffffu;

// The bookkeeping of a block of up to HALF sources and HALF destinations (rows of LDS 0 .. HALF-1 and HALF .. 2 HALF-1;
// token u is row (u & 1) * HALF + u / 2): which edges are kept, who merges into whom, where everything goes.
template <int HALF>
struct RoundLds {
  __attribute__((aligned(16))) uint32_t key[HALF];     // a source's score (rank_key)
  __attribute__((aligned(16))) int16_t kept[HALF];     // destination a kept source merges into, or -1
  __attribute__((aligned(16))) int16_t slot[2 * HALF]; // output row of a retained token
  int16_t dst[HALF], start[HALF], place[HALF];
  int32_t cnt[HALF];
  int32_t deg[2 * HALF];       // by row
  uint32_t word[2 * HALF];     // a row as the emit loops see it (the kernel's own encoding)
  uint32_t members[HALF];      // the words of the merged sources, list after list, ascending inside a list
  uint2 desc[2 * HALF];        // what to emit: word | output row, members << 10, first of them << 20
  int n_merged, n_copied, sel[2];
};

// A source's score as a number that orders like it, a NaN beyond the infinity of its sign: whatever the bits, exactly m
// edges are kept.  Below the largest number, so that there is a next larger one.
__device__ __forceinline__ uint32_t rank_key(float score) { return min(order_key(score), 0xfffffffeu); }

// In: key, dst (-1: nothing to merge into), deg and word of every row; cnt, desc, n_merged, n_copied zero, keys of
// sources that do not exist zero.  Chunks of `chunk` tokens, the last one of the block possibly short: m_full / m_tail
// edges of a whole / short one are merged.  Begins and ends with a barrier.
template <int HALF, int THREADS>
__device__ __forceinline__ void round_lists(RoundLds<HALF>& s, int n_tok, int chunk, int m_full, int m_tail,
                                            const RoundMap& map, int64_t bh, int u0, int out_base) {
  constexpr int LPA = THREADS / HALF;              // lanes that share the bookkeeping of one source
  static_assert(LPA >= 1 && LPA <= 8, "lanes per source");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nA = (n_tok + 1) >> 1;
  // the map's entries of a block's two original tokens to each of its own are requested here: waited for after the
  // lists, 64 x 32768 tokens, chunk 256, took 445 us for 437
  constexpr int EARLY = 4 * HALF > THREADS ? 4 * HALF / THREADS : 1;
  int part_of[EARLY];
  int32_t* originals = nullptr;
  int n_orig = 0;
  if (map.p && map.fold == 1) {
    originals = map.p + bh * map.stride + 2 * (int64_t)u0;
    n_orig = min(4 * HALF, map.len - 2 * u0);
#pragma unroll
    for (int i = 0; i < EARLY; ++i) part_of[i] = originals[min(tid + i * THREADS, n_orig - 1)];
  }
  __syncthreads();

  // ---- top-r of every chunk: rank by counting (score descending, index ascending) ---------------
  const int a = tid / LPA, sub = tid % LPA;
  const int a_lo = a & ~((chunk >> 1) - 1), nAc = min(chunk >> 1, nA - a_lo);
  const int m = (nAc == (chunk >> 1) && 2 * a_lo + chunk <= n_tok) ? m_full : m_tail;
  int d = -1;
  if (a < nA && m > 0) {
    d = s.dst[a];
    if (HALF <= 128 && m < nAc) {
      // an equal score of an earlier source ranks above: those are counted from the key itself on, the later
      // ones from the next larger number on (sources that do not exist hold 0 and come later)
      const uint32_t key = s.key[a], above = key + 1;
      int rank = 0;
      for (int o = a_lo + 4 * sub; o < a_lo + nAc; o += 4 * LPA) {
        const uint4 so = *reinterpret_cast<const uint4*>(&s.key[o]);
        rank += (so.x >= (o < a ? key : above)) + (so.y >= (o + 1 < a ? key : above)) +
                (so.z >= (o + 2 < a ? key : above)) + (so.w >= (o + 3 < a ? key : above));
      }
      rank = group_sum<LPA>(rank);
      if (rank >= m) d = -1;
    }
  }
  if constexpr (HALF > 128) {
    // one chunk: the key of its m-th best edge by a radix select, equal ones by position (ranks by counting grow with
    // the square: 512 sources take 4 us of the vector units)
    if (m > 0 && m < nAc) {
      uint32_t* histogram = s.members;             // (not in use yet)
      const uint32_t key = s.key[a];
      uint32_t cut = 0;
      int left = m, equal = 0;
#pragma unroll 1
      for (int shift = 24; shift >= 0; shift -= 8) {
        if (tid < 256) histogram[tid] = 0;
        __syncthreads();
        if (sub == 0 && d >= 0 && (shift == 24 || (key ^ cut) >> (shift + 8) == 0)) atomicAdd(&histogram[key >> shift & 255u], 1u);
        __syncthreads();
        if (wave == 0) {                           // lane l: bins 255 - 4l downwards
          int c[4], sum = 0;
#pragma unroll
          for (int e = 0; e < 4; ++e) sum += c[e] = (int)histogram[255 - 4 * lane - e];
          const int inc = (int)wave_inclusive_scan((uint32_t)sum);
          int above = inc - sum;
          if (above < left && inc >= left) {       // the bin of the left-th largest is one of this lane's
            int e = 0;
            while (e < 3 && above + c[e] < left) above += c[e++];
            s.sel[0] = (255 - 4 * lane - e) | c[e] << 8;
            s.sel[1] = left - above;
          }
        }
        __syncthreads();
        cut |= (uint32_t)(s.sel[0] & 255) << shift;
        equal = s.sel[0] >> 8;
        left = s.sel[1];
      }
      if (d >= 0 && key <= cut) {
        int earlier = 0;
        if (key == cut && left < equal)
          for (int o = 0; o < a; ++o) earlier += s.key[o] == cut;
        if (key < cut || earlier >= left) d = -1;
      }
    }
  }
  if (sub == 0) {
    s.kept[a] = (int16_t)d;
    if (d >= 0) atomicAdd(&s.cnt[d], 1);
  }
  __syncthreads();

  // ---- member lists (ascending inside a list) and the retained tokens' output rows ---------------
  if (wave == 0) {                                 // where every destination's list starts, and its place among the merged rows
    // one scan of three sums, ten bits each: members, lists of two or more, lists of one
    constexpr int PER = HALF >= 64 ? HALF / 64 : 1;
    auto sums = [](int c) -> uint32_t { return (uint32_t)c | (uint32_t)(c > 1) << 10 | (uint32_t)(c == 1) << 20; };
    int c[PER];
    uint32_t mine = 0;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      c[e] = lane * PER + e < HALF ? s.cnt[lane * PER + e] : 0;
      mine += sums(c[e]);
    }
    const uint32_t inc = wave_inclusive_scan(mine);
    const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    const int n_long = (int)(all >> 10 & 1023u);
    uint32_t before = inc - mine;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int j = lane * PER + e;
      if (j < HALF) {
        s.start[j] = (int16_t)(before & 1023u);
        s.place[j] = (int16_t)(c[e] > 1 ? before >> 10 & 1023u : n_long + (before >> 20));
      }
      before += sums(c[e]);
    }
    if (lane == 0) s.n_merged = n_long + (int)(all >> 20);
  } else if (wave == 1) {
    constexpr int PER = 2 * HALF / 64;             // neighbouring tokens per lane
    int keep[PER], mine = 0;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int u = lane * PER + e;
      keep[e] = u < n_tok && ((u & 1) || s.kept[u >> 1] < 0);
      mine += keep[e];
    }
    int at = (int)wave_inclusive_scan((uint32_t)mine) - mine;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      s.slot[lane * PER + e] = (int16_t)at;
      at += keep[e];
    }
  }
  int pos = 0;                                     // earlier sources of the same list
  if (HALF > 128) {
    // slots handed out by atomics (in the descriptors' place, still zero) and every short list sorted below, so that no
    // atomic decides an order; lists beyond eight (degenerate inputs) are placed by counting
    if (sub == 0 && d >= 0 && s.cnt[d] > 1) {
      if (s.cnt[d] <= 8) pos = (int)atomicAdd(&s.desc[d].x, 1u);
      else for (int o = 0; o < a; ++o) pos += s.kept[o] == d;
    }
  } else if (d >= 0 && s.cnt[d] > 1) {
    for (int o = a_lo + 8 * sub; o < a; o += 8 * LPA) {
      struct { int16_t v[8]; } x = *reinterpret_cast<const decltype(x)*>(&s.kept[o]);
#pragma unroll
      for (int i = 0; i < 8; ++i) pos += (x.v[i] == d) && (o + i < a);
    }
    pos = group_sum<LPA>(pos);
  }
  __syncthreads();
  // Rows with two or more members come first, then those with one, then the copies: the row groups of a wave
  // then do the same work side by side (in output order nine waves in ten carried some row to merge).
  if (sub == 0 && d >= 0) s.members[s.start[d] + pos] = s.word[a];
  if (tid < 2 * HALF) {                            // (whole waves)
    const int u = tid, j = u >> 1, row = (u & 1) * HALF + j;
    const int into = (u & 1) || u >= n_tok ? -1 : (int)s.kept[j];
    const int n = (u & 1) ? s.cnt[j] : 0;
    const bool copied = u < n_tok && into < 0 && n == 0;
    const uint64_t mask = __ballot(copied);
    int at = 0;
    if (lane == 0) at = atomicAdd(&s.n_copied, __popcll(mask));
    at = s.n_merged + __builtin_amdgcn_readfirstlane(at) + __popcll(mask & ((1ull << lane) - 1));
    const uint32_t o = (uint32_t)s.slot[u];
    if (copied) s.desc[at] = make_uint2(s.word[row], o);
    else if (u < n_tok && into < 0) s.desc[s.place[j]] = make_uint2(s.word[row], o | (uint32_t)n << 10 | (uint32_t)s.start[j] << 20);
    if (map.p && map.fold == 0 && u < n_tok)
      map.p[bh * map.stride + u0 + u] = map.offset + out_base + (into < 0 ? s.slot[u] : s.slot[2 * into + 1]);
  }
  if (map.p && map.fold > 0) {
    auto place = [&](int u) -> int {
      const int into = (u & 1) ? -1 : (int)s.kept[u >> 1];
      return map.offset + out_base + s.slot[into < 0 ? u : 2 * into + 1];
    };
    if (map.fold == 1) {
#pragma unroll
      for (int i = 0; i < EARLY; ++i)
        if (tid + i * THREADS < n_orig) originals[tid + i * THREADS] = place(part_of[i] - u0);
    } else {
      fold_map(map, bh, u0, 2 * HALF, THREADS, tid, place);
    }
  }
  __syncthreads();
  if constexpr (HALF > 128) {
    const int n = tid < HALF ? s.cnt[tid] : 0;
    if (n > 1 && n <= 8) {
      uint32_t* list = &s.members[s.start[tid]];   // (a word's place in LDS, its low 17 bits, grows with the row)
      for (int x = 1; x < n; ++x) {
        const uint32_t v = list[x];
        int y = x - 1;
        while (y >= 0 && (list[y] & kPlace) > (v & kPlace)) { list[y + 1] = list[y]; --y; }
        list[y + 1] = v;
      }
    }
    __syncthreads();
  }
}

// A lane's value as if it were new: what is worked out from it is then not kept in registers around a loop.
__device__ __forceinline__ int lane_anew(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// TOK: tokens of a workgroup; above kTok its one chunk.
template <int D, int TOK, bool PAGED, bool EDGES>
__global__ __launch_bounds__(TOK * D / 64, 4) void round_small_kernel(
    const __bf16* __restrict__ K, const __bf16* __restrict__ V, const int32_t* __restrict__ deg_in, TensorView in,
    int seq, int chunk, int blocks_per_seq, int m_full, int m_tail, __bf16* __restrict__ K_out,
    __bf16* __restrict__ V_out, int32_t* __restrict__ deg_out, TensorView out, int64_t deg_out_stride,
    RoundMap map, int64_t deg_in_stride, PagedSide pin,
    PagedSide pout, int out_k_paged, int out_v_paged, EdgeBlocks<EDGES> edges) {
  constexpr int THREADS = TOK * D / 64, HALF = TOK / 2;
  constexpr int WPT = THREADS / 64 / (HALF / 32);  // waves per 32-row tile of sources: 2 or 1
  constexpr int OCT = D / 8, ROWB = D * 2, KEYSHIFT = (ROWB == 256) ? 0 : 1, KSTEPS = D / 16;
  constexpr int NRG = THREADS / OCT;               // rows per pass = row groups
  constexpr int PASSES = TOK / NRG;
  static_assert(PASSES == 8 && NRG % 32 == 0 && TOK * ROWB <= 1 << 17, "whole swizzle periods, places of 17 bits");
  if constexpr (EDGES) {
    if ((int)blockIdx.x < edges.blocks) {
      copy_edges(edges.copy, (int64_t)blockIdx.x * THREADS + threadIdx.x);
      return;
    }
  }
  // rows 0 .. HALF-1: the A tokens, the others: the B tokens
  extern __shared__ __attribute__((aligned(16))) unsigned char s_rows[];
  // (a row's word: where its first piece sits in LDS - a lane XORs its own piece number in - and above those 17 bits
  // its degree as bf16, exact up to 256; a positive number has 15)
  __shared__ RoundLds<HALF> s_;
  __shared__ __attribute__((aligned(16))) float s_ib[HALF];
  __shared__ float s_best2[WPT == 2 ? HALF : 1];
  __shared__ int16_t s_dst2[WPT == 2 ? HALF : 1];
  __shared__ int s_wide;
  __shared__ int32_t s_rb_in[PAGED ? TOK / 8 + 2 : 1], s_rb_out[PAGED ? TOK / 8 + 2 : 1];

  int w = (int)blockIdx.x;
  if constexpr (EDGES) w -= edges.blocks;
  const int sb = w % blocks_per_seq, bh = w / blocks_per_seq;
  const int t0 = sb * TOK;
  const int n_tok = min(TOK, seq - t0);
  const int nA = (n_tok + 1) >> 1, nB = n_tok >> 1;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int piece = tid % OCT, rg = tid / OCT;
  const int n_whole = n_tok / chunk, tail = n_tok - n_whole * chunk;   // (a short chunk ends the sequence)
  const int n_out = n_tok - n_whole * m_full - (tail ? m_tail : 0);
  const int out_base = (t0 / chunk) * (chunk - m_full);

  RowBases rb_in{}, rb_out{};
  const bool in_paged = PAGED && pin.table != nullptr;
  const bool ok_paged = PAGED && out_k_paged, ov_paged = PAGED && out_v_paged;
  if (PAGED) {
    const int b = bh / in.heads, h = bh % in.heads;
    if (in_paged) rb_in = stage_row_bases(s_rb_in, pin, b, h, in.heads, pin.tok0 + t0, pin.tok0 + t0 + n_tok - 1, tid, THREADS);
    if (ok_paged || ov_paged)
      rb_out = stage_row_bases(s_rb_out, pout, b, h, in.heads, pout.tok0 + out_base, pout.tok0 + out_base + n_out - 1, tid, THREADS);
    if (in_paged) __syncthreads();
  }

  // ---- every load of the block, before the first use ------------------------------------------
  const int64_t seq_at = in_paged ? 0 : in.seq_base(bh) + (int64_t)t0 * in.stride_s;
  const __bf16* Kp = K + seq_at + piece * 8;
  const __bf16* Vp = V + seq_at + piece * 8;
  auto row_at = [&](int u) -> int64_t {            // rows past the block's end re-read its last one
    const int t = min(u, n_tok - 1);
    return in_paged ? (int64_t)rb_in.row(pin.tok0 + t0 + t) * D : (int64_t)t * in.stride_s;
  };
  Piece kx[PASSES];
  uint4 vx[PASSES];
#pragma unroll
  for (int it = 0; it < PASSES; ++it) kx[it].u = ldg16_stream(Kp + row_at(it * NRG + rg));
  int dg = 1;
  if (deg_in && tid < n_tok) dg = in_paged ? deg_in[rb_in.row(pin.tok0 + t0 + tid)] : deg_in[(int64_t)bh * deg_in_stride + t0 + tid];
#pragma unroll
  for (int it = 0; it < PASSES; ++it) vx[it] = ldg16_stream(Vp + row_at(it * NRG + rg));

  auto swz = [](int row, int pc) -> int { return row * ROWB + (((pc ^ (row >> KEYSHIFT)) & (OCT - 1)) << 4); };
  const int row0 = (rg & 1) * HALF + (rg >> 1);      // LDS row of token rg; 32 tokens on: 16 rows on, same XOR
  const int lds0 = swz(row0, piece);
  if (tid < HALF) { s_.cnt[tid] = 0; s_.key[tid] = 0; }
  if (tid < TOK) {
    const int row = (tid & 1) * HALF + (tid >> 1);
    s_.deg[row] = dg;
    s_.word[row] = (uint32_t)swz(row, 0) | (__float_as_uint((float)dg) & 0x7fff0000u) << 1;
    s_.desc[tid] = make_uint2(0, 0);
  }
  if (tid == 0) { s_wide = 0; s_.n_merged = 0; s_.n_copied = 0; }
#pragma unroll
  for (int it = 0; it < PASSES; ++it) {
    if (it * NRG + rg >= n_tok) kx[it].u = make_uint4(0, 0, 0, 0);
    const float ss = row_sum<OCT>(sumsq8(kx[it]));
    *reinterpret_cast<uint4*>(s_rows + lds0 + it * (NRG / 2) * ROWB) = kx[it].u;
    if (piece == 0 && (rg & 1)) s_ib[it * (NRG / 2) + (rg >> 1)] = inv_norm(ss);
  }
  __syncthreads();
  if (tid < TOK && dg > 256) s_wide = 1;

  // ---- similarity and matching: a 32-row tile of sources against the tiles of its own chunk -------
  const int half = lane >> 5, col = lane & 31;
  {
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    const int at = wv / WPT, hb = wv % WPT;
    const int tpc = chunk >> 6, first = at & -tpc;                         // tiles per chunk (a power of two); its first tile
    const int lo = WPT == 2 ? (hb * tpc + 1) / 2 : 0, hi = WPT == 2 && hb == 0 ? (tpc + 1) / 2 : tpc;
    float best = -INFINITY, inva = 0.f;
    int bestj = first * 32;                        // (where no score compares: the first row of its own chunk)
    if (at * 32 < nA && lo < hi) {                 // (the same for the whole wave)
      // two tiles at a time where there are two: their MFMA chains run side by side.  The source operands pass
      // through (the values wait in 32 registers): the sum of their squares is taken as they do, in the order of
      // inv_norm_of_operand_row
      float ss = 0.f;
      auto tiles = [&](auto count_c, int tt) {
        constexpr int C = decltype(count_c)::value;
        f32x16 acc[C];
        ss = 0.f;
#pragma unroll
        for (int c = 0; c < C; ++c) acc[c] = f32x16{0};
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) {
          const int off = swz(TOK == 256 ? col : lane_anew(col), 2 * s + half);
          Piece afrag;
          afrag.u = *reinterpret_cast<const uint4*>(s_rows + at * 32 * ROWB + off);
#pragma unroll
          for (int c = 0; c < C; ++c)
            acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                *reinterpret_cast<const bf16x8*>(s_rows + (HALF + (first + tt + c) * 32) * ROWB + off), afrag.v, acc[c],
                0, 0, 0);
          ss += sumsq8(afrag);
          // (operands requested further ahead, or kept for the sum, push the values into scratch)
          if (s % 2 == 1) asm volatile("" : "+v"(ss) : : "memory");
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
          const int bt = first + tt + c;
          f32x4 ib[4];
#pragma unroll
          for (int qd = 0; qd < 4; ++qd) ib[qd] = *reinterpret_cast<const f32x4*>(s_ib + bt * 32 + 4 * half + 8 * qd);
          const int valid = nB - bt * 32;          // rows of this tile that exist (>= 32: all)
          if (valid >= 32) tile_argmax<false>(acc[c], ib, bt * 32, half, 32, best, bestj);
          else if (valid > 0) tile_argmax<true>(acc[c], ib, bt * 32, half, valid, best, bestj);
          __builtin_amdgcn_sched_barrier(0);       // (one fold after the other)
        }
      };
      if (hi - lo == 1) tiles(std::integral_constant<int, 1>{}, lo);
      else tiles(std::integral_constant<int, 2>{}, lo);
      if constexpr (TOK == 256) {                  // (at most four; a loop would keep sixteen offsets for both)
        if (WPT == 1 && hi - lo == 4) tiles(std::integral_constant<int, 2>{}, lo + 2);
      } else {
#pragma unroll 1
        for (int tt = lo + 2; tt < hi; tt += 2) tiles(std::integral_constant<int, 2>{}, tt);
      }
      inva = inv_norm(ss + __shfl_xor(ss, 32));
      const float ob = __shfl_xor(best, 32);
      const int oj = __shfl_xor(bestj, 32);
      if (ob > best || (ob == best && oj < bestj)) { best = ob; bestj = oj; }
    }
    const int a = at * 32 + col;
    if (WPT == 2) {
      if (hb == 1 && half == 0) { s_best2[a] = best; s_dst2[a] = (int16_t)bestj; }
      __syncthreads();
      if (hb == 0 && s_best2[a] > best) { best = s_best2[a]; bestj = s_dst2[a]; }   // (the other wave's rows come later)
    }
    if (hb == 0 && half == 0 && a < nA) {
      s_.dst[a] = (nB <= first * 32) ? (int16_t)-1 : (int16_t)bestj;  // a one-token tail chunk: nothing to match
      s_.key[a] = rank_key(best * inva);
    }
  }
  round_lists<HALF, THREADS>(s_, n_tok, chunk, m_full, m_tail, map, bh, t0, out_base);

  // ---- emit the rows of one tensor: keys first, then the values in their place ---------------------
  const int64_t out_at = out.seq_base(bh) + (int64_t)out_base * out.stride_s;
  const int u_out0 = pout.tok0 + out_base;
  const int n_merged = s_.n_merged;
  const uint32_t lane_piece = (uint32_t)piece << 4;
  auto row_of = [&](uint32_t word) -> uint4 {
    return *reinterpret_cast<const uint4*>(s_rows + ((word & kPlace) ^ lane_piece));
  };
  auto degree_of = [&](uint32_t word) -> int { return s_.deg[(word & kPlace) / ROWB]; };
  auto weighed = [&](float* acc, const uint4& x, uint32_t word) {      // + degree * row, degrees up to 256
    const uint32_t w = word >> 17;
    const bf16x2 lo = __builtin_bit_cast(bf16x2, w), hi = __builtin_bit_cast(bf16x2, w << 16);
    const uint32_t v[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      acc[2 * i] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v[i]), lo, acc[2 * i], false);
      acc[2 * i + 1] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, v[i]), hi, acc[2 * i + 1], false);
    }
  };
  auto emit = [&](auto wide_c, auto keys_c) {
    constexpr bool WIDE = decltype(wide_c)::value, KEYS = decltype(keys_c)::value;
    const bool o_paged = KEYS ? ok_paged : ov_paged;
    __bf16* O = (KEYS ? K_out : V_out) + piece * 8 + (o_paged ? 0 : out_at);
    auto put = [&](int o, const uint4& x, int nd) {
      if (PAGED && (ok_paged || ov_paged) && rb_out.base_of(u_out0 + o) < 0) return;   // a block outside the pool
      stg16_stream(O + (o_paged ? (int64_t)rb_out.row(u_out0 + o) * D : (int64_t)o * out.stride_s), x);
      if (KEYS && piece == 0) {
        if (ov_paged) deg_out[rb_out.row(u_out0 + o)] = nd;
        else deg_out[(int64_t)bh * deg_out_stride + out_base + o] = nd;
      }
    };
    for (int i = rg; i < n_merged; i += NRG) {
      const uint2 w = s_.desc[i];
      const int o = (int)(w.y & 1023u), n = (int)(w.y >> 10 & 1023u);
      const uint32_t* list = s_.members + (w.y >> 20);
      const uint4 x = row_of(w.x);
      float acc[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = 0.f;
      if constexpr (WIDE) {
        int nd = degree_of(w.x);
        fma_bf16x8_t<true>(acc, x, nd);
#pragma unroll 1
        for (int q = 0; q < n; ++q) {
          const int dm = degree_of(list[q]);
          fma_bf16x8_t<true>(acc, row_of(list[q]), dm);
          nd += dm;
        }
        put(o, round_div_pack_bf16(acc, nd), nd);
      } else {
        float nd = __uint_as_float(w.x >> 17 << 16);
        uint32_t wm = list[0];
        weighed(acc, x, w.x);
        weighed(acc, row_of(wm), wm);
        nd += __uint_as_float(wm >> 17 << 16);
#pragma unroll 1
        for (int q = 1; q < n; ++q) {
          wm = list[q];
          weighed(acc, row_of(wm), wm);
          nd += __uint_as_float(wm >> 17 << 16);
        }
        put(o, round_div_pack_bf16(acc, nd), (int)nd);
      }
    }
    // untouched tokens, bit by bit (the row groups that had one merged row less start)
    for (int i = n_merged + (rg + NRG - n_merged % NRG) % NRG; i < n_out; i += NRG) {
      const uint2 w = s_.desc[i];
      put((int)(w.y & 1023u), row_of(w.x), degree_of(w.x));
    }
  };
  const bool wide = s_wide != 0;
#pragma unroll
  for (int it = 0; it < PASSES; ++it)              // the values are here by now: waited for before any store is counted
    asm volatile("" : "+v"(vx[it].x), "+v"(vx[it].y), "+v"(vx[it].z), "+v"(vx[it].w));
  if (wide) emit(std::true_type{}, std::true_type{});
  else emit(std::false_type{}, std::true_type{});
  __syncthreads();
#pragma unroll
  for (int it = 0; it < PASSES; ++it) *reinterpret_cast<uint4*>(s_rows + lds0 + it * (NRG / 2) * ROWB) = vx[it];
  __syncthreads();
  if (wide) emit(std::true_type{}, std::false_type{});
  else emit(std::false_type{}, std::false_type{});
}

// The same for fp32 caches, one chunk per workgroup: keys in LDS (rows padded by 16 bytes, so that consecutive rows
// start four banks apart), every dot product and norm one chain of fused multiply-adds over the channels as in
// match_f32_kernel, centroids in 64 bits as in merge_kernel: same bits.  These caches are small, so what counts is
// the chain of one workgroup: every load is requested at the start, and the products are taken NI x NJ rows per
// thread from registers.  (With more than one row a thread the compiler holds the waiting values in scratch, 48 to 144 bytes a
// lane: they are waited for before the similarity starts, stored there, and read back once the keys are out.)  1024 tokens of dim 64, chunk 64: 10.0 us, the two launches, with loads element by element and
// two LDS reads to a product, 11.6 + 7.3; 4 x 8192 tokens of dim 128, chunk 256, two rounds 75 us a call (157); 64 x 16384
// of dim 64, chunk 64 198 us (526).
template <int D, int CHUNK>
constexpr int f32_threads() { return CHUNK * D / 32 > 256 ? CHUNK * D / 32 : 256; }

template <int D, int CHUNK, int THREADS = f32_threads<D, CHUNK>()>
__global__ __launch_bounds__(THREADS) void round_f32_kernel(
    const float* __restrict__ K, const float* __restrict__ V, const int32_t* __restrict__ deg_in, TensorView in, int seq,
    int blocks_per_seq, int m_full, int m_tail, float* __restrict__ K_out, float* __restrict__ V_out,
    int32_t* __restrict__ deg_out, TensorView out, int64_t deg_out_stride, RoundMap map,
    int64_t deg_in_stride, EdgeBlocks<true> edges) {
  constexpr int HALF = CHUNK / 2;
  constexpr int LPR = D / 4, NRG = THREADS / LPR, PASSES = CHUNK / NRG;
  constexpr int PITCH = D + 4;
  constexpr int TX = 16, TY = THREADS / TX, NI = HALF / TY, NJ = HALF / TX;
  static_assert(PASSES >= 1 && PASSES <= 8 && NI >= 1 && NI * TY == HALF, "whole passes and tiles");
  if ((int)blockIdx.x < edges.blocks) {
    copy_edges(edges.copy, (int64_t)blockIdx.x * THREADS + threadIdx.x);
    return;
  }
  extern __shared__ __attribute__((aligned(16))) float s_f32[];   // rows 0 .. HALF-1: A tokens, HALF .. CHUNK-1: B tokens
  __shared__ RoundLds<HALF> s_;
  __shared__ float s_inv[CHUNK];

  const int w = (int)blockIdx.x - edges.blocks;
  const int g = w % blocks_per_seq, bh = w / blocks_per_seq;
  const int t0 = g * CHUNK, n_tok = min(CHUNK, seq - t0);
  const int nA = (n_tok + 1) >> 1, nB = n_tok >> 1;
  const int tid = threadIdx.x, piece = tid % LPR, rg = tid / LPR;
  const int n_out = n_tok - (n_tok == CHUNK ? m_full : m_tail);
  const int out_base = g * (CHUNK - m_full);
  const int64_t at = in.seq_base(bh) + (int64_t)t0 * in.stride_s + piece * 4;
  auto row_of = [](int u) { return (u & 1) * HALF + (u >> 1); };

  float4 kx[PASSES], vx[PASSES];
#pragma unroll
  for (int it = 0; it < PASSES; ++it)              // rows past the block's end re-read its last one
    kx[it] = *reinterpret_cast<const float4*>(K + at + (int64_t)min(it * NRG + rg, n_tok - 1) * in.stride_s);
  int dg = 1;
  if (deg_in && tid < n_tok) dg = deg_in[(int64_t)bh * deg_in_stride + t0 + tid];
#pragma unroll
  for (int it = 0; it < PASSES; ++it)
    vx[it] = *reinterpret_cast<const float4*>(V + at + (int64_t)min(it * NRG + rg, n_tok - 1) * in.stride_s);
  if (tid < HALF) { s_.cnt[tid] = 0; s_.key[tid] = 0; }
  if (tid < CHUNK) {
    const int row = row_of(tid);
    s_.deg[row] = dg;
    s_.word[row] = (uint32_t)row;
    s_.desc[tid] = make_uint2(0, 0);
  }
  if (tid == 0) { s_.n_merged = 0; s_.n_copied = 0; }
#pragma unroll
  for (int it = 0; it < PASSES; ++it) {
    const int u = it * NRG + rg;
    *reinterpret_cast<float4*>(s_f32 + row_of(u) * PITCH + piece * 4) = u < n_tok ? kx[it] : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  __syncthreads();
  if (tid < CHUNK) {                               // 1 / |k| of every row
    float ss = 0.f;
#pragma unroll 4
    for (int k = 0; k < D; k += 4) {
      const float4 x = *reinterpret_cast<const float4*>(s_f32 + tid * PITCH + k);
      ss = fmaf(x.x, x.x, ss); ss = fmaf(x.y, x.y, ss); ss = fmaf(x.z, x.z, ss); ss = fmaf(x.w, x.w, ss);
    }
    s_inv[tid] = inv_norm(ss);
  }
  const int tx = tid % TX, ty = tid / TX;
  float acc[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = 0.f;
#pragma unroll 2
  for (int k = 0; k < D; k += 4) {
    float4 a[NI], b[NJ];
#pragma unroll
    for (int i = 0; i < NI; ++i) a[i] = *reinterpret_cast<const float4*>(s_f32 + (ty + TY * i) * PITCH + k);
#pragma unroll
    for (int j = 0; j < NJ; ++j) b[j] = *reinterpret_cast<const float4*>(s_f32 + (HALF + tx + TX * j) * PITCH + k);
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        acc[i][j] = fmaf(a[i].x, b[j].x, acc[i][j]);
        acc[i][j] = fmaf(a[i].y, b[j].y, acc[i][j]);
        acc[i][j] = fmaf(a[i].z, b[j].z, acc[i][j]);
        acc[i][j] = fmaf(a[i].w, b[j].w, acc[i][j]);
      }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    float best = -INFINITY;
    int bestj = 0;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {                 // increasing rows: the first of equal ones stays
      const float sc = acc[i][j] * s_inv[HALF + tx + TX * j];
      if (tx + TX * j < nB && sc > best) { best = sc; bestj = tx + TX * j; }
    }
#pragma unroll
    for (int x = 1; x < TX; x <<= 1) {
      const float ob = __shfl_xor(best, x);
      const int oj = __shfl_xor(bestj, x);
      if (ob > best || (ob == best && oj < bestj)) { best = ob; bestj = oj; }
    }
    const int a = ty + TY * i;
    if (tx == 0 && a < nA) {
      s_.dst[a] = nB == 0 ? (int16_t)-1 : (int16_t)bestj;
      s_.key[a] = rank_key(best * s_inv[a]);
    }
  }
  round_lists<HALF, THREADS>(s_, n_tok, CHUNK, m_full, m_tail, map, bh, t0, out_base);

  const int n_merged = s_.n_merged;
  const int64_t out_at = out.seq_base(bh) + (int64_t)out_base * out.stride_s + piece * 4;
  auto emit = [&](float* __restrict__ O, bool keys) {
    for (int i = rg; i < n_out; i += NRG) {
      const uint2 w = s_.desc[i];
      const int o = (int)(w.y & 1023u), n = i < n_merged ? (int)(w.y >> 10 & 1023u) : 0;
      float4 x = *reinterpret_cast<const float4*>(s_f32 + w.x * PITCH + piece * 4);
      int nd = s_.deg[w.x];
      if (n > 0) {                                 // (an untouched token is copied bit by bit)
        double a[4] = {(double)nd * x.x, (double)nd * x.y, (double)nd * x.z, (double)nd * x.w};
        for (int q = 0; q < n; ++q) {
          const uint32_t row = s_.members[(w.y >> 20) + q];
          const float4 y = *reinterpret_cast<const float4*>(s_f32 + row * PITCH + piece * 4);
          const int dm = s_.deg[row];
          a[0] += (double)dm * y.x; a[1] += (double)dm * y.y; a[2] += (double)dm * y.z; a[3] += (double)dm * y.w;
          nd += dm;
        }
        const double dn = (double)nd;
        x = make_float4((float)(a[0] / dn), (float)(a[1] / dn), (float)(a[2] / dn), (float)(a[3] / dn));
      }
      *reinterpret_cast<float4*>(O + out_at + (int64_t)o * out.stride_s) = x;
      if (keys && piece == 0) deg_out[(int64_t)bh * deg_out_stride + out_base + o] = nd;
    }
  };
  emit(K_out, true);
  __syncthreads();
#pragma unroll
  for (int it = 0; it < PASSES; ++it) *reinterpret_cast<float4*>(s_f32 + row_of(it * NRG + rg) * PITCH + piece * 4) = vx[it];
  __syncthreads();
  emit(V_out, false);
}

template <int D, int CHUNK>
hipError_t launch_round_f32(const RoundCall& c, hipStream_t st) {
  constexpr int THREADS = f32_threads<D, CHUNK>();
  constexpr size_t lds = (size_t)CHUNK * (D + 4) * sizeof(float);
  static KernelSetup setup;
  if (hipError_t e = kernel_setup(reinterpret_cast<const void*>(&round_f32_kernel<D, CHUNK>), lds, setup); e != hipSuccess) return e;
  const int blocks = div_up(c.seq, CHUNK), tail = c.seq % CHUNK;
  const int64_t edge_blocks = c.edges ? (c.edges->total + THREADS - 1) / THREADS : 0;
  const int m_full = merge_count(c.r, CHUNK / 2), m_tail = tail >= 2 ? merge_count(c.r, (tail + 1) / 2) : 0;
  ScopedTimer t("round_f32", st);
  hipLaunchKernelGGL((round_f32_kernel<D, CHUNK>), dim3((unsigned)((int64_t)c.n_bh * blocks + edge_blocks)), dim3(THREADS), lds,
                     st, static_cast<const float*>(c.K), static_cast<const float*>(c.V), c.deg_in, c.in, c.seq, blocks, m_full,
                     m_tail, static_cast<float*>(c.K_out), static_cast<float*>(c.V_out), c.deg_out, c.out, c.deg_out_stride,
                     c.map, c.in.deg_stride,
                     EdgeBlocks<true>{(int)edge_blocks, c.edges ? *c.edges : EdgeCopy{}});
  return hipGetLastError();
}

template <int D, int TOK>
hipError_t launch_round_t(const RoundCall& c, hipStream_t st) {
  constexpr int THREADS = TOK * D / 64;
  constexpr size_t lds = (size_t)TOK * D * 2;
  const int blocks = div_up(c.seq, TOK);
  const int64_t total = (int64_t)c.n_bh * blocks;
  const int64_t edge_blocks = c.edges ? (c.edges->total + THREADS - 1) / THREADS : 0;
  const int nA_tail = (c.seq % c.chunk + 1) / 2;
  const int m_full = merge_count(c.r, c.chunk / 2), m_tail = c.seq % c.chunk >= 2 ? merge_count(c.r, nA_tail) : 0;
  const PagedSide pout = c.out_k.table ? c.out_k : c.out_v;
  ScopedTimer t("round_bf16", st);
#define CKV_ROUND(PG, ED, ...)                                                                                  \
  do {                                                                                                          \
    static KernelSetup setup;                                                                                   \
    if (hipError_t e = kernel_setup(reinterpret_cast<const void*>(&round_small_kernel<D, TOK, PG, ED>), lds, setup); \
        e != hipSuccess)                                                                                        \
      return e;                                                                                                 \
    hipLaunchKernelGGL((round_small_kernel<D, TOK, PG, ED>), dim3((unsigned)(total + edge_blocks)), dim3(THREADS), lds, st, \
                       static_cast<const __bf16*>(c.K), static_cast<const __bf16*>(c.V), c.deg_in, c.in, c.seq, c.chunk, \
                       blocks, m_full, m_tail, static_cast<__bf16*>(c.K_out), static_cast<__bf16*>(c.V_out), c.deg_out,  \
                       c.out, c.deg_out_stride, c.map, c.in.deg_stride, c.pin, pout,                                     \
                       c.out_k.table != nullptr, c.out_v.table != nullptr, EdgeBlocks<ED>{__VA_ARGS__});                 \
  } while (0)
  if (c.pin.table || pout.table) {
    if (c.edges) CKV_ROUND(true, true, (int)edge_blocks, *c.edges);
    else CKV_ROUND(true, false);
  } else {
    if (c.edges) CKV_ROUND(false, true, (int)edge_blocks, *c.edges);
    else CKV_ROUND(false, false);
  }
#undef CKV_ROUND
  return hipGetLastError();
}

}  // namespace

bool round_fits(int dtype, int dim, int n_bh, int seq, int chunk, const EdgeCopy* edges, bool paged) {
  if (!round_is_small(dtype, dim, chunk) || (paged && dtype != CKV_BF16)) return false;
  const int tokens = dtype == CKV_BF16 && chunk < kTok ? kTok : chunk;
  const int64_t threads = dtype == CKV_BF16 ? tokens * dim / 64 : chunk * dim / 32 > 256 ? chunk * dim / 32 : 256;
  return ((int64_t)n_bh * div_up(seq, tokens) + (edges ? edges->total / threads + 1 : 0)) * threads <= UINT32_MAX;
}

hipError_t launch_round(const RoundCall& c, int dtype, int dim, hipStream_t st) {
  if (dtype == CKV_BF16) {
    if (dim == 128) return c.chunk == 512 ? launch_round_t<128, 512>(c, st) : launch_round_t<128, 256>(c, st);
    return c.chunk == 1024 ? launch_round_t<64, 1024>(c, st) : c.chunk == 512 ? launch_round_t<64, 512>(c, st)
                                                                              : launch_round_t<64, 256>(c, st);
  }
#define CKV_ROUND_F32(D) \
  return c.chunk == 64 ? launch_round_f32<D, 64>(c, st) : c.chunk == 128 ? launch_round_f32<D, 128>(c, st) : launch_round_f32<D, 256>(c, st)
  if (dim == 128) CKV_ROUND_F32(128);
  if (dim == 64) CKV_ROUND_F32(64);
  if (dim == 32) CKV_ROUND_F32(32);
  CKV_ROUND_F32(16);
#undef CKV_ROUND_F32
}

}  // namespace ckv
