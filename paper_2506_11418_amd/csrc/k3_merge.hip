// Top-r selection, degree-weighted merge and order-preserving compaction of one clustering round
// (Sec. 5.3: candidate edges are ranked by similarity and only the best fraction r is merged; the
// centroid equation; values merged with the same weights).
//
// One workgroup per (sequence, chunk).  Integer bookkeeping lives in LDS:
//   keep[i]      source i is among the m = floor(r*|A|) best edges (score desc, index asc; radix select);
//   members[]    kept sources grouped by destination, ascending inside a group (rank by counting:
//                no atomics decide an order, so results are run-to-run identical);
//   local_out[]  prefix sum over retained tokens (all B tokens, unkept A tokens).
// Rows are then produced gather-style: 16-byte pieces, one row per group of row_bytes/16 lanes,
// fp32 accumulation for bf16 (fp64 for fp32 storage), one rounding to the storage type.
//
// What bounds it: large launches the HBM stream, at 0.82 to 0.86 of the copy rate; beside it origin mode has the vector ALU
// busy 58 % of the time at four waves per SIMD, keys-only mode 41 %.  Small ones the chain from the matches to the last row of
// one workgroup.  So the rows are emitted by the
// number of their sources, the row groups of a wave side by side, and nothing that a later step looks up waits
// for it: the matches, the map's entries and the lists of the round before are requested at the start.  us a
// launch, in output order with each requested where it is used / now: origin mode, 256 x 65536 tokens, chunk 1024
// 3559 / 3388; 8 x 524288, chunk 2048 925 / 865; over pages, 32 x 16384 80 / 76.
#include <type_traits>

#include "ckv_internal.h"
#include "ckv_device.h"

namespace ckv {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxHalf = 1024;  // max |A| = |B| (chunk <= 2048); chunks up to 1024 tokens take half the LDS

__device__ inline uint32_t block_exclusive_scan(uint32_t v, uint32_t* s_wave_tot, uint32_t* total) {
  // 256 threads = 4 waves
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t inc = wave_inclusive_scan(v);
  if (lane == 63) s_wave_tot[wave] = inc;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const uint32_t t = s_wave_tot[w];
    if (w < wave) base += t;
    tot += t;
  }
  __syncthreads();
  *total = tot;
  return base + inc - v;
}

template <typename T>
struct Row;  // per-lane 16-byte piece arithmetic

template <>
struct Row<__bf16> {
  static constexpr int E = 8;
  typedef float Acc;
  typedef uint4 Raw;
  __device__ static Raw load_raw(const __bf16* p) { return ldg16_stream(p); }
  __device__ static void store_raw(__bf16* p, const Raw& r) { stg16_stream(p, r); }
  template <bool WIDE>
  __device__ static void fma_into(Acc* acc, const Raw& u, int w) { fma_bf16x8_t<WIDE>(acc, u, w); }
  __device__ static Raw div_raw(const Acc* acc, int n) { return round_div_pack_bf16(acc, n); }
  __device__ static void store_div(__bf16* p, const Acc* acc, int n) { stg16_stream(p, div_raw(acc, n)); }
};

template <>
struct Row<float> {
  static constexpr int E = 4;
  typedef double Acc;
  typedef float4 Raw;
  __device__ static Raw load_raw(const float* p) { return *reinterpret_cast<const float4*>(p); }
  __device__ static void store_raw(float* p, const Raw& r) { *reinterpret_cast<float4*>(p) = r; }
  template <bool WIDE>
  __device__ static void fma_into(Acc* acc, const Raw& u, int wi) {
    const double w = (double)wi;
    acc[0] += w * (double)u.x; acc[1] += w * (double)u.y; acc[2] += w * (double)u.z; acc[3] += w * (double)u.w;
  }
  __device__ static Raw div_raw(const Acc* acc, int n) {
    const double dn = (double)n;
    return make_float4((float)(acc[0] / dn), (float)(acc[1] / dn), (float)(acc[2] / dn), (float)(acc[3] / dn));
  }
  __device__ static void store_div(float* p, const Acc* acc, int n) { *reinterpret_cast<float4*>(p) = div_raw(acc, n); }
};

constexpr int kRowsInFlight = 1;   // output rows of a row group per batch (two batches are in flight)
constexpr int kRowsInFlightOrigin = 2;   // ... when every value row is itself rebuilt from several rows

// MODE (two consecutive rounds whose first merges every edge, r = 1, can skip the intermediate
// VALUE cache: a round-0 chunk then keeps exactly its B tokens, so a round-1 chunk is fed by two
// round-0 chunks):
//   kMergeFull    keys and values of this round's input -> this round's output;
//   kMergeKeys    first round of such a pair: keys and degrees only, and the member lists of
//                 every chunk are exported (lists_out: per chunk cnt | start | members, int16);
//   kMergeOrigin  second round of the pair: keys as usual, while every value row of the input
//                 (a round-0 centroid that was never written) is rebuilt from the ORIGINAL values
//                 through the exported lists, in the same fp32 order and with the same single
//                 rounding the first round would have used, so the results are bit-identical.
enum { kMergeFull = 0, kMergeKeys = 1, kMergeOrigin = 2 };

// PAGED: some side of the launch lives in a block pool (PagedSide): the input rows (K, V, deg_in),
// the original values of kMergeOrigin (org.paged), the output keys (out_k_paged) or the output values
// and degrees (out_v_paged), each decided by its table pointer / flag at run time; the pool rows of the
// blocks a workgroup touches are staged in LDS (blocks of 8 tokens or more).
//
// EDGES: the first edge_blocks workgroups copy the tokens that bypass the clustering (none of the others
// touches those rows).
//
// Launch bounds: bf16 in full mode is to hold five waves per SIMD, the workgroups per CU that small launches are cut into
// (launch_merge_t).  It takes 92 to 96 registers, with or without being told; 97 would be four waves, and a fifth of the
// workgroups by themselves at the end.
template <typename T, int D, int MODE, int MH, bool PAGED, bool EDGES>   // MH: capacity of the per-chunk LDS arrays (|A| = |B| <= MH)
__global__ __launch_bounds__(kThreads, sizeof(T) == 2 && MODE == kMergeFull ? 5 : 1) void merge_kernel(
    const T* __restrict__ K, const T* __restrict__ V, const int32_t* __restrict__ deg_in, TensorView in,
    int seq, int chunk, int n_chunks, float r, const int32_t* __restrict__ dst_local,
    const float* __restrict__ score, T* __restrict__ K_out, T* __restrict__ V_out,
    int32_t* __restrict__ deg_out, TensorView out, int64_t deg_out_stride, RoundMap map,
    int64_t deg_in_stride, const int2* __restrict__ sel_table,
    int16_t* __restrict__ lists_out, ValueOrigin org, int parts, PagedSide pin, PagedSide pout, int out_k_paged,
    int out_v_paged, EdgeBlocks<EDGES> edges) {
  if constexpr (EDGES) {
    if ((int)blockIdx.x < edges.blocks) {
      copy_edges(edges.copy, (int64_t)blockIdx.x * kThreads + threadIdx.x);
      return;
    }
  }
  constexpr int E = Row<T>::E;
  constexpr int LPR = D / E;                 // lanes per row
  constexpr int NRG = kThreads / LPR;        // row groups per workgroup
  constexpr int U = (MODE == kMergeOrigin) ? kRowsInFlightOrigin : kRowsInFlight;
  typedef typename Row<T>::Acc Acc;
  typedef typename Row<T>::Raw Raw;

  // s_dstk[i]: destination (B index) of source i if its edge is kept, -1 otherwise
  __shared__ __attribute__((aligned(16))) int16_t s_dstk[MH];
  __shared__ __attribute__((aligned(16))) float s_score[MH];
  __shared__ int32_t s_cnt[MH];
  __shared__ __attribute__((aligned(16))) int32_t s_fill[MH];
  __shared__ int16_t s_start[MH];
  __shared__ int16_t s_members[MH];
  __shared__ __attribute__((aligned(16))) int16_t s_local_out[2 * MH];
  __shared__ int16_t s_src_of_place[2 * MH];
  __shared__ uint32_t s_wave_tot[4];
  // kMergeOrigin, chunks up to 1024 tokens: per output row, everything the emit loop would look up
  // through the lists, resolved once (three 8-byte words: the row's own sources, then where the
  // value rows of its own token and of its first merged source come from)
  constexpr bool DESC = (MODE == kMergeOrigin) && (MH <= 512);
  __shared__ uint2 s_desc[DESC ? 3 * 2 * MH : 1];
  __shared__ int16_t s_out_of_place[MODE == kMergeOrigin && !DESC ? 2 * MH : 1];
  __shared__ int32_t s_rb_in[PAGED ? 2 * MH / 8 + 2 : 1];
  __shared__ int32_t s_rb_org[(PAGED && MODE == kMergeOrigin) ? 4 * MH / 8 + 2 : 1];
  __shared__ int32_t s_rb_out[PAGED ? 2 * MH / 8 + 2 : 1];

  // `parts` workgroups share a chunk when the launch would otherwise leave most of the chip idle:
  // each repeats the (cheap) bookkeeping and emits every parts-th group of output rows.
  int id = (int)blockIdx.x;
  if constexpr (EDGES) id -= edges.blocks;
  const int part = id % parts, wg = id / parts;
  const int g = wg % n_chunks, bh = wg / n_chunks;
  const int tid = threadIdx.x;
  const int g0 = g * chunk, L = min(chunk, seq - g0);
  const int half = chunk >> 1;
  const int nA = (L + 1) >> 1, nB = L >> 1;
  // edges merged in this chunk and its first output row: fixed by r alone for per-chunk selection,
  // read from the table of the sequence-wide selection otherwise
  int m, out_base;
  if (sel_table) {
    const int2 e = sel_table[(int64_t)bh * n_chunks + g];
    m = e.x;
    out_base = e.y;
  } else {
    m = (nB > 0) ? merge_count(r, nA) : 0;
    out_base = g * chunk_out(chunk, r);
  }
  const int n_out = L - m;
  RowBases rb_in{}, rb_org{}, rb_out{};
  const bool in_paged = PAGED && pin.table != nullptr;
  const bool org_paged = PAGED && MODE == kMergeOrigin && org.paged.table != nullptr;
  const bool ok_paged = PAGED && out_k_paged, ov_paged = PAGED && out_v_paged;
  if (PAGED) {   // (the barriers of the bookkeeping below come before the first use)
    const int b = bh / in.heads, h = bh % in.heads;
    if (in_paged && L > 0) rb_in = stage_row_bases(s_rb_in, pin, b, h, in.heads, pin.tok0 + g0, pin.tok0 + g0 + L - 1, tid, kThreads);
    if (org_paged) {
      const int t_lo = 2 * g * chunk, t_hi = min(org.seq0, t_lo + 2 * chunk);
      if (t_hi > t_lo)
        rb_org = stage_row_bases(s_rb_org, org.paged, b, h, in.heads, org.paged.tok0 + t_lo, org.paged.tok0 + t_hi - 1, tid, kThreads);
    }
    if ((ok_paged || ov_paged) && n_out > 0)
      rb_out = stage_row_bases(s_rb_out, pout, b, h, in.heads, pout.tok0 + out_base, pout.tok0 + out_base + n_out - 1, tid, kThreads);
  }
  const int n_src = n_sources(seq, chunk);
  const int64_t src_base = (int64_t)bh * n_src + (int64_t)g * (chunk >> 1);
  // ---- top-r: the key of the m-th best edge by a radix select, equal ones by position -------------
  // (a rank by counting compares every score with every other one: 8 x 8448 tokens, chunk 1024, r = 0.8 43 us a launch,
  // one digit at a time 29)
  constexpr int PER = MH / kThreads;               // sources per thread
  int d_of[PER];
#pragma unroll
  for (int it = 0; it < PER; ++it) {
    const int i = tid + it * kThreads;
    d_of[it] = (i < nA && m > 0) ? dst_local[src_base + i] : -1;
  }
  // (so are the map's entries and the lists of the round before: each was a memory latency of its own further down)
  const int map_threads = parts * kThreads, map_hi = fold_end(map, g0, chunk), map_t = (g0 << map.fold) + part * kThreads + tid;
  FoldAhead map_ahead{};
  if (map.p != nullptr && map.fold > 0) map_ahead = fold_request(map, bh, map_hi, map_threads, map_t);
  constexpr int LP = (6 * MH / 8 + kThreads - 1) / kThreads;
  static_assert(LP == 2 || LP == 3, "pieces of the lists per thread");
  u32x4 piece0{}, piece1{}, piece2{};                // (an array of them ends up in scratch)
  const int n_list = MODE == kMergeOrigin ? min(2, org.n_chunks0 - 2 * g) * 3 * half : 0;   // of one or two chunks, side by side
  const int16_t* lists_in = MODE == kMergeOrigin ? org.lists + ((int64_t)bh * org.n_chunks0 + 2 * g) * 3 * half : nullptr;
  const bool by_piece = half % 8 == 0 && (reinterpret_cast<uintptr_t>(lists_in) & 15) == 0;
  if (MODE == kMergeOrigin && by_piece) {
    auto request = [&](int i) { return *reinterpret_cast<const u32x4*>(lists_in + 8 * min(tid + i * kThreads, n_list / 8 - 1)); };
    piece0 = request(0);
    piece1 = request(1);
    if (LP > 2) piece2 = request(2);
  }
  const bool ranked = m > 0 && m < nA;
  uint32_t key[PER];
  static_assert(MH >= 512 && kThreads == 256, "two histograms of a digit in either array");
  uint32_t* hist_of[4] = {reinterpret_cast<uint32_t*>(s_fill), reinterpret_cast<uint32_t*>(s_fill) + 256,
                          reinterpret_cast<uint32_t*>(s_score), reinterpret_cast<uint32_t*>(s_score) + 256};
  if (ranked) {
#pragma unroll
    for (int p = 0; p < 4; ++p) hist_of[p][tid] = 0;
#pragma unroll
    for (int it = 0; it < PER; ++it) {
      const int i = tid + it * kThreads;
      key[it] = i < nA ? order_key(score[src_base + i]) : 0u;
    }
  }
  for (int j = tid; j < nB; j += kThreads) s_cnt[j] = 0;
  if (PAGED) __syncthreads();                      // (the rows of the blocks)
  // Two versions of the emit loop: weights up to 256 ride in a packed bf16 operand (one v_dot2 per
  // element); a chunk that holds a larger degree takes the general route.  Same bits either way.
  // (asked here, so that the degrees' latency is the one of the matches)
  int big = 0;
  if (deg_in) {
    const int32_t* dc = in_paged ? deg_in : deg_in + (int64_t)bh * deg_in_stride + g0;
    for (int u = tid; u < L; u += kThreads) big |= dc[in_paged ? rb_in.row(pin.tok0 + g0 + u) : u] > 256;
  }
  if (MODE == kMergeOrigin && org.deg0) {
    const int32_t* dc = org_paged ? org.deg0 : org.deg0 + (int64_t)bh * org.view0.deg_stride;
    const int t_lo = 2 * g * chunk, t_hi = min(org.seq0, t_lo + 2 * chunk);
    for (int t = t_lo + tid; t < t_hi; t += kThreads) big |= dc[org_paged ? rb_org.row(org.paged.tok0 + t) : t] > 256;
  }
  const bool wide = __syncthreads_or(big) != 0;
  if (ranked) {
    const int lane = tid & 63;
    uint32_t cut = 0;
    int left = m, equal = 0;                       // of the keys that agree with the cut so far, the left best are kept
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int shift = 24 - 8 * p;
#pragma unroll
      for (int it = 0; it < PER; ++it)
        if (tid + it * kThreads < nA && (p == 0 || ((key[it] ^ cut) >> (shift + 8)) == 0))
          atomicAdd(&hist_of[p][key[it] >> shift & 255u], 1u);
      __syncthreads();
      // every wave finds the bin for itself; lane l: bins 255 - 4l downwards
      int c[4], sum = 0;
      const uint4 h = *reinterpret_cast<const uint4*>(&hist_of[p][252 - 4 * lane]);
      c[0] = (int)h.w; c[1] = (int)h.z; c[2] = (int)h.y; c[3] = (int)h.x;
#pragma unroll
      for (int e = 0; e < 4; ++e) sum += c[e];
      const int inc = (int)wave_inclusive_scan((uint32_t)sum);
      const int owner = __ffsll((unsigned long long)__ballot(inc >= left)) - 1;   // (the last lane's sum reaches it)
      int above = inc - sum, e = 0;
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (e == k && above + c[k] < left) { above += c[k]; ++e; }
      const int n = e == 0 ? c[0] : e == 1 ? c[1] : e == 2 ? c[2] : c[3];
      cut |= (uint32_t)__builtin_amdgcn_readlane(255 - 4 * lane - e, owner) << shift;
      left -= __builtin_amdgcn_readlane(above, owner);
      equal = __builtin_amdgcn_readlane(n, owner);
    }
    if (left < equal) {                            // (the same for every thread) only the earliest of the equal ones
      int16_t* at_cut = s_local_out;               // (not in use yet)
#pragma unroll
      for (int it = 0; it < PER; ++it) {
        const int i = tid + it * kThreads;
        if (i < nA) at_cut[i] = key[it] == cut;
      }
      __syncthreads();
#pragma unroll
      for (int it = 0; it < PER; ++it) {
        const int i = tid + it * kThreads;
        if (i < nA && key[it] == cut) {
          int earlier = 0;
          for (int o = 0; o < i; ++o) earlier += at_cut[o];
          if (earlier >= left) d_of[it] = -1;
        }
      }
    }
#pragma unroll
    for (int it = 0; it < PER; ++it)
      if (key[it] < cut) d_of[it] = -1;
  }

  // ---- kept sources grouped by destination, ascending within a group --------------------------
  // counts by integer atomics (order-free), then slots handed out by atomics in arbitrary order
  // and every destination's short list sorted: the final order is unique, so results stay
  // run-to-run identical.  Lists longer than kSortMax (degenerate inputs: many identical keys)
  // are placed by rank counting instead.
  constexpr int kSortMax = 8;
#pragma unroll
  for (int it = 0; it < PER; ++it) {
    const int i = tid + it * kThreads;
    if (i < nA) s_dstk[i] = (int16_t)d_of[it];
    if (d_of[it] >= 0) atomicAdd(&s_cnt[d_of[it]], 1);
  }
  __syncthreads();
  int longest = 0;
  {
    int c[4], sum = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int j = tid * 4 + e;
      c[e] = (j < nB) ? s_cnt[j] : 0;
      sum += c[e];
      longest = max(longest, c[e]);
    }
    uint32_t tot;
    uint32_t base = block_exclusive_scan((uint32_t)sum, s_wave_tot, &tot);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int j = tid * 4 + e;
      if (j < nB) { s_start[j] = (int16_t)base; s_fill[j] = 0; }
      base += c[e];
    }
  }
  const bool any_long = __syncthreads_or(longest > kSortMax);
#pragma unroll
  for (int it = 0; it < PER; ++it) {
    const int i = tid + it * kThreads;
    const int d = d_of[it];
    if (d >= 0) {
      int pos;
      if (any_long && s_cnt[d] > kSortMax) {        // rank among earlier sources of the same list
        pos = 0;
        for (int o = 0; o < i; ++o) pos += ((int)s_dstk[o] == d);
      } else {
        pos = atomicAdd(&s_fill[d], 1);
      }
      s_members[s_start[d] + pos] = (int16_t)i;
    }
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 4; ++e) {                     // insertion sort of the short lists
    const int j = tid * 4 + e;
    const int n = (j < nB) ? s_cnt[j] : 0;
    if (n > 1 && n <= kSortMax) {
      int16_t* lst = &s_members[s_start[j]];
      for (int a = 1; a < n; ++a) {
        const int16_t v = lst[a];
        int b2 = a - 1;
        while (b2 >= 0 && lst[b2] > v) { lst[b2 + 1] = lst[b2]; --b2; }
        lst[b2 + 1] = v;
      }
    }
  }

  // ---- retained tokens: prefix sum over the chunk --------------------------------------------
  // Their output rows, and the places at which they are emitted: rows of two or more sources first, then rows of
  // one, the copies last, so that the row groups of a wave do the same work side by side.  One scan of three sums
  // (10, 11 and 11 bits; 2048 copies, a whole chunk, pass theirs only in the total).
  // A launch with a row group for every row keeps them in output order: a wave is done with its longest row either way, and by
  // sources the rows of many stand together in a few workgroups.  us a compression of 8 sequences of dim 128 to a quarter, by
  // sources / in output order: 5000 tokens, chunk 1024 55.3 / 54.4; 4 of 6144, chunk 384 39.3 / 38.3; 8 of 3000, dim 64, chunk 384
  // 35.2 / 34.5.
  {
    const bool row_each = n_out <= parts * NRG * U;
    auto sums = [](int n) -> uint32_t { return n > 1 ? 1u : n == 1 ? 1u << 10 : 1u << 21; };
    const bool sources_left = m < nA;               // (else no source is looked at: every workgroup of a chunk does this)
    int n[4];                                       // sources of the destinations, -1: past the end
    bool left[4];
    uint32_t mine = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int u = tid * 8 + 2 * e;
      left[e] = sources_left && u < L && s_dstk[u >> 1] < 0;
      n[e] = u + 1 < L ? s_cnt[u >> 1] : -1;
      mine += ((uint32_t)left[e] << 21) + (n[e] >= 0 ? sums(n[e]) : 0u);
    }
    uint32_t tot;
    const uint32_t before = block_exclusive_scan(mine, s_wave_tot, &tot);
    const int n_long = (int)(tot & 1023u), n_merged = n_long + (int)(tot >> 10 & 2047u);
    int at2 = (int)(before & 1023u), at1 = (int)(before >> 10 & 2047u), at0 = (int)(before >> 21), o = at2 + at1 + at0;
    at1 += n_long;
    at0 += n_merged;
    auto put = [&](int u, int place) {
      if (row_each) place = o;
      s_local_out[u] = (int16_t)o;
      s_src_of_place[place] = (int16_t)u;
      if constexpr (DESC) s_desc[3 * place].y = (uint32_t)o;        // (s_local_out is overwritten below)
      else if constexpr (MODE == kMergeOrigin) s_out_of_place[place] = (int16_t)o;
      ++o;
    };
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int u = tid * 8 + 2 * e;
      if (left[e]) put(u, at0++);
      if (n[e] >= 0) put(u + 1, n[e] > 1 ? at2 : n[e] == 1 ? at1 : at0);
      at2 += n[e] > 1;
      at1 += n[e] == 1;
      at0 += n[e] == 0;
    }
  }
  __syncthreads();

  // Lists and map of a whole chunk are written by the last of its workgroups, whose rows, by sources, are the copies: by the first
  // one, they stood before the longest rows (us a compression, first / last: 8 sequences of 8192 tokens of dim 64, chunk 2048, to a
  // half 31.1 / 30.2; 2048 tokens of dim 128, chunk 2048 32.4 / 32.0, 5000, chunk 1024, to a quarter 55.9 / 55.3).
  if (MODE == kMergeKeys && part == parts - 1) {   // member lists of this chunk for the next round's value rebuild
    int16_t* lst = lists_out + ((int64_t)bh * n_chunks + g) * 3 * half;
    for (int i = tid; i < half; i += kThreads) {
      lst[i] = (i < nB) ? (int16_t)s_cnt[i] : (int16_t)0;
      lst[half + i] = (i < nB) ? s_start[i] : (int16_t)0;
      lst[2 * half + i] = (i < m) ? s_members[i] : (int16_t)0;
    }
  }

  // ---- assignment map of this round ----------------------------------------------------------
  if (map.p != nullptr) {
    auto place = [&](int u) -> int {
      const int d = (u & 1) ? -1 : (int)s_dstk[u >> 1];
      return map.offset + out_base + ((d < 0) ? s_local_out[u] : s_local_out[2 * d + 1]);
    };
    if (map.fold > 0) {
      fold_map(map, bh, g0, map_hi, map_threads, map_t, map_ahead, place);
    } else if (part == parts - 1) {
      int32_t* mp = map.p + (int64_t)bh * map.stride + g0;
      for (int u = tid; u < L; u += kThreads) mp[u] = place(u);
    }
  }

  // kMergeOrigin: the member lists of the two previous-round chunks that feed this chunk, staged in
  // LDS arrays the bookkeeping above no longer needs (scores, fill counters, local output slots)
  int16_t (*s0_cnt)[MH] = reinterpret_cast<int16_t (*)[MH]>(s_score);
  int16_t (*s0_start)[MH] = reinterpret_cast<int16_t (*)[MH]>(s_fill);
  int16_t (*s0_mem)[MH] = reinterpret_cast<int16_t (*)[MH]>(s_local_out);
  if (MODE == kMergeOrigin) {
    __syncthreads();
    auto list_at = [&](int e) -> int16_t* {          // where element e of the lists goes
      const int h = e >= 3 * half, i = e - h * 3 * half;
      return i < half ? &s0_cnt[h][i] : i < 2 * half ? &s0_start[h][i - half] : &s0_mem[h][i - 2 * half];
    };
    if (by_piece) {                                  // (no piece straddles two of them)
      auto park = [&](int i, u32x4 x) {
        const int e = 8 * (tid + i * kThreads);
        if (e < n_list) *reinterpret_cast<u32x4*>(list_at(e)) = x;
      };
      park(0, piece0);
      park(1, piece1);
      if (LP > 2) park(2, piece2);
    } else {
      for (int e = tid; e < n_list; e += kThreads) *list_at(e) = lists_in[e];
    }
    __syncthreads();
    if constexpr (DESC) {
      // token indices are kept relative to the first token of previous-round chunk 2g
      auto value_words = [&](int p) -> uint2 {
        const int h = (p >= half) ? 1 : 0, jj = p - h * half;
        const bool single = (org.seq0 - (2 * g + h) * chunk) == 1;
        const int tb = h * chunk + (single ? 0 : 2 * jj + 1);
        const int n = single ? 0 : (int)s0_cnt[h][jj];
        const int off = h * MH + (int)s0_start[h][jj];
        const int ta = (n > 0) ? h * chunk + 2 * (int)(&s0_mem[0][0])[off] : tb;
        return make_uint2((uint32_t)tb | ((uint32_t)ta << 16), (uint32_t)n | ((uint32_t)off << 16));
      };
      for (int o = tid; o < n_out; o += kThreads) {
        const int tok = s_src_of_place[o];
        const bool isB = tok & 1;
        const int nmem = isB ? s_cnt[tok >> 1] : 0;
        const int first = isB ? (int)s_start[tok >> 1] : 0;
        const int mem0 = (nmem > 0) ? 2 * (int)s_members[first] : tok;
        s_desc[3 * o] = make_uint2((uint32_t)tok | ((uint32_t)mem0 << 16),
                                   (uint32_t)nmem | ((uint32_t)first << 10) | (s_desc[3 * o].y << 20));
        s_desc[3 * o + 1] = value_words(tok);
        s_desc[3 * o + 2] = value_words(mem0);
      }
      __syncthreads();
    }
  }

  // ---- emit rows: every row group works on U output rows at once; the loads of their own rows
  // and of their first merged source are all in flight before anything is consumed ---------------
  const int rg = tid / LPR, piece = tid % LPR;
  const T* Kin = in_paged ? K + piece * E : K + in.seq_base(bh) + (int64_t)g0 * in.stride_s + piece * E;
  const T* Vin = (MODE != kMergeFull) ? nullptr
                 : in_paged ? V + piece * E : V + in.seq_base(bh) + (int64_t)g0 * in.stride_s + piece * E;
  T* Ko = ok_paged ? K_out + piece * E : K_out + out.seq_base(bh) + (int64_t)out_base * out.stride_s + piece * E;
  T* Vo = (MODE == kMergeKeys) ? nullptr
          : ov_paged ? V_out + piece * E : V_out + out.seq_base(bh) + (int64_t)out_base * out.stride_s + piece * E;
  const int32_t* dseq = !deg_in ? nullptr : in_paged ? deg_in : deg_in + (int64_t)bh * deg_in_stride + g0;
  int32_t* dout = ov_paged ? deg_out : deg_out + (int64_t)bh * deg_out_stride + out_base;
  // element offset of input row u / output row o of this chunk from Kin, Vin / Ko, Vo, and the index
  // of their degrees in dseq / dout.  An output row whose block lies outside the pool is not written.
  const int u_in0 = pin.tok0 + g0, u_out0 = pout.tok0 + out_base;
  auto in_off = [&](int u) -> int64_t { return in_paged ? (int64_t)rb_in.row(u_in0 + u) * D : (int64_t)u * in.stride_s; };
  auto in_deg = [&](int u) -> int { return in_paged ? dseq[rb_in.row(u_in0 + u)] : dseq[u]; };
  auto ok_off = [&](int o) -> int64_t { return ok_paged ? (int64_t)rb_out.row(u_out0 + o) * D : (int64_t)o * out.stride_s; };
  auto ov_off = [&](int o) -> int64_t { return ov_paged ? (int64_t)rb_out.row(u_out0 + o) * D : (int64_t)o * out.stride_s; };
  auto out_ok = [&](int o) -> bool { return !(ok_paged || ov_paged) || rb_out.base_of(u_out0 + o) >= 0; };
  auto put_deg = [&](int o, int d) {
    if (ov_paged) dout[rb_out.row(u_out0 + o)] = d;
    else dout[o] = d;
  };

  // The value row of input row p of this chunk.  kMergeFull: a load.  kMergeOrigin: the previous
  // round's centroid p, rebuilt: p is B token j of previous-round chunk 2g+h (a one-token tail chunk
  // kept its only token); its own row and its first member are loaded at once, the rest on demand.
  const T* V0p = (MODE != kMergeOrigin) ? nullptr
                 : org_paged ? static_cast<const T*>(org.V0) + piece * E
                             : static_cast<const T*>(org.V0) + org.view0.seq_base(bh) + piece * E;
  const int32_t* d0p = (MODE == kMergeOrigin && org.deg0)
                           ? (org_paged ? org.deg0 : org.deg0 + (int64_t)bh * org.view0.deg_stride) : nullptr;
  // original value row / degree of token t of the first round's clustered range
  auto v0_off = [&](int t) -> int64_t {
    return org_paged ? (int64_t)rb_org.row(org.paged.tok0 + t) * D : (int64_t)t * org.view0.stride_s;
  };
  auto d0_at = [&](int t) -> int { return org_paged ? d0p[rb_org.row(org.paged.tok0 + t)] : d0p[t]; };
  constexpr int kEager = 1;   // members of a previous-round cluster loaded together with its own row
  struct VLoad {
    Raw b, m[kEager];
    int db, dm[kEager], n, base;
    const int16_t* mem;
  };
  struct NoVLoad {};   // keys-only mode carries no value rows
  auto v_issue = [&](int p) -> VLoad {
    VLoad x;
    if (MODE == kMergeFull) {
      x.b = Row<T>::load_raw(Vin + in_off(p));
      x.n = 0;
    } else if (MODE == kMergeOrigin) {
      const int h = (p >= half) ? 1 : 0, jj = p - h * half;
      x.base = (2 * g + h) * chunk;
      const bool single = (org.seq0 - x.base) == 1;
      const int tb = x.base + (single ? 0 : 2 * jj + 1);
      x.n = single ? 0 : (int)s0_cnt[h][jj];
      x.mem = &s0_mem[h][s0_start[h][jj]];
      x.b = Row<T>::load_raw(V0p + v0_off(tb));
      x.db = d0p ? d0_at(tb) : 1;
#pragma unroll
      for (int q = 0; q < kEager; ++q) {
        if (q < x.n) {
          const int ta = x.base + 2 * (int)x.mem[q];
          x.m[q] = Row<T>::load_raw(V0p + v0_off(ta));
          x.dm[q] = d0p ? d0_at(ta) : 1;
        }
      }
    }
    return x;
  };
  auto v_issue_resolved = [&](uint2 w) -> VLoad {
    VLoad x;
    if constexpr (MODE == kMergeOrigin) {
      const int t0 = 2 * g * chunk;
      const int tb_rel = (int)(w.x & 0xffffu);
      const int tb = t0 + tb_rel, ta = t0 + (int)(w.x >> 16);
      x.base = t0 + ((tb_rel >= chunk) ? chunk : 0);
      x.n = (int)(w.y & 0xffffu);
      x.mem = &s0_mem[0][0] + (w.y >> 16);
      x.b = Row<T>::load_raw(V0p + v0_off(tb));
      x.db = d0p ? d0_at(tb) : 1;
      static_assert(kEager == 1, "one resolved member per cluster");
      if (x.n > 0) {
        x.m[0] = Row<T>::load_raw(V0p + v0_off(ta));
        x.dm[0] = d0p ? d0_at(ta) : 1;
      }
    }
    return x;
  };
  auto v_finish = [&](auto wide_c, const VLoad& x) -> Raw {
    constexpr bool WIDE = decltype(wide_c)::value;
    if (MODE != kMergeOrigin || x.n == 0) return x.b;
    Acc a[E];
#pragma unroll
    for (int e = 0; e < E; ++e) a[e] = 0;
    Row<T>::template fma_into<WIDE>(a, x.b, x.db);
    int nd = x.db;
#pragma unroll
    for (int q = 0; q < kEager; ++q)
      if (q < x.n) {
        Row<T>::template fma_into<WIDE>(a, x.m[q], x.dm[q]);
        nd += x.dm[q];
      }
    for (int q = kEager; q < x.n; ++q) {
      const int ta = x.base + 2 * (int)x.mem[q];
      const int da = d0p ? d0_at(ta) : 1;
      Row<T>::template fma_into<WIDE>(a, Row<T>::load_raw(V0p + v0_off(ta)), da);
      nd += da;
    }
    return Row<T>::div_raw(a, nd);
  };

  // One batch = U output rows per row group: where they come from (LDS lookups) and the loads of
  // their own rows and first merged sources, all issued before anything is consumed.
  struct Batch {
    int o[U], tok[U], nmem[U], first[U], du[U], dm[U];
    bool valid[U];
    Raw kb[U], km[U];
    typename std::conditional<MODE == kMergeKeys, NoVLoad, VLoad>::type vb[U], vm[U];
  };
  struct Where {
    int o[U], tok[U], mem0[U], nmem[U], first[U];
    bool valid[U];
    uint2 wb[U], wm[U];
  };
  auto lookup = [&](int ob) -> Where {
    Where w;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int at = ob + u * NRG + rg;
      w.valid[u] = at < n_out;
      const int place = w.valid[u] ? at : n_out - 1;
      if constexpr (DESC) {
        const uint2 k = s_desc[3 * place];
        w.wb[u] = s_desc[3 * place + 1];
        w.wm[u] = s_desc[3 * place + 2];
        w.tok[u] = (int)(k.x & 0xffffu);
        w.mem0[u] = (int)(k.x >> 16);
        w.nmem[u] = (int)(k.y & 1023u);
        w.first[u] = (int)(k.y >> 10 & 1023u);
        w.o[u] = (int)(k.y >> 20);
      } else {
        w.tok[u] = s_src_of_place[place];
        w.o[u] = MODE == kMergeOrigin ? s_out_of_place[place] : s_local_out[w.tok[u]];
        const bool isB = w.tok[u] & 1;
        w.nmem[u] = isB ? s_cnt[w.tok[u] >> 1] : 0;
        w.first[u] = isB ? (int)s_start[w.tok[u] >> 1] : 0;
        w.mem0[u] = (w.nmem[u] > 0) ? 2 * (int)s_members[w.first[u]] : w.tok[u];   // no source: re-read own row
      }
    }
    return w;
  };
  auto issue = [&](const Where& w) -> Batch {
    Batch x;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      x.valid[u] = w.valid[u];
      x.tok[u] = w.tok[u];
      x.o[u] = w.o[u];
      x.nmem[u] = w.nmem[u];
      x.first[u] = w.first[u];
      x.kb[u] = Row<T>::load_raw(Kin + in_off(w.tok[u]));
      if constexpr (DESC) x.vb[u] = v_issue_resolved(w.wb[u]);
      else if constexpr (MODE != kMergeKeys) x.vb[u] = v_issue(w.tok[u]);
      x.du[u] = dseq ? in_deg(w.tok[u]) : 1;
      if (MODE != kMergeOrigin || w.nmem[u] > 0) {
        x.km[u] = Row<T>::load_raw(Kin + in_off(w.mem0[u]));
        if constexpr (DESC) x.vm[u] = v_issue_resolved(w.wm[u]);
        else if constexpr (MODE != kMergeKeys) x.vm[u] = v_issue(w.mem0[u]);
        x.dm[u] = dseq ? in_deg(w.mem0[u]) : 1;
      }
    }
    return x;
  };
  auto fetch = [&](int ob) -> Batch { return issue(lookup(ob)); };
  auto finish = [&](auto wide_c, const Batch& x) {
    constexpr bool WIDE = decltype(wide_c)::value;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!x.valid[u]) continue;
      const int o = x.o[u];
      if (PAGED && !out_ok(o)) continue;
      if (x.nmem[u] == 0) {  // untouched token: bit copy
        Row<T>::store_raw(Ko + ok_off(o), x.kb[u]);
        if constexpr (MODE != kMergeKeys) Row<T>::store_raw(Vo + ov_off(o), v_finish(wide_c, x.vb[u]));
        if (piece == 0) put_deg(o, x.du[u]);
        continue;
      }
      Acc ak[E], av[E];
#pragma unroll
      for (int e = 0; e < E; ++e) { ak[e] = 0; av[e] = 0; }
      Row<T>::template fma_into<WIDE>(ak, x.kb[u], x.du[u]);
      Row<T>::template fma_into<WIDE>(ak, x.km[u], x.dm[u]);
      if constexpr (MODE != kMergeKeys) {
        Row<T>::template fma_into<WIDE>(av, v_finish(wide_c, x.vb[u]), x.du[u]);
        Row<T>::template fma_into<WIDE>(av, v_finish(wide_c, x.vm[u]), x.dm[u]);
      }
      int ndeg = x.du[u] + x.dm[u];
      // (two at a time: rows of several sources meet in few waves, which waited for them one by one)
      for (int q = 1; q < x.nmem[u]; q += 2) {
        const bool two = q + 1 < x.nmem[u];
        int ua[2], da[2];
        Raw kx[2], vx[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          ua[i] = 2 * (int)s_members[x.first[u] + q + (two ? i : 0)];
          da[i] = dseq ? in_deg(ua[i]) : 1;
          kx[i] = Row<T>::load_raw(Kin + in_off(ua[i]));
          if constexpr (MODE == kMergeFull) vx[i] = Row<T>::load_raw(Vin + in_off(ua[i]));
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          if (i == 1 && !two) break;
          Row<T>::template fma_into<WIDE>(ak, kx[i], da[i]);
          if constexpr (MODE == kMergeFull) Row<T>::template fma_into<WIDE>(av, vx[i], da[i]);
          ndeg += da[i];
        }
      }
      Row<T>::store_div(Ko + ok_off(o), ak, ndeg);
      if constexpr (MODE != kMergeKeys) Row<T>::store_div(Vo + ov_off(o), av, ndeg);
      if (piece == 0) put_deg(o, ndeg);
    }
  };
  // kMergeOrigin: the same sums in the same order as v_finish, for several clusters in lock step.
  // A row group that walks one cluster after the other waits a full memory latency per extra member
  // while the rest of its wave idles; here the q-th extra member of every cluster handed in is
  // requested at once, so the wave waits as often as the longest of them has members, not the sum.
  // Called per output row with its two clusters (own token, first merged source): handing in all
  // four of a batch measured the same and needs 15 more registers.
  auto v_finish_all = [&](auto wide_c, auto count_c, const VLoad* cl, const bool* on, Raw* res) {
    constexpr bool WIDE = decltype(wide_c)::value;
    constexpr int C = decltype(count_c)::value;
    Acc a[C][E];
    int nd[C], n[C], longest = 0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      n[c] = on[c] ? cl[c].n : 0;
      nd[c] = 0;
#pragma unroll
      for (int e = 0; e < E; ++e) a[c][e] = 0;
      if (n[c] > 0) {
        Row<T>::template fma_into<WIDE>(a[c], cl[c].b, cl[c].db);
        Row<T>::template fma_into<WIDE>(a[c], cl[c].m[0], cl[c].dm[0]);
        nd[c] = cl[c].db + cl[c].dm[0];
      }
      longest = max(longest, n[c]);
    }
    for (int q = kEager; q < longest; ++q) {
      Raw r[C];
      int d[C];
#pragma unroll
      for (int c = 0; c < C; ++c)
        if (q < n[c]) {
          const int ta = cl[c].base + 2 * (int)cl[c].mem[q];
          r[c] = Row<T>::load_raw(V0p + v0_off(ta));
          d[c] = d0p ? d0_at(ta) : 1;
        }
#pragma unroll
      for (int c = 0; c < C; ++c)
        if (q < n[c]) {
          Row<T>::template fma_into<WIDE>(a[c], r[c], d[c]);
          nd[c] += d[c];
        }
    }
#pragma unroll
    for (int c = 0; c < C; ++c)
      if (on[c]) res[c] = (n[c] == 0) ? cl[c].b : Row<T>::div_raw(a[c], nd[c]);
  };
  auto finish_origin = [&](auto wide_c, const Batch& x) {
    constexpr bool WIDE = decltype(wide_c)::value;
    if constexpr (MODE == kMergeOrigin) {
      bool on[2 * U];
      Raw vr[2 * U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const VLoad cl[2] = {x.vb[u], x.vm[u]};
        on[2 * u] = x.valid[u];
        on[2 * u + 1] = x.valid[u] && x.nmem[u] > 0;
        v_finish_all(wide_c, std::integral_constant<int, 2>{}, cl, on + 2 * u, vr + 2 * u);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (!x.valid[u]) continue;
        const int o = x.o[u];
        if (PAGED && !out_ok(o)) continue;
        if (x.nmem[u] == 0) {  // untouched token: bit copy of the key; its value row is one cluster
          Row<T>::store_raw(Ko + ok_off(o), x.kb[u]);
          Row<T>::store_raw(Vo + ov_off(o), vr[2 * u]);
          if (piece == 0) put_deg(o, x.du[u]);
          continue;
        }
        Acc ak[E], av[E];
#pragma unroll
        for (int e = 0; e < E; ++e) { ak[e] = 0; av[e] = 0; }
        Row<T>::template fma_into<WIDE>(ak, x.kb[u], x.du[u]);
        Row<T>::template fma_into<WIDE>(ak, x.km[u], x.dm[u]);
        Row<T>::template fma_into<WIDE>(av, vr[2 * u], x.du[u]);
        Row<T>::template fma_into<WIDE>(av, vr[2 * u + 1], x.dm[u]);
        int ndeg = x.du[u] + x.dm[u];
        for (int q = 1; q < x.nmem[u]; ++q) {
          const int ua = 2 * (int)s_members[x.first[u] + q];
          const int da = dseq ? in_deg(ua) : 1;
          const Raw kx = Row<T>::load_raw(Kin + in_off(ua));
          Row<T>::template fma_into<WIDE>(ak, kx, da);
          Row<T>::template fma_into<WIDE>(av, v_finish(wide_c, v_issue(ua)), da);
          ndeg += da;
        }
        Row<T>::store_div(Ko + ok_off(o), ak, ndeg);
        Row<T>::store_div(Vo + ov_off(o), av, ndeg);
        if (piece == 0) put_deg(o, ndeg);
      }
    }
  };
  // The loop over batches is software-pipelined (the next batch's loads are in flight while this
  // one is merged and stored) except in origin mode, whose batches are too large to hold twice.
  auto emit = [&](auto wide_c) {
    const int step = parts * NRG * U;
    int ob = part * NRG * U;
    if (ob >= n_out) return;
    if (MODE == kMergeOrigin) {
      for (; ob < n_out; ob += step) finish_origin(wide_c, fetch(ob));
      return;
    }
    Batch a = fetch(ob);
    for (;;) {
      ob += step;
      if (ob >= n_out) { finish(wide_c, a); break; }
      Batch b2 = fetch(ob);
      finish(wide_c, a);
      ob += step;
      if (ob >= n_out) { finish(wide_c, b2); break; }
      a = fetch(ob);
      finish(wide_c, b2);
    }
  };
  if (wide) emit(std::true_type{});
  else emit(std::false_type{});
}

// assign[bh][t] <- map[bh][assign[bh][t]]: four consecutive tokens per thread (one 16-byte access when
// the rows allow it), one workgroup per piece of 1024 tokens of one sequence
__global__ void compose_kernel(int32_t* __restrict__ assign, const int32_t* __restrict__ map, int seq0,
                               int map_len, int pieces, int vec) {
  const int bh = blockIdx.x / pieces, pc = blockIdx.x % pieces;
  int32_t* a = assign + (int64_t)bh * seq0;
  const int32_t* m = map + (int64_t)bh * map_len;
  const int t = (pc * (int)blockDim.x + (int)threadIdx.x) * 4;
  if (t >= seq0) return;
  if (vec && t + 4 <= seq0) {
    int4 v = *reinterpret_cast<const int4*>(a + t);
    v.x = m[v.x];
    v.y = m[v.y];
    v.z = m[v.z];
    v.w = m[v.w];
    *reinterpret_cast<int4*>(a + t) = v;
  } else {
    for (int i = t; i < min(t + 4, seq0); ++i) a[i] = m[a[i]];
  }
}

__global__ void copy_rows_kernel(const unsigned char* __restrict__ src, TensorView in,
                                 unsigned char* __restrict__ dst, TensorView out, int seq, int pieces_per_row,
                                 int elem_bytes, int64_t total) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const int piece = (int)(e % pieces_per_row);
  const int64_t row = e / pieces_per_row;
  const int t = (int)(row % seq), bh = (int)(row / seq);
  const int64_t so = (in.seq_base(bh) + (int64_t)t * in.stride_s) * elem_bytes + piece * 16;
  const int64_t dof = (out.seq_base(bh) + (int64_t)t * out.stride_s) * elem_bytes + piece * 16;
  *reinterpret_cast<uint4*>(dst + dof) = *reinterpret_cast<const uint4*>(src + so);
}

__global__ void edges_kernel(EdgeCopy ed) { copy_edges(ed, (int64_t)blockIdx.x * blockDim.x + threadIdx.x); }

// Cache update of a decode step (Algorithm 1, decoding part): the new token of every (batch, head)
// goes to row lens[b] (or `pos`) with degree 1.  A sequence already at capacity is left alone.
// One workgroup per sequence: all of its threads read lens[b], meet, write the rows of all heads, and
// one of them then advances lens[b] - no other workgroup reads or writes that entry, so the update
// needs no launch of its own.
__global__ void append_kernel(const unsigned char* __restrict__ k_new, const unsigned char* __restrict__ v_new,
                              unsigned char* __restrict__ K, unsigned char* __restrict__ V,
                              int32_t* __restrict__ deg, TensorView cache, int capacity,
                              int32_t* __restrict__ lens, int pos, int pieces_per_row, int elem_bytes) {
  const int b = blockIdx.x;
  const int t = lens ? lens[b] : pos;
  __syncthreads();
  if (t < 0 || t >= capacity) return;      // the same for every thread of the workgroup
  const int per_seq = cache.heads * pieces_per_row;
  for (int e = threadIdx.x; e < per_seq; e += blockDim.x) {
    const int piece = e % pieces_per_row, bh = b * cache.heads + e / pieces_per_row;
    const int64_t so = ((int64_t)bh * pieces_per_row + piece) * 16;
    const int64_t dof = (cache.seq_base(bh) + (int64_t)t * cache.stride_s) * elem_bytes + piece * 16;
    *reinterpret_cast<uint4*>(K + dof) = *reinterpret_cast<const uint4*>(k_new + so);
    *reinterpret_cast<uint4*>(V + dof) = *reinterpret_cast<const uint4*>(v_new + so);
    if (piece == 0 && deg) deg[(int64_t)bh * cache.deg_stride + t] = 1;
  }
  if (lens && threadIdx.x == 0) lens[b] = t + 1;
}

__global__ void fill_deg_kernel(const int32_t* __restrict__ deg_in, int64_t in_stride, int32_t* __restrict__ deg_out,
                                int64_t out_stride, int32_t* __restrict__ assign, int seq, int64_t total) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= total) return;
  const int t = (int)(e % seq);
  const int64_t bh = e / seq;
  deg_out[bh * out_stride + t] = deg_in ? deg_in[bh * in_stride + t] : 1;
  if (assign) assign[e] = t;
}

template <typename T, int D>
hipError_t launch_merge_t(const void* K, const void* V, const int32_t* deg_in, TensorView in, int n_bh,
                          int seq, int chunk, float r, const int32_t* dst_local, const float* score,
                          void* K_out, void* V_out, int32_t* deg_out, TensorView out,
                          int64_t deg_out_stride, RoundMap map, int64_t deg_in_stride, const int32_t* sel_table, int16_t* lists_out, const ValueOrigin* org,
                          hipStream_t st, PagedSide pin, PagedSide pok, PagedSide pov, const EdgeCopy* edges) {
  const int n_chunks = div_up(seq, chunk);
  const int64_t total = (int64_t)n_bh * n_chunks;
  if (total > (1 << 30)) return hipErrorInvalidValue;
  const ValueOrigin o = org ? *org : ValueOrigin{};
  // Small launches: split every chunk's rows over several workgroups, five per CU in all, none without a batch of rows
  // and no more than 32 (every one repeats the bookkeeping).  Compression of 8 sequences of dim 128 to a quarter, us, with
  // at most 8 a chunk in powers of two until there were 1024 / 1024 in all / 1280 / 1700 (256 CUs): 2048 tokens, chunk 1024: 63.4 /
  // 50.6 / 50.4 / 50.6; 5000: 66.3 / 58.0 / 56.9 / 56.8; 12000: 75.1 / 71.4 / 74.4 / 79.6; 20001: 91.1 / 91.1 / 88.1 / 100.8;
  // 32768: 114.6 / 114.8 / 113.8 / 128.5; 5000, chunk 2048: 101.0 / 79.6 / 79.6 / 82.7; 20001, chunk 384: 89.1 / 79.3 / 76.5 /
  // 86.1; one round of 30000, chunk 1024, r = 0.8: 84.5 / 74.5 / 73.2 / 85.3.
  // fp32 over pages in full mode holds 99 registers and so four per CU: with five, 8 sequences of 16384 tokens of dim 128, chunk 1024,
  // r = 0.5, one workgroup in five ran by itself at the end, 68.7 us a launch, 56.9 now (held to 96 registers, 12 bytes of scratch:
  // 58.1, and 32 such sequences at chunk 512, one workgroup a chunk, 120.5 -> 126.5).
  const bool full_f32_paged = sizeof(T) == 4 && !org && !lists_out && (pin.table || pok.table || pov.table);
  const int64_t workgroups = (full_f32_paged ? 4 : 5) * (int64_t)cu_count();
  const int row_groups = kThreads / (D * (int)sizeof(T) / 16);
  const int batches = div_up(chunk_out(min(chunk, seq), r), row_groups * (org ? kRowsInFlightOrigin : kRowsInFlight));
  const int parts = (int)max((int64_t)1, min((int64_t)min(32, batches), workgroups / total));
  // The copy of the set-aside tokens rides in the merge launch (a launch of its own costs 4 to 6 us a round),
  // unless the two together pass the 2^32 threads of a launch.
  const int64_t edge_blocks = edges ? (edges->total + kThreads - 1) / kThreads : 0;
  const bool ride = edges && (total * parts + edge_blocks) * kThreads <= UINT32_MAX;
  // any side in a block pool: the kernel variant that stages block tables (blocks of 8 tokens or more)
  const bool any_paged = pin.table || pok.table || pov.table || o.paged.table;
  if (any_paged && ((pin.table && pin.shift < 3) || (pok.table && pok.shift < 3) || (pov.table && pov.shift < 3) ||
                    (o.paged.table && o.paged.shift < 3)))
    return hipErrorInvalidValue;
  const PagedSide pout = pok.table ? pok : pov;
#define CKV_LAUNCH_MH(MODE, MH, PG, ED, edge_blocks, ...)                                                     \
  hipLaunchKernelGGL((merge_kernel<T, D, MODE, MH, PG, ED>), dim3((unsigned)(total * parts + (edge_blocks))), \
                     dim3(kThreads), 0, st,                                                                   \
                     static_cast<const T*>(K), static_cast<const T*>(V), deg_in, in, seq, chunk, n_chunks, r, \
                     dst_local, score, static_cast<T*>(K_out), static_cast<T*>(V_out), deg_out, out,          \
                     deg_out_stride, map, deg_in_stride,                                                      \
                     reinterpret_cast<const int2*>(sel_table), lists_out, o, parts, pin, pout,                \
                     pok.table != nullptr, pov.table != nullptr, EdgeBlocks<ED>{__VA_ARGS__})
  // (fp32, the small caches: one kernel for both; with two, 1024 tokens of dim 64, chunk 64, take as long: 7.27 against
  // 7.30 us a launch, for 48 kernels more)
#define CKV_LAUNCH_PG(MODE, MH, PG)                                                                          \
  do {                                                                                                       \
    if constexpr (sizeof(T) == 4)                                                                            \
      CKV_LAUNCH_MH(MODE, MH, PG, true, ride ? edge_blocks : 0, ride ? (int)edge_blocks : 0, ride ? *edges : EdgeCopy{}); \
    else if (ride) CKV_LAUNCH_MH(MODE, MH, PG, true, edge_blocks, (int)edge_blocks, *edges);                 \
    else CKV_LAUNCH_MH(MODE, MH, PG, false, 0);                                                              \
  } while (0)
  // smaller LDS arrays for chunks of up to 1024 tokens: more workgroups per CU
#define CKV_LAUNCH(MODE)                                                    \
  do {                                                                      \
    if (any_paged) {                                                        \
      if (chunk <= kMaxHalf) CKV_LAUNCH_PG(MODE, kMaxHalf / 2, true);       \
      else CKV_LAUNCH_PG(MODE, kMaxHalf, true);                             \
    } else {                                                                \
      if (chunk <= kMaxHalf) CKV_LAUNCH_PG(MODE, kMaxHalf / 2, false);      \
      else CKV_LAUNCH_PG(MODE, kMaxHalf, false);                            \
    }                                                                       \
  } while (0)
  if (org) {
    ScopedTimer t(sizeof(T) == 2 ? "merge_origin_bf16" : "merge_origin_f32", st);
    CKV_LAUNCH(kMergeOrigin);
  } else if (lists_out) {
    ScopedTimer t(sizeof(T) == 2 ? "merge_keys_bf16" : "merge_keys_f32", st);
    CKV_LAUNCH(kMergeKeys);
  } else {
    ScopedTimer t(sizeof(T) == 2 ? "merge_bf16" : "merge_f32", st);
    CKV_LAUNCH(kMergeFull);
  }
#undef CKV_LAUNCH
#undef CKV_LAUNCH_PG
#undef CKV_LAUNCH_MH
  const hipError_t err = hipGetLastError();
  return err == hipSuccess && edges && !ride ? launch_edges(*edges, st) : err;
}

}  // namespace

hipError_t launch_merge(const void* K, const void* V, const int32_t* deg_in, int dtype, int dim,
                        TensorView in, int n_bh, int seq, int chunk, float r,
                        const int32_t* dst_local, const float* score, void* K_out, void* V_out,
                        int32_t* deg_out, TensorView out, int64_t deg_out_stride, RoundMap map,
                        int64_t deg_in_stride, const int32_t* sel_table,
                        int16_t* lists_out, const ValueOrigin* org, hipStream_t st, PagedSide paged_in,
                        PagedSide paged_out_k, PagedSide paged_out_v, const EdgeCopy* edges) {
#define CKV_MERGE(T, DD)                                                                             \
  return launch_merge_t<T, DD>(K, V, deg_in, in, n_bh, seq, chunk, r, dst_local, score, K_out, V_out, \
                               deg_out, out, deg_out_stride, map, deg_in_stride, \
                               sel_table, lists_out, org, st, paged_in, paged_out_k, paged_out_v, edges)
  if (dtype == CKV_BF16) {
    if (dim == 128) CKV_MERGE(__bf16, 128);
    if (dim == 64) CKV_MERGE(__bf16, 64);
  } else {
    if (dim == 128) CKV_MERGE(float, 128);
    if (dim == 64) CKV_MERGE(float, 64);
    if (dim == 32) CKV_MERGE(float, 32);
    if (dim == 16) CKV_MERGE(float, 16);
  }
#undef CKV_MERGE
  return hipErrorInvalidValue;
}

hipError_t launch_compose(int32_t* assign, const int32_t* map, int n_bh, int seq0, int map_len,
                          hipStream_t st) {
  if (n_bh <= 0 || seq0 <= 0) return hipSuccess;
  const int vec = (seq0 % 4 == 0) && (reinterpret_cast<uintptr_t>(assign) % 16 == 0);
  ScopedTimer t("compose_assign", st);
  const int pieces = (seq0 + 1023) / 1024;
  if ((int64_t)n_bh * pieces > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(compose_kernel, dim3((unsigned)(n_bh * pieces)), dim3(256), 0, st, assign, map, seq0,
                     map_len, pieces, vec);
  return hipGetLastError();
}

hipError_t launch_copy_rows(const void* src, TensorView in, void* dst, TensorView out, int n_bh, int seq,
                            int row_bytes, int elem_bytes, hipStream_t st) {
  const int ppr = row_bytes / 16;
  const int64_t total = (int64_t)n_bh * seq * ppr;
  ScopedTimer t("copy_rows", st);
  hipLaunchKernelGGL(copy_rows_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                     static_cast<const unsigned char*>(src), in, static_cast<unsigned char*>(dst), out, seq,
                     ppr, elem_bytes, total);
  return hipGetLastError();
}

hipError_t launch_edges(const EdgeCopy& ed, hipStream_t st) {
  if (ed.total == 0) return hipSuccess;
  ScopedTimer t("edges_copy", st);
  hipLaunchKernelGGL(edges_kernel, dim3((unsigned)((ed.total + 255) / 256)), dim3(256), 0, st, ed);
  return hipGetLastError();
}

hipError_t launch_append(const void* k_new, const void* v_new, void* K, void* V, int32_t* deg, TensorView cache,
                         int batch, int capacity, int32_t* lens, int pos, int row_bytes, int elem_bytes,
                         hipStream_t st) {
  const int ppr = row_bytes / 16;
  ScopedTimer t("append", st);
  hipLaunchKernelGGL(append_kernel, dim3((unsigned)batch), dim3(256), 0, st,
                     static_cast<const unsigned char*>(k_new), static_cast<const unsigned char*>(v_new),
                     static_cast<unsigned char*>(K), static_cast<unsigned char*>(V), deg, cache, capacity, lens,
                     pos, ppr, elem_bytes);
  return hipGetLastError();
}

hipError_t launch_fill_deg(const int32_t* deg_in, int64_t in_stride, int32_t* deg_out, int64_t out_stride,
                           int32_t* assign, int n_bh, int seq, hipStream_t st) {
  const int64_t total = (int64_t)n_bh * seq;
  ScopedTimer t("fill_deg", st);
  hipLaunchKernelGGL(fill_deg_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, deg_in,
                     in_stride, deg_out, out_stride, assign, seq, total);
  return hipGetLastError();
}

}  // namespace ckv
