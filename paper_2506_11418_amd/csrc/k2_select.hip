// Top-r over ALL chunks of a sequence: the reading of Sec. 5.2-5.3 in which the candidate edges of
// every chunk of a sequence enter one common ranking and the best fraction r of them is merged.
//
// One workgroup per (batch, head) sequence finds the cut of the ranking (score descending, position
// ascending) below its m = floor(r * edges) best edges with a 3-pass radix select over the fp32
// scores, then counts for every chunk how many of its edges lie above the cut and prefix-sums the
// chunks' output offsets.  The merge kernel then keeps, in each chunk, that many of the chunk's
// best edges under the same order, which is exactly the part of the global top-m that falls into
// the chunk.  Everything is integer work on the stored scores: the result is deterministic.
//
// What bounds it: one workgroup walks its sequence's scores four times (three passes of digits and the
// count per chunk), so the latency of its loads, not their bytes.  Every thread therefore has eight scores
// in flight, the digits are wide (11, 11 and 10 bits: one pass less than with 8), and the wanted bin is
// found by a scan over all threads.  With one load in flight, 8-bit digits, plain atomics and one thread
// walking the bins it took, against now (us a launch; sequences x tokens, chunk): 8 x 1048576, 1024:
// 1688 -> 417; 8 x 1048576, 64: 1926 -> 654; 64 x 131072, 1024: 222 -> 63; 256 x 32768, 512: 77 -> 28;
// 8 x 16384, 256: 46 -> 20; 1 x 2000, 64: 24 -> 14.
#include "ckv_internal.h"
#include "ckv_device.h"

namespace ckv {
namespace {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kSelBins = 2 * kSelThreads;   // digits of 11, 11 and 10 bits; a thread scans two bins
constexpr int kSelFlight = 8;               // scores a thread requests before it looks at the first

__device__ inline int block_scan_excl(int v, int* s_wave, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int inc = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(inc, d);
    if (lane >= d) inc += o;
  }
  if (lane == 63) s_wave[wave] = inc;
  __syncthreads();
  int base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kSelWaves; ++w) {
    const int t = s_wave[w];
    if (w < wave) base += t;
    tot += t;
  }
  __syncthreads();
  *total = tot;
  return base + inc - v;
}

// Counts one digit per lane into the histogram.  Similarities crowd into a few values of the top digit
// (sign, exponent, two bits of mantissa), and atomics of a wave on one LDS word go one after the other:
// the lanes that share the first counted lane's digit add themselves up and count as one.
__device__ inline void count_digit(int* hist, int digit, bool in, int lane) {
  const uint64_t todo = __ballot(in);
  if (todo == 0) return;
  const int leader = __ffsll((unsigned long long)todo) - 1;
  const bool same = in && digit == __shfl(digit, leader);
  const int n = __popcll(__ballot(same));
  if (lane == leader) atomicAdd(&hist[digit], n);
  if (in && !same) atomicAdd(&hist[digit], 1);
}

// table[bh * n_chunks + g] = (edges of chunk g that are merged, first output row of chunk g)
__global__ __launch_bounds__(kSelThreads) void global_select_kernel(const float* __restrict__ score, int seq,
                                                                    int chunk, int n_chunks, float r,
                                                                    int2* __restrict__ table) {
  __shared__ int s_hist[kSelBins];
  __shared__ int s_wave[kSelWaves];
  __shared__ uint32_t s_digit;
  __shared__ int s_k;

  const int bh = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_src = n_sources(seq, chunk);
  const int half = chunk >> 1;
  const int tail = seq % chunk;
  const int n_edges = n_src - (tail == 1 ? 1 : 0);      // a one-token tail chunk has no B token
  const int m = merge_count(r, n_edges);
  const float* sc = score + (int64_t)bh * n_src;
  int2* tab = table + (int64_t)bh * n_chunks;

  uint32_t cut = 0;      // key of the m-th best edge
  int quota = 0;         // edges with key == cut that are merged (the lowest positions)
  const bool all = (m >= n_edges), none = (m == 0);
  if (!all && !none) {
    uint32_t prefix = 0, known = 0;      // the digits found so far and the bits they cover
    int k = m;                           // rank wanted among the edges that share the prefix
#pragma unroll
    for (int pass = 0; pass < 3; ++pass) {
      const int bits = pass == 2 ? 10 : 11, shift = pass == 0 ? 21 : pass == 1 ? 10 : 0;
      const uint32_t digit_mask = (1u << bits) - 1u;
      for (int i = tid; i < kSelBins; i += kSelThreads) s_hist[i] = 0;
      __syncthreads();
      for (int i0 = 0; i0 < n_edges; i0 += kSelThreads * kSelFlight) {
        float x[kSelFlight];
#pragma unroll
        for (int e = 0; e < kSelFlight; ++e) x[e] = sc[min(i0 + e * kSelThreads + tid, n_edges - 1)];
#pragma unroll
        for (int e = 0; e < kSelFlight; ++e) {
          const uint32_t key = order_key(x[e]);
          const bool in = (i0 + e * kSelThreads + tid < n_edges) && (key & known) == prefix;
          count_digit(s_hist, (int)((key >> shift) & digit_mask), in, lane);
        }
      }
      __syncthreads();
      // thread t holds the bins 2047 - 2t and 2046 - 2t: the scan runs from the top digit down
      const int hi = s_hist[kSelBins - 1 - 2 * tid], lo = s_hist[kSelBins - 2 - 2 * tid];
      int total;
      const int above = block_scan_excl(hi + lo, s_wave, &total);
      if (above < k && k <= above + hi + lo) {
        const bool in_hi = k <= above + hi;
        s_digit = (uint32_t)(kSelBins - (in_hi ? 1 : 2) - 2 * tid);
        s_k = k - above - (in_hi ? 0 : hi);
      }
      __syncthreads();
      prefix |= s_digit << shift;
      known |= digit_mask << shift;
      k = s_k;
    }
    cut = prefix;
    quota = k;
  }

  // ---- per chunk: edges above the cut and edges on it -----------------------------------------
  // table is used as scratch first: (.x = above, .y = on the cut)
  if (half > 64) {       // a wave per chunk, its scores 512 at a time
    for (int g = wave; g < n_chunks; g += kSelWaves) {
      const int L = min(chunk, seq - g * chunk);
      const int nA = (L >= 2) ? (L + 1) >> 1 : 0;
      int gt = 0, eq = 0;
      if (all) gt = nA;
      else if (!none)
        for (int i0 = 0; i0 < nA; i0 += 64 * kSelFlight) {
          float x[kSelFlight];
#pragma unroll
          for (int e = 0; e < kSelFlight; ++e) x[e] = sc[g * half + min(i0 + e * 64 + lane, nA - 1)];
#pragma unroll
          for (int e = 0; e < kSelFlight; ++e) {
            const uint32_t k = order_key(x[e]);
            const bool in = i0 + e * 64 + lane < nA;
            gt += __popcll(__ballot(in && k > cut));
            eq += __popcll(__ballot(in && k == cut));
          }
        }
      if (lane == 0) tab[g] = make_int2(gt, eq);
    }
  } else if (half >= 32) {   // a wave per chunk, the scores of eight chunks at a time
    for (int g0 = wave; g0 < n_chunks; g0 += kSelWaves * kSelFlight) {
      float x[kSelFlight];
      int nA[kSelFlight];
#pragma unroll
      for (int e = 0; e < kSelFlight; ++e) {
        const int g = g0 + e * kSelWaves;
        const int L = g < n_chunks ? min(chunk, seq - g * chunk) : 0;
        nA[e] = (L >= 2) ? (L + 1) >> 1 : 0;
        x[e] = (lane < nA[e]) ? sc[g * half + lane] : 0.f;
      }
#pragma unroll
      for (int e = 0; e < kSelFlight; ++e) {
        const int g = g0 + e * kSelWaves;
        const uint32_t k = order_key(x[e]);
        const bool in = lane < nA[e] && !none;
        const int gt = all ? nA[e] : __popcll(__ballot(in && k > cut));
        const int eq = all ? 0 : __popcll(__ballot(in && k == cut));
        if (lane == 0 && g < n_chunks) tab[g] = make_int2(gt, eq);
      }
    }
  } else {               // a thread per chunk
    for (int g = tid; g < n_chunks; g += kSelThreads) {
      const int L = min(chunk, seq - g * chunk);
      const int nA = (L >= 2) ? (L + 1) >> 1 : 0;
      int gt = 0, eq = 0;
      if (all) gt = nA;
      else if (!none)
        for (int i = 0; i < nA; ++i) {
          const uint32_t k = order_key(sc[g * half + i]);
          gt += (k > cut);
          eq += (k == cut);
        }
      tab[g] = make_int2(gt, eq);
    }
  }
  __syncthreads();

  // ---- chunks in order: hand the quota of on-the-cut edges to the earliest ones, offsets ------
  int eq_before = 0, out_before = 0;
  for (int g0 = 0; g0 < n_chunks; g0 += kSelThreads) {
    const int g = g0 + tid;
    int2 c = make_int2(0, 0);
    int L = 0;
    if (g < n_chunks) { c = tab[g]; L = min(chunk, seq - g * chunk); }
    int tot_eq, tot_out;
    const int eq_excl = eq_before + block_scan_excl(c.y, s_wave, &tot_eq);
    const int take = max(0, min(c.y, quota - eq_excl));
    const int kept = c.x + take;
    const int out_excl = out_before + block_scan_excl(L - kept, s_wave, &tot_out);
    if (g < n_chunks) tab[g] = make_int2(kept, out_excl);
    eq_before += tot_eq;
    out_before += tot_out;
  }
}

}  // namespace

hipError_t launch_global_select(const float* score, int n_bh, int seq, int chunk, float r, int32_t* table,
                                hipStream_t st) {
  ScopedTimer t("global_select", st);
  hipLaunchKernelGGL(global_select_kernel, dim3(n_bh), dim3(kSelThreads), 0, st, score, seq, chunk,
                     div_up(seq, chunk), r, reinterpret_cast<int2*>(table));
  return hipGetLastError();
}

}  // namespace ckv
