// The k best of a long list by one workgroup, as a device function for the prediction kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace slide {

constexpr int kSelectThreads = 256;      // threads of a selecting workgroup
constexpr int kSelectGather = 1024;      // entries at or above the bar that fit its LDS

struct SelectLds {
  alignas(16) uint64_t keys[kSelectGather];
  uint64_t last;
  int cnt;
};

// Sort key of (score, id): ascending keys = descending scores, ties to the lower id.  ~0 = no entry.
__device__ __forceinline__ uint32_t score_bits(float score) {         // orders like the float
  const uint32_t u = __float_as_uint(score);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ uint64_t topk_key(float score, uint32_t id) { return ((uint64_t)(~score_bits(score)) << 32) | id; }
__device__ __forceinline__ float topk_score(uint64_t key) {
  const uint32_t asc = ~(uint32_t)(key >> 32);
  return __uint_as_float((asc & 0x80000000u) ? (asc & 0x7fffffffu) : ~asc);
}

// The `topk` (<= 64) smallest keys of a list, in order: emit(place, key) for every place below the
// returned count, each by one thread.  sweep(f) calls f(key) for the calling thread's share of the list
// (keys distinct, ~0 = no entry) and gives the same keys every time.  The list is read twice: first every
// thread keeps the best of its (interleaved) share, and the topk-th best of these 256 is a bar that at
// least topk entries reach; then the entries that reach it -- topk and a few more -- are gathered in LDS
// and each finds its place by counting the better ones.  When one gather cannot hold them (the best
// entries all sit in a few threads' shares) the best entry is handed out and the search repeated.
// Bound by the latency of the two sweeps and a handful of barriers (one pass over the list per entry, which
// this replaced, took 22.7 us for the best 10 of 1,300 retrieved neurons and 200 us for 32 of 6,400; now 7.3
// and 15.8).  A single best entry needs neither bar nor gather: one sweep and a reduction.
// Every thread of the workgroup (kSelectThreads) calls.
template <typename Sweep, typename Emit>
__device__ __forceinline__ int select_topk(SelectLds& s, int topk, Sweep&& sweep, Emit&& emit) {
  const int tid = threadIdx.x;
  if (topk == 1) {
    uint64_t best = ~0ull;
    sweep([&](uint64_t k) { best = k < best ? k : best; });
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
      const uint64_t other = __shfl_xor((unsigned long long)best, d);
      best = other < best ? other : best;
    }
    if ((tid & 63) == 0) s.keys[tid >> 6] = best;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSelectThreads / 64; ++w) best = s.keys[w] < best ? s.keys[w] : best;
    if (best == ~0ull) return 0;
    if (tid == 0) emit(0, best);
    return 1;
  }
  uint64_t done = 0;                                     // keys up to here have been handed out
  int out = 0;
  while (out < topk) {
    const int want = topk - out;
    uint64_t best = ~0ull;
    sweep([&](uint64_t k) { if ((out == 0 || k > done) && k < best) best = k; });
    __syncthreads();                                     // (the last round's keys are no longer read)
    s.keys[tid] = best;
    if (tid == 0) { s.last = ~0ull - 1; s.cnt = 0; }
    __syncthreads();
    int rank = 0;
    const ulonglong2* pairs = (const ulonglong2*)s.keys;
#pragma unroll 8
    for (int q = 0; q < kSelectThreads / 2; ++q) {
      const ulonglong2 two = pairs[q];
      rank += (two.x < best ? 1 : 0) + (two.y < best ? 1 : 0);
    }
    if (best != ~0ull && rank == want - 1) s.last = best;  // (fewer than `want` threads with an entry: no bar)
    __syncthreads();
    const uint64_t bar = s.last;
    sweep([&](uint64_t k) {
      if ((out == 0 || k > done) && k <= bar) {
        const int c = atomicAdd(&s.cnt, 1);
        if (c < kSelectGather) s.keys[c] = k;
      }
    });
    __syncthreads();
    const bool whole = s.cnt <= kSelectGather;           // everything that reaches the bar is in the LDS
    int c = s.cnt, sure = min(want, c);
    if (!whole) {
      __syncthreads();
      s.keys[tid] = best;                                // the threads' bests: the best of all is among them
      c = kSelectThreads;
      sure = 1;
      __syncthreads();
    }
    for (int e = tid; e < c; e += kSelectThreads) {
      const uint64_t k = s.keys[e];
      int place = 0;
      for (int q = 0; q < c; ++q) place += s.keys[q] < k ? 1 : 0;
      if (k != ~0ull && place < sure) {
        emit(out + place, k);
        if (place == sure - 1) s.last = k;
      }
    }
    __syncthreads();
    out += sure;
    done = s.last;
    if (whole) break;
  }
  return out;
}

}  // namespace slide
