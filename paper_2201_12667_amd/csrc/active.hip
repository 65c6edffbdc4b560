// Active-set retrieval (paper Algorithm 1, the retrieval step of the loop body; Figure 1: the union of the
// neurons returned by every table) and the index structures the float kernels consume.
//
//  lookup_union : one workgroup per sample.  Reads one bucket per table, sets one bit per candidate
//                 and per label in an LDS bitmap over the neuron ids (deduplication and sorting
//                 are free: the bitmap is swept in id order), writes per-tile population counts
//                 (their prefix splits the sample's id list into one segment per tile of rows).
//                 It also emits the compact ascending id list per sample + the labels' slots and hands
//                 the sample its forward work items (chunks of kChunk active neurons).
#include "slide_internal.h"
#include "launch_rules.h"
#include "lookup_plan.h"
#include "spmm.h"
#include "wave_ops.h"

namespace slide {

// Counter-based random numbers of the sampling budget (Section 3.7): the 32-bit finaliser of
// MurmurHash3, a bijection, keyed by (seed, step, sample) and then by neuron or draw number.
__device__ __forceinline__ uint32_t sample_mix(uint32_t x) {
  x ^= x >> 16; x *= 0x85EBCA6Bu; x ^= x >> 13; x *= 0xC2B2AE35u; x ^= x >> 16;
  return x;
}
__device__ __forceinline__ uint32_t sample_prio(uint32_t base, uint32_t j) { return sample_mix(base + 0x9E3779B1u * (j + 1u)); }
__device__ __forceinline__ uint32_t sample_draw(uint32_t base, uint32_t d, uint32_t N) {
  return __umulhi(sample_mix((base ^ 0xA5A5A5A5u) + 0x632BE5ABu * (d + 1u)), N);
}

// Exclusive scan over a workgroup of up to 1024 threads; sm: 17 words of LDS.
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* sm, uint32_t& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const uint32_t inc = wave_incl_scan_add(v);
  __syncthreads();
  if (lane == 63) sm[wave] = inc;
  __syncthreads();
  uint32_t base = 0, tot = 0;
  for (int w = 0; w < nw; ++w) { const uint32_t x = sm[w]; if (w < wave) base += x; tot += x; }
  total = tot;
  return base + inc - v;
}

// Position of bitmap word w of sample i in the copy of the bitmaps that the row lists are built from (where a
// call builds them so): tile-major, [tile][sample][TW
// words], so that the transposition reads one contiguous block per tile; the per-sample writer
// pays the stride instead (full 4*TW-byte records).
__device__ __forceinline__ size_t act_index(const ActiveDev& ad, int i, int w) {
  const int tws = __ffs(ad.TW) - 1;
  return ((size_t)(w >> tws) * ad.B + i) * ad.TW + (w & (ad.TW - 1));
}

// A coordinate as DWTA compares it: ascending like the values, 0 for zeros and NaN, which no bin's winner can be.
// (The bits of a non-negative number that is no NaN will do as they are, where all of a vector's are.)
__device__ __forceinline__ uint32_t dwta_key(float x) {
  const uint32_t u = __float_as_uint(x);
  return x == 0.0f || x != x ? 0u : (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// The first words of the thread's hash functions, requested before the vector to hash is there: SimHash, sixteen words
// (32 coordinates) of its first function; DWTA with bins of eight, the coordinates of its first four bins.
constexpr int kHashAhead = 16;
template <int KIND>
__device__ __forceinline__ void sample_hash_request(const HashDev& hd, uint32_t (&ahead)[kHashAhead]) {
  const int tid = threadIdx.x, nthr = blockDim.x;
  if constexpr (KIND == SLIDE_HASH_SIMHASH) {
    const uint32_t* __restrict__ sw = hd.wordsT + min(tid, hd.NH - 1);
    const int half = hd.Spad / 2;
#pragma unroll
    for (int u = 0; u < kHashAhead; ++u) ahead[u] = sw[(size_t)min(u, half - 1) * hd.NH];
  } else if (hd.m == 8) {
    const uint4* __restrict__ bins = (const uint4*)hd.words;
#pragma unroll
    for (int u = 0; u < kHashAhead / 4; ++u) {
      const uint4 w = bins[min(tid + u * nthr, hd.NH - 1)];
      ahead[4 * u] = w.x; ahead[4 * u + 1] = w.y; ahead[4 * u + 2] = w.z; ahead[4 * u + 3] = w.w;
    }
  }
}

// Hash codes of one vector held in LDS, one thread per elementary hash (same arithmetic, in the
// same order, as the row-tile kernel in hash.hip); DWTA: its dwta_key bits.  raw[e]: DWTA winner position or -1, SimHash bit.
template <int KIND>
__device__ __forceinline__ void sample_hash_codes(const HashDev& hd, const uint32_t (&ahead)[kHashAhead], const float* hvec, int8_t* raw,
                                  uint32_t* codes_out) {
  const int tid = threadIdx.x, nthr = blockDim.x;
  if constexpr (KIND == SLIDE_HASH_SIMHASH) {
    // eight words (sixteen coordinates) at a time, sixteen words ahead of the sum, which is a chain
    const int half = hd.Spad / 2;
    uint32_t w[8], next[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) { w[u] = ahead[u]; next[u] = ahead[8 + u]; }
    for (int e = tid; e < hd.NH; e += nthr) {
      const uint32_t* __restrict__ sw = hd.wordsT + e;
      if (e != tid) {
#pragma unroll
        for (int u = 0; u < 8; ++u) { w[u] = sw[(size_t)min(u, half - 1) * hd.NH]; next[u] = sw[(size_t)min(8 + u, half - 1) * hd.NH]; }
      }
      float acc = 0.0f;
      for (int s0 = 0; s0 < half; s0 += 8) {
        float x[16];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const float x0 = hvec[w[u] & 0x7fffu], x1 = hvec[(w[u] >> 16) & 0x7fffu];
          x[2 * u] = (w[u] & 0x8000u) ? -x0 : x0;        // (a - x is a + (-x) bit for bit)
          x[2 * u + 1] = (w[u] & 0x80000000u) ? -x1 : x1;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) { w[u] = next[u]; next[u] = sw[(size_t)min(s0 + 16 + u, half - 1) * hd.NH]; }
#pragma unroll
        for (int u = 0; u < 16; ++u)
          if (2 * s0 + u < hd.S) acc += x[u];
      }
      raw[e] = acc > 0.0f ? 1 : 0;
    }
    __syncthreads();
    for (int t = tid; t < hd.L; t += nthr) {
      uint32_t c = 0;
      for (int k = 0; k < hd.K; ++k) c |= (uint32_t)raw[t * hd.K + k] << k;
      codes_out[t] = c;
    }
  } else {
    const int half = hd.m / 2;
    const uint32_t* key = (const uint32_t*)hvec;         // (order-preserving, 0 for an entry that does not count)
    if (hd.m == 8) {
      // a bin's coordinates in one read; the thread's first four bins have been requested already
      const uint4* __restrict__ bins = (const uint4*)hd.words;
      uint4 w[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) w[u] = make_uint4(ahead[4 * u], ahead[4 * u + 1], ahead[4 * u + 2], ahead[4 * u + 3]);
      for (int e0 = tid; e0 < hd.NH; e0 += 4 * nthr) {
        if (e0 != tid) {
#pragma unroll
          for (int u = 0; u < 4; ++u) w[u] = bins[min(e0 + u * nthr, hd.NH - 1)];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int e = e0 + u * nthr;
          if (e >= hd.NH) continue;
          const uint32_t k[8] = {key[w[u].x & 0xffffu], key[w[u].x >> 16], key[w[u].y & 0xffffu], key[w[u].y >> 16],
                                 key[w[u].z & 0xffffu], key[w[u].z >> 16], key[w[u].w & 0xffffu], key[w[u].w >> 16]};
          const uint32_t best = max(max(max(k[0], k[1]), max(k[2], k[3])), max(max(k[4], k[5]), max(k[6], k[7])));
          int pos = 7;                                   // the lowest position that holds it
#pragma unroll
          for (int q = 6; q >= 0; --q) pos = k[q] == best ? q : pos;
          raw[e] = (int8_t)(best ? pos : -1);
        }
      }
    } else {
      for (int e = tid; e < hd.NH; e += nthr) {
        int pos = -1;
        uint32_t best = 0;
        for (int p2 = 0; p2 < half; ++p2) {
          const uint32_t w = hd.words[(size_t)e * half + p2], k0 = key[w & 0xffffu], k1 = key[w >> 16];
          if (k0 > best) { best = k0; pos = 2 * p2; }
          if (k1 > best) { best = k1; pos = 2 * p2 + 1; }
        }
        raw[e] = (int8_t)pos;
      }
    }
    __syncthreads();
    for (int t = tid; t < hd.L; t += nthr) {
      uint32_t c = 0;
      for (int k = 0; k < hd.K; ++k) {
        const int e = t * hd.K + k;
        int val = raw[e];
        if (val < 0) {                                   // empty bin: borrow from the probe sequence
          val = 0;
          for (uint32_t tr = 1; tr <= 100; ++tr) {
            const uint32_t u = hd.dens_a * (uint32_t)(e + 1) + hd.dens_b * tr;
            const int r2 = raw[(u >> 8) % (uint32_t)hd.NH];
            if (r2 >= 0) { val = r2; break; }
          }
        }
        c |= (uint32_t)val << (k * hd.lgm);
      }
      codes_out[t] = c;
    }
  }
  __syncthreads();
}

// The bitmap of a sample in LDS: quads of four words, permuted within each stretch of eight quads, so that threads
// which own neighbouring stretches of 4, 8, 16 or 32 words read their k-th quads from different banks.
__device__ __forceinline__ int bitmap_quad(int q) { return q ^ ((q >> 3) & 7); }
__device__ __forceinline__ int bitmap_word(int w) { return w ^ (((w >> 5) & 7) << 2); }
__device__ __forceinline__ int popc4(const uint4& w) { return __popc(w.x) + __popc(w.y) + __popc(w.z) + __popc(w.w); }

// One workgroup per sample: hidden activations, hash codes, buckets, and the union of the buckets and labels as an
// ascending id list, by way of a bitmap in LDS (or of several in turn, for stretches of `segw` words of the ids).
// All of it is latency: three dependent reads to the hidden activations, two more to the bucket contents, barriers
// between the phases, and the instructions that each of sixteen waves spends on what is the same for all.  Hash functions and
// labels are requested before they are needed; a table's bucket is read by 2^lg neighbouring lanes, eight entries each in
// flight, with no search for who reads what; a thread then counts 2^lcw consecutive words of the bitmap, and one scan over
// the threads gives the rank of every quad of words, from which every entry finds its own place in the list.
// Nothing is stored where only the store would be waited for (a store takes a microsecond to be acknowledged, and a wait
// for an older load waits for it too wherever the compiler cannot count what lies between).
// Call with this kernel as it was / is, us: 4 samples x 670K neurons x 400 tables 35.5 / 33.4, 32 x 2,000 x 8 44.4 / 41.8,
// 512 samples x 670K x 200 tables of 2^24 216 / 207.  Threads: 512 cost the wide shape 30 us, 256 the
// 670K one 12.
// ROUNDS: the batch is larger than the machine; then two workgroups share a compute unit (64 registers a
// thread, half of the LDS each), one of them at work while the other waits, and the hidden activations come from a launch of
// their own: 1,024 samples x 254K neurons x 50 tables 89 -> 62 us.  (2,048 samples x 670K x 400 tables 205 -> 194 in two
// pieces: those wait for 1.6 M buckets scattered over 1.5 GB.)
constexpr int kLookupArgs = 412;       // bytes of the kernel's arguments

template <bool ROUNDS, bool BUDGET, int KIND>
__global__ __launch_bounds__(kLookupThreads, ROUNDS ? 8 : 4) void lookup_union_kernel(
    ActiveDev ad, HashDev hd, const float* __restrict__ h, SpmmArgs sp, const uint32_t* __restrict__ off,
    const int32_t* __restrict__ ids, uint32_t nb, uint32_t* __restrict__ codes,
    const int32_t* __restrict__ y_indptr, const int32_t* __restrict__ y_indices, int include_labels,
    int32_t* __restrict__ ncand, Ctrl* ctrl, int segw, int lg, int lcw, LongRule lr) {
  // (BUDGET: a sampling budget applies; the whole bitmap is one segment then)
  extern __shared__ uint32_t lds[];
  uint32_t* bm = lds;                    // [segw] bitmap segment
  uint32_t* o0s = bm + segw;             // [L] bucket start inside its table (first: the table codes)
  uint32_t* blen = o0s + ad.L;           // [L] bucket lengths
  uint32_t* sm = blen + ad.L;            // [20] scan scratch + counters: [17] labels, [18] bucket entries, [19] long buckets
  float* hvec = (float*)(sm + 20);       // [H] the sample's hidden activations
  uint32_t* rk = (uint32_t*)(hvec + hd.H);     // [segw >> lcw] rank of every thread's first word
  uint16_t* qrk = (uint16_t*)(rk + (segw >> lcw));   // [segw / 4] entries of that thread's before a quad of words, or, BUDGET,
  uint32_t* sel = (uint32_t*)qrk;        // [kSelWords] digit histogram + counters of the sampling budget
  int8_t* raw = BUDGET ? (int8_t*)(sel + kSelWords) : (int8_t*)(qrk + segw / 4);   // [NH] elementary hash values
  const int i = blockIdx.x, tid = threadIdx.x;
  constexpr int nthr = kLookupThreads;
  const int lane = tid & 63;
  touch_kernarg<kLookupArgs>();
  uint32_t ahead[kHashAhead];
  if (!ROUNDS) sample_hash_request<KIND>(hd, ahead);           // (ROUNDS: no registers for it; the other workgroup covers the wait)
  if (tid == 0) { sm[17] = 0; sm[18] = 0; sm[19] = 0; }
  if (i == 0 && tid == 0) {                              // consumed after this kernel
    ctrl->nlong2 = 0; ctrl->max_nu2 = 0;
    if (sp.W1) { ctrl->p1 = 0; ctrl->nlong1 = 0; ctrl->max_nu1 = 0; }
    for (int r = 0; r < kPairRegions; ++r) ctrl->p1r[r] = 0;
    for (uint32_t w = 0; w < kMaxWords; ++w) ctrl->max_nch[ad.par ^ 1][w][0] = 0;   // the previous call's: clear for the next call
  }

  // the sample's slice of the sample-major arrays: room for every candidate plus its labels
  int y0 = 0, nlab = 0;
  if (include_labels) {
    y0 = min(max(y_indptr[i], 0), ad.num_labels);
    nlab = min(max(y_indptr[i + 1], y0), ad.num_labels) - y0;
  }
  const int y_first = tid < nlab ? y_indices[y0 + tid] : -1;   // the thread's first label
  const int base_i = i * ad.PS + y0;
  const int tws = __ffs(ad.TW) - 1;                      // TW is a power of two >= 4
  auto label = [&](int q) { return q == tid ? y_first : y_indices[y0 + q]; };   // (q: of the thread's own)

  // The labels of bitmap segment [seg0, seg0 + sw) words (their "new bit" test counts the distinct
  // labels, so they go in before any candidate; under a sampling budget they go in after it).
  auto segment_labels = [&](int seg0, int sw) {
    if (BUDGET) return;
    const int64_t lo = (int64_t)seg0 * 32, hi = lo + (int64_t)sw * 32;
    for (int q = tid; q < nlab; q += nthr) {
      const int y = label(q);
      if (y < 0 || y >= ad.N) { if (seg0 == 0) atomicOr(&ctrl->status, SLIDE_FLAG_BAD_LABEL); continue; }
      if (y >= lo && y < hi) {
        const uint32_t bit = 1u << (y & 31);
        const uint32_t old = atomicOr(&bm[bitmap_word((int)(y - lo) >> 5)], bit);
        if (!(old & bit)) atomicAdd(&sm[17], 1u);       // distinct labels
      }
    }
  };
  auto clear_words = [&](int from, int to) {             // (multiples of four)
    uint32_t zero = 0;
    asm volatile("" : "+v"(zero));                       // (made here, not kept through the kernel)
    for (int q = from / 4 + tid; q < to / 4; q += nthr) ((uint4*)bm)[q] = make_uint4(zero, zero, zero, zero);
  };

  // a1 (sparse-input mode): the sample's hidden activations by the whole workgroup, their rows of W1 staged in a part
  // of the bitmap's room while the rest is cleared (non-negative and no NaN: their bits are their keys).  Dense-hidden
  // mode: the activations are read.
  const int sw0 = min(segw, ad.NWpad);
  const bool staged = !ROUNDS && sp.W1 && hd.H <= nthr && spmm_stage_rows(segw, hd.H, nthr) >= 32;
  if (staged) {
    const int stage = min(segw, 256 * (hd.H + 2) + 4) & ~3;
    clear_words(stage, sw0);
    spmm_sample_staged(sp, i, ad.B, (float*)bm, stage, hvec, ctrl, false);
    clear_words(0, min(stage, sw0));
  } else {
    clear_words(0, sw0);
    if (!ROUNDS && sp.W1) {
      const int wave = tid >> 6;
      if (wave * 128 < hd.H) spmm_sample(sp, i, ad.B, wave, lane, hvec, ctrl);
    } else {
      for (int c = tid; c < hd.H; c += nthr) {
        const float x = h[(size_t)i * hd.H + c];
        hvec[c] = KIND == SLIDE_HASH_DWTA ? __uint_as_float(dwta_key(x)) : x;
      }
    }
  }
  __syncthreads();                                       // (also orders the counters' reset before the labels)
  segment_labels(0, sw0);
  if (ROUNDS) sample_hash_request<KIND>(hd, ahead);
  // a2: hash codes of the hidden activations
  sample_hash_codes<KIND>(hd, ahead, hvec, raw, o0s);

  // Sampling budget: the bitmap holds the retrieved neurons.  The labels do not count (their bits are
  // taken out first and put back at the end); more than `budget` left: keep the `budget` of smallest
  // priority (a radix selection over the 32-bit priorities, which are distinct); fewer, with the fill
  // option: draws d = 0, 1, 2, ... accepted when new, in rounds that cannot overshoot.
  auto apply_budget = [&]() {
    uint32_t* hist = sel;                                // [256]
    uint32_t* misc = sel + 256;                          // [0] count, [1] prefix, [2] still to take, [3] new bits
    const uint32_t base = sample_mix(ad.sample_seed + 0x9E3779B9u * ad.step + 0x7F4A7C15u * (uint32_t)i);
    const int nq = ad.NWpad / 4;
    for (int q = tid; q < nlab; q += nthr) {
      const int y = y_indices[y0 + q];
      if (y >= 0 && y < ad.N) atomicAnd(&bm[bitmap_word(y >> 5)], ~(1u << (y & 31)));
    }
    if (tid == 0) { misc[0] = 0; misc[1] = 0; misc[2] = (uint32_t)ad.budget; }
    __syncthreads();
    uint32_t c = 0;
    for (int q = tid; q < nq; q += nthr) c += popc4(((const uint4*)bm)[q]);
    c = wave_sum(c);
    if (lane == 0 && c) atomicAdd(&misc[0], c);
    __syncthreads();
    const uint32_t have = misc[0];
    if (have > (uint32_t)ad.budget) {
      for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        for (int b = tid; b < 256; b += nthr) hist[b] = 0;
        __syncthreads();
        const uint32_t prefix = misc[1];
        for (int q = tid; q < nq; q += nthr) {
          const uint4 wd = ((const uint4*)bm)[bitmap_quad(q)];
          const uint32_t ww[4] = {wd.x, wd.y, wd.z, wd.w};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            uint32_t word = ww[k];
            while (word) {
              const int b = __ffs(word) - 1;
              word &= word - 1;
              const uint32_t p = sample_prio(base, (uint32_t)((4 * q + k) * 32 + b));
              const uint32_t upper = pass == 0 ? 0u : p >> ((shift + 8) & 31);   // the digits fixed so far
              if (upper == prefix) atomicAdd(&hist[(p >> shift) & 255u], 1u);
            }
          }
        }
        __syncthreads();
        if (tid < 64) {                                  // the digit that holds the misc[2]-th smallest: wave 0,
          const uint32_t h0 = hist[4 * lane], h1 = hist[4 * lane + 1], h2 = hist[4 * lane + 2], h3 = hist[4 * lane + 3];
          const uint32_t four = h0 + h1 + h2 + h3;       // four bins per lane
          const uint32_t inc = wave_incl_scan_add(four);
          const uint32_t take = misc[2];
          const unsigned long long reached = __ballot(inc >= take);
          if (reached && lane == __ffsll(reached) - 1) {
            uint32_t cum = inc - four;
            int bin = 4 * lane;
            if (cum + h0 < take) { cum += h0; ++bin;
              if (cum + h1 < take) { cum += h1; ++bin;
                if (cum + h2 < take) { cum += h2; ++bin; } } }
            misc[1] = (prefix << 8) | (uint32_t)bin;
            misc[2] = take - cum;
          }
        }
        __syncthreads();
      }
      const uint32_t last = misc[1];                     // the largest priority that stays
      for (int q = tid; q < nq; q += nthr) {
        const uint4 wd = ((const uint4*)bm)[bitmap_quad(q)];
        if (!(wd.x | wd.y | wd.z | wd.w)) continue;
        uint32_t ww[4] = {wd.x, wd.y, wd.z, wd.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          uint32_t word = ww[k];
          while (word) {
            const int b = __ffs(word) - 1;
            word &= word - 1;
            if (sample_prio(base, (uint32_t)((4 * q + k) * 32 + b)) > last) ww[k] &= ~(1u << b);
          }
        }
        ((uint4*)bm)[bitmap_quad(q)] = make_uint4(ww[0], ww[1], ww[2], ww[3]);
      }
    } else if (ad.fill && have < (uint32_t)ad.budget) {
      uint32_t need = (uint32_t)ad.budget - have, drawn = 0;
      const uint32_t dmax = 4u * (uint32_t)ad.budget + 64u;
      while (need > 0 && drawn < dmax) {                 // (uniform: both come from LDS values read after barriers)
        const uint32_t n = min(need, dmax - drawn);
        if (tid == 0) misc[3] = 0;
        __syncthreads();
        for (uint32_t d = tid; d < n; d += nthr) {
          const uint32_t j = sample_draw(base, drawn + d, (uint32_t)ad.N);
          bool is_label = false;
          for (int q = 0; q < nlab; ++q) is_label |= y_indices[y0 + q] == (int)j;
          if (!is_label) {
            const uint32_t bit = 1u << (j & 31);
            if (!(atomicOr(&bm[bitmap_word((int)(j >> 5))], bit) & bit)) atomicAdd(&misc[3], 1u);
          }
        }
        __syncthreads();
        need -= misc[3];
        drawn += n;
        __syncthreads();
      }
    }
    __syncthreads();
    for (int q = tid; q < nlab; q += nthr) {             // the labels, counted once each
      const int y = y_indices[y0 + q];
      if (y < 0 || y >= ad.N) { atomicOr(&ctrl->status, SLIDE_FLAG_BAD_LABEL); continue; }
      const uint32_t bit = 1u << (y & 31);
      if (!(atomicOr(&bm[bitmap_word(y >> 5)], bit) & bit)) atomicAdd(&sm[17], 1u);
    }
    __syncthreads();
  };

  // Buckets: 2^lg lanes to a table, in one go where the tables allow (then a lane keeps its first eight entries for
  // the passes to come).  What is beyond eight entries a lane is read by whole waves, four buckets at a time, or, where
  // that takes longer, by the tables' lanes (tables_of_wave).
  const int G = 1 << lg, tstep = nthr >> lg;
  const bool once = ad.L <= tstep;
  const int direct = kBucketAhead * G;
  int j[kBucketAhead];
  uint32_t entries = 0;                                  // (of the buckets this thread leads)
  uint32_t n = 0;                                        // active neurons in the segments so far
  for (int seg0 = 0; seg0 < ad.NWpad; seg0 += segw) {
    // (What only depends on these is worked out again for every segment: kept through the loop it would not fit the registers.)
    int me = tid, lanes = G, quads = 1 << (lcw - 2);
    asm volatile("" : "+v"(me), "+s"(lanes), "+s"(quads));
    const int sub = me & (lanes - 1), nq = quads;
    const int sw = min(segw, ad.NWpad - seg0);
    const int lo = seg0 * 32;
    const uint32_t span = (uint32_t)sw * 32u;            // (ids of the segment: id - lo < span)
    auto set_bit = [&](int id) {
      const uint32_t r = (uint32_t)id - (uint32_t)lo;    // (-1, no entry, is beyond every span: N is at most 2^30)
      if (r < span) atomicOr(&bm[bitmap_word((int)(r >> 5))], 1u << (r & 31));
    };
    if (seg0 > 0) { clear_words(0, sw); __syncthreads(); segment_labels(seg0, sw); __syncthreads(); }
    // Every entry of the buckets: f(id), -1 where a lane has none.  (again: the lane's entries, if it keeps them)
    auto for_direct = [&](bool again, auto&& f) __attribute__((always_inline)) {
      for (int t = me >> lg; t < ad.L; t += tstep) {
        uint32_t a = 0, len = 0;
        if (again && once) {
        } else if (seg0 == 0 && !again) {
          const uint32_t code = o0s[t];
          if (sub == 0) codes[(size_t)i * ad.L + t] = code;
          a = off[(size_t)t * (nb + 1) + code];
          len = min(off[(size_t)t * (nb + 1) + code + 1] - a, (uint32_t)ad.C);
          if (sub == 0) {                                // (the group's lanes sit in one wave: they have read the code)
            o0s[t] = a;
            blen[t] = len;
            entries += len;
            if ((int)len > direct) atomicAdd(&sm[19], 1u);
          }
        } else {
          a = o0s[t];
          len = blen[t];
        }
        const uint32_t first = (uint32_t)t * (uint32_t)ad.N + a + (uint32_t)sub;   // (L * N < 2^32)
        if (!(again && once)) {
#pragma unroll
          for (int u = 0; u < kBucketAhead; ++u) j[u] = -1;
#pragma unroll
          for (int u = 0; u < kBucketAhead; ++u)
            if (sub + u * lanes < (int)len) j[u] = ids[first + (uint32_t)(u * lanes)];
        }
#pragma unroll
        for (int u = 0; u < kBucketAhead; ++u) f(j[u]);
      }
    };
    // ... what of them is beyond the lanes' first: by the lanes of the table, or by whole waves, a wave the long ones of `per` tables
    auto for_rest = [&](auto&& f) __attribute__((always_inline)) {
      for (int t = me >> lg; t < ad.L; t += tstep) {
        const int most = (int)blen[t];
        const uint32_t first = (uint32_t)t * (uint32_t)ad.N + o0s[t];
        for (int at = direct + sub; at < most; at += 4 * lanes) {
          int x[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) x[u] = -1;
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (at + u * lanes < most) x[u] = ids[first + (uint32_t)(at + u * lanes)];
#pragma unroll
          for (int u = 0; u < 4; ++u) f(x[u]);
        }
      }
    };
    auto for_long = [&](int per, auto&& f) __attribute__((always_inline)) {
      for (int t0 = __builtin_amdgcn_readfirstlane(me >> 6) * per; t0 < ad.L; t0 += nthr / 64 * per) {
        unsigned long long left = __ballot(lane < per && t0 + lane < ad.L && (int)blen[min(t0 + lane, ad.L - 1)] > direct);
        while (left) {
          uint32_t from[4];
          int rest[4], most = 0;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int t = t0 + (left ? __ffsll((long long)left) - 1 : 0);
            rest[k] = left ? __builtin_amdgcn_readfirstlane((int)blen[t]) - direct : 0;
            from[k] = (uint32_t)t * (uint32_t)ad.N + (uint32_t)__builtin_amdgcn_readfirstlane((int)o0s[t]) + (uint32_t)direct;
            most = max(most, rest[k]);
            left &= left - 1;
          }
          for (int e = lane; e - lane < most; e += 128) {
            int v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = -1;
#pragma unroll
            for (int u = 0; u < 8; ++u)
              if (e + 64 * (u & 1) < rest[u >> 1]) v[u] = ids[from[u >> 1] + (uint32_t)(e + 64 * (u & 1))];
#pragma unroll
            for (int u = 0; u < 8; ++u) f(v[u]);
          }
        }
      }
    };
    // (What the kernel leaves in memory by the way is stored under these reads: a store of its own would be waited for.)
    if (staged && seg0 == 0 && tid < hd.H) sp.h[(size_t)i * hd.H + tid] = hvec[tid];
    for_direct(seg0 > 0, set_bit);
    if (seg0 == 0) {
      entries = wave_sum(entries);
      if (lane == 0 && entries) atomicAdd(&sm[18], entries);
    }
    __syncthreads();
    const int nlong = __builtin_amdgcn_readfirstlane((int)sm[19]), per = nlong == 0 ? -1 :
        tables_of_wave(lr, lg, nlong, __builtin_amdgcn_readfirstlane((int)sm[18]));
    if (per > 0) for_long(per, set_bit);
    if (per == 0) for_rest(set_bit);
    if (per >= 0) __syncthreads();
    if constexpr (BUDGET) apply_budget();

    // A thread takes 2^lcw consecutive words: their population, its exclusive prefix over the threads, and from these the
    // rank of every quad of words and of the tiles' ends.
    const int nchunk = sw >> lcw, tq = ad.TW >> 2;
    for (int c0 = 0; c0 < nchunk; c0 += nthr) {
      const int c = c0 + me;
      uint32_t cnt = 0, before[4] = {0, 0, 0, 0};        // entries before a quad, two to a word
#pragma unroll
      for (int hq = 0; hq < 2; ++hq) {
        if (4 * hq >= nq) break;
        uint4 wd[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int q = 4 * hq + k;
          wd[k] = c < nchunk && q < nq ? ((const uint4*)bm)[bitmap_quad(c * nq + q)] : make_uint4(0u, 0u, 0u, 0u);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          before[2 * hq + (k >> 1)] |= cnt << (16 * (k & 1));
          cnt += (uint32_t)popc4(wd[k]);
        }
      }
      uint32_t total;
      const uint32_t rank = n + block_excl_scan(cnt, sm, total);
      n += total;
      if (c0 + nthr >= nchunk && seg0 + segw >= ad.NWpad && tid == 0) {
        const uint32_t nch = (n + kChunk - 1) / kChunk;
        ad.cnt[i] = (int32_t)n; ad.ny[i] = (int32_t)sm[17]; ncand[i] = (int32_t)sm[18]; ad.as_base[i] = base_i;
        // forward work items of this sample: the partial results of its chunk c go to slot
        // base_i / kChunk + i + c (the samples' slices of the sample-major arrays do not overlap, so neither
        // do these), and the largest number of items of any sample bounds the forward launch's enumeration
        ad.chunk_ptr[i] = base_i / kChunk + i;
        atomicMax(&ctrl->max_nch[ad.par][i % kMaxWords][0], nch);
        ad.rankT[(size_t)ad.NT * ad.B + i] = n;          // closes the last tile's segment
      }
      if (c < nchunk) {
        rk[c] = rank;
#pragma unroll
        for (int q = 0; q < 8; q += 2) {
          if (BUDGET || q >= nq) break;
          if (nq == 1) qrk[c] = 0;
          else ((uint32_t*)qrk)[(c * nq + q) >> 1] = before[q >> 1];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {                    // rank of each tile's first active neuron
          if (q >= nq) break;
          const int quad = seg0 / 4 + c * nq + q;
          if ((quad & (tq - 1)) == 0)
            ad.rankT[(size_t)(quad >> (tws - 2)) * ad.B + i] = rank + ((before[q >> 1] >> (16 * (q & 1))) & 0xffffu);
        }
      }
    }
    __syncthreads();
    // Rank of id lo + r, which the bitmap holds.  (BUDGET: only the labels', so their threads' quads before them are counted.)
    auto rank_of = [&](uint32_t r) __attribute__((always_inline)) -> uint32_t {
      const int quad = (int)(r >> 7), b = (int)(r & 127u);
      const uint4 wd = ((const uint4*)bm)[bitmap_quad(quad)];
      const uint32_t ww[4] = {wd.x, wd.y, wd.z, wd.w};
      uint32_t at = rk[quad >> (lcw - 2)];
      if constexpr (BUDGET)
        for (int q = quad & -nq; q < quad; ++q) at += (uint32_t)popc4(((const uint4*)bm)[bitmap_quad(q)]);
      else at += qrk[quad];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int low = b - 32 * k;                      // bits of this word that come before
        at += __popc(low >= 32 ? ww[k] : low > 0 ? ww[k] & ((1u << low) - 1u) : 0u);
      }
      return at;
    };
    if (!BUDGET && (per < 0 || (per > 0 && 4 * __builtin_amdgcn_readfirstlane((int)n) < sw))) {
      // every entry puts itself in its place (those that several buckets hold more than once)
      auto place = [&](int id) __attribute__((always_inline)) {
        const uint32_t r = (uint32_t)id - (uint32_t)lo;
        if (r < span) ad.as_ids[base_i + (int)rank_of(r)] = id;
      };
      for_direct(true, place);
      if (per > 0) for_long(per, place);
    } else {
      // Drawn neurons are nowhere but in the bitmap, and what is beyond the lanes' first entries would have to be read again: every
      // thread lists what its words hold.  (Retrievals, us, long buckets read again / listed: 1,000 tables of 200 entries 356 / 227, 400
      // of 256 153 / 127, 254 of 20K neurons x 32 47.4 / 39.2.  Where none is long the lanes' entries are at hand, and listing takes longer,
      // the tiny step 42.0 / 43.0, and so it does where a few are and the bitmap is nearly empty, 4 samples of 670K neurons 32.5 / 33.0.)
      for (int c = me; c < nchunk; c += nthr) {
        int slot = base_i + (int)rk[c];
        for (int k0 = 0; k0 < nq; k0 += 4) {
          uint4 wd[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) wd[k] = k0 + k < nq ? ((const uint4*)bm)[bitmap_quad(c * nq + k0 + k)] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const uint32_t ww[4] = {wd[k].x, wd[k].y, wd[k].z, wd[k].w};
            if (!(ww[0] | ww[1] | ww[2] | ww[3])) continue;
#pragma unroll
            for (int w = 0; w < 4; ++w)
              for (uint32_t word = ww[w]; word; word &= word - 1)
                ad.as_ids[slot++] = (seg0 + 4 * (c * nq + k0 + k) + w) * 32 + __ffs(word) - 1;
          }
        }
      }
    }
    if (ad.write_act)                                    // the row lists are built from the bitmaps
      for (int q = tid; q < sw / 4; q += nthr)
        *(uint4*)&ad.act[act_index(ad, i, seg0 + 4 * q)] = ((const uint4*)bm)[bitmap_quad(q)];
    // for every label entry its slot (-1 for invalid or repeated entries): these slots are the label flags
    for (int q = tid; q < nlab; q += nthr) {
      const int y = label(q);
      if (y < 0 || y >= ad.N) { if (seg0 == 0) ad.ylist[y0 + q] = -1; continue; }
      const uint32_t r = (uint32_t)y - (uint32_t)lo;
      if (r >= span) continue;
      const int slot = base_i + (int)rank_of(r);
      bool repeated = false;
      if (nlab <= 64) {                                  // (all labels are in this wave's lanes)
        for (int k = 0; k < nlab; ++k) repeated |= __builtin_amdgcn_readlane(y_first, k) == y && k < q;
      } else {
        for (int q2 = 0; q2 < q && !repeated; ++q2) repeated = y_indices[y0 + q2] == y;
      }
      ad.as_ids[slot] = y;
      ad.ylist[y0 + q] = repeated ? -1 : slot;
    }
    __syncthreads();                                     // (before the next segment is cleared)
  }
}

static_assert(kernarg<decltype(lookup_union_kernel<false, false, SLIDE_HASH_DWTA>)>::bytes == kLookupArgs, "touch_kernarg reads them all");

hipError_t active_setup_attributes(size_t* lds_limit_out) {
  int dev = 0, lim = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  e = hipDeviceGetAttribute(&lim, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
  if (e != hipSuccess) return e;
  if (lim > 160 * 1024) lim = 160 * 1024;
  const void* kernels[] = {
      (const void*)lookup_union_kernel<false, false, SLIDE_HASH_DWTA>, (const void*)lookup_union_kernel<false, false, SLIDE_HASH_SIMHASH>,
      (const void*)lookup_union_kernel<false, true, SLIDE_HASH_DWTA>, (const void*)lookup_union_kernel<false, true, SLIDE_HASH_SIMHASH>,
      (const void*)lookup_union_kernel<true, false, SLIDE_HASH_DWTA>, (const void*)lookup_union_kernel<true, false, SLIDE_HASH_SIMHASH>};
  for (const void* k : kernels)
    if (e == hipSuccess) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, lim);
  if (e != hipSuccess) return e;
  *lds_limit_out = (size_t)lim;
  return hipSuccess;
}

hipError_t launch_lookup_union(const ActiveDev& ad, const HashDev& hd, const float* h, const SpmmArgs& sp,
                               const TablesDev& td, uint32_t* codes, const int32_t* y_indptr,
                               const int32_t* y_indices, int include_labels, int32_t* ncand, Ctrl* ctrl,
                               size_t lds_limit, int num_cus, hipStream_t s) {
  const bool budgeted = ad.budget > 0 && include_labels;
  const bool rounds = ad.B > num_cus && !sp.W1 && !budgeted;
  // (slide_init has refused configurations that leave no room for a segment worth sweeping, or, with a budget, for the bitmap)
  const LookupPlan plan = lookup_plan(ad.L, hd.H, hd.NH, ad.NWpad, budgeted, rounds, lds_limit);
  if (plan.segw == 0 || (budgeted && plan.segw < ad.NWpad)) return hipErrorInvalidValue;
  // lanes to a table
  int lg = 0;
  while (lg < 6 && (ad.L << (lg + 1)) <= kLookupThreads) ++lg;
  const bool dwta = hd.kind == SLIDE_HASH_DWTA;
  auto kernel = budgeted ? (dwta ? lookup_union_kernel<false, true, SLIDE_HASH_DWTA> : lookup_union_kernel<false, true, SLIDE_HASH_SIMHASH>)
                : rounds ? (dwta ? lookup_union_kernel<true, false, SLIDE_HASH_DWTA> : lookup_union_kernel<true, false, SLIDE_HASH_SIMHASH>)
                         : (dwta ? lookup_union_kernel<false, false, SLIDE_HASH_DWTA> : lookup_union_kernel<false, false, SLIDE_HASH_SIMHASH>);
  hipLaunchKernelGGL(kernel, dim3(ad.B), dim3(kLookupThreads), plan.bytes, s, ad, hd, h, sp, td.off, td.ids, td.nb,
                     codes, y_indptr, y_indices, include_labels, ncand, ctrl, plan.segw, lg, plan.lcw, long_rule(ad.L, ad.C, lg));
  return hipGetLastError();
}

}  // namespace slide
