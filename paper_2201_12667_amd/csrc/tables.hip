// Hash-table build / rebuild (paper Algorithm 1, the table-construction step before the loop, rebuilt on a
// schedule, Section 3.1).  Layout: per table a CSR over the 2^bits codes -- off[t][code] is the
// start of the bucket inside ids[t][0..N).  A bucket's first min(size, C) ids are its kept members,
// ascending by id; which members are kept when size > C is decided by the smallest
// (priority, id) keys.
//
// The build is a two-level counting sort with every counter in LDS (no global atomics on the tables) that keeps
// the order of the rows, so that nothing has to be sorted: (1) hash every row of W2, codes stored table-major;
// (2) every slab of up to 32,768 rows of a table is grouped by the high bits of the code in LDS and written back in
// place, with the run boundaries per (slab, digit); (3) one workgroup per (table, partition) gathers the partition's
// runs from the slabs, counts the low bits in LDS, writes that partition's offsets, places the ids and chooses the
// survivors of over-capacity buckets.  Partitions too large for its staging area are left to larger workgroups.
#include "slide_internal.h"
#include "wave_ops.h"

#include <algorithm>

namespace slide {

__global__ void fill_u32_kernel(uint32_t* p, size_t n, uint32_t v) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t step = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += step) p[i] = v;
}

// Plain streaming copy: the yardstick the HBM counters and the achievable bandwidth are calibrated
// against.  Of the plain forms tried (grid-stride with one, four or eight 16-byte words per thread in
// flight, cached or streaming accesses, 2 K to 256 K workgroups) this one -- four words per thread in
// flight, loads and stores past the caches -- is the fastest on a 1 GiB buffer (6.3 TB/s against
// 5.4 for the one-word cached loop).
typedef float copy_v4f __attribute__((ext_vector_type(4)));
constexpr size_t kCopyChunk = 1024;       // 16-byte words a workgroup of 256 moves per step
__global__ __launch_bounds__(256) void copy_kernel(copy_v4f* __restrict__ dst, const copy_v4f* __restrict__ src, size_t n16) {
  size_t base = (size_t)blockIdx.x * kCopyChunk;
  const size_t step = (size_t)gridDim.x * kCopyChunk;
  for (; base + kCopyChunk <= n16; base += step) {
    copy_v4f v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = __builtin_nontemporal_load(src + base + (size_t)u * 256 + threadIdx.x);
#pragma unroll
    for (int u = 0; u < 4; ++u) __builtin_nontemporal_store(v[u], dst + base + (size_t)u * 256 + threadIdx.x);
  }
  // (the last, partial chunk: only the workgroup whose turn it would have been gets here with base < n16)
  for (size_t i = base + threadIdx.x; i < n16; i += 256) dst[i] = src[i];
}

hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
  const size_t n16 = bytes / 16;
  if (n16 == 0) return hipSuccess;
  size_t blocks = (n16 + kCopyChunk - 1) / kCopyChunk;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(copy_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (copy_v4f*)dst, (const copy_v4f*)src, n16);
  return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, size_t n, uint32_t v, hipStream_t s) {
  if (n == 0) return hipSuccess;
  size_t blocks = (n + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

constexpr int kRowBits = 15;             // an entry is (low digit of the code << kRowBits) | row inside its slab

// Exclusive scan over a workgroup of 1024 threads; sm: 17 words of LDS.
__device__ uint32_t block_excl_scan1024(uint32_t v, uint32_t* sm, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t inc = wave_incl_scan_add(v);
  __syncthreads();
  if (lane == 63) sm[wave] = inc;
  __syncthreads();
  uint32_t base = 0, tot = 0;
  for (int w = 0; w < 16; ++w) { const uint32_t x = sm[w]; if (w < wave) base += x; tot += x; }
  *total = tot;
  return base + inc - v;
}

// One workgroup per (slab, table): the slab's rows grouped by the high digit of their code, in place
// -- the grouped entries of slab s stay in entries[t][s*slab_rows ..), so no table-wide histogram has to
// exist before this pass.  The rows of a digit stay in ascending order: a wave takes consecutive rows and
// has counters of its own (two waves to a word, 16 bits each), so that only the order in which the lanes
// of one instruction are served by an LDS word is left to the hardware (lane order: part_buckets_kernel
// checks what it gets and sorts where it does not hold).
// runs[t][s][d] = first entry of digit d inside the slab's stretch, runs[t][s][nbins] = rows of the slab.
// The grouping happens in LDS and the slab is written out as one coalesced stretch.
// RPT rows a thread: as many as leave room for the counters of nbins digits (slab_rpt).
template <int RPT>
__global__ __launch_bounds__(1024) void slab_group_kernel(const uint32_t* __restrict__ codes_t, int64_t N, int lb,
                                                          int nbins, uint32_t* __restrict__ runs, int nslab,
                                                          uint32_t* __restrict__ entries) {
  extern __shared__ uint32_t lds[];
  constexpr int kRows = RPT * 1024;
  uint32_t* stage = lds;                           // [kRows] entries grouped by digit
  uint32_t* cur = lds + kRows;                     // [8][nbins] counters, then cursors, of waves 2i (low half) and 2i + 1
  uint32_t* sm = cur + 8 * nbins;                  // [20]
  const int slab = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const size_t t = blockIdx.y;
  for (int b = tid; b < 8 * nbins; b += 1024) cur[b] = 0;
  __syncthreads();
  const int64_t j0 = (int64_t)slab * kRows;
  const int nvalid = (int)(N - j0 < kRows ? N - j0 : kRows);
  const int r0 = wave * (RPT * 64) + lane;
  uint32_t* mine = cur + (wave >> 1) * nbins;
  const uint32_t shift = 16u * (uint32_t)(wave & 1);
  uint32_t code[RPT];
  const uint32_t* own = codes_t + t * N + j0 + r0;
  // (only a table's last slab is not full: a test per row costs more than what it guards)
  const bool full = nvalid == kRows;
  if (full) {
#pragma unroll
    for (int k = 0; k < RPT; ++k) code[k] = own[k * 64];
#pragma unroll
    for (int k = 0; k < RPT; ++k) atomicAdd(&mine[code[k] >> lb], 1u << shift);
  } else {
#pragma unroll
    for (int k = 0; k < RPT; ++k) code[k] = r0 + k * 64 < nvalid ? own[k * 64] : 0u;
#pragma unroll
    for (int k = 0; k < RPT; ++k)
      if (r0 + k * 64 < nvalid) atomicAdd(&mine[code[k] >> lb], 1u << shift);
  }
  __syncthreads();
  uint32_t* rrow = runs + (t * nslab + slab) * (size_t)(nbins + 1);
  uint32_t carry = 0;
  for (int base = 0; base < nbins; base += 1024) {
    const int b = base + tid;
    uint32_t w[8], v = 0;
    if (b < nbins)
#pragma unroll
      for (int i = 0; i < 8; ++i) { w[i] = cur[i * nbins + b]; v += (w[i] & 0xffffu) + (w[i] >> 16); }
    uint32_t total;
    const uint32_t ex = block_excl_scan1024(v, sm, &total);
    if (b < nbins) {
      uint32_t at = carry + ex;
      rrow[b] = at;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t lo = w[i] & 0xffffu;
        cur[i * nbins + b] = at | (at + lo) << 16;
        at += lo + (w[i] >> 16);
      }
    }
    carry += total;
  }
  if (tid == 0) rrow[nbins] = (uint32_t)nvalid;
  __syncthreads();
  const uint32_t lowmask = (1u << lb) - 1u;
  auto put = [&](int k) {
    const uint32_t at = atomicAdd(&mine[code[k] >> lb], 1u << shift) >> shift & 0xffffu;
    stage[at] = ((code[k] & lowmask) << kRowBits) | (uint32_t)(r0 + k * 64);
  };
  if (full) {
#pragma unroll
    for (int k = 0; k < RPT; ++k) put(k);
  } else {
#pragma unroll
    for (int k = 0; k < RPT; ++k)
      if (r0 + k * 64 < nvalid) put(k);
  }
  __syncthreads();
  struct __attribute__((packed, aligned(4))) Words4 { uint32_t w[4]; };   // (in memory: word-aligned only)
  uint32_t* out = entries + t * N + j0;
  for (int k = 4 * tid; k < nvalid; k += 4096) {
    const uint4 q = *(const uint4*)(stage + k);
    if (k + 4 <= nvalid) *reinterpret_cast<Words4*>(out + k) = Words4{{q.x, q.y, q.z, q.w}};
    else
      for (int i = k; i < nvalid; ++i) out[i] = stage[i];
  }
}

__device__ __forceinline__ uint32_t overflow_prio(uint32_t j, uint32_t t, uint32_t r, uint32_t pa, uint32_t pb) {
  uint32_t u = pa * (j + 1u) + pb * (t * 65537u + r + 1u);
  u ^= u >> 15; u *= pa; u ^= u >> 13;
  return u;
}

constexpr int kStageIds = 4096;    // most ids of a partition staged in LDS by the bucket kernel (larger ones: its large form)
constexpr int kStageMin = 1024;    // the staging area is four mean partitions, within these two
constexpr int kLargeThreads = 1024;
constexpr int kMaxSlabs = 512;     // slabs of a layer whose partitions are staged (entry numbers of 24 bits)
constexpr int kPiece = 16;         // entries of a run a row of lanes takes at a time
constexpr int kBatch = 8;          // steps of four pieces a wave keeps in flight

__device__ __forceinline__ uint32_t lanes_before(uint64_t m) {   // set bits of m below the lane's
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// The C of the n members ids[0 .. n), ascending, with the smallest (priority, id) keys, ascending, to out: by a wave
// (WAVES = 1) or, each wave with a stretch of the members, by the workgroup (sums: 4 + 2 * WAVES words, the first two
// zero and zero again afterwards).  The C-th smallest priority is searched for between bounds: twice where evenly
// spread priorities would have it, then in the middle (the search ends when exactly C members are at or below a
// bound, nearly always after three to five looks).
template <int WAVES, int REGS = 0>
__device__ __forceinline__ void keep_smallest(const int32_t* ids, const uint32_t n, const uint32_t C, int32_t* out,
                                              uint32_t t, uint32_t r, uint32_t pa, uint32_t pb, uint32_t* sums) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wave = WAVES == 1 ? 0u : (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t per = WAVES == 1 ? n : ((n + 63u) / 64u + WAVES - 1u) / WAVES * 64u;   // members of a wave
  const uint32_t i0 = min(wave * per, n), m = min(per, n - i0);
  const bool held = per <= 64u * REGS;             // (the priorities in registers)
  const int32_t* own = ids + i0;
  auto prio = [&](uint32_t i) { return i < m ? overflow_prio((uint32_t)own[i], t, r, pa, pb) : ~0u; };
  uint32_t u[REGS > 0 ? REGS : 1];
  if (held)
#pragma unroll
    for (int k = 0; k < REGS; ++k) u[k] = k * 64u < m ? prio(k * 64u + lane) : ~0u;
  auto count_own = [&](uint32_t limit) {           // members of the wave at or below limit < 2^32 - 1
    uint32_t c = 0;
    if (held) {
#pragma unroll
      for (int k = 0; k < REGS; ++k)
        if (k * 64u < m) c += (uint32_t)__popcll(__ballot(u[k] <= limit));
    } else {
      for (uint32_t k = 0; k < m; k += 64) c += (uint32_t)__popcll(__ballot(prio(k + lane) <= limit));
    }
    return c;
  };
  auto count = [&](uint32_t limit, int look) {
    uint32_t c = count_own(limit);
    if (WAVES > 1) {                               // (three words in turn: the one after next is cleared behind the barrier)
      if (lane == 0) atomicAdd(&sums[look % 3], c);
      __syncthreads();
      c = (uint32_t)__builtin_amdgcn_readfirstlane((int)sums[look % 3]);
      if (threadIdx.x == 0) sums[(look + 2) % 3] = 0;
    }
    return c;
  };
  uint32_t lo = 0, hi = ~0u, below = 0, upto = n, ties = 0;   // members below lo, up to hi; the answer is between them
  for (int look = 0;; ++look) {
    if (lo == hi) { ties = C - below; break; }     // several members share the C-th priority: the lowest ids
    const float even = (float)(hi - lo) * ((float)(C - below) / (float)(upto - below));
    const uint32_t step = look % 3 == 2 ? (hi - lo) / 2u : min((uint32_t)fminf(even, 4294967040.f), hi - lo - 1u);
    const uint32_t mid = lo + step, c = count(mid, look);
    if (c == C) { lo = mid; ties = n; break; }
    if (c > C) { hi = mid; upto = c; }
    else { lo = mid + 1u; below = c; }
  }
  uint32_t at = 0, tied = 0;
  auto each = [&](auto&& f) {
    if (held) {
#pragma unroll
      for (int k = 0; k < REGS; ++k)
        if (k * 64u < m) f(k * 64u + lane, u[k]);
    } else {
      for (uint32_t k = 0; k < m; k += 64) f(k + lane, prio(k + lane));
    }
  };
  if (WAVES > 1) {                                 // what the waves before this one keep
    uint32_t under = 0, equal = 0;
    each([&](uint32_t i, uint32_t p) {
      under += (uint32_t)__popcll(__ballot(i < m && p < lo));
      equal += (uint32_t)__popcll(__ballot(i < m && p == lo));
    });
    if (lane == 0) { sums[4 + 2 * wave] = under; sums[5 + 2 * wave] = equal; }
    __syncthreads();
    if (threadIdx.x < 3) sums[threadIdx.x] = 0;
    for (uint32_t w = 0; w < wave; ++w) { at += sums[4 + 2 * w]; tied += sums[5 + 2 * w]; }
    at += min(tied, ties);
    __syncthreads();
  }
  each([&](uint32_t i, uint32_t p) {
    const uint64_t eq = __ballot(i < m && p == lo);
    const bool keep = i < m && (p < lo || (p == lo && tied + lanes_before(eq) < ties));
    const uint64_t kept = __ballot(keep);
    if (keep) out[at + lanes_before(kept)] = own[i];
    at += (uint32_t)__popcll(kept);
    tied += (uint32_t)__popcll(eq);
  });
}

// Over-capacity buckets of a partition, added to one of many words (one that every workgroup bumps serves an update per
// 8 ns or so: 100 us for the 12,800 partitions of 325K neurons in 50 tables).
__device__ __forceinline__ void count_over(Ctrl* c, uint32_t m, uint32_t n) { atomicAdd(&c->overflowed[m % kOverWords][0], n); }

struct PartArgs {
  const uint32_t* entries;
  const uint32_t* runs;
  uint32_t* large;                 // [2][L * nbins] partitions left to the large form, and those that it leaves in turn
  uint32_t* off;
  int32_t* ids;
  Ctrl* ctrl;
  int64_t N;
  uint32_t nb, r, pa, pb;
  int nslab, slab_rows, nbins, hb, lb, C, policy;
  int stage, slot_cap;             // ids of a partition that fit the staging area, pieces that fit their table
  int cut_bits;                    // lanes that cut a slab's run into pieces (log2)
  int nxcd, per_xcd, total;        // partitions per die (rounded up), partitions in all
};

static __host__ __device__ constexpr int part_misc(int threads) { return 8 + 4 + 2 * (threads / 64); }

constexpr int kSelStage = 4096;    // members of an over-capacity bucket staged in LDS while its survivors are chosen

template <int THREADS>
__device__ void bitonic_sort_u64(uint64_t* keys, int n) {
  for (int k = 2; k <= n; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = threadIdx.x; i < n / 2; i += THREADS) {
        const int a = 2 * j * (i / j) + (i % j), b = a + j;
        const bool up = (a & k) == 0;
        const uint64_t x = keys[a], y = keys[b];
        if ((x > y) == up) { keys[a] = y; keys[b] = x; }
      }
      __syncthreads();
    }
}

// The workgroup puts the s members p[0 .. s) of a bucket of table t, in any order, into the order of a bucket.
// s <= C: sort by id.  s > C: the survivors are the C members with the smallest (priority, id) keys.  The C-th
// smallest key is found digit by digit from the top (a 256-bin histogram of the candidates' next eight bits, a scan,
// the bin that holds rank C; the search ends as soon as the bins up to the chosen one hold exactly the wanted number,
// which with hashed priorities happens after two or three digits); then the members at or below it are gathered and
// put in id order.
template <int THREADS>
__device__ void finish_bucket(const PartArgs& g, uint32_t* lds, int32_t* p, const uint32_t s, const uint32_t t) {
  uint64_t* keys = (uint64_t*)lds;             // [kSortCap]
  uint32_t* sid = lds + 2 * kSortCap;          // [kSelStage]
  uint32_t* hist = sid + kSelStage;            // [256]
  uint32_t* pick = hist + 256;                 // chosen digit, rank left inside it, 1 when the search is over, survivors gathered
  const int tid = threadIdx.x, lane = tid & 63, C = g.C;
  int capp = 1;
  while (capp < C) capp <<= 1;
  if (s <= (uint32_t)C) {
    int n2 = 2;
    while ((uint32_t)n2 < s) n2 <<= 1;
    for (int i = tid; i < n2; i += THREADS) keys[i] = (uint32_t)i < s ? (uint64_t)(uint32_t)p[i] : ~0ull;
    __syncthreads();
    bitonic_sort_u64<THREADS>(keys, n2);
    for (uint32_t i = tid; i < s; i += THREADS) p[i] = (int32_t)(uint32_t)keys[i];
  } else {
    const bool in_lds = s <= (uint32_t)kSelStage;
    if (in_lds) for (uint32_t i = tid; i < s; i += THREADS) sid[i] = (uint32_t)p[i];
    if (tid < 256) hist[tid] = 0;
    if (tid == 0) pick[3] = 0;
    __syncthreads();
    auto member = [&](uint32_t i) { return in_lds ? sid[i] : (uint32_t)p[i]; };
    auto key_of = [&](uint32_t j) {
      const uint32_t pr = g.policy == SLIDE_KEEP_LOWEST_ID ? 0u : overflow_prio(j, t, g.r, g.pa, g.pb);
      return ((uint64_t)pr << 32) | j;
    };
    uint64_t prefix = 0;                      // the digits chosen so far, in place
    uint32_t want = (uint32_t)C;              // rank of the wanted key among the candidates (1-based)
    int shift = g.policy == SLIDE_KEEP_LOWEST_ID ? 24 : 56;   // (without priorities the upper half of every key is zero)
    for (;; shift -= 8) {
      // candidates: the members whose digits above this one equal the chosen ones
      for (uint32_t i = tid; i < s; i += THREADS) {
        const uint64_t k = key_of(member(i));
        if (shift == 56 || (k >> (shift + 8)) == (prefix >> (shift + 8))) atomicAdd(&hist[(uint32_t)(k >> shift) & 255u], 1u);
      }
      __syncthreads();
      if (tid < 64) {                         // lane l: bins 4l .. 4l + 3
        const uint32_t c0 = hist[4 * lane], c1 = hist[4 * lane + 1], c2 = hist[4 * lane + 2], c3 = hist[4 * lane + 3];
        hist[4 * lane] = 0; hist[4 * lane + 1] = 0; hist[4 * lane + 2] = 0; hist[4 * lane + 3] = 0;
        const uint32_t tot = c0 + c1 + c2 + c3, incl = wave_incl_scan_add(tot), excl = incl - tot;
        if (excl < want && want <= incl) {    // (one lane: the candidates number at least `want`)
          uint32_t before = excl, digit = 4u * (uint32_t)lane, in_bin = c0;
          if (before + in_bin < want) { before += in_bin; ++digit; in_bin = c1; }
          if (before + in_bin < want) { before += in_bin; ++digit; in_bin = c2; }
          if (before + in_bin < want) { before += in_bin; ++digit; in_bin = c3; }
          pick[0] = digit;
          pick[1] = want - before;
          pick[2] = (before + in_bin == want || shift == 0) ? 1u : 0u;
        }
      }
      __syncthreads();
      prefix |= (uint64_t)pick[0] << shift;
      want = pick[1];
      const bool found = pick[2] != 0u;
      if (found || shift == 0) break;         // (uniform; at shift 0 a bin holds one key, so the search ends there at the latest)
    }
    // every key up to the chosen digit with all lower digits set survives: exactly C of them
    const uint64_t limit = prefix | (shift ? ((uint64_t)1 << shift) - 1u : 0u);
    uint32_t* surv = reinterpret_cast<uint32_t*>(keys);
    for (uint32_t i = tid; i < s; i += THREADS) {
      const uint32_t j = member(i);
      if (key_of(j) <= limit) {
        const uint32_t slot = atomicAdd(&pick[3], 1u);
        if (slot < (uint32_t)C) surv[slot] = j;
      }
    }
    __syncthreads();
    uint64_t mine[(1024 + THREADS - 1) / THREADS];            // capp <= 1024
#pragma unroll
    for (int q = 0; q < (1024 + THREADS - 1) / THREADS; ++q) mine[q] = tid + q * THREADS < C ? (uint64_t)surv[tid + q * THREADS] : ~0ull;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < (1024 + THREADS - 1) / THREADS; ++q)
      if (tid + q * THREADS < capp) keys[tid + q * THREADS] = mine[q];
    __syncthreads();
    bitonic_sort_u64<THREADS>(keys, capp);
    for (int i = tid; i < C; i += THREADS) p[i] = (int32_t)(uint32_t)keys[i];
  }
  __syncthreads();
}

// Partitions of more ids than places of 16 bits count.  Grouped in the table itself, in arrival order, with one set of counters;
// then the buckets are put in order one by one, up to 64 ids by a wave.  A single over-capacity bucket (tables of few
// codes) is not grouped at all: of its n members, in order of the rows, the few hundred whose priorities are low
// enough to be among the C smallest are gathered, and chosen from.
constexpr int kTableIds = 65535;   // most ids of a partition grouped in the table itself (places of 16 bits)
constexpr int kBitWords = (kTableIds + 32) / 32;
constexpr int kRoomWords = 16384;  // LDS beside the counters: finish_bucket, or the gathered members

template <int WAVES>
__device__ __forceinline__ void unstaged_partition(const PartArgs& g, uint32_t* lds, uint32_t m) {
  constexpr int THREADS = WAVES * 64;
  const int nlo = 1 << g.lb, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t C = (uint32_t)g.C, t = m >> g.hb, d = m & ((uint32_t)g.nbins - 1u);
  uint32_t *room = lds, *csum = room + kRoomWords, *sums = csum + 64 /* [4 + 2 * WAVES] */, *misc = sums + 4 + 2 * WAVES;
  uint32_t* cnt = misc + 4;                        // [nlo]; misc: ids, first place, over capacity
  const uint32_t* tent = g.entries + (size_t)t * g.N;
  const uint32_t* truns = g.runs + (size_t)t * (size_t)g.nslab * (size_t)(g.nbins + 1) + d;
  auto run = [&](int q, uint32_t& a, uint32_t& len) {
    const uint32_t* p = truns + (size_t)q * (size_t)(g.nbins + 1);
    a = p[0];
    len = p[1] - a;
  };
  if (wave == 0) {
    uint32_t n = 0, s0 = 0;
    for (int q0 = 0; q0 < g.nslab; q0 += 64) {
      uint32_t a = 0, len = 0;
      if (q0 + lane < g.nslab) run(q0 + lane, a, len);
      n += wave_sum(len);
      s0 += wave_sum(a);
    }
    if (lane == 0) { misc[0] = n; misc[1] = s0; misc[2] = 0; }
    if (lane < 4) sums[lane] = 0;
  }
  for (int b = tid; b < nlo; b += THREADS) cnt[b] = 0;
  __syncthreads();
  const uint32_t n = __builtin_amdgcn_readfirstlane(misc[0]), s0 = __builtin_amdgcn_readfirstlane(misc[1]);
  int32_t* seg = g.ids + (size_t)t * g.N + s0;
  uint32_t* orow = g.off + (size_t)t * ((size_t)g.nb + 1) + ((size_t)d << g.lb);
  constexpr uint32_t kRowMask = (1u << kRowBits) - 1u;
  if (nlo == 1 && n > C && g.policy != SLIDE_KEEP_LOWEST_ID && g.nslab * WAVES + 1 <= kRoomWords / 2) {
    const float share = ((float)C + 8.f * sqrtf((float)C) + 32.f) / (float)n;
    const uint32_t limit = share < 1.f ? (uint32_t)fminf(share * 4294967296.f, 4294967040.f) : ~0u;
    uint32_t* counts = room;                       // [nslab][WAVES], then where they begin; then the gathered ids
    int32_t* few = (int32_t*)(room + g.nslab * WAVES + 1);
    const uint32_t cap = (uint32_t)(kRoomWords - g.nslab * WAVES - 1);
    auto each = [&](auto&& f) {                    // f(first place's index, rows' base, entries of the wave)
      for (int q = 0; q < g.nslab; ++q) {
        uint32_t a, len;
        run(q, a, len);
        const uint32_t share_len = ((len + 63u) / 64u + WAVES - 1u) / WAVES * 64u, e0 = min(wave * share_len, len), e1 = min(e0 + share_len, len);
        const uint32_t rowbase = (uint32_t)q * (uint32_t)g.slab_rows;
        f(q * WAVES + wave, rowbase, rowbase + a + e0, rowbase + a + e1);
      }
    };
    each([&](int at, uint32_t rowbase, uint32_t e0, uint32_t e1) {
      uint32_t c = 0;
      for (uint32_t e = e0; e < e1; e += 64)
        c += (uint32_t)__popcll(__ballot(e + lane < e1 && overflow_prio(rowbase + (tent[min(e + lane, e1 - 1u)] & kRowMask), t, g.r, g.pa, g.pb) <= limit));
      if (lane == 0) counts[at] = c;
    });
    __syncthreads();
    if (wave == 0) {
      uint32_t carry = 0;
      for (int c = 0; c < g.nslab * WAVES; c += 64) {
        const uint32_t v = c + lane < g.nslab * WAVES ? counts[c + lane] : 0u, inc = wave_incl_scan_add(v);
        if (c + lane < g.nslab * WAVES) counts[c + lane] = carry + inc - v;
        carry += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
      }
      if (lane == 0) counts[g.nslab * WAVES] = carry;
    }
    __syncthreads();
    const uint32_t gathered = __builtin_amdgcn_readfirstlane(counts[g.nslab * WAVES]);
    if (gathered >= C && gathered <= cap) {        // (nearly always)
      each([&](int at, uint32_t rowbase, uint32_t e0, uint32_t e1) {
        uint32_t to = (uint32_t)__builtin_amdgcn_readfirstlane(counts[at]);
        for (uint32_t e = e0; e < e1; e += 64) {
          const uint32_t row = rowbase + (tent[min(e + lane, e1 - 1u)] & kRowMask);
          const uint64_t m = __ballot(e + lane < e1 && overflow_prio(row, t, g.r, g.pa, g.pb) <= limit);
          if (m >> lane & 1u) few[to + lanes_before(m)] = (int32_t)row;
          to += (uint32_t)__popcll(m);
        }
      });
      if (tid == 0) { orow[0] = s0; count_over(g.ctrl, m, 1u); }
      __syncthreads();
      keep_smallest<WAVES>(few, gathered, C, seg, t, g.r, g.pa, g.pb, sums);
      return;
    }
  }
  auto entries = [&](auto&& f) {                   // f(row, low digit)
    for (int q = wave; q < g.nslab; q += WAVES) {
      uint32_t a, len;
      run(q, a, len);
      const uint32_t rowbase = (uint32_t)q * (uint32_t)g.slab_rows;
      for (uint32_t e = lane; e < len; e += 64) {
        const uint32_t y = tent[rowbase + a + e];
        f(rowbase + (y & kRowMask), y >> kRowBits);
      }
    }
  };
  entries([&](uint32_t, uint32_t low) { atomicAdd(&cnt[low], 1u); });
  __syncthreads();
  const int nch = (nlo + 255) / 256;               // chunks of 256 buckets, four per lane
  auto four = [&](int c, uint32_t (&tot)[4]) {
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      tot[i] = c * 256 + lane * 4 + i < nlo ? cnt[c * 256 + lane * 4 + i] : 0u;
      sum += tot[i];
    }
    return sum;
  };
  for (int c = wave; c < nch; c += WAVES) {
    uint32_t tot[4];
    const uint32_t sum = wave_sum(four(c, tot));
    if (lane == 0) csum[c] = sum;
  }
  __syncthreads();
  const uint32_t v = lane < nch ? csum[lane] : 0u, before = wave_incl_scan_add(v) - v;
  for (int c = wave; c < nch; c += WAVES) {
    uint32_t tot[4], nover = 0;
    const uint32_t sum = four(c, tot);
    uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)before, c) + wave_incl_scan_add(sum) - sum;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int b = c * 256 + lane * 4 + i;
      if (b < nlo) { cnt[b] = at; orow[b] = s0 + at; }
      at += tot[i];
      nover += (uint32_t)__popcll(__ballot(tot[i] > C));
    }
    if (nover && lane == 0) atomicAdd(&misc[2], nover);
  }
  __syncthreads();
  if (tid == 0 && misc[2]) count_over(g.ctrl, m, misc[2]);
  entries([&](uint32_t row, uint32_t low) { seg[atomicAdd(&cnt[low], 1u)] = (int32_t)row; });
  __syncthreads();
  auto buckets = [&](bool wave_sized, auto&& f) {  // of two ids and more; the end of a bucket is the start of the next
    for (int c = 0; c < nlo; c += 64) {
      const int b = c + lane;
      const uint32_t a = b < nlo && b ? cnt[b - 1] : 0u, sz = b < nlo ? cnt[b] - a : 0u;
      for (uint64_t todo = __ballot(sz >= 2u && (sz <= 64u && sz <= C) == wave_sized); todo; todo &= todo - 1) {
        const int l = __ffsll((long long)todo) - 1;
        f(seg + (uint32_t)__builtin_amdgcn_readlane((int)a, l), (uint32_t)__builtin_amdgcn_readlane((int)sz, l));
      }
    }
  };
  int nth = 0;
  buckets(true, [&](int32_t* p, uint32_t sz) {     // a bitonic sort across the lanes
    if (nth++ % WAVES != wave) return;
    int32_t key = (uint32_t)lane < sz ? p[lane] : 0x7fffffff;
#pragma unroll
    for (int k = 2; k <= 64; k <<= 1)
#pragma unroll
      for (int j = k >> 1; j > 0; j >>= 1) {
        const int32_t other = __shfl_xor(key, j);
        const bool up = (lane & k) == 0, lower = (lane & j) == 0;
        const int32_t mn = key < other ? key : other, mx = key < other ? other : key;
        key = (lower == up) ? mn : mx;
      }
    if ((uint32_t)lane < sz) p[lane] = key;
  });
  buckets(false, [&](int32_t* p, uint32_t sz) { finish_bucket<THREADS>(g, room, p, sz, t); });
}

// One partition: (d, t) holds the buckets (d << lb) .. (d << lb) + 2^lb - 1 of table t, and its entries are the runs
// of digit d of every slab, in order of the rows.  The ids are grouped by bucket in LDS, in the order they come: PW
// waves take consecutive stretches of the entries and have counters of their own, so the ids of a bucket end up
// ascending without being sorted.  (What is not ours to decide is the order in which an LDS word serves the lanes of
// one instruction.  It is lane order on this hardware; a partition in which it were not would be found out while it
// is copied to the table and put right by exchanges of neighbours: with the lanes of a piece reversed on purpose every
// table still came out right.)  The survivors of an over-capacity bucket are chosen
// here too, by a wave, or by the workgroup where there are many members.
// DIRECT: the entries are the codes themselves (one partition per table, one slab: no grouping pass has run).
// IN_TABLE: a partition of up to kTableIds ids that no staging area holds: the same, with the ids placed in the table
// and a bit per id in LDS for the first ones of the buckets.  Returns false where nothing has been done.
template <int PW, int V, int THREADS, bool DIRECT, bool IN_TABLE = false>
__device__ __forceinline__ bool build_partition(const PartArgs& g, uint32_t* lds, const uint32_t m) {
  constexpr bool kLarge = THREADS == kLargeThreads;
  constexpr int kWaves = THREADS / 64;
  constexpr int kSelRegs = kLarge ? 8 : 16;        // members per lane of an over-capacity bucket whose priorities stay in registers
  typedef uint32_t vec __attribute__((ext_vector_type(V)));
  struct __attribute__((packed, aligned(4))) Words { vec w; };      // (in memory: word-aligned only)
  struct __attribute__((packed, aligned(4))) Ids4 { int32_t w[4]; };
  const size_t t = m >> g.hb;
  const uint32_t d = m & ((uint32_t)g.nbins - 1u);
  const int lb = g.lb, nlo = 1 << lb, nlop = nlo < V ? V : nlo, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t N = g.N;
  const uint32_t C = (uint32_t)g.C;
  const int np = nlop + 64;                        // (a word per lane behind the counters: lanes without an entry)
  uint32_t* cnt = lds;                             // [PW/2][np] counters, then cursors, of waves 2i (low half) and 2i + 1
  int32_t* staged = (int32_t*)(cnt + (PW / 2 * np + 3) / 4 * 4);   // [stage + 4] the partition's ids grouped by bucket (bit 31: first of a bucket)
  uint32_t* bits = (uint32_t*)staged;              // (IN_TABLE) [kBitWords]
  uint2* slots = (uint2*)(staged + (IN_TABLE ? kBitWords : g.stage + 4));      // [slot_cap] pieces: entry inside the table | entries << 24, first row of the slab
  int32_t* survivors = (int32_t*)slots;            // (IN_TABLE) [waves][C]
  uint32_t* csum = (uint32_t*)(slots + g.slot_cap);   // [64] ids per chunk of buckets
  uint32_t* misc = csum + 64;                      // [0] pieces [1] ids [2] first place [3] out of order [4] over capacity
  uint32_t* sums = misc + 8;                       // [4 + 2 * waves] for keep_smallest
  const uint32_t* tent = g.entries + t * N;
  const uint32_t* truns = g.runs + t * (size_t)g.nslab * (size_t)(g.nbins + 1) + d;
  // (0) counters cleared; one wave looks up the runs and cuts them into pieces
#pragma unroll
  for (int h = 0; h < PW / 2; ++h) {
    for (int b = tid; b < nlop / 2; b += THREADS) ((uint2*)(cnt + h * np))[b] = make_uint2(0u, 0u);
    if (tid < 64) cnt[h * np + nlop + tid] = (uint32_t)tid * 0x10001u;   // (places of their own to put nothing into)
  }
  if (wave == 1) {
    if (lane >= 3 && lane < 12) misc[lane] = 0;    // (sums[0 .. 3] among them)
  }
  if (wave == 0) {
    uint32_t npieces = 0, n = 0, s0 = 0;
    const int cl = 1 << g.cut_bits, first = lane & (cl - 1);
    for (int q0 = 0; q0 < g.nslab; q0 += 64 >> g.cut_bits) {
      const int q = q0 + (lane >> g.cut_bits);
      uint32_t a = 0, len = 0;
      if (q < g.nslab) {
        if (DIRECT) len = (uint32_t)N;
        else { const uint32_t* p = truns + (size_t)q * (size_t)(g.nbins + 1); a = p[0]; len = p[1] - a; }
      }
      const uint32_t cuts = (len + kPiece - 1) / kPiece, inc = wave_incl_scan_add(first == 0 ? cuts : 0u);
      const uint32_t base = npieces + inc - cuts, rowbase = (uint32_t)q * (uint32_t)g.slab_rows;
      for (uint32_t j = (uint32_t)first; j < cuts; j += (uint32_t)cl)
        if (base + j < (uint32_t)g.slot_cap)
          slots[base + j] = make_uint2((rowbase + a + j * kPiece) | min((uint32_t)kPiece, len - j * kPiece) << 24, rowbase);
      npieces += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
      n += wave_sum(first == 0 ? len : 0u);
      s0 += wave_sum(first == 0 ? a : 0u);         // (the rows of the slab with a smaller digit)
    }
    if (lane < 3) misc[lane] = lane == 0 ? npieces : lane == 1 ? n : s0;
    if (lane < 4 * kBatch && npieces + lane < (uint32_t)g.slot_cap) slots[npieces + lane] = make_uint2(0u, 0u);   // (see load)
  }
  __syncthreads();
  const uint32_t npieces = __builtin_amdgcn_readfirstlane(misc[0]), n = __builtin_amdgcn_readfirstlane(misc[1]);
  const uint32_t s0 = __builtin_amdgcn_readfirstlane(misc[2]);
  const bool fits = g.nslab <= kMaxSlabs && npieces + 4u * kBatch <= (uint32_t)g.slot_cap;   // (entry numbers of 24 bits: kMaxSlabs)
  int32_t* seg = g.ids + t * N + s0;
  uint32_t* orow = g.off + t * ((size_t)g.nb + 1) + ((size_t)d << lb);
  if (d == (uint32_t)g.nbins - 1 && tid == 0) g.off[t * ((size_t)g.nb + 1) + g.nb] = (uint32_t)N;
  if (!fits || n > (uint32_t)(IN_TABLE ? kTableIds : g.stage) || (IN_TABLE && lb == 0)) {   // (lb = 0: see unstaged_partition)
    if (!IN_TABLE && tid == 0) {
      if (!kLarge || DIRECT) g.large[atomicAdd(&g.ctrl->nlarge, 1u)] = m;   // (DIRECT: never)
      else g.large[(uint32_t)g.total + atomicAdd(&g.ctrl->nunstaged, 1u)] = m;
    }
    return false;
  }
  int32_t* idl = IN_TABLE ? seg : staged;
  if (IN_TABLE) for (uint32_t p = tid; p <= n / 32u; p += THREADS) bits[p] = 0;
  else for (uint32_t p = tid; p < (n + 4u) / 4u; p += THREADS) ((int4*)staged)[p] = make_int4(0, 0, 0, 0);
  // A wave's entries: steps of four pieces, a row of lanes each.
  const int steps = (int)(npieces + 7) >> 3 << 1, per = (steps + 2 * PW - 1) / (2 * PW) * 2;   // (even)
  const int g0 = wave < PW ? min(wave * per, steps) : 0, g1 = wave < PW ? min(g0 + per, steps) : 0;
  uint32_t low[kBatch], id[kBatch];                // bucket (no entry: a word of the lane's own) and row (no entry: 0) of the entries in flight
  // (the pairs of steps that there are, compared anew in every loop: kept, the comparisons cost more than they do)
  auto live = [&](int base) { int e = g1 - base; asm("" : "+s"(e)); return e; };
  auto load = [&](int base) {
    // All pieces looked up, then all entries requested, without a branch between them (at its end a wave looks up the
    // next one's pieces, or the padding, for nothing: a branch per step would wait for the step before).
    const uint32_t l16 = (uint32_t)lane & 15u;
    const uint2* from = slots + (uint32_t)base * 4u + ((uint32_t)lane >> 4);
    uint2 piece[kBatch];
    uint32_t at[kBatch], x[kBatch];
#pragma unroll
    for (int k = 0; k < kBatch; ++k) piece[k] = from[k * 4];
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      at[k] = (piece[k].x & 0xffffffu) + (l16 < piece[k].x >> 24 ? l16 : 0u);
      x[k] = *(const uint32_t*)((const char*)tent + at[k] * 4u);
    }
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const bool has = l16 < piece[k].x >> 24;
      if (DIRECT) x[k] = x[k] << kRowBits | at[k];
      low[k] = has ? x[k] >> kRowBits : (uint32_t)(nlop + lane);   // (nlop >= 2)
      id[k] = has ? piece[k].y + (x[k] & ((1u << kRowBits) - 1u)) : 0u;
    }
  };
  uint32_t* mine = cnt + (wave >> 1) % (PW / 2) * np;
  const uint32_t shift = 16u * (uint32_t)(wave & 1);
  const bool few = lb <= 1;                        // one or two buckets: all lanes would queue at their counters
  // f(slot of the batch), for the steps of the batch
  auto steps_of = [&](int base, auto&& f) {
    const int e = live(base);
#pragma unroll
    for (int k = 0; k < kBatch; k += 2)
      if (k < e) { f(k); f(k + 1); }
  };
  // (1) count
  if (few) {
    uint32_t c0 = 0, c1 = 0;
    for (int base = g0; base < g1; base += kBatch) {
      load(base);
      steps_of(base, [&](int k) {
        c0 += (uint32_t)__popcll(__ballot(low[k] == 0u));
        c1 += (uint32_t)__popcll(__ballot(low[k] == 1u));
      });
    }
    if (wave < PW && lane < nlo) atomicAdd(&mine[lane], (lane ? c1 : c0) << shift);
  } else {
    for (int base = g0; base < g1; base += kBatch) {
      load(base);
      steps_of(base, [&](int k) { atomicAdd(&mine[low[k]], 1u << shift); });
    }
  }
  __syncthreads();
  // (2) bucket starts, from the sums of chunks of 64 * V buckets: a chunk a wave where they are that few, else
  // the sums first and every chunk again from where it begins
  const int nch = (nlo + 64 * V - 1) / (64 * V);
  auto counts = [&](int c, vec (&w)[PW / 2]) {
    const int b = c * 64 * V + lane * V;
#pragma unroll
    for (int h = 0; h < PW / 2; ++h) {
#pragma unroll
      for (int i = 0; i < V; ++i) w[h][i] = 0;
      if (b < nlop) w[h] = *(const vec*)(cnt + h * np + b);
    }
  };
  auto starts = [&](int c, vec (&w)[PW / 2], uint32_t at) {   // the lane's buckets begin at `at`
    const int b = c * 64 * V + lane * V;
    vec tot, first;
#pragma unroll
    for (int i = 0; i < V; ++i) {
      uint32_t cur = at;
      first[i] = s0 + at;
      if (b < nlop) {                              // (an empty bucket marks the start of the next one, or the word behind the ids)
        if (IN_TABLE) atomicOr(&bits[at >> 5], 1u << (at & 31u));
        else idl[at] = INT32_MIN;
      }
#pragma unroll
      for (int h = 0; h < PW / 2; ++h) {
        const uint32_t mid = cur + (w[h][i] & 0xffffu), end = mid + (w[h][i] >> 16);
        w[h][i] = cur | mid << 16;
        cur = end;
      }
      tot[i] = cur - at;
      at = cur;
    }
    uint32_t most = tot[0];
#pragma unroll
    for (int i = 1; i < V; ++i) most = max(most, tot[i]);
    if (__any(most > C)) {
      uint32_t nover = 0;
#pragma unroll
      for (int i = 0; i < V; ++i) nover += (uint32_t)__popcll(__ballot(tot[i] > C));
      if (lane == 0) atomicAdd(&misc[4], nover);
    }
    if (b < nlop)
#pragma unroll
      for (int h = 0; h < PW / 2; ++h) *(vec*)(cnt + h * np + b) = w[h];
    if (b + V <= nlo) reinterpret_cast<Words*>(orow + b)->w = first;
    else if (b < nlo) orow[b] = first[0];          // (V buckets or more, or a single one: nlo is a power of two)
  };
  auto sum_of = [&](const vec (&w)[PW / 2]) {      // (the halves of the words add up side by side: fewer than 2^16 ids)
    uint32_t both = 0;
#pragma unroll
    for (int h = 0; h < PW / 2; ++h)
#pragma unroll
      for (int i = 0; i < V; ++i) both += w[h][i];
    return (both & 0xffffu) + (both >> 16);
  };
  if (nch <= kWaves) {
    vec w[PW / 2];
    counts(wave, w);
    const uint32_t sum = sum_of(w), inc = wave_incl_scan_add(sum);
    if (lane == 63) csum[wave] = inc;
    __syncthreads();
    uint32_t at = inc - sum;
    for (int c = 0; c < wave; ++c) at += csum[c];
    if (wave < nch) starts(wave, w, at);
  } else {
    for (int c = wave; c < nch; c += kWaves) {
      vec w[PW / 2];
      counts(c, w);
      const uint32_t sum = wave_sum(sum_of(w));
      if (lane == 0) csum[c] = sum;
    }
    __syncthreads();
    const uint32_t v = lane < nch ? csum[lane] : 0u, before = wave_incl_scan_add(v) - v;
    for (int c = wave; c < nch; c += kWaves) {
      vec w[PW / 2];
      counts(c, w);
      const uint32_t sum = sum_of(w);
      starts(c, w, (uint32_t)__builtin_amdgcn_readlane((int)before, c) + wave_incl_scan_add(sum) - sum);
    }
  }
  __syncthreads();
  // (3) place
  const bool reload = g1 - g0 > kBatch;
  if (few) {
    uint32_t at0 = 0, at1 = 0;
    if (wave < PW) { at0 = mine[0] >> shift & 0xffffu; at1 = mine[1] >> shift & 0xffffu; }
    for (int base = g0; base < g1; base += kBatch) {
      if (reload) load(base);
      steps_of(base, [&](int k) {
        const uint64_t m0 = __ballot(low[k] == 0u), m1 = __ballot(low[k] == 1u);
        const uint32_t at = low[k] ? at1 + lanes_before(m1) : at0 + lanes_before(m0);
        if (low[k] <= 1u) { if (IN_TABLE) idl[at] = (int32_t)id[k]; else idl[at] |= (int32_t)id[k]; }
        at0 += (uint32_t)__popcll(m0);
        at1 += (uint32_t)__popcll(m1);
      });
    }
    if (wave == PW - 1 && lane < nlo)              // (the last wave's cursors end where their buckets end: see end_of)
      mine[lane] = (mine[lane] & 0xffffu) | (lane ? at1 : at0) << 16;
  } else {
    for (int base = g0; base < g1; base += kBatch) {
      if (reload) load(base);
      uint32_t at[kBatch];                         // (all places asked for before the first is used)
      steps_of(base, [&](int k) { at[k] = atomicAdd(&mine[low[k]], 1u << shift); });
      steps_of(base, [&](int k) {
        const uint32_t to = at[k] >> shift & 0xffffu;
        if (!IN_TABLE) atomicOr((uint32_t*)&idl[to], id[k]);
        else if (low[k] < (uint32_t)nlop) idl[to] = (int32_t)id[k];
      });
    }
  }
  __syncthreads();
  const uint32_t nover = __builtin_amdgcn_readfirstlane(misc[4]);
  if (nover && tid == 0) count_over(g.ctrl, m, nover);
  // (4) to the table, in one coalesced copy; an id not above the one before it must begin a bucket
  bool wrong = false;
  const bool select = nover != 0 && g.policy != SLIDE_KEEP_LOWEST_ID;   // (the lowest ids come first anyway)
  if (IN_TABLE) {
    for (uint32_t p = 1u + tid; p < n; p += THREADS) wrong |= idl[p - 1] >= idl[p] && !(bits[p >> 5] >> (p & 31u) & 1u);
  } else
  for (uint32_t p = 4u * tid; p < n; p += 4u * THREADS) {
    const int4 q = *(const int4*)(idl + p);        // (up to three words past the ids: zeros and a mark)
    const uint32_t v[5] = {(uint32_t)idl[max((int)p, 1) - 1], (uint32_t)q.x, (uint32_t)q.y, (uint32_t)q.z, (uint32_t)q.w};
    const uint32_t left = n - p;
    Ids4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o.w[i] = (int32_t)(v[i + 1] & 0x7fffffffu);
      wrong |= (v[i] & 0x7fffffffu) >= v[i + 1] && (uint32_t)i < left;   // (a marked id exceeds every unmarked one)
    }
    if (left >= 4u) *reinterpret_cast<Ids4*>(seg + p) = o;
    else
#pragma unroll
      for (int i = 0; i < 3; ++i)
        if ((uint32_t)i < left) seg[p + i] = o.w[i];
  }
  if (__any(wrong) && lane == 0) misc[3] = 1u;
  __syncthreads();
  const bool sorted = __builtin_amdgcn_readfirstlane(misc[3]) == 0u;
  if (sorted && !select) return true;
  if (!sorted) {
    // (lanes of an instruction were not served in lane order: neighbours change places until all are in order)
    for (uint32_t pass = 0, quiet = 0; quiet < 2; ++pass) {
      __syncthreads();
      if (tid == 0) misc[3] = 0;
      __syncthreads();
      for (uint32_t p = 2u * tid + (pass & 1u); p + 1u < n; p += 2u * THREADS) {
        const uint32_t a = (uint32_t)idl[p], b = (uint32_t)idl[p + 1];
        const bool first = IN_TABLE && (bits[(p + 1u) >> 5] >> ((p + 1u) & 31u) & 1u);
        if ((a & 0x7fffffffu) > b && !first) {     // (b is unmarked, then: the second of a bucket or later)
          idl[p] = (int32_t)(b | (a & 0x80000000u));
          idl[p + 1] = (int32_t)(a & 0x7fffffffu);
          misc[3] = 1u;
        }
      }
      __syncthreads();
      quiet = misc[3] ? 0u : quiet + 1u;
    }
    if (!IN_TABLE) for (uint32_t p = tid; p < n; p += THREADS) seg[p] = idl[p] & 0x7fffffff;
    __syncthreads();
    if (!select) return true;
  }
  if (!IN_TABLE) for (uint32_t p = tid; p < n; p += THREADS) idl[p] &= 0x7fffffff;
  __syncthreads();
  auto end_of = [&](int b) { return cnt[(PW / 2 - 1) * np + b] >> 16; };   // the end of bucket b = the start of bucket b + 1
  // (5) the survivors of the over-capacity buckets: the C members with the smallest (priority, id)
  auto over_capacity = [&](bool many, auto&& f) {
    for (int c = 0; c < nlo; c += 64) {
      const int b = c + lane;
      const uint32_t a = b < nlo && b ? end_of(b - 1) : 0u, sz = b < nlo ? end_of(b) - a : 0u;
      for (uint64_t todo = __ballot(sz > C && (sz > 64u * kSelRegs) == many); todo; todo &= todo - 1) {
        const int l = __ffsll((long long)todo) - 1;
        f((uint32_t)__builtin_amdgcn_readlane((int)a, l), (uint32_t)__builtin_amdgcn_readlane((int)sz, l));
      }
    }
  };
  int nth = 0;
  over_capacity(false, [&](uint32_t a, uint32_t sz) {
    if (nth++ % kWaves != wave) return;
    int32_t* to = IN_TABLE ? survivors + wave * (int)C : seg + a;
    keep_smallest<1, kSelRegs>(idl + a, sz, C, to, (uint32_t)t, g.r, g.pa, g.pb, nullptr);
    if (IN_TABLE) for (uint32_t i = lane; i < C; i += 64) seg[a + i] = to[i];
  });
  if (IN_TABLE) __syncthreads();
  over_capacity(true, [&](uint32_t a, uint32_t sz) {
    keep_smallest<kWaves>(idl + a, sz, C, IN_TABLE ? survivors : seg + a, (uint32_t)t, g.r, g.pa, g.pb, sums);
    __syncthreads();
    if (IN_TABLE) {
      for (uint32_t i = tid; i < C; i += THREADS) seg[a + i] = survivors[i];
      __syncthreads();
    }
  });
  return true;
}

// What bounds it: three dependent round trips to memory per partition and the instructions between them (57
// vector and 64 scalar ones per 64 ids; the scalar unit issues no more of them than each SIMD does vector ones).
// 670,091 ids x 400 tables, fresh weights: 840 us, against 1,390 and 64 for sorting what arrived in any order
// (skewed weights 905 + 128 for the large form, against 1,574 and 300); 325,056 ids x 50 tables in 25,600 buckets of
// 635: 110 us, half of them for the survivors, against 181 and 137.  A staging area of 2.5 mean partitions lets two more
// workgroups share a compute unit, 760 us, but leaves a skewed layer's partitions to the large form (905 + 128
// -> 789 + 215 us) and some of the 635-id buckets (4.5 -> 16 us): not taken.
// One workgroup per partition.  Neighbouring partitions share cache lines of entries and run boundaries: a die takes
// a contiguous stretch of them.  PW = 4 waves count with two words per bucket, or, from 4,096 buckets per partition
// on, where the counters decide how many workgroups share a compute unit, PW = 2 with one; V: buckets per lane in
// the passes over them.
// THREADS: 256, or 1,024 where a table of up to 512 codes is a single partition (2,000 ids, eight tables: 18 -> 12 us).
template <int PW, int V, bool DIRECT, int THREADS = 256>
__global__ __launch_bounds__(THREADS) void part_buckets_kernel(PartArgs g) {
  extern __shared__ uint4 part_lds[];
  const uint32_t k = blockIdx.x / (uint32_t)g.nxcd, m = (blockIdx.x % (uint32_t)g.nxcd) * (uint32_t)g.per_xcd + k;
  if (m < (uint32_t)g.total) build_partition<PW, V, THREADS, DIRECT>(g, (uint32_t*)part_lds, m);
}

// The partitions too large for that, as the digits of a layer in training are skewed: a workgroup of sixteen waves per
// compute unit goes through the list.
template <int PW, int V>
__global__ __launch_bounds__(kLargeThreads) void large_buckets_kernel(PartArgs g) {
  extern __shared__ uint4 part_lds[];
  const uint32_t count = g.ctrl->nlarge;
  for (uint32_t i = blockIdx.x; i < count; i += gridDim.x) {
    build_partition<PW, V, kLargeThreads, false>(g, (uint32_t*)part_lds, g.large[i]);
    __syncthreads();
  }
}

// And those that fit no staging area.
template <int PW, int V>
__global__ __launch_bounds__(kLargeThreads) void unstaged_buckets_kernel(PartArgs g) {
  extern __shared__ uint4 part_lds[];
  const uint32_t count = g.ctrl->nunstaged;
  for (uint32_t i = blockIdx.x; i < count; i += gridDim.x) {
    const uint32_t m = g.large[(uint32_t)g.total + i];
    if (!build_partition<PW, V, kLargeThreads, false, true>(g, (uint32_t*)part_lds, m)) {
      __syncthreads();
      unstaged_partition<kLargeThreads / 64>(g, (uint32_t*)part_lds, m);
    }
    __syncthreads();
  }
}

// Split of the code into partition digit (high hb bits) and in-partition digit (low lb bits).
void tables_split(int bits, int64_t N, int* hb, int* lb) {
  int want = 0;
  while (want < 11 && ((int64_t)2048 << want) < N) ++want;     // about 1024 to 2048 rows per partition
  int h = want < bits ? want : bits;
  if (bits - h > 13) h = bits - 13;                            // low digit counters must fit in LDS
  *hb = h;
  *lb = bits - h;
}

// Rows per thread of the slab grouping: entries and counters fill the LDS (160 KB).
static int slab_rpt(int nbins) { return nbins <= 512 ? 32 : nbins <= 1024 ? 30 : 22; }
static int64_t slab_count(int64_t N, int nbins) {
  const int64_t rows = (int64_t)slab_rpt(nbins) * 1024;
  return N > 0 ? (N + rows - 1) / rows : 1;
}

size_t tables_bh_words(int bits, int64_t N, int L) {      // run boundaries per (table, slab)
  int hb, lb;
  tables_split(bits, N, &hb, &lb);
  return (size_t)L * (size_t)slab_count(N, 1 << hb) * (((size_t)1 << hb) + 1);
}

size_t tables_list_words(int bits, int64_t N, int L) {    // two lists of partitions
  int hb, lb;
  tables_split(bits, N, &hb, &lb);
  return (size_t)2 * L << hb;
}

constexpr int kWideLb = 12;               // partitions of 2^12 buckets and more: one word of counters per bucket
static int large_ids(int lb) { return lb < 13 ? 30720 : 24576; }   // most ids of a partition staged by the large form
static int large_waves(int lb) { return lb <= 9 ? 16 : lb == 10 ? 8 : lb == 11 ? 4 : 2; }   // waves that count in the large form
static size_t part_buckets_lds(int lb, int waves, int slot_cap, int stage, int threads) {
  const size_t nlo = std::max<size_t>((size_t)1 << lb, 2);
  return (((nlo + 64) * (waves / 2) + 3) / 4 * 4 + stage + 4 + 2 * (size_t)slot_cap + 64 + part_misc(threads)) * 4;
}
// The staging area of the bucket kernel: four mean partitions (a fresh layer's partitions stay within a
// few percent of the mean, a trained one's within a few times), so that tables with many buckets per
// partition, whose counters take most of the LDS, still fit another workgroup per compute unit.
static int stage_ids(int64_t N, int nbins) {
  const int64_t want = 4 * ((N + nbins - 1) / nbins);
  const int64_t s = want < kStageMin ? kStageMin : (want > kStageIds ? kStageIds : want);
  return (int)((s + 63) / 64 * 64);
}
static int piece_slots(int stage, int64_t nslab) { return stage / kPiece + (int)std::min<int64_t>(nslab, kMaxSlabs) + 4 * kBatch; }
// (pieces, then the survivors of sixteen buckets of the largest capacity)
static int table_slots(int64_t nslab) { return std::max(piece_slots(kTableIds, nslab), kLargeThreads / 64 * 1024 / 2); }
static size_t in_table_lds(int lb, int waves, int slot_cap) { return part_buckets_lds(lb, waves, slot_cap, kBitWords, kLargeThreads); }
static size_t unstaged_lds(int lb) { return ((size_t)kRoomWords + 64 + 4 + 2 * (kLargeThreads / 64) + 4 + ((size_t)1 << lb)) * 4; }
static size_t slab_group_lds(int nbins) { return ((size_t)slab_rpt(nbins) * 1024 + 8 * (size_t)nbins + 20) * 4; }

// Rows of W2 touched since the last build (one byte each, set by the training step) -> a list of
// their ids and its length; the marks are cleared.  One thread per row, one counter update per
// workgroup (ascending ids within a workgroup's stretch; stretches in arrival order).
__global__ __launch_bounds__(1024) void collect_touched_kernel(uint8_t* __restrict__ touched, int64_t N,
                                                               int32_t* __restrict__ rows, uint32_t* count) {
  __shared__ uint32_t wsum[17];
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool hit = j < N && touched[j] != 0;
  const uint64_t m = __ballot(hit);
  if (lane == 0) wsum[wave] = (uint32_t)__popcll(m);
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t run = 0;
    for (int w = 0; w < 16; ++w) { const uint32_t c = wsum[w]; wsum[w] = run; run += c; }
    wsum[16] = run ? atomicAdd(count, run) : 0u;
  }
  __syncthreads();
  if (hit) {
    rows[wsum[16] + wsum[wave] + __popcll(m & ((1ull << lane) - 1))] = (int32_t)j;
    touched[j] = 0;
  }
}

// When most rows were touched, hashing all of them in place is cheaper than hashing them through
// the list (whole lines of codes instead of scattered words): the count becomes N, which the hash
// kernels take as "no list".  Then the count goes to the one of the two that takes as many rows.
__global__ void split_listed_kernel(uint32_t* count, uint32_t N, uint32_t ranked_from, uint32_t* listed, Ctrl* ctrl) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  for (uint32_t w = 0; w < kOverWords; ++w) ctrl->overflowed[w][0] = 0;
  ctrl->nlarge = 0; ctrl->nunstaged = 0;
  if ((uint64_t)*count * 4 > (uint64_t)N * 3) *count = N;
  const uint32_t n = *count;
  listed[0] = n < ranked_from ? n : 0u;
  listed[1] = n < ranked_from ? 0u : n;
}

hipError_t tables_setup_attributes() {
  hipError_t e;
#define SLIDE_SET(K, BYTES) \
  e = hipFuncSetAttribute((const void*)&K, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(BYTES)); \
  if (e != hipSuccess) return e;
  SLIDE_SET((part_buckets_kernel<4, 2, false>), part_buckets_lds(kWideLb - 1, 4, piece_slots(kStageIds, kMaxSlabs), kStageIds, 256))
  SLIDE_SET((part_buckets_kernel<2, 4, false>), part_buckets_lds(13, 2, piece_slots(kStageIds, kMaxSlabs), kStageIds, 256))
  SLIDE_SET((part_buckets_kernel<16, 2, true, kLargeThreads>), part_buckets_lds(9, 16, piece_slots(kStageIds, kMaxSlabs), kStageIds, kLargeThreads))
  SLIDE_SET((part_buckets_kernel<4, 2, true>), part_buckets_lds(kWideLb - 1, 4, piece_slots(kStageIds, kMaxSlabs), kStageIds, 256))
  SLIDE_SET((part_buckets_kernel<2, 4, true>), part_buckets_lds(13, 2, piece_slots(kStageIds, kMaxSlabs), kStageIds, 256))
  SLIDE_SET((large_buckets_kernel<16, 2>), part_buckets_lds(9, 16, piece_slots(large_ids(9), kMaxSlabs), large_ids(9), kLargeThreads))
  SLIDE_SET((large_buckets_kernel<8, 2>), part_buckets_lds(10, 8, piece_slots(large_ids(10), kMaxSlabs), large_ids(10), kLargeThreads))
  SLIDE_SET((large_buckets_kernel<4, 2>), part_buckets_lds(11, 4, piece_slots(large_ids(11), kMaxSlabs), large_ids(11), kLargeThreads))
  SLIDE_SET((large_buckets_kernel<2, 4>), std::max(part_buckets_lds(12, 2, piece_slots(large_ids(12), kMaxSlabs), large_ids(12), kLargeThreads),
                                              part_buckets_lds(13, 2, piece_slots(large_ids(13), kMaxSlabs), large_ids(13), kLargeThreads)))
  SLIDE_SET((unstaged_buckets_kernel<8, 2>), std::max(unstaged_lds(10), in_table_lds(10, 8, table_slots(kMaxSlabs))))
  SLIDE_SET((unstaged_buckets_kernel<4, 2>), std::max(unstaged_lds(11), in_table_lds(11, 4, table_slots(kMaxSlabs))))
  SLIDE_SET((unstaged_buckets_kernel<2, 4>), std::max(unstaged_lds(13), in_table_lds(13, 2, table_slots(kMaxSlabs))))
  SLIDE_SET(slab_group_kernel<32>, slab_group_lds(512))
  SLIDE_SET(slab_group_kernel<30>, slab_group_lds(1024))
  SLIDE_SET(slab_group_kernel<22>, slab_group_lds(2048))
#undef SLIDE_SET
  return hipSuccess;
}

hipError_t launch_build_tables(const HashDev& hd, const TablesDev& td, const float* W2, uint32_t* codes_t,
                               uint32_t* entries, uint32_t* bh, uint32_t* large_list, Ctrl* ctrl, int policy, uint32_t r, uint32_t prio_a,
                               uint32_t prio_b, uint8_t* touched, int32_t* touched_rows, bool only_touched,
                               int nxcd, hipStream_t s) {
  hipError_t e;
  int bits = 0, hb, lb;
  while ((1u << bits) < td.nb) ++bits;
  tables_split(bits, td.N, &hb, &lb);
  const int nbins = 1 << hb;
  const int nslab = (int)slab_count(td.N, nbins), rpt = slab_rpt(nbins);
  // (1) codes of every row, or -- when codes_t still holds the codes of the last build -- only of the
  // rows whose weights changed since; the grouping below always runs in full, so the tables are the
  // same either way.  The first kernel that comes here clears the counters of the queues.
  if (only_touched) {
    if ((e = launch_fill_u32(&ctrl->rehashed, 1, 0u, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(collect_touched_kernel, dim3((unsigned)ceil_div(td.N, 1024)), dim3(1024), 0, s, touched, td.N,
                       touched_rows, &ctrl->rehashed);
    hipLaunchKernelGGL(split_listed_kernel, dim3(1), dim3(64), 0, s, &ctrl->rehashed, (uint32_t)td.N,
                       (uint32_t)std::min<int64_t>(hash_ranked_from(hd), UINT32_MAX), ctrl->listed, ctrl);
    if ((e = launch_hash(hd, W2, td.N, codes_t, 1, td.N, touched_rows, ctrl->listed, hd.L, nullptr, s)) != hipSuccess) return e;
  } else {
    if (touched && (e = launch_fill_u32((uint32_t*)touched, (size_t)ceil_div(td.N, 4), 0u, s)) != hipSuccess) return e;
    if ((e = launch_hash(hd, W2, td.N, codes_t, 1, td.N, nullptr, nullptr, hd.L, ctrl, s)) != hipSuccess) return e;
  }
  // (2) every slab grouped by the high digit (nothing to group where a table is one partition), (3) buckets
  PartArgs g;
  const bool direct = nbins == 1 && nslab == 1;        // (at most 2,048 rows: never too many for the staging area)
  if (!direct) {
#define SLIDE_SLAB(RPT) \
    case RPT: \
      hipLaunchKernelGGL((slab_group_kernel<RPT>), dim3(nslab, td.L), dim3(1024), slab_group_lds(nbins), s, codes_t, td.N, \
                         lb, nbins, bh, nslab, entries); \
      break;
    switch (rpt) { SLIDE_SLAB(32) SLIDE_SLAB(30) SLIDE_SLAB(22) }
#undef SLIDE_SLAB
  }
  g.entries = direct ? codes_t : entries; g.runs = bh; g.off = td.off; g.ids = td.ids;
  g.ctrl = ctrl; g.N = td.N; g.nb = td.nb; g.r = r; g.pa = prio_a; g.pb = prio_b;
  g.nslab = nslab; g.slab_rows = rpt * 1024; g.nbins = nbins; g.hb = hb; g.lb = lb; g.C = td.C; g.policy = policy;
  g.stage = stage_ids(td.N, nbins); g.slot_cap = piece_slots(g.stage, nslab);
  g.cut_bits = 0;
  while (g.cut_bits < 6 && nslab << (g.cut_bits + 1) <= 64) ++g.cut_bits;
  g.total = nbins * td.L; g.nxcd = nxcd; g.per_xcd = ceil_div(g.total, nxcd); g.large = large_list;
  const dim3 grid((unsigned)(g.per_xcd * nxcd));
  const bool wide = direct && lb <= 9;
  const size_t lds = wide ? part_buckets_lds(lb, 16, g.slot_cap, g.stage, kLargeThreads) : part_buckets_lds(lb, lb < kWideLb ? 4 : 2, g.slot_cap, g.stage, 256);
#define SLIDE_PART(PW, V, DIRECT) hipLaunchKernelGGL((part_buckets_kernel<PW, V, DIRECT>), grid, dim3(256), lds, s, g)
  if (wide)
    hipLaunchKernelGGL((part_buckets_kernel<16, 2, true, kLargeThreads>), grid, dim3(kLargeThreads), lds, s, g);
  else if (lb < kWideLb) { if (direct) SLIDE_PART(4, 2, true); else SLIDE_PART(4, 2, false); }
  else { if (direct) SLIDE_PART(2, 4, true); else SLIDE_PART(2, 4, false); }
#undef SLIDE_PART
  if (td.N <= g.stage) return hipGetLastError();         // (no partition is larger than the layer)
  g.stage = (int)std::min<int64_t>((td.N + 63) / 64 * 64, large_ids(lb));
  g.slot_cap = piece_slots(g.stage, nslab);
  const int waves = large_waves(lb);
  const size_t large_lds = part_buckets_lds(lb, waves, g.slot_cap, g.stage, kLargeThreads);
  const dim3 large(std::min(hd.num_cus, g.total));
#define SLIDE_LARGE(PW, V) hipLaunchKernelGGL((large_buckets_kernel<PW, V>), large, dim3(kLargeThreads), large_lds, s, g)
  switch (waves) {
    case 16: SLIDE_LARGE(16, 2); break;
    case 8: SLIDE_LARGE(8, 2); break;
    case 4: SLIDE_LARGE(4, 2); break;
    default: SLIDE_LARGE(2, 4); break;
  }
#undef SLIDE_LARGE
  if (td.N <= large_ids(lb)) return hipGetLastError();
  g.slot_cap = table_slots(nslab);
  const int table_waves = std::min(waves, 8);
  const size_t table_lds = std::max(unstaged_lds(lb), in_table_lds(lb, table_waves, g.slot_cap));
#define SLIDE_TABLE(PW, V) hipLaunchKernelGGL((unstaged_buckets_kernel<PW, V>), large, dim3(kLargeThreads), table_lds, s, g)
  switch (table_waves) {
    case 8: SLIDE_TABLE(8, 2); break;
    case 4: SLIDE_TABLE(4, 2); break;
    default: SLIDE_TABLE(2, 4); break;
  }
#undef SLIDE_TABLE
  return hipGetLastError();
}

}  // namespace slide
