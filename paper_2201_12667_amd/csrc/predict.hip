// Inference over all output neurons: scores z[i][j] = b2[j] + W2[j,:].h_i for every neuron j, and
// the k best per sample.  This is the dense evaluation the paper compares the hashed retrieval
// against (Section 2.1: the tables are meant to return the neurons with the highest activations;
// Section 4: accuracy is measured on full predictions).  Unlike the training path it is a dense
// contraction, run on the matrix cores.
//
// Launches: (1) the samples' hidden activations, split for the matrix cores; (2) the scores of an evenly
// spaced sample of about 8,192 neurons, of which the best of every 32 are kept; (3) per sample the topk-th best of
// these, which is a bar that at least topk neurons of the layer reach; (4) the scores of all neurons, of which only
// those that reach their sample's bar are kept (about topk * N / 8,192 of them: the scores themselves are never
// written); (5) per sample the topk best of these.  For layers of fewer than 16,384 neurons all scores are written
// and the topk best of them chosen.  The bar comes from the whole id range, and so does every group of 32, so an order of the
// ids (by frequency, say) does not matter: 8 samples x 670K neurons whose scores fall with the id take 73 us where random order
// takes 61 (32 coordinates, 10 best), and took 106 us to 15 ms (32 best) when a group was 32 neighbours.
#include "slide_internal.h"
#include "spmm.h"
#include "topk.h"
#include "wave_ops.h"

#include <algorithm>
#include <cmath>

namespace slide {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kScoreThreads = 512;         // eight waves, 32 neurons each
constexpr int kTileNeurons = kScoreThreads / 2;
constexpr int kSampled = 8192;             // neurons the bars are taken from (up to twice as many)
constexpr int kStreamNeurons = 131072;     // layers from which on up to 32 samples take the form kStream
constexpr int kMaxGroups = 2 * kSampled / 32;   // groups of 32 of them
constexpr int kCandMax = 16384;            // candidate keys per sample and launch
constexpr int kCntPitch = 16;              // words between the candidate counters of two samples (one line each)
constexpr int kFrag = 512;                 // values of an operand fragment: 32 rows x 16 coordinates
// (row block, coordinate block) pairs of h that may stay in LDS for good.  Two workgroups of 48 KB share a compute unit; 128
// samples of up to 160 coordinates take one with 120 KB, and more samples than that such workgroups side by side: against 256
// samples staged in turns, a barrier per stage, calls of 256 x 670K x 128 take 284 us instead of 319, 100 x 400K x 32 74 instead
// of 98, 300 x 670K x 128 389 instead of 527, 2,000 x 670K x 128 1,900 instead of 2,030.  The blocks read W2 once each, from wherever
// it is by then: they share a die's L2 only where the grid's width is a multiple of the dies, and rounding it down to that is
// slower by what it leaves idle (300 x 670K x 32 185 -> 194 us, 700 x 200K x 128 266 -> 275, 520 x 9K x 128 41 -> 51; 300 x 670K x 128 the same).
__host__ __device__ constexpr int res_frags(int NIB) { return NIB == 4 ? 40 : 16; }
constexpr int kBlockPad = 8;               // coordinate blocks are padded (with zeros) to a multiple of this
constexpr int kListed = 128;               // scores a wave lists before it hands them over
constexpr int kCornerWords = 512 + 3 * kListed;    // LDS words of a wave: half a block of scores and that list
constexpr size_t kCorners = (size_t)kScoreThreads / 64 * kCornerWords * 4;
constexpr size_t kTriple = 3 * kFrag * 2;  // bytes of a fragment's three parts
// Coordinate blocks of h staged at a time when it does not all fit.
__host__ __device__ constexpr int stage_blocks(int NIB) { return NIB == 8 ? 2 : NIB == 1 ? 8 : 4; }

// Eight floats as three bf16 vectors whose sum they are exactly (8 + 8 + 8 significand bits, each part
// rounded to nearest, so that what a product of parts leaves out has either sign).  Values so large that
// the first part rounds to infinity, infinities and NaN give a score of NaN or infinity, which the caller evaluates
// again in plain arithmetic (see settled).
__device__ __forceinline__ void split8(const float4& a, const float4& b, bf16x8 (&out)[3]) {
  const f32x2 x[4] = {{a.x, a.y}, {a.z, a.w}, {b.x, b.y}, {b.z, b.w}};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const bf16x2 hi = __builtin_convertvector(x[q], bf16x2);
    const f32x2 r1 = x[q] - __builtin_convertvector(hi, f32x2);
    const bf16x2 mid = __builtin_convertvector(r1, bf16x2);
    const f32x2 r2 = r1 - __builtin_convertvector(mid, f32x2);
    const bf16x2 lo = __builtin_convertvector(r2, bf16x2);
    out[0][2 * q] = hi[0]; out[0][2 * q + 1] = hi[1];
    out[1][2 * q] = mid[0]; out[1][2 * q + 1] = mid[1];
    out[2][2 * q] = lo[0]; out[2][2 * q + 1] = lo[1];
  }
}

// (1) One workgroup per sample (rows past the batch: zeros): the hidden activations -- computed here in
// sparse-input mode -- and their three parts in fragment order: fragment (row block, coordinate block, part)
// is the 1 KB a wave reads as one operand, lane l holding row l % 32, coordinates 8 * (l / 32) .. + 7.
__global__ __launch_bounds__(1024) void dense_prepare_kernel(int B, int H, int nkb, const float* __restrict__ h,
                                                             SpmmArgs sp, bf16x8* __restrict__ frags, Ctrl* ctrl,
                                                             int stage_words) {
  extern __shared__ float lds[];                         // [stage_words] rows of W1, [H] the sample's activations
  float* hvec = lds + stage_words;
  const int i = blockIdx.x, tid = threadIdx.x, nthr = blockDim.x;
  if (i < B) {
    if (sp.W1 && H <= nthr && spmm_stage_rows(stage_words, H, nthr) >= 32) {
      spmm_sample_staged(sp, i, B, lds, stage_words, hvec, ctrl);
    } else if (sp.W1) {
      const int wave = tid >> 6;
      if (wave * 128 < H) spmm_sample(sp, i, B, wave, tid & 63, hvec, ctrl);
    } else {
      for (int c = tid; c < H; c += nthr) hvec[c] = h[(size_t)i * H + c];
    }
  }
  __syncthreads();
  for (int c8 = tid; c8 < 2 * nkb; c8 += nthr) {          // (nkb: padded)
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = (i < B && 8 * c8 + e < H) ? hvec[8 * c8 + e] : 0.f;
    bf16x8 part[3];
    split8(make_float4(x[0], x[1], x[2], x[3]), make_float4(x[4], x[5], x[6], x[7]), part);
    const int kb = c8 >> 1, lane = (c8 & 1) * 32 + (i & 31);
#pragma unroll
    for (int p = 0; p < 3; ++p) frags[((size_t)((i >> 5) * nkb + kb) * 3 + p) * 64 + lane] = part[p];
  }
}

// A score in plain arithmetic, for the few that come out as NaN or plus infinity on the matrix cores.
__device__ __forceinline__ float plain_score(const float* __restrict__ h, const float* __restrict__ w, float bias, int H) {
  float s = 0.f;
  for (int k = 0; k < H; ++k) s = fmaf(h[k], w[k], s);
  return s + bias;
}
// Whether a matrix-core score stands as it is: a number, or minus infinity (a sum that left the range at that end
// has left it in any order but for a rounding; the passes have to agree, or a neuron could set a bar that it does not
// reach itself).  NaN and plus infinity may come of the parts of ordinary values and are evaluated again.
__device__ __forceinline__ bool settled(float z) { return z < INFINITY; }
// Key of the others while they wait for that (before every other key, so it passes every bar).
__device__ __forceinline__ uint64_t open_key(uint32_t id) { return id; }
__device__ __forceinline__ bool is_open(uint64_t key) { return (key >> 32) == 0; }

// (2), (4) Scores of the neurons j0 + c * stride, c < nc (clamped to the layer), for all samples.
// The 32-bit product is formed from bf16 products: with x = x0 + x1 + x2 the six products of parts whose
// indices add up to at most two are accumulated in 32 bits; the three left out are below 2^-25 of |h||w| each,
// the size of one rounding of the 32-bit chain this replaced.  The six products of a coordinate block are summed by
// themselves and then added to the rest (the bias last), the same way in every variant: the sampled neurons' scores have
// to be what the pass over all neurons finds.  Relative error against 64 bits, chain / six products added to the
// whole sum / this: 1.2e-7, 1.3e-7 and 5.5e-8 with 128 coordinates, 1.7e-7, 1.8e-7 and 6.8e-8 with 256, 3.2e-7, 3.6e-7 and
// 1.2e-7 with 1,024; it costs 5 % of the call with 256 samples (this kernel 298 -> 313 us), 1 % and less below 128.
// Six bf16 passes at 1/16 of the cost each against one pass at the 32-bit matrix rate: those 44 GFLOP took 564 us
// there, 110 of them for writing the scores, and 304 here in stages of 256 samples (matrix cores busy 41 % of the time), 260 in resident blocks of 128.
// Product rows are samples, columns neurons.  A wave owns 32 neurons and all NIB * 32 samples of the
// workgroup: its W2 values come straight from memory, two coordinate blocks ahead (also across tiles: the
// workgroups are persistent), and are split in registers; h, split once in advance, is staged in LDS in
// fragment order -- RES: it all fits (res_frags), is staged once, and the waves never meet again; otherwise the next stage is fetched under the products of this one.
// kStore: every score goes to zs; kGroupBest: the best of every 32 neurons does, as a key (the sampled neurons);
// kCandidates: the scores that reach their sample's bar go to its candidate buffer.
enum { kCandidates, kStore, kGroupBest };
// Forms.  kStages: h is staged in LDS in turns; kResident: it all fits (res_frags), is staged once, and the waves never meet
// again; kStream: the same for up to 32 samples, which are bound by reading W2: the wave reads its rows 128 bytes at a time
// (eight lanes to a row), streaming, and turns them over through its corner of the LDS.  8 samples x 670K neurons: 64.7 us
// (5.3 TB/s) against 75 (4.6) for lanes that read their own rows 32 bytes at a time -- a plain read of W2 in either pattern takes 52 and 61 us,
// and streaming loads of half lines 101, so the rows have to be whole lines (launch_dense_topk).  A wave has a stretch of
// neighbouring neurons, as long as any other's, instead of tiles dealt out in turn (5.1 rounds of them took as long as 6).
enum { kStages, kResident, kStream };
__host__ __device__ constexpr int score_threads(int MODE, int FORM) { return FORM != kStream ? kScoreThreads : MODE == kCandidates ? 1024 : 256; }
__host__ __device__ constexpr int score_waves_per_simd(int NIB, int MODE, int FORM) {
  return FORM == kStream ? (MODE == kCandidates ? 4 : 2) : FORM == kStages || NIB == 4 ? 2 : NIB == 2 && MODE != kCandidates ? 3 : 4;
}
template <int NIB, int MODE, int FORM>
__global__ __launch_bounds__(score_threads(MODE, FORM), score_waves_per_simd(NIB, MODE, FORM)) void dense_scores_kernel(
    int B, int64_t N, int H, int nkbp, const float4* frags, const float* __restrict__ W2, const float* __restrict__ b2, int64_t j0, int nc, int stride, float* __restrict__ zs,
    const uint64_t* __restrict__ bars, uint64_t* __restrict__ cand, uint32_t* ccnt, int cand_cap, int per_wave, const float* __restrict__ h) {
  // (The order of the arguments: what every form reads first is in the first line of them.  With h before frags the last of these
  // were read behind the first barrier, and all scores of 3,192 neurons x 296 for 473 samples took 18.6 us for 18.1.)
  constexpr bool RES = FORM != kStages, STREAM = FORM == kStream;
  constexpr int THREADS = score_threads(MODE, FORM);
  constexpr int MB = NIB * 32;                           // samples per workgroup
  constexpr int KS = stage_blocks(NIB);                  // coordinate blocks per stage
  constexpr int PIECES = NIB * KS * 192;                 // 16-byte pieces of a stage
  constexpr int PPT = (RES ? res_frags(NIB) * 192 : PIECES) / THREADS;   // ... per thread
  extern __shared__ f32x4 hs[];                          // [row block][coordinate block][part][lane], twice unless RES; the waves' corners
  __shared__ uint64_t bar_s[MB];
  __shared__ float thr[MB];                              // score of the bar
  __shared__ __attribute__((aligned(16))) float thr4[MB / 4];   // lowest of four samples' (row block, half, group)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, half = lane >> 5;
  const int i0 = blockIdx.y * MB, rows = min(B - i0, MB);
  const int ntiles = (nc + kTileNeurons - 1) / kTileNeurons;
  if (!STREAM && (int)blockIdx.x >= ntiles) return;
  // kGroupBest: group g of 32 is columns g, g + ngroups, ...: a stride apart, or where scores follow the ids the best of a
  // stretch of the layer would be the best of a few groups only, and the bar as low as the worst of them.
  const int ngroups = (nc + 31) / 32, npos = MODE == kGroupBest ? ngroups * 32 : nc;
  auto column_at = [&](int pos) { return MODE == kGroupBest ? (pos & 31) * ngroups + (pos >> 5) : pos; };
  // kStream: the wave's neurons are at positions c_lo .. c_hi - 1, in tiles of 32
  const int c_lo = STREAM ? min((int)(blockIdx.x * (THREADS / 64) + wave) * per_wave, npos) : 0, c_hi = STREAM ? min(c_lo + per_wave, npos) : npos;
  auto position = [&](int tile) { return STREAM ? c_lo + tile * 32 + col : tile * kTileNeurons + wave * 32 + col; };
  // coordinate blocks to go through (at least four where they are staged: the loads run two blocks ahead, and no
  // further than the next tile)
  const int nkb = RES ? (H + 15) / 16 : max(4, (H + 16 * KS - 1) / (16 * KS) * KS);
  const f32x4* mine = (const f32x4*)frags + (size_t)blockIdx.y * NIB * nkbp * 192;

  // The stage that starts at block kb0 (RES: everything), a fragment part (1 KB) per wave and step: part q % per
  // of row block q / per.
  constexpr int WAVES = THREADS / 64;
  const int per = RES ? nkb * 3 : KS * 3;
  auto fetch = [&](int kb0, int u) -> f32x4 {
    const int q = min(u * WAVES + wave, NIB * per - 1), ib = q / per, r = q - ib * per;
    return mine[((size_t)(ib * nkbp + kb0) * 3 + r) * 64 + lane];
  };
  auto put = [&](int buf, int u, const f32x4& x) {
    const int q = u * WAVES + wave;
    if (!RES || q < NIB * per) hs[(RES ? 0 : buf * PIECES) + q * 64 + lane] = x;
  };
  auto neuron_of = [&](int tile) -> int64_t {
    const int64_t j = j0 + (int64_t)column_at(position(tile)) * stride;
    return j < N ? j : N - 1;                            // (columns past the end are not looked at)
  };
  // The W2 values to come: block lk of tile lt.  (Loads are unconditional, so that the waits for them can be
  // counted: past the end of the row the last four values are read again, against zeros of h.)
  int lt = blockIdx.x, lk = 0;
  const float* wrow = W2 + (size_t)neuron_of(lt) * H;
  const float* wnext = wrow;                             // the row of the workgroup's next tile (!RES)
  const int kmax = H - 4;
  float4 wb0[2], wb1[2];
  auto issue = [&](float4 (&w)[2]) {
    const int k = lk * 16 + 8 * half;
    w[0] = *(const float4*)(wrow + min(k, kmax));
    w[1] = *(const float4*)(wrow + min(k + 4, kmax));
    if (RES) {
      if (++lk == nkb) {
        lk = 0;
        lt = lt + (int)gridDim.x < ntiles ? lt + (int)gridDim.x : lt;
        wrow = W2 + (size_t)neuron_of(lt) * H;
      }
    } else {                                             // (a branch would let the compiler move the stage's loads behind it)
      const bool wrap = lk + 1 == nkb;
      lk = wrap ? 0 : lk + 1;
      wrow = wrap ? wnext : wrow;
    }
  };
  // kStream: a stage is two coordinate blocks of the wave's 32 rows, 8 lanes of 16 bytes to a row; DEPTH of them ahead.
  constexpr int DEPTH = !STREAM ? 1 : MODE == kGroupBest ? 4 : 2;
  const int nst = nkb / 2;                               // (kStream: H is a multiple of 32)
  f32x4 sb[DEPTH][4];
  int st = 0, ss = 0;                                    // tile and stage to come
  const int piece = lane & 7, row8 = lane >> 3;
  auto issue_stage = [&](f32x4 (&x)[4]) {
    const int k = ss * 32 + 4 * piece;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      int64_t j = j0 + (int64_t)column_at(max(min(c_lo + st * 32 + d * 8 + row8, c_hi - 1), 0)) * stride;
      if (MODE == kGroupBest) j = min(j, N - 1);         // (a group's last column may lie past the end)
      const f32x4* at = (const f32x4*)(W2 + (size_t)j * H + k);
      x[d] = MODE == kCandidates ? __builtin_nontemporal_load(at) : *at;
    }
    const bool wrap = ss + 1 == nst;
    ss = wrap ? 0 : ss + 1;
    st += wrap ? 1 : 0;                                  // (past the last tile: its last row again)
  };
  if constexpr (STREAM) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) issue_stage(sb[d]);
  } else {
    issue(wb0);
    issue(wb1);
  }
  if (MODE == kCandidates)
    for (int q = tid; q < MB; q += THREADS) {
      const uint64_t bar = q < rows ? bars[i0 + q] : 0ull;
      bar_s[q] = bar;
      thr[q] = q >= rows ? INFINITY : bar == ~0ull ? -INFINITY : topk_score(bar);
    }
  for (int u = 0; u < PPT; ++u) put(0, u, fetch(0, u));
  __syncthreads();
  if constexpr (MODE == kCandidates) {
    if (tid < MB / 4) {
      const float* t = thr + (tid >> 3) * 32 + 8 * (tid & 3) + 4 * ((tid >> 2) & 1);
      thr4[tid] = fminf(fminf(t[0], t[1]), fminf(t[2], t[3]));
      if (t[0] != t[0] || t[1] != t[1] || t[2] != t[2] || t[3] != t[3]) thr4[tid] = -INFINITY;   // (a bar of NaN)
    }
    __syncthreads();
  }

  // the wave's corner: half a 32x32 block of scores, and the scores that passed the first test (score, column,
  // sample), handed to the samples' buffers together when the list fills and at the end: the exact test (ties by
  // id) and a lane's counter update and store each
  constexpr int BOUNCE = STREAM ? 1024 : 512;            // (kStream: the wave's rows pass through it, too)
  float* bounce = (float*)(hs + (RES ? NIB * nkb * 192 : 2 * PIECES)) + wave * (BOUNCE + (MODE == kCandidates ? 3 * kListed : 0));
  float* list_z = bounce + BOUNCE;
  int* list_c = (int*)list_z + kListed;
  int* list_i = list_c + kListed;
  int listed = 0;
  auto flush = [&]() {
    __builtin_amdgcn_wave_barrier();
    for (int q = lane; q < listed; q += 64) {
      const float z = list_z[q];
      const int il = list_i[q];
      const uint32_t id = (uint32_t)(j0 + (int64_t)list_c[q] * stride);
      const uint64_t key = settled(z) ? topk_key(z, id) : open_key(id);
      // (rows past the batch have no buffer; a non-finite weight times their zeros is NaN and passes the first test)
      if (il < rows && key <= bar_s[il]) {
        const uint32_t pos = atomicAdd(&ccnt[(size_t)(i0 + il) * kCntPitch], 1u);
        if (pos < (uint32_t)cand_cap) cand[(size_t)(i0 + il) * cand_cap + pos] = key;
      }
    }
    __builtin_amdgcn_wave_barrier();
    listed = 0;
  };

  f32x16 acc[NIB];
  // the products of one coordinate block: block kl of what hb points at
  auto contract = [&](float4 (&wr)[2], const bf16x8* hb, int ib_pitch) {
    bf16x8 w[3];
    split8(wr[0], wr[1], w);
    if (!STREAM) issue(wr);
    if (!RES) asm volatile("" ::: "memory");             // (not later: see below)
    constexpr int G = NIB < 2 || (RES && NIB < 4) ? 1 : 2;            // row blocks interleaved (independent sums)
#pragma unroll
    for (int ib = 0; ib < NIB; ib += G) {
      bf16x8 a[G][3];
      f32x16 t[G];
#pragma unroll
      for (int g = 0; g < G; ++g) {
#pragma unroll
        for (int p = 0; p < 3; ++p) a[g][p] = hb[(ib + g) * ib_pitch + p * 64];
#pragma unroll
        for (int r = 0; r < 16; ++r) t[g][r] = 0.f;
      }
#pragma unroll
      for (int pr = 0; pr < 6; ++pr) {
        constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};   // small products first
#pragma unroll
        for (int g = 0; g < G; ++g)
          t[g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[g][pa[pr]], w[pb[pr]], t[g], 0, 0, 0);
      }
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[ib + g][r] += t[g][r];
    }
  };
  auto clear = [&]() {
#pragma unroll
    for (int ib = 0; ib < NIB; ++ib)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[ib][r] = 0.f;
  };
  auto finish = [&](int tile, float bias) {
    // lane holds column `col`, rows 8*(r/4) + 4*half + r%4 of each 32x32 block
    const int pos = position(tile), c = column_at(pos);
    const bool live = pos < c_hi && c < nc;
    if constexpr (MODE == kStore) {
#pragma unroll
      for (int ib = 0; ib < NIB; ++ib)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int il = ib * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
          if (live && il < rows) zs[(size_t)(i0 + il) * nc + c] = acc[ib][r] + bias;
        }
    } else if constexpr (MODE == kGroupBest) {
      // the best of the wave's 32 neurons for every sample, as its key (~0: none)
      const int group = STREAM ? c_lo / 32 + tile : tile * (kTileNeurons / 32) + wave;
#pragma unroll
      for (int ib = 0; ib < NIB; ++ib) {
        float z[16];
        bool open = false;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          z[r] = acc[ib][r] + bias;
          open |= !settled(z[r]);
        }
        if (__any(open)) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int il = ib * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
            if (live && il < rows && !settled(z[r]))
              z[r] = plain_score(h + (size_t)(i0 + il) * H, W2 + (size_t)neuron_of(tile) * H, bias, H);
          }
        }
        const uint32_t none = live ? 0u : ~0u, id = (uint32_t)(j0 + (int64_t)c * stride) | none;
        uint64_t v[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = topk_key(z[r], id) | (uint64_t)none << 32;
        // 32 lanes and 16 rows: every step halves the rows that a lane goes on with and takes the best of two lanes
        auto halve = [&](int n, bool upper, auto&& other) {
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            if (q >= n) break;
            const uint64_t keep = upper ? v[n + q] : v[q], give = upper ? v[q] : v[n + q];
            v[q] = min(keep, (uint64_t)other((uint32_t)(give >> 32)) << 32 | other((uint32_t)give));
          }
        };
        auto swap16 = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, 16 << 10 | 0x1f); };
        halve(8, lane & 1, [](uint32_t x) { return dpp_u32<kDppQuadSwap1>(x, x); });
        halve(4, lane & 2, [](uint32_t x) { return dpp_u32<kDppQuadSwap2>(x, x); });
        halve(2, lane & 8, [](uint32_t x) { return dpp_u32<kDppRowRor + 8>(x, x); });
        halve(1, lane & 4, [](uint32_t x) { return (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, 4 << 10 | 0x1f); });
        const uint64_t best = min(v[0], (uint64_t)swap16((uint32_t)(v[0] >> 32)) << 32 | swap16((uint32_t)v[0]));
        const int r = (lane & 1 ? 8 : 0) + (lane & 2 ? 4 : 0) + (lane & 8 ? 2 : 0) + (lane & 4 ? 1 : 0);
        const int il = ib * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
        if (col < 16 && il < rows && group < ngroups) ((uint64_t*)zs)[(size_t)(i0 + il) * ngroups + group] = best;
      }
    } else {
      // First test, whole blocks: the largest of four consecutive samples' scores (NaN counts as largest) against
      // the lowest of their bars.  The blocks in which something passes (about half of them) go through the wave's
      // corner of the LDS, half a block at a time, and every lane hands on what reaches its own bar.
      uint32_t todo = 0;
#pragma unroll
      for (int ib = 0; ib < NIB; ++ib) {
        const float4 low = *(const float4*)&thr4[(ib * 2 + half) * 4];
        const float t[4] = {low.x, low.y, low.z, low.w};
        bool pass = false;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float top = __builtin_elementwise_maximum(__builtin_elementwise_maximum(acc[ib][4 * g], acc[ib][4 * g + 1]),
                                                          __builtin_elementwise_maximum(acc[ib][4 * g + 2], acc[ib][4 * g + 3]));
          pass |= !(top + bias < t[g]);                  // (the rounded sum grows with its first operand)
        }
        if (__any(live && pass)) todo |= 1u << ib;
      }
#pragma unroll 1
      while (todo) {
        const int ib = __ffs(todo) - 1;
        todo &= todo - 1;
#pragma unroll 1
        for (int hf = 0; hf < 2; ++hf) {
          uint32_t mask = 0;                             // rows of this half block that the lane hands on
#pragma unroll
          for (int I = 0; I < 2 * NIB; ++I)
            if (2 * ib + hf == I) {
#pragma unroll
              for (int q = 0; q < 8; ++q) {
                const int r = 8 * (I & 1) + q, il = (I >> 1) * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                const float z = acc[I >> 1][r] + bias;
                bounce[q * 64 + lane] = z;
                mask |= !(z < thr[il]) ? 1u << q : 0u;
              }
            }
          if (!live) mask = 0;
#pragma unroll 1
          while (true) {
            const unsigned long long m = __ballot(mask != 0u);
            if (!m) break;
            if (listed + 64 > kListed) flush();
            if (mask) {
              const int q = __ffs(mask) - 1, r = 8 * hf + q;
              mask &= mask - 1;
              const int at = listed + __popcll(m & ((1ull << lane) - 1ull));
              list_z[at] = bounce[q * 64 + lane];
              list_c[at] = c;
              list_i[at] = ib * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
            }
            listed += __popcll(m);
          }
        }
      }
    }
  };
  const bf16x8* hb = (const bf16x8*)hs + lane;
  if constexpr (STREAM) {
    const int units = (c_hi - c_lo + 31) / 32 * nst;
    int tile = 0, kb = 0;
    float bias = 0.f, bias_next = b2[neuron_of(0)];
    // pieces of a row are permuted among each other by the row's number, so that neither eight lanes with a row
    // nor eight lanes with a row each meet in a bank
    f32x4* put_at = (f32x4*)bounce + row8 * 8 + (piece ^ row8);
    const f32x4* get_at = (const f32x4*)bounce + col * 8;
    auto unit = [&](f32x4 (&x)[4]) {
      if (kb == 0) {
        clear();
        bias = bias_next;
        bias_next = b2[neuron_of(tile + 1)];
      }
#pragma unroll
      for (int d = 0; d < 4; ++d) put_at[d * 64] = x[d];
      issue_stage(x);
      asm volatile("" ::: "memory");                     // (a wave's accesses to its corner are in order)
      __builtin_amdgcn_wave_barrier();
      f32x4 y[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) y[q] = get_at[((q >> 1) * 4 + half * 2 + (q & 1)) ^ (col & 7)];
      asm volatile("" ::: "memory");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        float4 w[2] = {make_float4(y[2 * b][0], y[2 * b][1], y[2 * b][2], y[2 * b][3]),
                       make_float4(y[2 * b + 1][0], y[2 * b + 1][1], y[2 * b + 1][2], y[2 * b + 1][3])};
        contract(w, hb + (kb + b) * 192, nkb * 192);
      }
      kb += 2;
      if (kb < nkb) return;
      finish(tile, bias);
      kb = 0;
      ++tile;
    };
    for (int u = 0; u < units; u += DEPTH) {
#pragma unroll
      for (int d = 0; d < DEPTH; ++d)
        if (u + d < units) unit(sb[d]);
    }
  } else if constexpr (RES) {
    const int units = ((ntiles - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x) * nkb;
    int tile = blockIdx.x, kb = 0;
    float bias, bias_next = b2[neuron_of(tile)];
    auto unit = [&](float4 (&wr)[2]) {
      if (kb == 0) {
        clear();
        bias = bias_next;
        bias_next = b2[neuron_of(tile + (int)gridDim.x < ntiles ? tile + (int)gridDim.x : tile)];
      }
      contract(wr, hb + kb * 192, nkb * 192);
      if (++kb < nkb) return;
      finish(tile, bias);
      kb = 0;
      tile += gridDim.x;
    };
    for (int u = 0; u < units; u += 2) {
      unit(wb0);
      if (u + 1 < units) unit(wb1);
    }
  } else {
    int buf = 0;
    float bias_next = b2[neuron_of(blockIdx.x)];
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {   // (the same for every wave of the workgroup)
      const int64_t next = neuron_of(tile + (int)gridDim.x < ntiles ? tile + (int)gridDim.x : tile);
      wnext = W2 + (size_t)next * H;
      const float bias = bias_next;
      bias_next = b2[next];
      clear();
      for (int kb = 0; kb < nkb; kb += KS) {
        // the next stage (after the last: the next tile's first)
        const int nkb0 = kb + KS < nkb ? kb + KS : 0;
        static_assert(PPT == 3 || PPT == 6, "fragment parts per wave and stage");
        f32x4 n3, n4, n5;
        const f32x4 n0 = fetch(nkb0, 0), n1 = fetch(nkb0, 1), n2 = fetch(nkb0, 2);
        if constexpr (PPT == 6) { n3 = fetch(nkb0, 3); n4 = fetch(nkb0, 4); n5 = fetch(nkb0, 5); }
        asm volatile("" ::: "memory");                   // These loads stay ahead of the products (the compiler would move
        __builtin_amdgcn_sched_barrier(0);               // them to their use, and does so with pointers it knows to be
                                                         // read-only: frags and W2 are not __restrict__).
#pragma unroll
        for (int kl = 0; kl < KS; kl += 2) {
          contract(wb0, hb + buf * PIECES + kl * 192, KS * 192);
          contract(wb1, hb + buf * PIECES + (kl + 1) * 192, KS * 192);
        }
        __builtin_amdgcn_sched_barrier(0);
        put(buf ^ 1, 0, n0); put(buf ^ 1, 1, n1); put(buf ^ 1, 2, n2);
        if constexpr (PPT == 6) { put(buf ^ 1, 3, n3); put(buf ^ 1, 4, n4); put(buf ^ 1, 5, n5); }
        __syncthreads();
        buf ^= 1;
      }
      finish(tile, bias);
    }
  }
  if constexpr (MODE == kCandidates) flush();
}

// (3) Per sample, when every neuron was sampled: the topk best of the scores.  (Column c is neuron c * stride.  The stride is 1
// here, but a compiler that knows it keeps the addresses of all rows that may have to be read again: 138 registers for 80 and,
// for 473 samples x 3,192 neurons, 11.6 us for 11.1.)
__global__ __launch_bounds__(kSelectThreads) void dense_select_kernel(int H, const float* __restrict__ h,
                                                                      const float* __restrict__ W2,
                                                                      const float* __restrict__ b2, int nc, int stride,
                                                                      const float* __restrict__ zs, int topk,
                                                                      int32_t* __restrict__ out_ids,
                                                                      float* __restrict__ out_scores) {
  __shared__ SelectLds lds;
  const int i = blockIdx.x, tid = threadIdx.x;
  const float* row = zs + (size_t)i * nc;
  constexpr int UN = 16;                                 // scores per thread in flight
  const int found = select_topk(lds, topk, [&](auto&& f) {
    for (int c0 = tid; c0 < nc; c0 += UN * kSelectThreads) {
      float z[UN];
#pragma unroll
      for (int u = 0; u < UN; ++u) z[u] = row[min(c0 + u * kSelectThreads, nc - 1)];
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        const int c = c0 + u * kSelectThreads;
        if (c >= nc) continue;
        const uint32_t j = (uint32_t)c * (uint32_t)stride;
        if (!settled(z[u])) z[u] = plain_score(h + (size_t)i * H, W2 + (size_t)j * H, b2[j], H);
        f(topk_key(z[u], j));
      }
    }
  }, [&](int place, uint64_t key) {
    out_ids[(size_t)i * topk + place] = (int32_t)(uint32_t)key;
    out_scores[(size_t)i * topk + place] = topk_score(key);
  });
  for (int k = found + tid; k < topk; k += kSelectThreads) {
    out_ids[(size_t)i * topk + k] = -1;
    out_scores[(size_t)i * topk + k] = -INFINITY;
  }
}

// (3) Per sample: the topk-th best of the groups' bests as the bar, which at least topk neurons reach (one of each of
// as many groups; the topk-th best of all sampled neurons is hardly higher: groups hold 32 of them from all over the layer,
// 256 groups and more).
// A wave per sample; the bar's score is found bit by bit, by counting the groups that reach what is tried, and then its id
// among the groups that are tied there.  (The bar is a key, id and all: where many neurons share the bar's score only those of
// lower ids pass.  With the score alone a sample whose scores were all the same took 27 ms for 90 us.  The topk-th
// best of the scores themselves, which this replaced, took two sweeps over 8,192 of them, 14 us.)
__global__ __launch_bounds__(64) void dense_bar_kernel(int ngroups, const uint64_t* __restrict__ best, int topk,
                                                       uint64_t* __restrict__ bars, uint32_t* __restrict__ ccnt) {
  constexpr int U = kMaxGroups / 64;
  const int i = blockIdx.x, lane = threadIdx.x;
  uint32_t v[U], id[U];                                  // keys: bits that ascend as scores fall, and ids
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint64_t key = u * 64 + lane < ngroups ? best[(size_t)i * ngroups + u * 64 + lane] : ~0ull;
    v[u] = (uint32_t)(key >> 32);
    id[u] = (uint32_t)key;
  }
  auto count = [&](auto&& has) {
    int n = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) n += __popcll(__ballot(has(u)));
    return n;
  };
  // the smallest value that topk groups are within, or any that just topk are
  uint32_t bar = 0, within = 0;
  bool found = false;
  for (int bit = 31; bit >= 0 && !found; --bit) {
    within = bar | ((1u << bit) - 1u);
    const int n = count([&](int u) { return v[u] <= within; });
    found = n == topk;
    if (n < topk) bar |= 1u << bit;
  }
  uint32_t bar_id = 0;
  if (found) {                                           // the last of these
    uint32_t m = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) m = max(m, v[u] <= within ? v[u] : 0u);
    bar = wave_max(m);
    m = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) m = max(m, v[u] == bar ? id[u] : 0u);
    bar_id = wave_max(m);
  } else {                                               // more than that are tied at the bar: the lowest id that enough of them are within
    const int need = topk - count([&](int u) { return v[u] < bar; });
    for (int bit = 31; bit >= 0; --bit) {
      const uint32_t trial = bar_id | ((1u << bit) - 1u);
      if (count([&](int u) { return v[u] == bar && id[u] <= trial; }) < need) bar_id |= 1u << bit;
    }
  }
  if (lane == 0) {
    bars[i] = bar == ~0u ? ~0ull : (uint64_t)bar << 32 | bar_id;   // (~0: fewer groups have a score, everything passes)
    ccnt[(size_t)i * kCntPitch] = 0;
  }
}

// The same for neurons j0 .. j0 + 255 (before j1; H a multiple of four), one for every thread of the workgroup: neuron
// j0 + 16 * (thread % 16) + thread / 16.  Sixteen lanes read a row together.
__device__ __forceinline__ float plain_scores(const float* __restrict__ h, const float* __restrict__ W2, const float* __restrict__ b2,
                                              int64_t j0, int64_t j1, int H) {
  static_assert(kSelectThreads == 256, "sixteen rows of sixteen lanes");
  const int l = threadIdx.x & 15, g = threadIdx.x >> 4;
  float mine = 0.f;
  for (int s0 = 0; s0 < 16; s0 += 8) {
    float p[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) p[u] = 0.f;
    for (int c = 4 * l; c < H; c += 64) {
      const float4 a = *(const float4*)(h + c);
      float4 b[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) b[u] = *(const float4*)(W2 + (size_t)min(j0 + (s0 + u) * 16 + g, j1 - 1) * H + c);
#pragma unroll
      for (int u = 0; u < 8; ++u) p[u] = fmaf(a.w, b[u].w, fmaf(a.z, b[u].z, fmaf(a.y, b[u].y, fmaf(a.x, b[u].x, p[u]))));
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
#pragma unroll
      for (int d = 1; d < 16; d <<= 1) p[u] += __shfl_xor(p[u], d);
      if (l == s0 + u) mine = p[u];
    }
  }
  return mine + b2[min(j0 + l * 16 + g, j1 - 1)];
}

// (5) Per sample: folds the candidates of one launch of scores into the running list of the topk best
// (best[i][0..64), read when `first` is 0); the last launch writes the result.  A sample with more candidates
// than its buffer holds (most scores are no numbers, as after divergence, or the neurons that reach the bar sit between
// the sampled ones: see launch_dense_topk for how unlikely chance makes that) evaluates the launch's neurons itself,
// twice or more: tens of milliseconds for a layer of 670K x 128, which one workgroup reads at 20 GB/s (8 and 256 such
// samples: 36 and 48; a row per thread took 98 and 118).
__global__ __launch_bounds__(kSelectThreads) void dense_merge_kernel(int H, const float* __restrict__ h,
                                                                     const float* __restrict__ W2,
                                                                     const float* __restrict__ b2, int64_t j0, int nc, int topk,
                                                                     uint64_t* __restrict__ best, uint64_t* __restrict__ bars,
                                                                     int first, int last, const uint64_t* __restrict__ cand,
                                                                     uint32_t* ccnt, int cand_cap,
                                                                     int32_t* __restrict__ out_ids,
                                                                     float* __restrict__ out_scores) {
  __shared__ SelectLds lds;
  __shared__ uint64_t list[64];
  const int i = blockIdx.x, tid = threadIdx.x;
  const uint32_t ncand = ccnt[(size_t)i * kCntPitch];
  if (tid < 64) list[tid] = !first && tid < topk ? best[(size_t)i * 64 + tid] : ~0ull;
  __syncthreads();
  const uint64_t* mine = cand + (size_t)i * cand_cap;
  constexpr int UN = 4;
  const int found = select_topk(lds, topk, [&](auto&& f) {
    if (tid < 64) f(list[tid]);
    if (ncand <= (uint32_t)cand_cap) {
      for (uint32_t q0 = tid; q0 < ncand; q0 += UN * kSelectThreads) {
        uint64_t k[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) k[u] = mine[min(q0 + (uint32_t)(u * kSelectThreads), ncand - 1u)];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
          if (q0 + (uint32_t)(u * kSelectThreads) >= ncand) continue;
          const uint32_t j = (uint32_t)k[u];
          if (is_open(k[u])) k[u] = topk_key(plain_score(h + (size_t)i * H, W2 + (size_t)j * H, b2[j], H), j);
          f(k[u]);
        }
      }
    } else {
      for (int64_t c = j0; c < j0 + nc; c += kSelectThreads) {   // (every thread of the workgroup)
        const float z = plain_scores(h + (size_t)i * H, W2, b2, c, j0 + nc, H);
        const int64_t j = c + (tid & 15) * 16 + (tid >> 4);
        if (j < j0 + nc) f(topk_key(z, (uint32_t)j));
      }
    }
  }, [&](int place, uint64_t key) {
    if (last) {
      out_ids[(size_t)i * topk + place] = (int32_t)(uint32_t)key;
      out_scores[(size_t)i * topk + place] = topk_score(key);
    } else {
      best[(size_t)i * 64 + place] = key;
      if (place == topk - 1 && key < bars[i]) bars[i] = key;
    }
  });
  for (int k = found + tid; k < topk; k += kSelectThreads) {
    if (last) {
      out_ids[(size_t)i * topk + k] = -1;
      out_scores[(size_t)i * topk + k] = -INFINITY;
    } else {
      best[(size_t)i * 64 + k] = ~0ull;
    }
  }
  if (tid == 0) ccnt[(size_t)i * kCntPitch] = 0;
}

// ---- host side --------------------------------------------------------------------------------------
static int dense_stride(int64_t N) { return (int)std::max<int64_t>(1, N / kSampled); }
static int64_t dense_sampled(int64_t N) { return (N + dense_stride(N) - 1) / dense_stride(N); }
static int dense_cand_cap(int64_t N) { return (int)std::min<int64_t>(N, kCandMax); }
static int padded_blocks(int H) { return ceil_div(ceil_div(H, 16), kBlockPad) * kBlockPad; }
static int dense_row_blocks(int B) { return B <= 32 ? 1 : B <= 64 ? 2 : B <= 128 ? 4 : 8; }

DenseLayout dense_layout(int Bmax, int64_t N, int H) {
  DenseLayout d;
  size_t o = 0;
  auto take = [&](size_t bytes) { const size_t at = o; o = (o + bytes + 255) / 256 * 256; return at; };
  const size_t B = (size_t)Bmax, MB = (size_t)dense_row_blocks(Bmax) * 32, rows = (B + MB - 1) / MB * MB;
  d.frags = take(rows * (size_t)padded_blocks(H) * 16 * 6);
  d.zs = take(B * (size_t)dense_sampled(N) * 4);
  d.bars = take(B * 8);
  d.best = take(B * 64 * 8);
  d.cand = take(B * (size_t)dense_cand_cap(N) * 8);
  d.ccnt = take(B * kCntPitch * 4);
  d.total = o;
  return d;
}

// Whether blocks of 128 samples stay in LDS for more than 64 samples (staged in turns otherwise, up to 256 to a workgroup).  A
// workgroup has to fetch them all before it starts.  With one tile of neurons it has nothing to make that up with, unless
// the stages would be padded: 128 samples x 40,000 neurons staged / resident, us: 128 coordinates 51.6 / 53.6, 64 1 %
// for staged, 96 50.5 / 48.5, 160 2 % for resident.  Up to 192 samples as two such blocks need a round of
// tiles to be saved against one of 256: 129 x 65,000 x 128 4 % for staged, x 70,000 (three rounds of 128, two of 256) 11 % for
// resident; from 193 on their second block is full enough (-1 to +7 %).
static bool blocks_stay(int B, int nkb, int ntiles, int num_cus) {
  if (4 * nkb > res_frags(4)) return false;
  if (B <= 128) return ntiles > num_cus || nkb % stage_blocks(4) != 0;
  if (B > 192 || ntiles > 2 * num_cus || nkb % stage_blocks(8) != 0) return true;
  return ceil_div(ntiles, std::max(1, num_cus / 2)) < 2 * ceil_div(ntiles, num_cus);
}

// LDS of a launch: of a resident block (nkb: its coordinate blocks), of the stages otherwise.
static constexpr size_t resident_lds(int NIB, int nkb, bool store) { return (size_t)NIB * nkb * kTriple + (store ? 0 : kCorners); }
// (More than 32 samples: the sampled neurons 14.7 us resident, 19.5 streamed for 256 samples; all of 400K x 64 for 64
// samples 50.6 and 57.6, 670K x 128 about the same.)
static constexpr bool streams(int NIB, int MODE) { return MODE != kStore && NIB == 1; }
static constexpr size_t stream_lds(int NIB, int nkb, int MODE) {
  return (size_t)NIB * nkb * kTriple + (size_t)score_threads(MODE, kStream) / 64 * (1024 + (MODE == kCandidates ? 3 * kListed : 0)) * 4;
}
static constexpr size_t staged_lds(int NIB, bool store) { return (size_t)2 * NIB * stage_blocks(NIB) * kTriple + (store ? 0 : kCorners); }

template <int NIB, int MODE>
static hipError_t launch_scores(bool stay, int B, int64_t N, int H, const float* h, const float4* frags, const float* W2, const float* b2,
                                int64_t j0, int nc, int stride, float* zs, const uint64_t* bars, uint64_t* cand,
                                uint32_t* ccnt, int cand_cap, int num_cus, hipStream_t s) {
  const int nkb = ceil_div(H, 16), nkbp = padded_blocks(H), gy = ceil_div(B, NIB * 32), ntiles = ceil_div(nc, kTileNeurons);
  const bool res = stay && NIB <= 4 && NIB * nkb <= res_frags(NIB);
  // as many workgroups as fit: two of up to 64 resident samples per compute unit (registers; their LDS is half of the unit's at
  // most, H = 256), one otherwise
  const int per_cu = res && NIB < 4 ? 2 : 1;
  const int gx = std::max(1, std::min(ntiles, num_cus * per_cu / std::min(gy, num_cus)));
  const dim3 grid(gx, gy), block(kScoreThreads);
  if constexpr (streams(NIB, MODE)) {
    // whole lines of W2, neurons enough that a wave's stretch is more than a tile or two
    if (res && H % 32 == 0 && ((uintptr_t)W2 & 127) == 0 && (MODE == kGroupBest || nc >= kStreamNeurons)) {
      constexpr int WAVES = score_threads(MODE, kStream) / 64;
      const int groups = MODE == kGroupBest ? ceil_div(ceil_div(nc, 32), WAVES) : num_cus;
      const int per_wave = MODE == kGroupBest ? 32 : ceil_div(nc, groups * WAVES);
      hipLaunchKernelGGL((dense_scores_kernel<NIB, MODE, kStream>), dim3(groups, gy), dim3(WAVES * 64), stream_lds(NIB, nkb, MODE), s, B, N, H,
                         nkbp, frags, W2, b2, j0, nc, stride, zs, bars, cand, ccnt, cand_cap, per_wave, h);
      return hipGetLastError();
    }
  }
  if constexpr (NIB <= 4) {
    if (res) {
      hipLaunchKernelGGL((dense_scores_kernel<NIB, MODE, kResident>), grid, block, resident_lds(NIB, nkb, MODE != kCandidates), s, B, N, H, nkbp, frags, W2, b2,
                         j0, nc, stride, zs, bars, cand, ccnt, cand_cap, 0, h);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((dense_scores_kernel<NIB, MODE, kStages>), grid, block, staged_lds(NIB, MODE != kCandidates), s, B, N, H, nkbp, frags, W2,
                     b2, j0, nc, stride, zs, bars, cand, ccnt, cand_cap, 0, h);
  return hipGetLastError();
}

template <int NIB, int MODE>
static hipError_t scores_attr() {
  constexpr bool STORE = MODE != kCandidates;
  hipError_t e = hipFuncSetAttribute((const void*)dense_scores_kernel<NIB, MODE, kStages>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)staged_lds(NIB, STORE));
  if constexpr (NIB <= 4)
    if (e == hipSuccess) e = hipFuncSetAttribute((const void*)dense_scores_kernel<NIB, MODE, kResident>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)resident_lds(NIB, res_frags(NIB) / NIB, STORE));
  if constexpr (streams(NIB, MODE))
    if (e == hipSuccess) e = hipFuncSetAttribute((const void*)dense_scores_kernel<NIB, MODE, kStream>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)stream_lds(NIB, res_frags(NIB) / NIB, MODE));
  return e;
}

// words of LDS for the rows of W1 of one sample: 64 KB, more for rows so long that 32 of them need it
static int prepare_stage_words(int H) { return (H <= 448 ? 64 : 144) * 256; }

hipError_t predict_setup_attributes() {
  hipError_t e = hipFuncSetAttribute((const void*)dense_prepare_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 156 * 1024);
  if (e == hipSuccess) e = scores_attr<1, kStore>();
  if (e == hipSuccess) e = scores_attr<2, kStore>();
  if (e == hipSuccess) e = scores_attr<1, kGroupBest>();
  if (e == hipSuccess) e = scores_attr<2, kGroupBest>();
  if (e == hipSuccess) e = scores_attr<1, kCandidates>();
  if (e == hipSuccess) e = scores_attr<2, kCandidates>();
  if (e == hipSuccess) e = scores_attr<4, kCandidates>();
  if (e == hipSuccess) e = scores_attr<8, kCandidates>();
  return e;
}

hipError_t launch_dense_prepare(int B, int H, const float* h, const SpmmArgs& sp, char* scratch, const DenseLayout& d,
                                Ctrl* ctrl, hipStream_t s) {
  const int MB = dense_row_blocks(B) * 32, words = sp.W1 ? prepare_stage_words(H) : 0;
  hipLaunchKernelGGL(dense_prepare_kernel, dim3(ceil_div(B, MB) * MB), dim3(sp.W1 ? 1024 : 256), (size_t)(words + H) * 4, s, B, H,
                     padded_blocks(H), h, sp, (bf16x8*)(scratch + d.frags), ctrl, words);
  return hipGetLastError();
}

hipError_t launch_dense_topk(int B, int64_t N, int H, const float* h, const float* W2, const float* b2, int topk,
                             char* scratch, const DenseLayout& d, int num_cus, int32_t* out_ids, float* out_scores,
                             hipStream_t s) {
  const float4* frags = (const float4*)(scratch + d.frags);
  float* zs = (float*)(scratch + d.zs);
  uint64_t *bars = (uint64_t*)(scratch + d.bars), *best = (uint64_t*)(scratch + d.best), *cand = (uint64_t*)(scratch + d.cand);
  uint32_t* ccnt = (uint32_t*)(scratch + d.ccnt);
  const int stride = dense_stride(N), ns = (int)dense_sampled(N), cap = dense_cand_cap(N);
  const bool all = stride == 1;
  // the sampled neurons are few: small row blocks, so that the samples spread over the machine
#define SLIDE_SAMPLED(NIB, MODE) launch_scores<NIB, MODE>(true, B, N, H, h, frags, W2, b2, 0, ns, stride, zs, nullptr, nullptr, nullptr, 0, num_cus, s)
  if (all) {
    const hipError_t e = B <= 32 ? SLIDE_SAMPLED(1, kStore) : SLIDE_SAMPLED(2, kStore);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(dense_select_kernel, dim3(B), dim3(kSelectThreads), 0, s, H, h, W2, b2, ns, stride, zs, topk, out_ids, out_scores);
    return hipGetLastError();
  }
  hipError_t e = B <= 32 ? SLIDE_SAMPLED(1, kGroupBest) : SLIDE_SAMPLED(2, kGroupBest);
#undef SLIDE_SAMPLED
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(dense_bar_kernel, dim3(B), dim3(64), 0, s, ceil_div(ns, 32), (const uint64_t*)zs, topk, bars, ccnt);
  // The bar is about the r-th best of the sampled neurons: r = topk and a few more, those drawn until topk of the g groups
  // have one (64 of 256: 74).  About r * nc / ns of nc neurons reach it, spread like a sum of r exponentials: with that
  // mean at cap * r / (r + 4 sqrt(r) + 16) -- a 21st of the candidate buffer for topk = 1, 0.59 of it for 64 -- chance
  // overflows it for less than one sample in a million.  A launch takes as many neurons as that allows (6.4 M and 1.1 M).
  const double g = ceil_div(ns, 32), r = std::max<double>(topk, g * std::log(g / (g - topk)));
  const int64_t fit = (int64_t)((double)ns * cap / (r + 4.0 * std::sqrt(r) + 16.0));
  const int64_t most = std::max<int64_t>(kTileNeurons, fit / kTileNeurons * kTileNeurons);
  for (int64_t j0 = 0; j0 < N; j0 += most) {
    const int nc = (int)std::min<int64_t>(std::min<int64_t>(most, (int64_t)1 << 30), N - j0);
#define SLIDE_SCORES(NIB) launch_scores<NIB, kCandidates>(stay, B, N, H, h, frags, W2, b2, j0, nc, 1, nullptr, bars, cand, ccnt, cap, num_cus, s)
    const bool stay = B <= 64 || blocks_stay(B, ceil_div(H, 16), ceil_div(nc, kTileNeurons), num_cus);
    switch (std::min(dense_row_blocks(B), stay ? 4 : 8)) {
      case 1: e = SLIDE_SCORES(1); break;
      case 2: e = SLIDE_SCORES(2); break;
      case 4: e = SLIDE_SCORES(4); break;
      default: e = SLIDE_SCORES(8); break;
    }
#undef SLIDE_SCORES
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(dense_merge_kernel, dim3(B), dim3(kSelectThreads), 0, s, H, h, W2, b2, j0, nc, topk, best, bars,
                       j0 == 0 ? 1 : 0, j0 + nc >= N ? 1 : 0, cand, ccnt, cap, out_ids, out_scores);
  }
  return hipGetLastError();
}

}  // namespace slide
