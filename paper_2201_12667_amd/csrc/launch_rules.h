// Rules that size launches, apart from the kernels so that they can be checked without a GPU (constexpr: host and device).
#pragma once

#include <algorithm>
#include <cstdint>

namespace slide {

constexpr int kForwardWaves = 8;          // waves of a logit workgroup

// Logit workgroups that stay, of the `nworkers` launched, when `ntiles` tiles of row lists ride in their launch and the
// samples have up to `items` work items.  With several items per wave the workers would hold every slot of the machine until
// the end and the tiles would run after them: then the last of them leave at once and make room, more of them when the tiles are
// many for the amount of logit work.  What stays is a multiple of the dies (nxcd > 1): only then can every die keep to its own
// stretch of the neurons.  Launch, us, three workgroups a compute unit cut to 512 or 640 / two cut to 341 or 426 / two cut to
// 336 or 424: 400K x 256 x 200 182 / 217 / 166, 600K x 512 x 180 621 / 636 / 568, 300K x 128 x 150 70 / 77 / 69.
// (Inlined by force: a call costs the kernel three registers, and with them the sixth wave of a SIMD: 24.8 -> 27.3 us for 256
// samples of 256 neurons of 670K x 128.)
__attribute__((always_inline)) inline constexpr int logit_workers(int nworkers, int items, int ntiles, int nxcd) {
  int workers = (ntiles == 0 || items <= 2 * nworkers * kForwardWaves) ? nworkers
                : (items < 20 * ntiles ? nworkers * 2 / 3 : nworkers * 5 / 6);
  if (nxcd > 1 && workers > nxcd) workers -= workers % nxcd;
  return workers;
}

constexpr int kBucketAhead = 8;           // entries of a bucket that a lane of the lookup kernel requests at once

// How a lookup's workgroup of sixteen waves reads what is beyond the first eight entries of every lane (8 << lg of a bucket) in the
// `nlong` buckets that have more, of L tables, at most C entries each, `entries` in all.
//   0: by the lanes of their tables, four entries each at a time.  All buckets at once, but a lane's reads are a chain, and from 512
//      tables on the lanes of an instruction ask for as many lines.
//   else: by waves, four buckets of 128 entries at a time, a wave the long ones of that many tables: of a sixteenth of them, or, of 256
//      tables and more of which few have one, an eighth (a few full waves are faster than many with a bucket each).
// Few long buckets (64) go by waves: by lanes 4 samples of 670K neurons with a few each take 39 us for 33.  More go by lanes where
// these take fewer steps of their longest bucket, which is taken for twice the mean, than waves take for all: three half steps for
// each four buckets of a wave.  Retrievals, us, by lanes / by waves (when long buckets were read twice, for the bitmap and for the
// list): 400 tables of up to 32 entries (SimHash) 49.7 / 61.3, of 64 70.6 / 74.0, of 256 194 / 152, 400 of 670K x 128 in a few directions, up
// to 128 entries 109 / 93, up to 256 169 / 120, 200 of 64 54.0 / 58.1, of 256 128 / 117, 68 of 256 69 / 63, 1,000 of 16 82 / 114, of 64 203 / 164.
// (Before, up to 64 long ones were shared out by 64 tables to a wave, one wave for all of them with 68 tables: 94 us a call
// that takes 45, and by lanes beyond that.)
struct LongRule {
  int even, few;       // tables of a wave
  int all;             // from that many long buckets on they go by lanes, however long: none is longer than C
  float steps;         // lanes' steps for an entry, in waves' steps for a bucket
};
inline LongRule long_rule(int L, int C, int lg) {
  const int even = std::min((L + 15) / 16, 64), rounds = (L + (1024 >> lg) - 1) >> (10 - lg);
  const float steps = 64.0f * (float)rounds * (float)std::max(512, std::min(L, 1024)) / (512.0f * (float)(6 << lg));
  return {even, L >= 256 ? std::min(2 * even, 64) : even, (int)std::min(1e9f, (float)std::max(0, C - (kBucketAhead << lg)) * steps), steps};
}
// (All waves work this out, with one scalar unit for all of them; the whole rule in the kernel cost every call 0.3 to 0.8 us, most
// of it for the scalar registers that it took.)
__attribute__((always_inline)) inline constexpr int tables_of_wave(const LongRule r, int lg, int nlong, int entries) {
  if (nlong <= 64) return r.few;
  const float beyond = (float)(2 * entries - (kBucketAhead << lg) * nlong);
  return nlong >= r.all || beyond * r.steps <= (float)nlong * (float)nlong ? 0 : r.even;
}

// Whether the update launch streams about `rows` weight rows of H floats past the caches, like their moments (aligned: to 128
// bytes).  Rows that together exceed the memory-side cache (256 MB) do not stay there from the logits to the update, nor from one
// step to the next.  That takes whole lines, parts of which would come and go several times, and from 512 floats on, where a wave
// takes a row, lanes that are all at work.  Steps, us, cached / streamed: 670K x 128, 642K rows 944 / 930, x 160, 540K 769 / 742,
// 600K x 256, 358K 596 / 586, x 320, 539K 1,237 / 1,207, x 192, 579K 1,014 / 997, 400K x 480, 331K 1,022 / 1,017; 300K x 384, 178K (261 MB)
// 431 / 436.  Parts of lines: 353K x 356, 170K 436 / 481, 650K x 300, 220K 541 / 572, 500K x 200, 480K 973 / 1,032, 670K x 120,
// 668K 1,640 / 1,677.  Longer rows: 250K x 544, 208K 878 / 997, x 672 978 / 1,056, x 928 1,258 / 1,297; x 1,024 1,344 / 1,341 (the launch
// alone, 190K rows, 586 / 551), 100K rows (391 MB) 639 / 654.
inline bool streams_weights(double rows, int H, bool aligned) {
  const double mb = rows * H * 4 / (1 << 20);
  if (!aligned || H % 32 != 0) return false;
  return H <= 512 ? mb > 288 : H % 1024 == 0 && mb > 512;
}

}  // namespace slide
