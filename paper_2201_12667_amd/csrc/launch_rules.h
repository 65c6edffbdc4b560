// Rules that size launches, apart from the kernels so that they can be checked without a GPU (constexpr: host and device).
#pragma once

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

}  // namespace slide
