// LDS of a lookup launch (lookup_union_kernel): what slide_query_memory and slide_init accept, and how a launch divides what
// there is.  Plain C++, so that both limits can be compared without a GPU.
#pragma once

#include <algorithm>
#include <cstddef>

namespace slide {

constexpr int kLookupThreads = 1024;      // of a sample's workgroup
constexpr int kLookupMinSegment = 1024;   // bitmap words the lookup kernel must be able to hold at a time
constexpr int kSelWords = 264;            // 256 histogram bins + counters of the sampling-budget selection

// Segments of `segw` bitmap words, 2^lcw of them to a thread; bytes: LDS of the launch.  segw = 0: there is no room.
struct LookupPlan {
  int segw, lcw;
  size_t bytes;
};

// Besides the segment: bucket starts and lengths, 20 words for scans and counters, the hidden activations, the hash values,
// the rank of every thread's first word, and without a sampling budget those of its quads of words (16 bits each).  With a
// budget, which needs the whole bitmap in one segment, the histogram of the selection takes their place and the ranks of
// quads are counted when they are asked for: that keeps the limit on the classes where the bitmap sets it.
inline size_t lookup_lds(int L, int H, int NH, bool budgeted, int segw, int lcw) {
  const size_t fixed = ((size_t)2 * L + 20 + H + (budgeted ? kSelWords : 0)) * 4 + (((size_t)NH + 3) & ~(size_t)3);
  return fixed + (size_t)segw * 4 + (size_t)(segw >> lcw) * 4 + (budgeted ? 0 : (size_t)segw / 2);
}

// LDS that the configurations are accepted by: a bitmap segment of `words` and a word for each of the NT tiles of a sample.
// No launch takes more for the same segment (a tile has at most 32 words) but one without a budget, whose segment may be
// smaller: with room for kLookupMinSegment words here it has at least as many there.
inline size_t lookup_accepted_lds(int L, int H, int NT, int NH, int words) {
  return ((size_t)2 * L + 1 + 20 + H + NT + kSelWords + words) * 4 + (((size_t)NH + 3) & ~(size_t)3);
}

inline LookupPlan lookup_plan(int L, int H, int NH, int NWpad, bool budgeted, bool rounds, size_t limit) {
  auto words_in = [&](size_t lds) {                       // (at most 148 bytes for 32 words)
    const size_t fixed = lookup_lds(L, H, NH, budgeted, 0, 5);
    return (int)std::min<size_t>(lds > fixed ? (lds - fixed) / 148 * 32 : 0, NWpad);
  };
  LookupPlan p = {budgeted ? NWpad : words_in(limit), 2, 0};
  // two workgroups to a compute unit, where that takes at most four segments instead of one (calls, us, with the ranks of a
  // segment chosen against all of the LDS, which cost some of them the second workgroup / against half of it: a step of 1,024
  // samples x 515K neurons 444 / 433, of 600 samples x 520K 361 / 350, 1,000 samples' retrieval from 515K 177 / 166)
  size_t room = limit;                                    // (of a workgroup; half of it then, also for the ranks)
  if (rounds && !budgeted) {
    const int half = words_in(limit / 2);
    if (half > 0) {
      const int segments = (NWpad + half - 1) / half;
      if (segments <= 4) { p.segw = ((NWpad + segments - 1) / segments + 31) / 32 * 32; room = limit / 2; }
    }
  }
  // words to a thread: the fewest that let all threads together take the segment at once (and its ranks fit)
  while (p.lcw < 5 && ((p.segw >> p.lcw) > kLookupThreads || lookup_lds(L, H, NH, budgeted, p.segw, p.lcw) > room)) ++p.lcw;
  p.bytes = lookup_lds(L, H, NH, budgeted, p.segw, p.lcw);
  if (p.segw < 32 || p.bytes > limit) p.segw = 0;
  return p;
}

}  // namespace slide
