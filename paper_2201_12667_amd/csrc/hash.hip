// Locality-sensitive hash codes of fp32 vectors (hidden activations when the tables are
// queried, rows of W2 when they are built; paper Sections 2.1, 3.1, 4.1).
//
// Mapping: one lane owns one vector; the workgroup stages a tile of vectors in LDS transposed
// ([coordinate][vector], odd row pitch), so for a given elementary hash every lane reads the
// same coordinate of its own vector: the coordinate tables are wave-uniform (scalar loads) and
// the LDS reads hit consecutive banks.  The waves of a workgroup take different tables; when a
// tile holds fewer than 64 vectors (long vectors), the lane groups of a wave take different tables
// too, and the workgroup has more waves to cover the LDS latency.
// For DWTA the tile holds order-preserving integer keys instead of floats (0 = entry absent: zero or
// NaN), so that a comparison is one unsigned compare and two selects.
#include "slide_internal.h"
#include "wave_ops.h"

#include <algorithm>
#include <cstring>
#include <vector>

namespace slide {

// Vectors per tile of the row-tile kernel: 64 (a wave per table) while two tiles fit a compute unit's LDS;
// beyond that 16, so that two workgroups still share a compute unit and one reads its tile while the
// other hashes (with 32 vectors of 1,024 coordinates a single workgroup filled the LDS and the unit
// idled through every tile read).
static int rows_per_tile(int H) { return H <= 512 ? 64 : 16; }
size_t hash_lds_bytes(int H) { return ((size_t)H + 1) * (rows_per_tile(H) + 1) * sizeof(float); }
int hash_tile_pitch(int H) { return rows_per_tile(H) + 1; }

// Key of a coordinate: 0 if it cannot win (zero of either sign, NaN), else an unsigned integer that
// orders like the float (equal floats <-> equal keys), at least 1.
__device__ __forceinline__ uint32_t dwta_key(float x) {
  const uint32_t u = __float_as_uint(x);
  const uint32_t k = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return (x != 0.0f && x == x) ? k : 0u;
}

// The row-tile kernel reads its coordinates from a second parameter table, offs: one 32-bit entry
// per coordinate = its byte offset in the transposed tile (coordinate * pitch * 4), so that an LDS
// address is one add (the 16-bit coordinate table would cost a mask, a multiply and a shift per
// element); SimHash entries carry the sign in bit 31, and a bit's entries are padded to a multiple
// of eight with pointers to a row of zeros behind the tile (adding +0 changes no sum).
//
// Winner position of elementary hash e for the vector whose keys start at byte address col0 of the
// tile; -1 when the bin has no entry.  Strictly greater wins, so ties keep the lowest position.
// Eight keys of the lane's vector at the (wave-uniform) byte offsets o[0..8) of the tile, whose vector
// of lane l starts 4*l bytes into every coordinate's row: the read that adds the lane number to a scalar
// base address, so that no lane spends an instruction on the address (a wait state between the write of
// the base register and the read is required on this family).  tile_base: LDS address of the tile.
__device__ __forceinline__ void read8_lane_rows(uint32_t (&k)[8], const uint32_t* __restrict__ o, uint32_t tile_base) {
  asm volatile(
      "s_add_u32 m0, %16, %8\n\ts_nop 0\n\tds_read_addtid_b32 %0\n\t"
      "s_add_u32 m0, %16, %9\n\ts_nop 0\n\tds_read_addtid_b32 %1\n\t"
      "s_add_u32 m0, %16, %10\n\ts_nop 0\n\tds_read_addtid_b32 %2\n\t"
      "s_add_u32 m0, %16, %11\n\ts_nop 0\n\tds_read_addtid_b32 %3\n\t"
      "s_add_u32 m0, %16, %12\n\ts_nop 0\n\tds_read_addtid_b32 %4\n\t"
      "s_add_u32 m0, %16, %13\n\ts_nop 0\n\tds_read_addtid_b32 %5\n\t"
      "s_add_u32 m0, %16, %14\n\ts_nop 0\n\tds_read_addtid_b32 %6\n\t"
      "s_add_u32 m0, %16, %15\n\ts_nop 0\n\tds_read_addtid_b32 %7\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(k[0]), "=&v"(k[1]), "=&v"(k[2]), "=&v"(k[3]), "=&v"(k[4]), "=&v"(k[5]), "=&v"(k[6]), "=&v"(k[7])
      : "s"(o[0]), "s"(o[1]), "s"(o[2]), "s"(o[3]), "s"(o[4]), "s"(o[5]), "s"(o[6]), "s"(o[7]), "s"(tile_base)
      : "m0", "scc", "memory");
}

// The same for two bins at once (sixteen reads in flight before the wait).
__device__ __forceinline__ void read16_lane_rows(uint32_t (&a)[8], uint32_t (&b)[8], const uint32_t* __restrict__ oa,
                                                 const uint32_t* __restrict__ ob, uint32_t tile_base) {
  asm volatile(
      "s_add_u32 m0, %16, %8\n\ts_nop 0\n\tds_read_addtid_b32 %0\n\t"
      "s_add_u32 m0, %16, %9\n\ts_nop 0\n\tds_read_addtid_b32 %1\n\t"
      "s_add_u32 m0, %16, %10\n\ts_nop 0\n\tds_read_addtid_b32 %2\n\t"
      "s_add_u32 m0, %16, %11\n\ts_nop 0\n\tds_read_addtid_b32 %3\n\t"
      "s_add_u32 m0, %16, %12\n\ts_nop 0\n\tds_read_addtid_b32 %4\n\t"
      "s_add_u32 m0, %16, %13\n\ts_nop 0\n\tds_read_addtid_b32 %5\n\t"
      "s_add_u32 m0, %16, %14\n\ts_nop 0\n\tds_read_addtid_b32 %6\n\t"
      "s_add_u32 m0, %16, %15\n\ts_nop 0\n\tds_read_addtid_b32 %7"
      : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3]), "=&v"(a[4]), "=&v"(a[5]), "=&v"(a[6]), "=&v"(a[7])
      : "s"(oa[0]), "s"(oa[1]), "s"(oa[2]), "s"(oa[3]), "s"(oa[4]), "s"(oa[5]), "s"(oa[6]), "s"(oa[7]), "s"(tile_base)
      : "m0", "scc", "memory");
  asm volatile(
      "s_add_u32 m0, %16, %8\n\ts_nop 0\n\tds_read_addtid_b32 %0\n\t"
      "s_add_u32 m0, %16, %9\n\ts_nop 0\n\tds_read_addtid_b32 %1\n\t"
      "s_add_u32 m0, %16, %10\n\ts_nop 0\n\tds_read_addtid_b32 %2\n\t"
      "s_add_u32 m0, %16, %11\n\ts_nop 0\n\tds_read_addtid_b32 %3\n\t"
      "s_add_u32 m0, %16, %12\n\ts_nop 0\n\tds_read_addtid_b32 %4\n\t"
      "s_add_u32 m0, %16, %13\n\ts_nop 0\n\tds_read_addtid_b32 %5\n\t"
      "s_add_u32 m0, %16, %14\n\ts_nop 0\n\tds_read_addtid_b32 %6\n\t"
      "s_add_u32 m0, %16, %15\n\ts_nop 0\n\tds_read_addtid_b32 %7\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(b[0]), "=&v"(b[1]), "=&v"(b[2]), "=&v"(b[3]), "=&v"(b[4]), "=&v"(b[5]), "=&v"(b[6]), "=&v"(b[7])
      : "s"(ob[0]), "s"(ob[1]), "s"(ob[2]), "s"(ob[3]), "s"(ob[4]), "s"(ob[5]), "s"(ob[6]), "s"(ob[7]), "s"(tile_base)
      : "m0", "scc", "memory");
  // (the first eight registers are filled only once the wait above has passed: nothing may read them earlier)
  asm volatile("" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]));
}

// Winner position among the M keys of a bin, and the winning key (0: the bin has no entry).
template <int M>
__device__ __forceinline__ uint32_t dwta_winner(const uint32_t (&k)[M], uint32_t& best) {
  best = k[0];                                       // the largest key first (three-operand maxima) ...
#pragma unroll
  for (int p = 1; p < M; ++p) best = max(best, k[p]);
  bool eq[M];                                        // ... then the lowest position that holds it
#pragma unroll
  for (int p = 0; p < M; ++p) eq[p] = k[p] == best;
  uint32_t best_p = M - 1;
#pragma unroll
  for (int p = M - 2; p >= 0; --p) best_p = eq[p] ? (uint32_t)p : best_p;
  return best_p;
}

template <int M, bool UNI>
__device__ __forceinline__ int dwta_raw(const char* col0, const uint32_t* __restrict__ offs, int e, uint32_t tile_base = 0) {
  const uint32_t* o = offs + (size_t)(UNI ? __builtin_amdgcn_readfirstlane(e) : e) * M;
  uint32_t k[M];
  if constexpr (M == 8 && UNI) {
    read8_lane_rows(k, o, tile_base);
  } else {
#pragma unroll
    for (int p = 0; p < M; ++p) k[p] = *(const uint32_t*)(col0 + o[p]);
  }
  uint32_t best = k[0];                              // the largest key first (three-operand maxima) ...
#pragma unroll
  for (int p = 1; p < M; ++p) best = max(best, k[p]);
  bool eq[M];                                        // ... then the lowest position that holds it
#pragma unroll
  for (int p = 0; p < M; ++p) eq[p] = k[p] == best;
  int best_p = M - 1;
#pragma unroll
  for (int p = M - 2; p >= 0; --p) best_p = eq[p] ? p : best_p;
  return best == 0u ? -1 : best_p;
}

template <int M, bool UNI>
__device__ __forceinline__ uint32_t dwta_code(const HashDev& hd, const uint32_t* __restrict__ offs, const char* col0,
                                              int pitch_bytes, int t, int& rowstate, uint32_t tile_base) {
  // Empty bin: borrow the winner of another elementary hash (rare, per lane).
  auto borrow = [&](int e) -> int {
    if (rowstate < 0) {
      rowstate = 0;
      for (int c = 0; c < hd.H; ++c) if (*(const uint32_t*)(col0 + (size_t)c * pitch_bytes) != 0u) { rowstate = 1; break; }
    }
    if (rowstate == 1)
      for (uint32_t tr = 1; tr <= 100; ++tr) {
        const uint32_t u = hd.dens_a * (uint32_t)(e + 1) + hd.dens_b * tr;
        const int e2 = (int)((u >> 8) % (uint32_t)hd.NH);
        const int r2 = dwta_raw<M, false>(col0, offs, e2);
        if (r2 >= 0) return r2;
      }
    return 0;
  };
  uint32_t code = 0;
  const int e0 = UNI ? __builtin_amdgcn_readfirstlane(t * hd.K) : t * hd.K;   // uniform over the lanes of a table
  int k = 0;
  for (; k + 1 < hd.K; k += 2) {                     // two independent argmax chains in flight
    if constexpr (M == 8 && UNI) {
      const uint32_t* o = offs + (size_t)(e0 + k) * 8;
      uint32_t ka[8], kb[8], ba, bb;
      read16_lane_rows(ka, kb, o, o + 8, tile_base);
      uint32_t v0 = dwta_winner<8>(ka, ba), v1 = dwta_winner<8>(kb, bb);
      if (__any(min(ba, bb) == 0u)) {                // (an empty bin in some lane: rare)
        if (ba == 0u) v0 = (uint32_t)borrow(e0 + k);
        if (bb == 0u) v1 = (uint32_t)borrow(e0 + k + 1);
      }
      code |= (v0 << (k * hd.lgm)) | (v1 << ((k + 1) * hd.lgm));
    } else {
      int v0 = dwta_raw<M, UNI>(col0, offs, e0 + k, tile_base);
      int v1 = dwta_raw<M, UNI>(col0, offs, e0 + k + 1, tile_base);
      if (v0 < 0) v0 = borrow(e0 + k);
      if (v1 < 0) v1 = borrow(e0 + k + 1);
      code |= ((uint32_t)v0 << (k * hd.lgm)) | ((uint32_t)v1 << ((k + 1) * hd.lgm));
    }
  }
  if (k < hd.K) {
    int v0 = dwta_raw<M, UNI>(col0, offs, e0 + k, tile_base);
    if (v0 < 0) v0 = borrow(e0 + k);
    code |= (uint32_t)v0 << (k * hd.lgm);
  }
  return code;
}

template <bool UNI>
__device__ __forceinline__ uint32_t simhash_code(const HashDev& hd, const uint32_t* __restrict__ offs, const char* col0,
                                                 int t) {
  uint32_t code = 0;
  for (int k = 0; k < hd.K; ++k) {
    const int e = UNI ? __builtin_amdgcn_readfirstlane(t * hd.K + k) : t * hd.K + k;
    const uint32_t* __restrict__ o = offs + (size_t)e * hd.So;        // So is a multiple of 8
    float acc = 0.0f;
    for (int q = 0; q < hd.So; q += 8) {             // sequential sum: a - x is a + (-x) bit for bit
      uint32_t w[8], x[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) w[j] = o[q + j];
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = *(const uint32_t*)(col0 + (w[j] & 0x7fffffffu));
#pragma unroll
      for (int j = 0; j < 8; ++j) acc += __uint_as_float(x[j] ^ (w[j] & 0x80000000u));
    }
    code |= (acc > 0.0f ? 1u : 0u) << k;
  }
  return code;
}

// ---------------------------------------------------------------------------------------------
// DWTA (bins of eight) of many vectors when the functions are many: the winner of a bin depends on the order of
// the coordinates only, so every vector's coordinates are replaced by their ranks first (equal values get
// equal ranks), and a bin is then decided on 16-bit keys, two vectors to a lane: key = (rank + 128) << 3 | (7 -
// position), so that one maximum gives the winner and, among equals, the lowest position.  Per bin and 128
// vectors: 8 LDS reads, 7 ORs, 4 three-operand packed maxima and 5 more instructions, against twice 8 reads and
// 25 instructions with 32-bit keys.  (The maximum is the packed 16-bit floating one: the keys of present
// coordinates are ordinary positive numbers and order like integers.)
//
// The ranks: a wave sorts a vector's 128 keys in its registers (a bitonic network, two keys a lane, exchanges by
// DPP moves and half-wave swaps: 104 instructions), puts them in LDS, and every coordinate finds its place by
// bisection.  That costs about as much as it saves on 500 functions, and a workgroup takes 128 vectors through all
// tables, hence the rule in launch_hash.
// 670,091 vectors of 128 coordinates, 2,400 functions: 1,311 -> 739 us, about 200 of them for the ranks.  The bins
// issue 50 instructions each, 17 of them vector ones; with eight waves a SIMD (four workgroups' LDS just fits a
// compute unit: with three it took 853) the waits for offsets and keys are the rest.
// ---------------------------------------------------------------------------------------------
constexpr int kRankThreads = 512;
constexpr int kRankRows = 128;             // vectors per workgroup
constexpr int kRankPitch = 65;             // words between consecutive coordinates (the pitch the byte offsets are for)
constexpr int kRankMaxH = 128;
static size_t ranked_lds(int H) { return ((size_t)H * kRankPitch + kRankThreads / 64 * 128) * 4; }
constexpr uint32_t kRankBase = 128;        // (keys of present coordinates start at 1024: normal 16-bit floats)

__device__ __forceinline__ uint32_t med3(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t d;
  asm("v_med3_u32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}
__device__ __forceinline__ uint32_t max3_pk(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t d;
  asm("v_pk_maximum3_f16 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t min_pk(uint32_t a, uint32_t b) {
  const u16x2 r = __builtin_elementwise_min(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b));
  return __builtin_bit_cast(uint32_t, r);
}

// Ascending sort of 128 keys, lane l holding elements 2l (a) and 2l + 1 (b).  A lane keeps the smaller of a pair
// where its mask is 0 and the larger where it is ~0: the median of both and the mask.
struct SortMasks { uint32_t m1, m2, m4, m8, d16, d32; };   // ~0 in lanes with that bit set
__device__ __forceinline__ SortMasks sort_masks(int lane) {
  return {(lane & 1) ? ~0u : 0u, (lane & 2) ? ~0u : 0u, (lane & 4) ? ~0u : 0u, (lane & 8) ? ~0u : 0u,
          (lane & 16) ? ~0u : 0u, (lane & 32) ? ~0u : 0u};
}
template <int CTRL> __device__ __forceinline__ uint32_t dpp0(uint32_t v) { return dpp_u32<CTRL>(0u, v); }
__device__ __forceinline__ uint32_t lane_xor4(uint32_t v) { return dpp0<0x1B>(dpp0<kDppRowHalfMirror>(v)); }   // (7 ^ 3)
template <int CTRL> __device__ __forceinline__ void exchange(uint32_t& a, uint32_t& b, uint32_t k) {   // same element of lane ^ x
  const uint32_t pa = dpp0<CTRL>(a), pb = dpp0<CTRL>(b);
  a = med3(a, pa, k); b = med3(b, pb, k);
}
template <int CTRL> __device__ __forceinline__ void exchange_mirror(uint32_t& a, uint32_t& b, uint32_t k) {   // the other element
  const uint32_t pa = dpp0<CTRL>(b), pb = dpp0<CTRL>(a);
  a = med3(a, pa, k); b = med3(b, pb, k);
}
__device__ __forceinline__ void exchange_xor4(uint32_t& a, uint32_t& b, uint32_t k) {
  const uint32_t pa = lane_xor4(a), pb = lane_xor4(b);
  a = med3(a, pa, k); b = med3(b, pb, k);
}
__device__ __forceinline__ void exchange_own(uint32_t& a, uint32_t& b, uint32_t dir) {
  const uint32_t x = med3(a, b, dir), y = med3(a, b, ~dir);
  a = x; b = y;
}
__device__ __forceinline__ void swap16(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  a = r[0]; b = r[1];
}
__device__ __forceinline__ void swap32(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0]; b = r[1];
}
__device__ __forceinline__ void tail16(uint32_t& a, uint32_t& b, const SortMasks& m, uint32_t dir) {   // distances 16 .. 1
  exchange<kDppRowRor + 8>(a, b, m.m8 ^ dir);
  exchange_xor4(a, b, m.m4 ^ dir);
  exchange<kDppQuadSwap2>(a, b, m.m2 ^ dir);
  exchange<kDppQuadSwap1>(a, b, m.m1 ^ dir);
  exchange_own(a, b, dir);
}
__device__ __forceinline__ void sort128(uint32_t& a, uint32_t& b, const SortMasks& m) {
  exchange_own(a, b, 0u);                                // runs of 2
  exchange_mirror<kDppQuadSwap1>(a, b, m.m1);            // 4
  exchange_own(a, b, 0u);
  exchange_mirror<0x1B>(a, b, m.m2);                     // 8: quad_perm [3,2,1,0]
  exchange<kDppQuadSwap1>(a, b, m.m1);
  exchange_own(a, b, 0u);
  exchange_mirror<kDppRowHalfMirror>(a, b, m.m4);        // 16
  exchange<kDppQuadSwap2>(a, b, m.m2);
  exchange<kDppQuadSwap1>(a, b, m.m1);
  exchange_own(a, b, 0u);
  exchange_mirror<kDppRowMirror>(a, b, m.m8 ^ m.d16);    // 32, every other run descending
  exchange_xor4(a, b, m.m4 ^ m.d16);
  exchange<kDppQuadSwap2>(a, b, m.m2 ^ m.d16);
  exchange<kDppQuadSwap1>(a, b, m.m1 ^ m.d16);
  exchange_own(a, b, m.d16);
  swap16(a, b);                                          // 64 (lane ^ 16: both elements face each other after the swap)
  exchange_own(a, b, m.d32);
  swap16(a, b);
  tail16(a, b, m, m.d32);
  swap32(a, b);                                          // 128
  exchange_own(a, b, 0u);
  swap32(a, b);
  swap16(a, b);
  exchange_own(a, b, 0u);
  swap16(a, b);
  tail16(a, b, m, 0u);
}

__global__ __launch_bounds__(kRankThreads, 8) void dwta_ranked_kernel(HashDev hd, const uint32_t* __restrict__ offs,
                                                                      const float* __restrict__ V, int64_t rows,
                                                                      uint32_t* __restrict__ codes, int64_t row_stride,
                                                                      int64_t tab_stride, const int32_t* __restrict__ rowlist,
                                                                      const uint32_t* __restrict__ nrows_dev, Ctrl* build) {
  // [H][kRankPitch] keys of two vectors per word (vector l low, 64 + l high); then, while the ranks are found, the
  // sorted keys of a vector per wave
  extern __shared__ uint32_t rk[];
  const int H = hd.H, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int NW = kRankThreads / 64, PER = kRankRows / NW;   // vectors per wave
  if (build && blockIdx.x == 0 && tid == 0) start_build(build, rows);
  if (rowlist) {
    const int64_t listed = (int64_t)*nrows_dev;
    if (listed == rows) rowlist = nullptr;               // every vector: in place, without the list
    rows = listed;
  }
  const int64_t row0 = (int64_t)blockIdx.x * kRankRows;
  if (row0 >= rows) return;
  auto row_of = [&](int r) -> int64_t {                  // vector r of the workgroup, -1 = none
    const int64_t q = row0 + r;
    return q < rows ? (rowlist ? (int64_t)rowlist[q] : q) : -1;
  };
  {
    const SortMasks m = sort_masks(lane);
    uint32_t* sorted = rk + H * kRankPitch + wave * 128;
    const bool own = 2 * lane < H;                       // (H is a multiple of eight)
    float2 x[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int64_t row = row_of(wave * PER + u);
      x[u] = own && row >= 0 ? *(const float2*)(V + (size_t)row * H + 2 * lane) : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int u = 0; u < PER; u += 2) {                   // two vectors at a time: their sorts overlap
      uint32_t key[4], sa[2], sb[2];
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        key[2 * v] = own ? dwta_key(x[u + v].x) : ~0u;
        key[2 * v + 1] = own ? dwta_key(x[u + v].y) : ~0u;
        sa[v] = key[2 * v]; sb[v] = key[2 * v + 1];
      }
#pragma unroll
      for (int v = 0; v < 2; ++v) sort128(sa[v], sb[v], m);
      uint32_t pos[4] = {0u, 0u, 0u, 0u};                // keys of the vector below this one
#pragma unroll
      for (int v = 0; v < 2; ++v) {                      // (one set of sorted keys: four workgroups fit a compute unit)
        *(uint2*)(sorted + 2 * lane) = make_uint2(sa[v], sb[v]);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int d = 64; d > 0; d >>= 1)
#pragma unroll
          for (int q = 2 * v; q < 2 * v + 2; ++q) pos[q] += sorted[pos[q] + d - 1] < key[q] ? (uint32_t)d : 0u;
        __builtin_amdgcn_wave_barrier();
      }
      if (own) {
        const int r = wave * PER + u;                    // (PER is even and divides 64: both vectors in the same half)
        uint16_t* out = (uint16_t*)(rk + 2 * lane * kRankPitch + (r & 63)) + (r >> 6);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          out[(q & 1) * 2 * kRankPitch + (q >> 1) * 2] = (uint16_t)(key[q] ? (pos[q] + 1u + kRankBase) << 3 : 0u);
      }
    }
  }
  __syncthreads();
  const uint32_t tile_base = (uint32_t)(uintptr_t)rk;    // (the low half of a generic LDS address is the LDS address)
  const int64_t lo_row = row_of(lane), hi_row = row_of(64 + lane);
  const uint32_t codemask = (1u << (3 * hd.K)) - 1u;
  for (int t = wave; t < hd.L; t += NW) {
    uint32_t c0 = 0, c1 = 0, least = ~0u;
    for (int k = hd.K - 1; k >= 0; --k) {
      uint32_t key[8];
      read8_lane_rows(key, offs + (size_t)(t * hd.K + k) * 8, tile_base);
#pragma unroll
      for (int p = 0; p < 7; ++p) key[p] |= (uint32_t)(7 - p) * 0x10001u;
      const uint32_t best = max3_pk(max3_pk(key[0], key[1], key[2]), max3_pk(key[3], key[4], key[5]), max3_pk(key[6], key[7], key[7]));
      c0 = (c0 << 3) | (best & 7u);
      c1 = (c1 << 3) | ((best >> 16) & 7u);
      least = min_pk(least, best);
    }
    c0 ^= codemask;
    c1 ^= codemask;
    // a bin without an entry in some vector (rare): that vector's code again, its empty bins borrowing from the
    // probe sequence
    const bool e0 = lo_row >= 0 && (least & 0xffffu) < (kRankBase << 3), e1 = hi_row >= 0 && (least >> 16) < (kRankBase << 3);
    if (__any(e0 || e1)) {
      for (int h = 0; h < 2; ++h) {
        if (!(h ? e1 : e0)) continue;
        const uint16_t* col = (const uint16_t*)(rk + lane) + h;
        auto raw = [&](int e) -> int {                   // winner of elementary hash e, -1 = no entry
          uint32_t best = 0;
          for (int p = 0; p < 8; ++p) {
            const uint32_t v = *(const uint16_t*)((const char*)col + offs[(size_t)e * 8 + p]);
            if (v) best = max(best, v | (uint32_t)(7 - p));
          }
          return best ? 7 - (int)(best & 7u) : -1;
        };
        bool any = false;
        for (int c = 0; c < H && !any; ++c) any = col[c * 2 * kRankPitch] != 0;
        uint32_t code = 0;
        for (int k = 0; k < hd.K && any; ++k) {
          const int e = t * hd.K + k;
          int v = raw(e);
          for (uint32_t tr = 1; tr <= 100 && v < 0; ++tr)
            v = raw((int)(((hd.dens_a * (uint32_t)(e + 1) + hd.dens_b * tr) >> 8) % (uint32_t)hd.NH));
          code |= (uint32_t)(v < 0 ? 0 : v) << (3 * k);
        }
        if (h) c1 = code; else c0 = code;
      }
    }
    if (lo_row >= 0) codes[lo_row * row_stride + (int64_t)t * tab_stride] = c0;
    if (hi_row >= 0) codes[hi_row * row_stride + (int64_t)t * tab_stride] = c1;
  }
}

// ---------------------------------------------------------------------------------------------
// SimHash of many vectors on the matrix cores.  A bit is the sign of the 32-bit running sum of S signed
// coordinates, in storage order; the order only matters when the sum is within its rounding errors of zero.  So
// the sums are formed as a matrix product of the vectors, split into two bf16 parts, with a matrix of 0 and
// +-1, and where the product is further from zero than both evaluations' errors together its sign is the bit.
// The rest (2 in 10,000 for S = 43) is summed exactly as documented, by the whole wave.
//
// Errors, with M = the vector's largest magnitude and u = 2^-24: the running sum is off by at most S * S*M*u; the
// two parts leave 2^-18 of each coordinate out, S*M*2^-18 in all; the matrix cores add 2S non-zero terms, each
// addition off by at most 2u of a partial sum below S*M (they may truncate).  Together S*M * (5*S*u + 2^-18);
// the bound used has 6 in place of 5.
//
// A wave holds the fragments of 32 vectors in registers (columns of the product) and goes through the hash
// matrix, 32 rows at a time, which its workgroup keeps in LDS.  The 16 rows whose results land in a lane are 16
// consecutive bits of the lane's stream, K per table from the most significant: the lower half wave has its own
// tables, the upper half its own.  The matrix holds the negated signs, so that a set sign bit is a set bit.
// 325,056 vectors of 128 coordinates, 450 bits of 43 coordinates: 607 us with the kernel below (a lane per
// vector, three vector instructions and an LDS read per coordinate), 110 here: 75 GFLOP, 32 us at the MFMA rate;
// the rest is the bits summed exactly (a fifth of the 32 x 32 blocks holds one).  253,855 vectors of 200: 790 -> 212.
// Vectors longer than 256 coordinates (128 registers of fragments) stay with the kernel below.
// ---------------------------------------------------------------------------------------------
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Waves per workgroup (one fills a compute unit's LDS): as many as the registers of their fragments allow without
// spilling, 16, 12 or 8.
constexpr int simhash_threads(int nkb) { return nkb <= 6 ? 1024 : nkb <= 10 ? 768 : 512; }

// NKB: blocks of 16 coordinates held (H <= 16 * NKB), rounded up to an even number, so that at most one block of zeros
// is multiplied (builds of 325,056 vectors, 450 bits: 96 coordinates 434 us, 128 465, 160 519, 192 570, 256 685).  hd.smat: [chunk][nblk][NKB][64 lanes][8]; a chunk holds
// tph tables per half wave.
template <int NKB>
__global__ __launch_bounds__(simhash_threads(NKB)) void simhash_rows_kernel(HashDev hd, const float* __restrict__ V,
                                                                             int64_t rows, uint32_t* __restrict__ codes,
                                                                             int64_t row_stride, int64_t tab_stride,
                                                                             const int32_t* __restrict__ rowlist,
                                                                             const uint32_t* __restrict__ nrows_dev,
                                                                             int nblk, int tph, Ctrl* build) {
  extern __shared__ float4 smat[];                       // [nblk][NKB][64]
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, H = hd.H, S = hd.S, K = hd.K;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
  if (build && (blockIdx.x | blockIdx.y) == 0 && tid == 0) start_build(build, rows);
  if (rowlist) {
    const int64_t listed = (int64_t)*nrows_dev;
    if (listed == rows) rowlist = nullptr;               // every vector: in place, without the list
    rows = listed;
  }
  const int64_t ngroups = (rows + 31) / 32;
  if ((int64_t)blockIdx.x >= ngroups) return;
  const float4* src = (const float4*)hd.smat + (size_t)blockIdx.y * nblk * NKB * 64;
  for (int q = tid; q < nblk * NKB * 64; q += blockDim.x) smat[q] = src[q];
  __syncthreads();
  const int t_half = (blockIdx.y * 2 + half) * tph;      // first table of the lane's half
  const int t_own = max(0, min(tph, hd.L - t_half));     // tables it has
  // (a workgroup's waves take groups far apart: when the groups do not divide evenly every workgroup has some of
  // the waves with one group more)
  for (int64_t g = (int64_t)wave * gridDim.x + blockIdx.x; g < ngroups; g += (int64_t)nw * gridDim.x) {
    const int64_t q = g * 32 + (lane & 31);
    const bool live = q < rows;
    const int64_t row = rowlist ? (int64_t)rowlist[live ? q : rows - 1] : (live ? q : rows - 1);
    const float* v = V + (size_t)row * H;
    bf16x8 hi[NKB], mid[NKB];
    float top = 0.f;
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
      const int k = kb * 16 + 8 * half;                  // (past the end: the last coordinates again, against zeros)
      const float4 a = *(const float4*)(v + min(k, H - 4)), b = *(const float4*)(v + min(k + 4, H - 4));
      const f32x2 x[4] = {{a.x, a.y}, {a.z, a.w}, {b.x, b.y}, {b.z, b.w}};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bf16x2 h2 = __builtin_convertvector(x[e], bf16x2);
        const bf16x2 m2 = __builtin_convertvector(x[e] - __builtin_convertvector(h2, f32x2), bf16x2);
        hi[kb][2 * e] = h2[0]; hi[kb][2 * e + 1] = h2[1];
        mid[kb][2 * e] = m2[0]; mid[kb][2 * e + 1] = m2[1];
        top = __builtin_elementwise_maximum(top, __builtin_elementwise_maximum(fabsf(x[e][0]), fabsf(x[e][1])));   // (NaN stays)
      }
    }
    top = __builtin_elementwise_maximum(top, __shfl_xor(top, 32));
    // magnitudes whose parts would overflow or lose bits: every bit in storage order (as where top * S leaves the
    // range, which makes the bound infinite: only then can a partial sum of either order)
    const bool zero = top == 0.f, plain = !(top < 1e37f) || (!zero && top < 1e-30f);
    const float bound = zero ? -1.f : plain ? INFINITY : top * (float)S * (3.8146973e-6f + 6.f * 5.9604645e-8f * (float)S);
    uint64_t stream = 0;
    int held = 0, t = 0;                                 // bits in the stream, tables done (uniform)
#pragma unroll 1
    for (int blk = 0; blk < nblk; ++blk) {
      const bf16x8* m = (const bf16x8*)(smat + blk * NKB * 64) + lane;
      f32x16 acc;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
        const bf16x8 a = m[kb * 64];
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, mid[kb], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, hi[kb], acc, 0, 0, 0);
      }
      uint32_t bits = 0;
      float low = INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(acc[r]), 31);   // bits << 1 | sign
        low = __builtin_elementwise_minimum(low, fabsf(acc[r]));               // (NaN stays)
      }
      if (__any(live && !(low > bound))) {
        uint32_t open = 0;                               // bits too close to call
#pragma unroll
        for (int r = 0; r < 16; ++r) open |= !(fabsf(acc[r]) > bound) ? 0x8000u >> r : 0u;
        const int filled = t_own * K - blk * 16;         // (the rows past the half's tables are zeros)
        open &= filled >= 16 ? 0xffffu : filled > 0 ? 0xffffu & ~(0xffffu >> filled) : 0u;
        if (!live) open = 0;
        while (true) {
          const unsigned long long any = __ballot(open != 0u);
          if (!any) break;
          const int src_lane = __ffsll((long long)any) - 1;
          const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)open, src_lane);
          const int r = __clz((int)o) - 16, s = blk * 16 + r;                   // the stream's s-th bit
          const int ti = s / K, tt = (blockIdx.y * 2 + (src_lane >> 5)) * tph + ti;
          float sum = 0.f;
          const int e = tt * K + (K - 1 - (s - ti * K));
          const uint64_t rr = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(row >> 32), src_lane) << 32) |
                              (uint32_t)__builtin_amdgcn_readlane((int)row, src_lane);
          const float* vr = V + (size_t)rr * H;
          const uint32_t* words = hd.words + (size_t)e * (hd.Spad / 2);
          for (int s0 = 0; s0 < S; s0 += 64) {
            const int mine = min(s0 + lane, S - 1);
            const uint32_t w = words[mine >> 1] >> (16 * (mine & 1));
            const float x = vr[w & 0x7fffu];
            const int signed_x = __float_as_int((w & 0x8000u) ? -x : x);
            for (int k = 0; k < min(64, S - s0); ++k) sum += __int_as_float(__builtin_amdgcn_readlane(signed_x, k));
          }
          if (lane == src_lane) {
            bits = (bits & ~(0x8000u >> r)) | (sum > 0.f ? 0x8000u >> r : 0u);
            open &= ~(0x8000u >> r);
          }
        }
      }
      if (zero) bits = 0;
      stream = (stream << 16) | bits;
      held += 16;
      while (held >= K && t < tph) {
        held -= K;
        const uint32_t code = (uint32_t)(stream >> held) & ((1u << K) - 1u);
        if (live && t < t_own) codes[row * row_stride + (int64_t)(t_half + t) * tab_stride] = code;
        ++t;
      }
    }
  }
}

constexpr int kSimhashMaxBlocks = 16;      // coordinate blocks of the longest vectors taken
constexpr size_t kSimhashLds = 128 * 1024; // LDS for the hash matrix

SimhashSplit simhash_split(int H, int K, int L) {
  SimhashSplit p{};
  const int nkb = (H + 15) / 16;
  if (nkb > kSimhashMaxBlocks) return p;
  p.nkb = (nkb + 1) / 2 * 2;
  const int most = (int)(kSimhashLds / 1024) / p.nkb, per_half = (L + 1) / 2;      // blocks of a chunk; tables of a half
  const int tables = most * 16 / K > 0 ? most * 16 / K : 1;                        // ... that a chunk can hold
  p.chunks = (per_half + tables - 1) / tables;
  p.tph = (per_half + p.chunks - 1) / p.chunks;
  p.nblk = (p.tph * K + 15) / 16;
  return p;
}

// The hash matrix in fragment order: lane l of block (chunk, blk, kb) holds row l % 32, coordinates
// 16*kb + 8*(l / 32) .. + 7.  Row 8*(r/4) + 4*half + r%4 of a block is bit 16*blk + r of the half's stream.
void simhash_matrix(const SimhashSplit& p, int H, int K, int L, int S, const int32_t* idx, const int8_t* sign, uint16_t* out) {
  std::vector<int> sum(H);
  for (int c = 0; c < p.chunks; ++c)
    for (int half = 0; half < 2; ++half)
      for (int s = 0; s < p.tph * K; ++s) {
        const int t = (c * 2 + half) * p.tph + s / K;
        if (t >= L) continue;
        const int e = t * K + (K - 1 - s % K), blk = s / 16, r = s % 16, m = 8 * (r / 4) + 4 * half + r % 4;
        std::fill(sum.begin(), sum.end(), 0);
        for (int q = 0; q < S; ++q) sum[idx[(size_t)e * S + q]] -= sign[(size_t)e * S + q];
        for (int k = 0; k < H; ++k) {                    // (a coordinate listed more than once: small integers, exact in bf16)
          if (!sum[k]) continue;
          const float f = (float)sum[k];
          uint32_t u;
          memcpy(&u, &f, 4);
          const int kb = k / 16, lane = ((k % 16) / 8) * 32 + m;
          out[((((size_t)c * p.nblk + blk) * p.nkb + kb) * 64 + lane) * 8 + k % 8] = (uint16_t)(u >> 16);
        }
      }
}

template <int NKB>
static hipError_t launch_simhash(const HashDev& hd, const SimhashSplit& p, const float* V, int64_t rows, uint32_t* codes,
                                 int64_t row_stride, int64_t tab_stride, const int32_t* rowlist, const uint32_t* nrows_dev,
                                 int num_cus, Ctrl* build, hipStream_t s) {
  const int per = num_cus / p.chunks > 0 ? num_cus / p.chunks : 1;
  const int64_t groups = (rows + 31) / 32;
  hipLaunchKernelGGL((simhash_rows_kernel<NKB>), dim3((unsigned)(groups < per ? groups : per), p.chunks),
                     dim3(simhash_threads(NKB)), (size_t)p.nblk * NKB * 1024, s, hd, V, rows, codes, row_stride, tab_stride,
                     rowlist, nrows_dev, p.nblk, p.tph, build);
  return hipGetLastError();
}

// MODE 0: SimHash; 2,4,8,16: DWTA with that bin size.  UNI: a tile holds 64 vectors, so a wave works
// on one table at a time and reads its coordinates through scalar loads.
// rowlist == nullptr: vectors 0 .. rows-1 of V.  Otherwise the vectors rowlist[0 .. *nrows_dev) of V
// (the grid covers rows; tiles past the device-side count leave at once; a count equal to rows means
// all of them, and the list is not read).
template <int MODE, bool UNI>
__global__ __launch_bounds__(1024) void hash_rows_kernel(HashDev hd, const uint32_t* __restrict__ offs,
                                                        const float* __restrict__ V,
                                                        int64_t rows, int RPT, uint32_t* __restrict__ codes,
                                                        int64_t row_stride, int64_t tab_stride,
                                                        const int32_t* __restrict__ rowlist,
                                                        const uint32_t* __restrict__ nrows_dev, int tpb, Ctrl* build) {
  extern __shared__ float tile[];                    // [H + 1][RPT + 1]; the last row is zero
  __shared__ int64_t rid[64];                        // vector held by tile column r, -1 = none
  const int stride = RPT + 1, H = hd.H;
  const int64_t row0 = (int64_t)blockIdx.x * RPT;
  if (build && (blockIdx.x | blockIdx.y) == 0 && threadIdx.x == 0) start_build(build, rows);
  if (rowlist) {
    const int64_t listed = (int64_t)*nrows_dev;
    if (listed == rows) rowlist = nullptr;           // every vector: in place, without the list
    rows = listed;
  }
  if (row0 >= rows) return;
  if ((int)threadIdx.x < RPT) {
    const int64_t q = row0 + threadIdx.x;
    rid[threadIdx.x] = q < rows ? (rowlist ? (int64_t)rowlist[q] : q) : -1;
  }
  if ((int)threadIdx.x < stride) tile[H * stride + threadIdx.x] = 0.0f;
  __syncthreads();
  // coalesced reads, eight per thread in flight (a tile of long vectors is tens of elements per thread,
  // and one at a time would be as many round trips to memory); conflict-free stores
  constexpr int kTileBatch = 8;
  const int total = RPT * H;
  for (int base = 0; base < total; base += kTileBatch * (int)blockDim.x) {
    float x[kTileBatch];
    int at[kTileBatch];
#pragma unroll
    for (int u = 0; u < kTileBatch; ++u) {
      const int idx = base + u * (int)blockDim.x + (int)threadIdx.x;
      x[u] = 0.0f;
      at[u] = -1;
      if (idx < total) {
        const int r = idx / H, c = idx - r * H;
        const int64_t row = rid[r];
        at[u] = c * stride + r;
        if (row >= 0) x[u] = V[row * H + c];
      }
    }
#pragma unroll
    for (int u = 0; u < kTileBatch; ++u)
      if (at[u] >= 0) tile[at[u]] = MODE == 0 ? x[u] : __uint_as_float(dwta_key(x[u]));
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const int tps = 64 / RPT;                          // tables per wave and step (RPT is 16, 32 or 64)
  const int r = lane & (RPT - 1), sub = lane / RPT;
  const int64_t row = rid[r];
  const char* col0 = (const char*)(tile + r);
  const uint32_t tile_base = (uint32_t)(uintptr_t)tile;   // (the low half of a generic LDS address is the LDS address)
  const int t_end = min((int)(blockIdx.y + 1) * tpb, hd.L);
  int rowstate = -1;
  for (int t0 = blockIdx.y * tpb + wave * tps; t0 < t_end; t0 += nw * tps) {
    const int t = t0 + sub;
    if (t >= t_end) continue;
    uint32_t code;
    if (MODE == 0) code = simhash_code<UNI>(hd, offs, col0, t);
    else code = dwta_code<(MODE == 0 ? 2 : MODE), UNI>(hd, offs, col0, stride * 4, t, rowstate, tile_base);
    if (row >= 0) codes[row * row_stride + (int64_t)t * tab_stride] = code;
  }
}

template <int MODE>
static hipError_t launch_mode(const HashDev& hd, const float* V, int64_t rows, uint32_t* codes,
                              int64_t row_stride, int64_t tab_stride, const int32_t* rowlist,
                              const uint32_t* nrows_dev, int tpb, Ctrl* build, hipStream_t s) {
  const int RPT = rows_per_tile(hd.H);
  dim3 grid((unsigned)ceil_div(rows, RPT), (unsigned)ceil_div(hd.L, tpb));
  if (RPT == 64)
    hipLaunchKernelGGL((hash_rows_kernel<MODE, true>), grid, dim3(1024), hash_lds_bytes(hd.H), s, hd, hd.offs, V, rows,
                       RPT, codes, row_stride, tab_stride, rowlist, nrows_dev, tpb, build);
  else
    hipLaunchKernelGGL((hash_rows_kernel<MODE, false>), grid, dim3(1024), hash_lds_bytes(hd.H), s, hd, hd.offs, V, rows,
                       RPT, codes, row_stride, tab_stride, rowlist, nrows_dev, tpb, build);
  return hipGetLastError();
}

// On ranks from 600 functions on (1,000 for vectors of up to 96 coordinates: finding the ranks costs the same there,
// reading a tile less) and where their workgroups of 128 vectors fill the machine, five for every two compute units
// (82K vectors).  Table builds, row tiles and ranks, us: 2,400 functions of 128 coordinates 355 and 399 for 32K
// vectors, 522 and 509 for 64K, 611 and 539 for 82K, 1,027 and 911 for 200K; 600 of them 171 and 178 (64K), 204 and
// 190 (82K), 311 and 319 (200K), 436 and 421 (300K); 1,000 of 64 coordinates 192 and 196 (64K), 222 and 231 (72K), 257
// and 239 (82K), 528 and 488 (200K); 600 of 72 coordinates 286 and 297 (82K), 385 and 391 (150K).
// How long a list of rows is only the device knows: both kernels are launched then, and one of them finds a count of 0
// and leaves (split_listed_kernel).
int64_t hash_ranked_from(const HashDev& hd) {
  const bool fits = hd.kind == SLIDE_HASH_DWTA && hd.m == 8 && hd.H <= kRankMaxH && hd.NH >= (hd.H > 96 ? 600 : 1000);
  return fits ? (int64_t)320 * hd.num_cus : INT64_MAX;
}

hipError_t launch_hash(const HashDev& hd, const float* V, int64_t rows, uint32_t* codes,
                       int64_t row_stride, int64_t tab_stride, const int32_t* rowlist,
                       const uint32_t* nrows_dev, int tables_per_block, Ctrl* build, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  const int tpb = tables_per_block < 1 ? 1 : tables_per_block;
  if (hd.kind == SLIDE_HASH_SIMHASH && hd.smat) {
    const SimhashSplit p = simhash_split(hd.H, hd.K, hd.L);
#define SLIDE_SRP(NKB) return launch_simhash<NKB>(hd, p, V, rows, codes, row_stride, tab_stride, rowlist, nrows_dev, hd.num_cus, build, s)
    switch (p.nkb) {
      case 2: SLIDE_SRP(2);
      case 4: SLIDE_SRP(4);
      case 6: SLIDE_SRP(6);
      case 8: SLIDE_SRP(8);
      case 10: SLIDE_SRP(10);
      case 12: SLIDE_SRP(12);
      case 14: SLIDE_SRP(14);
      case 16: SLIDE_SRP(16);
    }
#undef SLIDE_SRP
  }
  if (hd.kind == SLIDE_HASH_SIMHASH)
    return launch_mode<0>(hd, V, rows, codes, row_stride, tab_stride, rowlist, nrows_dev, tpb, build, s);
  const int64_t ranked_from = hash_ranked_from(hd);
  if (rows >= ranked_from) {                             // (a list of rows may still be shorter: see hash_ranked_from)
    hipLaunchKernelGGL(dwta_ranked_kernel, dim3((unsigned)ceil_div(rows, kRankRows)), dim3(kRankThreads), ranked_lds(hd.H), s, hd,
                       hd.offs, V, rows, codes, row_stride, tab_stride, rowlist, rowlist ? nrows_dev + 1 : nullptr, build);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !rowlist) return e;
  }
  switch (hd.m) {
    case 2: return launch_mode<2>(hd, V, rows, codes, row_stride, tab_stride, rowlist, nrows_dev, tpb, build, s);
    case 4: return launch_mode<4>(hd, V, rows, codes, row_stride, tab_stride, rowlist, nrows_dev, tpb, build, s);
    case 8: return launch_mode<8>(hd, V, rows, codes, row_stride, tab_stride, rowlist, nrows_dev, tpb, build, s);
    case 16: return launch_mode<16>(hd, V, rows, codes, row_stride, tab_stride, rowlist, nrows_dev, tpb, build, s);
  }
  return hipErrorInvalidValue;
}

hipError_t hash_setup_attributes(int H) {
  const int bytes = (int)hash_lds_bytes(H);
  hipError_t e;
#define SLIDE_SET(K) \
  e = hipFuncSetAttribute((const void*)&K, hipFuncAttributeMaxDynamicSharedMemorySize, bytes); \
  if (e != hipSuccess) return e;
  SLIDE_SET((hash_rows_kernel<0, true>))
  SLIDE_SET((hash_rows_kernel<2, true>))
  SLIDE_SET((hash_rows_kernel<4, true>))
  SLIDE_SET((hash_rows_kernel<8, true>))
  SLIDE_SET((hash_rows_kernel<16, true>))
  SLIDE_SET((hash_rows_kernel<0, false>))
  SLIDE_SET((hash_rows_kernel<2, false>))
  SLIDE_SET((hash_rows_kernel<4, false>))
  SLIDE_SET((hash_rows_kernel<8, false>))
  SLIDE_SET((hash_rows_kernel<16, false>))
#undef SLIDE_SET
#define SLIDE_SET(NKB) \
  e = hipFuncSetAttribute((const void*)&simhash_rows_kernel<NKB>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSimhashLds); \
  if (e != hipSuccess) return e;
  e = hipFuncSetAttribute((const void*)&dwta_ranked_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)ranked_lds(kRankMaxH));
  if (e != hipSuccess) return e;
  SLIDE_SET(2) SLIDE_SET(4) SLIDE_SET(6) SLIDE_SET(8) SLIDE_SET(10) SLIDE_SET(12) SLIDE_SET(14) SLIDE_SET(16)
#undef SLIDE_SET
  return hipSuccess;
}

}  // namespace slide
