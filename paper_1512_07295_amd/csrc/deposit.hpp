// Shared by the two deposit kernels: the fixed-point formats and the lookup
// of a candidate's bucket run.
#pragma once

#include "particles.hpp"

namespace fsest {

// ------------------------------------------------------------------ formats
// Fixed-point accumulation.  LDS float atomics are ~20x slower than integer
// ones on gfx950, so a workgroup sums its tile in unsigned integers: a weight
// product w in [0, 1] adds floor(w * S + 1/2).  Two formats:
//  * wide (64-bit): S = 2^32 - 2^8; a grid sums to N_P < 2^31 units, so no
//    cell can overflow;
//  * narrow (32-bit): S = 2^F with F chosen on the device from the largest
//    bucket count M of this deposit.  A cell only receives particles whose
//    first grid's first stencil cell lies within p + 1 cells of it per axis
//    (at most 2 buckets per axis for p <= 4, 3 for p = 5, 6), and one
//    particle gives a cell at most w_max^3 (w_max the largest 1D weight of
//    the order: 1, 1, 3/4, 2/3, 115/192, 11/20), so its sum is at most
//    K (w_max^3 S + 1/2) units with K = 8 M (27 M) possible contributors; F
//    is the largest value keeping that below 2^32.  F >= 22 is required
//    (24 with masses, where the unit is the largest mass), or the wide
//    kernel runs instead (both are launched; the one not selected returns
//    at once).  Each contribution is rounded to 2^-(F+1) <= 2^-23 of a unit
//    mass; F < 24 only happens when the largest bucket (64 cells) holds more
//    than 32 (NGP) to 108 (PCS) particles, where cells sum several units and
//    float32 accumulation would round each addition at least as coarsely.
// Integer sums are exact, so deposits are bitwise reproducible.
constexpr float kFixWide = 4294967040.0f;  // 2^32 - 2^8
// fraction bits the narrow format needs, without and with masses
constexpr int kNarrowMinBits = 22;
constexpr int kNarrowMinBitsMass = 24;

// The narrow format's fraction bits for a largest bucket count: the largest F
// with K (w_max^3 2^F + 1/2) < 2^32 - 1, found from the logarithm and settled
// by the condition itself.  Every workgroup computes it (a kernel of its own
// for it cost 4 us per deposit).
template <int P>
__device__ __forceinline__ int narrow_bits(uint32_t maxcount) {
  // w_max^3 of the order, with a margin for the float32 rounding of the
  // weight products; the base cells of the particles that reach one cell span
  // p + 1 cells per axis (both grids), so they meet at most 2 buckets per axis
  // for p <= 4 and 3 for p = 5, 6
  constexpr double wmax = P <= 2 ? 1.0 : (P == 3 ? 0.75 : (P == 4 ? 2.0 / 3.0 : (P == 5 ? 115.0 / 192.0 : 0.55)));
  constexpr double w3 = wmax * wmax * wmax * (1.0 + 1e-6);
  const double k = (P <= 4 ? 8.0 : 27.0) * (double)(maxcount > 0 ? maxcount : 1);
  auto fits = [&](int f) { return k * (w3 * ldexp(1.0, f) + 0.5) < 4294967295.0; };
  int f = (int)(32.0f - __log2f((float)(k * w3)));
  f = f < 0 ? 0 : (f > 31 ? 31 : f);
  while (f > 0 && !fits(f)) --f;
  while (f < 31 && fits(f + 1)) ++f;
  return f;
}

// ------------------------------------------------------------------ runs
// A tile's candidates: runs of bucket-ordered records, run t holding the
// candidates pref[t] .. pref[t + 1] - 1 from record start[t] on.
struct DepRanges {
  uint32_t start[72];
  uint32_t pref[73];
  int count;
};

// Segment of each lane's candidate `item` (the wave's candidates are c0 ..
// c0 + 63): the last t < nr with pref[t] <= item, i.e. the number of
// starts pref[0..nr] at or below it, minus one (pref[nr] = total lies above
// every candidate; empty pieces repeat a start and count twice, which
// still lands on the non-empty piece).  Lane t holds starts t and t + 64:
// one ballot counts those at or below c0 for the whole wave, and the few
// inside the window are added lane by lane.
__device__ __forceinline__ int find_segment(const DepRanges& rg, int nr, uint32_t c0,
                                            uint32_t item, int lane) {
  const uint32_t pa = lane <= nr ? rg.pref[lane] : 0xFFFFFFFFu;
  const uint32_t pb = lane + 64 <= nr ? rg.pref[lane + 64] : 0xFFFFFFFFu;
  int cnt = __popcll(__ballot(pa <= c0)) + __popcll(__ballot(pb <= c0));
  unsigned long long ia = __ballot(pa > c0 && pa <= c0 + 63);
  unsigned long long ib = __ballot(pb > c0 && pb <= c0 + 63);
  while (ia) {
    const int t = __builtin_ctzll(ia);
    cnt += item >= (uint32_t)__builtin_amdgcn_readlane((int)pa, t) ? 1 : 0;
    ia &= ia - 1;
  }
  while (ib) {
    const int t = __builtin_ctzll(ib);
    cnt += item >= (uint32_t)__builtin_amdgcn_readlane((int)pb, t) ? 1 : 0;
    ib &= ib - 1;
  }
  return cnt - 1;
}

// The z-walking deposit (deposit_walk.hip): orders 1..4 on grids larger than
// a tile; where g.walk is not set the 64-bit format only.  q, ma, mb: slab and
// shift masks of interlacing codes 2 and 3.
hipError_t launch_deposit_walk(const Geom& g, const Buffers& b, const Tune& tu, const float* sw,
                               int q, int ma, int mb, hipStream_t s);

}  // namespace fsest
