// Mass assignment of orders 1..4 on grids larger than a tile (every N > 16):
// workgroups walk columns of 16 x 16 x 8-cell tiles in z.  Orders 5 and 6,
// grids of one tile and the 32-bit format on sparse grids take the general
// kernel of deposit.hip.
//
// What bounds it (gfx950): LDS integer atomics and VALU together.  A 32-bit
// LDS atomic takes at least 4 cycles per wave instruction and CU (16 active
// lanes a cycle), or as many as the most lanes that meet in one of 32 banks;
// a 64-bit one 6; lanes on one address cost 2 each.  A contribution is two
// VALU instructions and one atomic, and a particle's stencil falls on 1.4
// tiles of each grid.  At 256^3 (16.8M particles, PCS pair) the VALU issues
// in 79 % and the LDS works in 76 % of the cycles.  What the layout does
// about it: whole work items in LDS (no record read again, no unpacking per
// item), two barriers per round of candidates, several small workgroups per
// CU in different phases, bucket runs and records loaded a tile ahead.
// Against the general kernel of deposit.hip (one or two workgroups of 16^3
// tiles per CU), PCS pair, same box: 1024^3 with 2^27 particles 6.41 -> 5.73
// ms, 480^3 with 360^3 1.93 -> 1.62 ms, 256^3 with 256^3 0.65 -> 0.60 ms; in
// the 64-bit format 64 clustered sets on 128^3 6.71 -> 5.12 ms, one CIC grid
// of 512^3 0.58 -> 0.47 ms; 5000 particles on 32^3 32 -> 19 us.
#include <type_traits>

#include "deposit.hpp"

namespace fsest {

// Tile: kWalkT cells in x and y, kWalkTZ in z.  A row of LDS accumulators
// holds kZOff margin cells (a unit's first tile adds what reaches it from
// below there, never read), the tile's cells and up to four cells above
// them (rz <= kWalkTZ, plus p - 1), which the walk carries to the next tile.
// kRow and kPlane make the 64 offsets i kPlane + k kRow + l (i, k, l < 4)
// distinct mod 64: stencils whose bases differ mod 64 ("bank class") do not
// share an LDS bank in one instruction.
constexpr int kWalkT = kTileMax;
constexpr int kWalkTZ = 8;
constexpr int kZOff = 4;
constexpr int kRow = 16;
constexpr int kPlane = kWalkT * kRow + 4;
constexpr int kGridElems = kWalkT * kPlane;
constexpr int kWalkThreads = 512;
constexpr int kWalkWaves = kWalkThreads / 64;
constexpr int kPad = 64;  // elements around the regions that masked rows may address

constexpr bool walk_offsets_cover_banks() {
  bool seen[64] = {};
  for (int i = 0; i < 4; ++i)
    for (int k = 0; k < 4; ++k)
      for (int l = 0; l < 4; ++l) {
        const int r = (i * kPlane + k * kRow + l) % 64;
        if (seen[r]) return false;
        seen[r] = true;
      }
  return true;
}
static_assert(walk_offsets_cover_banks(), "stencil offsets must cover the 64 banks");
static_assert(kZOff + kWalkTZ + 3 < kRow, "a row holds the cells above the tile");
static_assert(kWalkThreads == 2 * kWalkT * kWalkT, "write-out: half a row per thread");
// a base address lies at least 3 rows and 3 cells below a region (masked y rows add zeros there)
static_assert(kPad >= 3 * kRow + 3 - kZOff &&
                  kGridElems + kPad > (kWalkT - 1) * kPlane + (kWalkT + 2) * kRow + kZOff + kWalkTZ + 3,
              "masked rows stay inside the accumulators and their pads");

// A work item is one grid's stencil of one particle: three words, per axis
// the 24-bit offset fraction on that grid (0 .. 2^24) and, above bit 25, the
// first cell relative to the tile plus p - 1 (0 .. 18); the grid in bit 31
// of the first word; a fourth word with the mass for weighted deposits.
constexpr uint32_t kItemFrac = (1u << 25) - 1u;

// IL: 0 one grid; 1 the interlaced pair; 2 a pair with run-time masks.
// POW2: N is a power of two (cells wrap with a mask).  WT: masses.
//
// Per tile: (1) candidates, NC per thread and round, become work items in
// registers, ranked inside their bank class by a returning LDS atomic;
// (2) every wave scans the class counts for itself, and the items go to LDS
// in class order such that the 32 lanes of a half wave take items spread
// evenly over the classes; (3) each lane adds its item's stencil with LDS
// atomics; (4) the finished cells are written, the cells above move down.
// A unit is a segment of up to seg_len tiles of one column; a particle's items
// go, whole in z, to the tile that holds its first z cell, and a unit's first
// tile also takes the bucket layers below it, whose stencils reach into it
// (the carry of its last tile is dropped: the next unit takes those
// particles again).  `dynamic`: units come from a counter (stats[1], zeroed
// with the sort), one workgroup per resident slot; else each workgroup has
// one unit.
template <int P, int IL, bool WIDE, bool POW2, bool WT>
__global__ __launch_bounds__(kWalkThreads) __attribute__((amdgpu_waves_per_eu(WIDE && IL ? 4 : 6))) void k_deposit_walk(
    const uint4* __restrict__ recs, const uint32_t* __restrict__ boff,
    const uint32_t* __restrict__ bcnt, float* __restrict__ grid, Geom g,
    uint32_t* __restrict__ stats, int exclusive, int dynamic, const float* __restrict__ sw, int q,
    int mask_a, int mask_b, int seg_len) {
  using AT = typename std::conditional<WIDE, unsigned long long, unsigned>::type;
  constexpr int NG = IL ? 2 : 1;
  // candidates per thread and round: a grid alone takes two, for as many items
  // as a pair has.  The half waves of a round then reach over more of the
  // tile's buckets, and a clump narrower than a cell meets itself on fewer
  // lanes: PCS on one grid, 16 clumped sets of 128^3, 0.88 -> 0.67 ms (32-bit,
  // a particle in two cells) and 2.08 -> 1.57 (64-bit, one per cell); uniform
  // particles 512^3, one per cell, 2.67 -> 2.46 ms.
  constexpr int NC = IL ? 1 : 2;
  // candidates per round: fewer where 64-bit pairs with masses would leave
  // room for one workgroup per CU only
  constexpr int kCand = (WIDE && WT && NG == 2) ? 384 : NC * kWalkThreads;
  constexpr int kItems = NG * kCand;
  constexpr int kItemWords = WT ? 4 : 3;
  // y rows outside the tile add zeros in the 32-bit format (no test per row:
  // 6.22 -> 6.06 ms at 1024^3), and are skipped in the 64-bit one, whose
  // atomics are the scarcer (64 clustered sets: 6.09 against 5.65 ms)
  constexpr bool kZeroRows = !WIDE;
  __shared__ __align__(16) AT acc[kPad + NG * kGridElems + kPad];
  __shared__ uint32_t items[kItemWords * kItems];
  __shared__ DepRanges rgs[2];           // runs of this tile and of the next, in turn
  __shared__ int cls_cnt[2][64];
  __shared__ uint32_t unit_ring[4];      // units by their order in this workgroup (o mod 4)

  const int nbits = __builtin_amdgcn_readfirstlane(narrow_bits<P>(stats[0]));
  constexpr int kMinBits = WT ? kNarrowMinBitsMass : kNarrowMinBits;
  if (!WIDE && nbits < kMinBits) return;                // the wide kernel does it
  if (WIDE && !exclusive && nbits >= kMinBits) return;  // the narrow one does it
  const float scale = WIDE ? kFixWide : ldexpf(1.0f, nbits);
  const double inv_scale = 1.0 / (double)scale;
  const float inv_f = (float)inv_scale;
  // masses: items carry w / w_max and the tile is multiplied back by w_max;
  // an invalid mass makes it NaN
  float wmul = 1.0f;
  if constexpr (WT) wmul = stats[5] ? __builtin_nanf("") : __uint_as_float(stats[4]);

  constexpr int off = (P % 2 == 0) ? (P / 2 - 1) : (P - 1) / 2;
  constexpr int kLow = (P - 1 + (IL ? 1 : 0) + kBucket - 1) / kBucket;  // bucket layers below a tile
  const int n = g.n, nb = g.nb;
  const int tpa = (n + kWalkT - 1) / kWalkT;     // tiles per axis in x, y
  const int tpz = (n + kWalkTZ - 1) / kWalkTZ;   // and in z
  const int upc = (tpz + seg_len - 1) / seg_len;  // units per column
  const uint32_t units_per_set = (uint32_t)(tpa * tpa * upc);
  const uint32_t nunits = (uint32_t)g.batch * units_per_set;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  struct Tile {
    int mock, tx, ty, tz, tz1;
    bool first;
  };
  auto first_tile = [&](uint32_t unit) {
    Tile t;
    t.mock = (int)(unit / units_per_set);
    const int urem = (int)(unit % units_per_set);
    t.tx = urem / (tpa * upc);
    t.ty = (urem / upc) % tpa;
    t.tz = (urem % upc) * seg_len;
    t.tz1 = min(tpz, t.tz + seg_len);
    t.first = true;
    return t;
  };
  // bucket columns of a tile: those whose particles can reach it in x and y
  // (first cells in [t0 - (p - 1) - S, t0 + extent - 1])
  auto columns = [&](int t0, int ext, int& b0, int& cnt) {
    cnt = ext / kBucket + kLow;
    if (cnt >= nb) {
      cnt = nb;
      b0 = 0;
    } else {
      b0 = t0 / kBucket - kLow;
      b0 = b0 < 0 ? b0 + nb : b0;
    }
  };
  // wave 0: lane l's bucket run of column l, in up to two pieces (a run is
  // contiguous except across a super-bucket edge)
  uint32_t s0 = 0, e0 = 0, s1 = 0, e1 = 0;
  int ncol = 0;
  auto load_runs = [&](const Tile& t) {
    int bx0, cx, by0, cy;
    columns(t.tx * kWalkT, min(kWalkT, n - t.tx * kWalkT), bx0, cx);
    columns(t.ty * kWalkT, min(kWalkT, n - t.ty * kWalkT), by0, cy);
    const int t0z = t.tz * kWalkTZ, zlow = t.first ? kLow : 0;
    const int cntz = min(kWalkTZ, n - t0z) / kBucket + zlow;
    int b0z = t0z / kBucket - zlow;
    b0z = b0z < 0 ? b0z + nb : b0z;
    s0 = e0 = s1 = e1 = 0;
    ncol = cx * cy;  // <= 25
    if (lane < ncol) {
      int bx = bx0 + lane / cy, by = by0 + lane % cy;
      bx = bx >= nb ? bx - nb : bx;
      by = by >= nb ? by - nb : by;
      const int64_t row = (((int64_t)t.mock * nb + bx) * nb + by) * nb;
      const int z1 = b0z + cntz;               // exclusive end, may pass nb
      const int zs = (b0z / g.fb + 1) * g.fb;  // next super-bucket edge
      const int za = z1 < zs ? z1 : zs;        // end of the first piece
      s0 = boff[row + b0z];
      e0 = boff[row + za - 1] + bcnt[row + za - 1];
      if (z1 > zs) {
        const int zb = zs >= nb ? zs - nb : zs, ze = zb + (z1 - zs);
        s1 = boff[row + zb];
        e1 = boff[row + ze - 1] + bcnt[row + ze - 1];
      }
    }
  };
  // wave 0: the loaded runs as starts and prefixes
  auto put_runs = [&](DepRanges& rg) {
    const uint32_t la = e0 - s0, lb = e1 - s1;
    uint32_t incl = la + lb;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t v = (uint32_t)__shfl_up((int)incl, o, 64);
      if (lane >= o) incl += v;
    }
    if (lane < ncol) {
      const uint32_t excl = incl - la - lb;
      rg.start[2 * lane] = s0;
      rg.start[2 * lane + 1] = s1;
      rg.pref[2 * lane + 1] = excl + la;
      rg.pref[2 * lane + 2] = incl;
    }
    if (lane == 0) {
      rg.pref[0] = 0;
      rg.count = 2 * ncol;
    }
  };

  // wave 0 runs ahead of the others: at a tile's start it stores the next
  // tile's runs (loaded during the previous tile) and loads those of the one
  // after.  `it` is that tile, `it_unit` and `it_ord` its unit and the unit's
  // order in this workgroup.
  Tile it;
  uint32_t it_unit = 0;
  int it_ord = 0;
  auto grab = [&](bool start) {
    // without the counter a workgroup has one unit
    uint32_t nx = start ? blockIdx.x : 0xFFFFFFFFu;
    if (dynamic) {
      if (lane == 0) nx = atomicAdd(&stats[1], 1u);
      nx = (uint32_t)__builtin_amdgcn_readfirstlane((int)nx);
    }
    return nx;
  };
  auto advance = [&]() {
    if (it_unit >= nunits) {
      // past the end: no runs
    } else if (it.tz + 1 < it.tz1) {
      ++it.tz;
      it.first = false;
    } else {
      it_unit = grab(false);
      ++it_ord;
      if (lane == 0) unit_ring[it_ord & 3] = it_unit;
      if (it_unit < nunits) it = first_tile(it_unit);
    }
    s0 = e0 = s1 = e1 = 0;
    ncol = 0;
    if (it_unit < nunits) load_runs(it);
  };
  {
    uint4* z4 = reinterpret_cast<uint4*>(acc);
    constexpr int kZero4 = (2 * kPad + NG * kGridElems) * (int)sizeof(AT) / 16;
    for (int i = threadIdx.x; i < kZero4; i += kWalkThreads) z4[i] = make_uint4(0u, 0u, 0u, 0u);
    if (threadIdx.x < 64) cls_cnt[0][threadIdx.x] = 0;
    if (wave == 0) {
      it_unit = grab(true);
      if (lane == 0) unit_ring[0] = it_unit;
      if (it_unit < nunits) {
        it = first_tile(it_unit);
        load_runs(it);
        put_runs(rgs[0]);
        advance();
      }
    }
  }
  __syncthreads();
  int ord = 0;  // this tile's unit in order
  uint32_t b = unit_ring[0];
  if (b >= nunits) return;
  Tile t = first_tile(b);
  int cur = 0;  // which of rgs holds this tile's runs
  int par = 0;  // which class counters the next round uses
  // candidates rb + e kWalkThreads + threadIdx.x (e < NC) of a tile with runs rg, their records loaded
  uint4 cr[NC];
  float cmass[NC];
#pragma unroll
  for (int e = 0; e < NC; ++e) {
    cr[e] = make_uint4(0u, 0u, 0u, 0u);
    cmass[e] = 0.0f;
  }
  auto fetch = [&](const DepRanges& rg, uint32_t rb) __attribute__((always_inline)) {
    const int nr = rg.count;
    const uint32_t total = rg.pref[nr];
#pragma unroll
    for (int e = 0; e < NC; ++e) {
      const uint32_t c0 = rb + (uint32_t)(e * kWalkThreads + wave * 64), cand = c0 + lane;
      uint32_t j = 0;
      if (c0 < total && wave < kCand / NC / 64) {
        const int seg = find_segment(rg, nr, c0, cand, lane);
        if (cand < total) j = rg.start[seg] + (cand - rg.pref[seg]);
      }
      cr[e] = recs[j];
      if constexpr (WT) cmass[e] = sw[j];
    }
  };
  fetch(rgs[0], 0);

  for (;;) {
    const int t0x = t.tx * kWalkT, t0y = t.ty * kWalkT, t0z = t.tz * kWalkTZ;
    // cells of this tile per axis
    const int ex = min(kWalkT, n - t0x), ey = min(kWalkT, n - t0y), ez = min(kWalkTZ, n - t0z);
    const bool last = t.tz + 1 == t.tz1;
    const uint32_t total = rgs[cur].pref[rgs[cur].count];
    if (wave == 0) {
      put_runs(rgs[cur ^ 1]);
      advance();
    }
    // the next tile's first candidates (its runs are complete after a barrier)
    if (total == 0) {
      __syncthreads();
      fetch(rgs[cur ^ 1], 0);
    }

    for (uint32_t rb = 0; rb < total; rb += kCand) {
      // (1) this thread's candidates
      constexpr int NI = NG * NC;  // their items: e NG + grid
      uint32_t w[NI][3];
      bool ok[NI];
      int cls[NI], rank[NI];
      float mass[NC];
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        ok[i] = false;
        cls[i] = rank[i] = 0;
      }
#pragma unroll
      for (int e = 0; e < NC; ++e) {
        mass[e] = cmass[e];
        if (rb + (uint32_t)(e * kWalkThreads) + threadIdx.x >= total || wave >= kCand / NC / 64) continue;
        const uint4 r = cr[e];
        // first cells of the first grid, relative to the tile, plus p - 1
        const int ux = (int)(r.x & 1023u) - off - t0x + (P - 1);
        const int uy = (int)((r.x >> 10) & 1023u) - off - t0y + (P - 1);
        const int uz = (int)((r.x >> 20) & 1023u) - off - t0z + (P - 1);
        auto wrap = [&](int v) {
          if constexpr (POW2) return v & (n - 1);
          else {
            v = v < 0 ? v + n : v;
            return v >= n ? v - n : v;
          }
        };
        // own buckets always count (the cells above the tile are carried),
        // the look-back buckets if the stencil reaches into the tile from
        // below, i.e. starts in [-(p - 1), 0]
        const bool own = !t.first || wrap(uz - (P - 1)) < ez;
#pragma unroll
        for (int gi = 0; gi < NG; ++gi) {
          const int i = e * NG + gi;
          const int mk = (IL == 2) ? (gi ? mask_b : mask_a) : (gi ? 7 : 0);
          const int stx = (int)((r.x >> 30) & 1u), sty = (int)(r.x >> 31), stz = (int)((r.y >> 24) & 1u);
          const bool hx = (mk & 1) != 0, hy = (mk & 2) != 0, hz = (mk & 4) != 0;
          const int qx = wrap(ux + (hx ? stx : 0)), qy = wrap(uy + (hy ? sty : 0));
          const int qz = wrap(uz + (hz ? stz : 0));
          ok[i] = qx < ex + P - 1 && qy < ey + P - 1 && (own || qz <= P - 1);
          // the offset on this grid, as record_offset (particles.hpp)
          auto frac = [](uint32_t word, int step, bool shifted) {
            int v = (int)(word & kFracMask);
            if (shifted) v += step ? -(1 << (kFracBits - 1)) : (1 << (kFracBits - 1));
            return (uint32_t)v;
          };
          w[i][0] = frac(r.y, stx, hx) | ((uint32_t)qx << 25) | ((uint32_t)gi << 31);
          w[i][1] = frac(r.z, sty, hy) | ((uint32_t)qy << 25);
          w[i][2] = frac(r.w, stz, hz) | ((uint32_t)qz << 25);
          cls[i] = (qx * (kPlane & 63) + qy * kRow + qz) & 63;
          if constexpr (WIDE) cls[i] = ((cls[i] << 1) & 63) | (cls[i] >> 5);
          if (ok[i]) rank[i] = atomicAdd(&cls_cnt[par][cls[i]], 1);
        }
      }
      __syncthreads();
      // (2) class starts (every wave for itself), then the items in class
      // order: sorted position p goes to lane p / H of half wave p % H
      const int c = cls_cnt[par][lane];
      int incl = c;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
      }
      const int m = __builtin_amdgcn_readlane(incl, 63);
      const int W = (m + 63) >> 6, H = 2 * W;
      const uint32_t hm = 0xFFFFFFFFu / (uint32_t)(H > 0 ? H : 2) + 1u;  // p / H by a high multiply
      const int start = incl - c;
      par ^= 1;
      if (wave == 0) cls_cnt[par][lane] = 0;  // next used after this round's last barrier
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int st = __shfl(start, cls[i], 64);
        if (ok[i]) {
          const uint32_t p = (uint32_t)(st + rank[i]);
          const uint32_t l = __umulhi(p, hm);
          const uint32_t slot = (p - l * (uint32_t)H) * 32u + l;
          items[slot] = w[i][0];
          items[kItems + slot] = w[i][1];
          items[2 * kItems + slot] = w[i][2];
          if constexpr (WT) items[3 * kItems + slot] = __float_as_uint(mass[i / NG]);
        }
      }
      __syncthreads();
      // the next round's (or tile's) records are loaded during the stencils, from
      // one place in the code and, without a candidate, from record 0: with two
      // places or a load in a branch the compiler copies the registers at the
      // join, and waits for the loads there (512^3, one particle in eight
      // cells, one grid: 0.57 -> 0.51 ms)
      {
        const bool more = rb + kCand < total;
        fetch(rgs[more ? cur : cur ^ 1], more ? rb + kCand : 0u);
      }
      // (3) the stencils
      for (int v = wave; v < W; v += kWalkWaves) {
        if (2 * v + (lane >> 5) + (lane & 31) * H >= m) continue;
        const int slot = v * 64 + lane;
        const uint32_t w0 = items[slot], w1 = items[kItems + slot], w2 = items[2 * kItems + slot];
        float sc = scale;
        if constexpr (WT) sc *= __uint_as_float(items[3 * kItems + slot]);
        auto offset = [](uint32_t word) {
          float f = (float)(int)(word & kItemFrac) * (1.0f / 16777216.0f);
          if constexpr (P % 2 == 1) f -= 0.5f;
          return f;
        };
        float wx[P], wy[P], wz[P];
        weights_from_offset<P>(offset(w0), wx);
        weights_from_offset<P>(offset(w1), wy);
        weights_from_offset<P>(offset(w2), wz);
        const int rx = (int)((w0 >> 25) & 31u) - (P - 1), ry = (int)(w1 >> 25) - (P - 1);
        const int rz = (int)(w2 >> 25) - (P - 1);
        AT* base = acc + kPad + (NG == 2 && (w0 >> 31) ? kGridElems : 0) + rx * kPlane + ry * kRow +
                   rz + kZOff;
#pragma unroll
        for (int k = 0; k < P; ++k) wy[k] = (kZeroRows && (unsigned)(ry + k) >= (unsigned)kWalkT) ? 0.0f : wy[k];
#pragma unroll
        for (int i = 0; i < P; ++i) wx[i] *= sc;
#pragma unroll
        for (int i = 0; i < P; ++i) {
          if ((unsigned)(rx + i) >= (unsigned)kWalkT) continue;
#pragma unroll
          for (int k = 0; k < P; ++k) {
            if (!kZeroRows && (unsigned)(ry + k) >= (unsigned)kWalkT) continue;
            const float wxy = wx[i] * wy[k];
#pragma unroll
            for (int l = 0; l < P; ++l)
              atomicAdd(&base[i * kPlane + k * kRow + l], (AT)(uint32_t)__builtin_fmaf(wxy, wz[l], 0.5f));
          }
        }
      }
      // the next round writes items only after its first barrier
    }
    __syncthreads();

    // (4) write-out: half a row (four cells) per thread, narrow scale a power
    // of two, so float(sum) * 2^-F rounds exactly like the double product.
    // The half at the row's start then takes the four cells above the tile
    // (zero after a unit's last tile), the rest of the row is cleared.
    {
      // lanes: half rows, 4 planes, 8 rows; waves: 2 groups of rows, 4 of
      // planes (the planes' shift by 4 words spreads the 16-word rows over
      // the LDS banks)
      const int zq = lane & 1, lx = ((lane >> 1) & 3) + 4 * (wave >> 1);
      const int ly = (lane >> 3) + 8 * (wave & 1), lz = 4 * zq;
      constexpr int kV = (int)sizeof(AT) / 4;  // uint4 per four cells
      float v[NG][4];
#pragma unroll
      for (int gi = 0; gi < NG; ++gi) {
        uint4* rowp = reinterpret_cast<uint4*>(acc + kPad + gi * kGridElems + lx * kPlane + ly * kRow);
        uint4* cellp = rowp + kV * (kZOff / 4 + zq);
        uint4* upp = rowp + kV * (kZOff + kWalkTZ) / 4;
        union {
          uint4 u[kV];
          AT e[4];
        } cell;
        uint4 up[kV];
#pragma unroll
        for (int e = 0; e < kV; ++e) {
          cell.u[e] = cellp[e];
          up[e] = (zq == 0 && !last) ? upp[e] : make_uint4(0u, 0u, 0u, 0u);
        }
#pragma unroll
        for (int e = 0; e < kV; ++e) {
          cellp[e] = up[e];
          if (zq == 0) upp[e] = make_uint4(0u, 0u, 0u, 0u);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
          v[gi][e] = (WIDE ? (float)((double)cell.e[e] * inv_scale) : (float)cell.e[e] * inv_f) * wmul;
      }
      if (lx < ex && ly < ey && lz < ez) {  // inside a ragged tile
        const int slab = (IL == 2) ? t.mock * g.npair + q : t.mock;
        if constexpr (IL) {
          float4* dst = reinterpret_cast<float4*>(reinterpret_cast<float2*>(grid) +
                                                  complex_index(g, slab, t0x + lx, t0y + ly, t0z + lz));
          dst[0] = make_float4(v[0][0], v[NG - 1][0], v[0][1], v[NG - 1][1]);
          dst[1] = make_float4(v[0][2], v[NG - 1][2], v[0][3], v[NG - 1][3]);
        } else {
          *reinterpret_cast<float4*>(grid + real_cell_index(g, slab, t0x + lx, t0y + ly, t0z + lz)) =
              make_float4(v[0][0], v[0][1], v[0][2], v[0][3]);
        }
      }
    }
    if (last) {
      ++ord;
      b = unit_ring[ord & 3];
      if (b >= nunits) break;
      t = first_tile(b);
    } else {
      ++t.tz;
      t.first = false;
    }
    cur ^= 1;
    __syncthreads();
  }
}

// Workgroups of one instantiation that a CU holds, by LDS (160 KB) and by the
// registers the kernel is compiled for (4 or 6 waves per SIMD; 8 for one
// 32-bit grid spills: CIC at 512^3 0.459 against 0.442 ms).
template <int IL, bool WIDE>
constexpr int walk_groups_per_cu() {
  return WIDE && IL ? 2 : 3;
}

// Segment length of the z walk in tiles: of 1..16 the one with the smallest
// rounds of units over the resident workgroups times their length, half a
// tile added per unit for its look-back, and three quarters of a unit for
// the uneven end when there are several rounds.  256^3 (768 workgroups of
// the pair): 11 tiles, one unit each, 0.60 ms against 0.64 with 4 tiles per
// unit; 64 uneven clustered sets of 128^3: 8 tiles, 5.1 ms against 5.6 with 16.
static int walk_segment(const Geom& g, int64_t slots) {
  const int tpa = (g.n + kWalkT - 1) / kWalkT, tpz = (g.n + kWalkTZ - 1) / kWalkTZ;
  const int64_t cols = (int64_t)g.batch * tpa * tpa;
  int best = 1;
  int64_t cost = -1;
  for (int len = 1; len <= 16 && len <= tpz; ++len) {
    const int64_t units = cols * ((tpz + len - 1) / len);
    const int64_t rounds = (units + slots - 1) / slots;
    const int64_t c = rounds * (4 * len + 2) + (rounds > 1 ? 3 * len : 0);
    if (cost < 0 || c <= cost) {
      cost = c;
      best = len;
    }
  }
  return best;
}

template <int P, int IL, bool WIDE, bool POW2, bool WT>
static hipError_t walk_launch(const Geom& g, const Buffers& b, const Tune& tu, bool exclusive,
                              const float* sw, int q, int ma, int mb, hipStream_t s) {
  const int tpa = (g.n + kWalkT - 1) / kWalkT, tpz = (g.n + kWalkTZ - 1) / kWalkTZ;
  const int64_t slots = (int64_t)tu.cus * walk_groups_per_cu<IL, WIDE>();
  const int seg = walk_segment(g, slots);
  const int64_t nunits = (int64_t)g.batch * tpa * tpa * ((tpz + seg - 1) / seg);
  const bool dynamic = nunits > slots;
  hipLaunchKernelGGL((k_deposit_walk<P, IL, WIDE, POW2, WT>),
                     dim3((unsigned)(dynamic ? slots : nunits)), dim3(kWalkThreads), 0, s,
                     (const uint4*)b.recs, b.boff, b.bcnt, (float*)b.grid, g, b.stats,
                     exclusive ? 1 : 0, dynamic ? 1 : 0, sw, q, ma, mb, seg);
  return hipGetLastError();
}

template <int P, int IL, bool POW2, bool WT>
static hipError_t walk_formats(const Geom& g, const Buffers& b, const Tune& tu, const float* sw, int q,
                               int ma, int mb, hipStream_t s) {
  const bool narrow = tu.dep_narrow != 0;
  if (narrow && g.walk) {
    const hipError_t e = walk_launch<P, IL, false, POW2, WT>(g, b, tu, false, sw, q, ma, mb, s);
    if (e != hipSuccess) return e;
  }
  return walk_launch<P, IL, true, POW2, WT>(g, b, tu, !narrow, sw, q, ma, mb, s);
}

template <int P, int IL>
static hipError_t walk_dispatch(const Geom& g, const Buffers& b, const Tune& tu, const float* sw, int q,
                                int ma, int mb, hipStream_t s) {
  const bool pow2 = (g.n & (g.n - 1)) == 0;
  if (pow2) {
    return sw ? walk_formats<P, IL, true, true>(g, b, tu, sw, q, ma, mb, s)
              : walk_formats<P, IL, true, false>(g, b, tu, sw, q, ma, mb, s);
  }
  return sw ? walk_formats<P, IL, false, true>(g, b, tu, sw, q, ma, mb, s)
            : walk_formats<P, IL, false, false>(g, b, tu, sw, q, ma, mb, s);
}

template <int P>
static hipError_t walk_order(const Geom& g, const Buffers& b, const Tune& tu, const float* sw, int q,
                             int ma, int mb, hipStream_t s) {
  if (g.code == 0) return walk_dispatch<P, 0>(g, b, tu, sw, q, ma, mb, s);
  if (g.code == 1) return walk_dispatch<P, 1>(g, b, tu, sw, q, ma, mb, s);
  return walk_dispatch<P, 2>(g, b, tu, sw, q, ma, mb, s);
}

hipError_t launch_deposit_walk(const Geom& g, const Buffers& b, const Tune& tu, const float* sw,
                               int q, int ma, int mb, hipStream_t s) {
  switch (g.order) {
    case 1: return walk_order<1>(g, b, tu, sw, q, ma, mb, s);
    case 2: return walk_order<2>(g, b, tu, sw, q, ma, mb, s);
    case 3: return walk_order<3>(g, b, tu, sw, q, ma, mb, s);
    case 4: return walk_order<4>(g, b, tu, sw, q, ma, mb, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace fsest
