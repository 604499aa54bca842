// Which kernel takes a Gram matrix, and the work split of more than 64 columns (ortho_f64.h).  Plain C++, so that it can be
// tested without a GPU.
#pragma once
#include <algorithm>
#include <cstdint>

#define GRAM_SLICES 8
#define GRAM_MAX_BLOCKS 5
#define GRAM_MAX_UNITS (GRAM_MAX_BLOCKS * (GRAM_MAX_BLOCKS + 1) / 2)
#define GRAM_WAVES 8             // two per SIMD (registers: 128 of accumulators), one workgroup per CU
#define GRAM_STEP (4 * GRAM_WAVES)   // rows that a workgroup's waves take at a time
#define GRAM_MAX_WGS 32          // per slice (fewer slices than XCDs have one step each)

// Work split of a Gram matrix, made on the host.  Unit u: pair of blocks (bi >= bj) of qi and qj tiles from columns ci, cj.
// The work of a slice is the list of (unit, GRAM_STEP rows), unit major, each as long as the unit has tiles; workgroup w of
// `wgs` takes the w-th equal share of its length: from step `step` of unit `unit` of bound[w] up to those of bound[w + 1].
struct GramUnit {
  short ci, cj;
  signed char qi, qj;
  short tiles;                   // qi qj, of a diagonal pair the lower qi (qi + 1) / 2
  short tile0;                   // tiles of the units before
  short wg0, wgs;                // workgroups of a slice that have a share of it (one set of partial tiles each)
  int part_at;                   // its partial tiles, in tiles
};
struct GramBound { int unit, step; };
struct GramPlan {
  int64_t m;
  int steps;                     // groups of GRAM_STEP rows per slice
  int kp, units, slices, wgs, tiles;
  int part_tiles;
  GramUnit unit[GRAM_MAX_UNITS];
  GramBound bound[GRAM_MAX_WGS + 1];
};

static inline int64_t gram_ceil(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Up to 64 columns: gram_narrow_kernel.
static inline bool gram_is_narrow(int kp) { return kp <= 64; }
// More columns and few rows: gram_short_kernel; the rest: gram_mfma_kernel with a gram_plan.  Product and sum, us, rocprofv3, first with
// gram_mfma_kernel, then with gram_short_kernel:
//   rows    80 columns   96           128          192          256          320
//   200     8.8   7.3    9.1   7.6    10.6  7.9    11.4  9.1
//   1000    9.2   7.3    9.6   8.0    11.7  9.4    13.5  11.0   15.1  12.7   15.6  14.4
//   2000    9.6   8.1    10.1  8.4    13.5  10.5   15.1  12.6   16.8  15.9   17.6  16.5
//   2500    9.8   8.8    10.6  9.5    13.4  10.9   14.8  13.2   17.2  16.8   17.9  18.2
//   4096    10.2  9.5    11.3  10.4   14.1  11.4   16.0  15.7   18.8  19.0   20.6  22.1
//   6000    9.9   10.1   11.4  10.9   14.8  12.7   16.6  16.8   21.0  21.8   24.4  27.5
//   8192    10.4  10.6   11.4  11.7   14.9  14.3   18.4  18.6   22.9  25.3   27.7  34.2
static inline bool gram_is_short(int64_t m, int kp) {
  return !gram_is_narrow(kp) && m <= (kp <= 128 ? 6144 : (kp <= 256 ? 4096 : 2048));
}
static inline bool gram_is_planned(int64_t m, int kp) { return !gram_is_narrow(kp) && !gram_is_short(m, kp); }
// Rows of a wave of gram_short_kernel: four waves per CU, one per SIMD, at least 32 rows each, whole trips of 16.
static inline int gram_short_blocks(int kp) { const int nb32 = (kp / 16 + 1) / 2; return nb32 * (nb32 + 1) / 2; }
static inline int gram_short_rows(int64_t m, int kp) {
  const int64_t chunks = std::max(1, 4 * 256 / gram_short_blocks(kp));
  return (int)std::max<int64_t>(32, gram_ceil(gram_ceil(m, chunks), 16) * 16);
}

// What a second unit costs a workgroup -- its first loads, the sum of the waves' tiles and their way out -- in tiles times steps
// of matrix instructions (some 3 us): shares that keep to one unit may be longer by that much.  Kernel, us, with 0, 48 and any
// length: 6500 x 112 11.6, 9.3, 9.0; 8192 x 192 16.8, 13.2, 13.5, x 256 19.3, 16.9, 17.4; 16384 x 96 11.4, 9.1, 9.3; 32768 x 256 42.2,
// 42.0, 44.1; 65536 x 160 34.6, 34.6, 36.2, x 256 73.4, 73.5, 80.5, x 320 108, 108, 125.  (16: 8192 x 192 16.9; 128: 32768 x 256 44.1.)
#define GRAM_UNIT_COST 48
// Work split of the Gram matrix of more than 64 columns (kp: a multiple of 16, at most 320).
static GramPlan gram_plan(int64_t m, int kp) {
  GramPlan g;
  g.m = m; g.kp = kp;
  // columns: as few blocks of up to four tiles as there can be, the larger ones first
  const int nj = kp / 16, nblk = (nj + 3) / 4;
  int q[GRAM_MAX_BLOCKS], c[GRAM_MAX_BLOCKS];
  for (int b = 0, at = 0; b < nblk; ++b) {
    q[b] = nj / nblk + (b < nj % nblk);
    c[b] = at;
    at += 16 * q[b];
  }
  g.tiles = nj * (nj + 1) / 2;
  g.units = 0;
  for (int bi = 0; bi < nblk; ++bi)
    for (int bj = 0; bj <= bi; ++bj) {
      GramUnit& u = g.unit[g.units++];
      u.ci = c[bi]; u.cj = c[bj]; u.qi = q[bi]; u.qj = q[bj];
      u.tiles = bi == bj ? q[bi] * (q[bi] + 1) / 2 : q[bi] * q[bj];
    }
  // Rows: a slice per XCD, a share a step of 8 tiles at least.
  g.slices = (int)std::min<int64_t>(GRAM_SLICES, gram_ceil(m, GRAM_STEP));
  g.steps = (int)gram_ceil(m, (int64_t)g.slices * GRAM_STEP);
  int tile = 0;
  for (int n = 0; n < g.units; ++n) {
    g.unit[n].tile0 = (short)tile;
    tile += g.unit[n].tiles;
  }
  const int work = g.steps * g.tiles;      // (32 bits hold it for 2^31 rows; divisions in 64 took most of the time of this, on every call)
  g.wgs = std::max(1, std::min(work / 8, 256 / g.slices));
  // Shares that keep to one unit: every unit one workgroup, the next one always to the unit whose shares are the longest.
  int count[GRAM_MAX_UNITS], len[GRAM_MAX_UNITS], total = g.units, longest = 0;
  for (int n = 0; n < g.units; ++n) {
    count[n] = 1;
    len[n] = g.steps * g.unit[n].tiles;
  }
  for (;;) {
    int at = 0;
    longest = len[0];
#ifdef __clang__                             // (whole vectors are loaded over the entry that was stored last, which waits for it)
#pragma clang loop vectorize(disable) unroll(disable)
#endif
    for (int n = 1; n < g.units; ++n)
      if (len[n] > longest) { longest = len[n]; at = n; }
    if (total >= g.wgs || count[at] >= g.steps) break;
    ++count[at];
    ++total;
    len[at] = (g.steps + count[at] - 1) / count[at] * g.unit[at].tiles;
  }
  int w = 0;
  if (total <= GRAM_MAX_WGS && longest <= (work + g.wgs - 1) / g.wgs + GRAM_UNIT_COST) {
    for (int n = 0; n < g.units; ++n) {
      g.unit[n].wg0 = (short)w;
      g.unit[n].wgs = (short)count[n];
      for (int i = 0; i < count[n]; ++i) g.bound[w++] = GramBound{n, g.steps * i / count[n]};
    }
    g.wgs = total;
  } else {
    // equal shares of the whole list; one that begins where a unit ends begins with the next
    const int each = work / g.wgs, over = work % g.wgs;
    auto begins = [&](int share) { return each * share + over * share / g.wgs; };
    g.bound[0] = GramBound{0, 0};
    for (int n = 0; n < g.units; ++n) {
      GramUnit& u = g.unit[n];
      const int begin = g.steps * u.tile0, end = begin + g.steps * u.tiles;
      u.wg0 = (short)w;
      while (w + 1 < g.wgs && begins(w + 1) < end) {
        const int step = (begins(w + 1) - begin + u.tiles - 1) / u.tiles;
        if (step >= g.steps) break;
        g.bound[++w] = GramBound{n, step};
      }
      u.wgs = (short)(w - u.wg0 + 1);
      if (w + 1 < g.wgs && begins(w + 1) <= end) g.bound[++w] = GramBound{n + 1, 0};
    }
  }
  g.bound[g.wgs] = GramBound{g.units - 1, g.steps};
  g.part_tiles = 0;
  for (int n = 0; n < g.units; ++n) {
    g.unit[n].part_at = g.part_tiles;
    g.part_tiles += g.unit[n].wgs * g.slices * g.unit[n].qi * g.unit[n].qj;
  }
  return g;
}
