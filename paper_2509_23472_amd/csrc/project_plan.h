// Rules of the projection's work split (stream_bf16.h).  Plain C++, so that they can be tested without a GPU.
#pragma once
#include <cstdint>

#ifdef __HIPCC__
#define PJ_FN __host__ __device__ __forceinline__
#else
#define PJ_FN inline
#endif

// Shares [first, end) of the items that reach into an output tile; share w begins at item floor(items w / wgs).  Only the first of
// them may begin in a tile before, first_tile.  (Closed forms: walked share by share with a 64-bit division each, this was 2 us
// of the launch that adds the partial tiles.)
struct ProjectShares { int64_t first, end, first_tile; };
template <typename T>
PJ_FN ProjectShares project_shares_of(T items, T wgs, T slabs, T tile) {
  const T lo = tile * slabs, hi = lo + slabs;
  const T first = ((lo + 1) * wgs + items - 1) / items - 1;
  return ProjectShares{(int64_t)first, (int64_t)((hi * wgs + items - 1) / items), (int64_t)(items * first / wgs / slabs)};
}
// In 32 bits where the numbers allow it (wgs <= PJ_MAX_WGS).
#define PJ_MAX_WGS 512
#define PJ_ITEMS_32 ((1ll << 31) / (PJ_MAX_WGS + 1))
PJ_FN ProjectShares project_shares(int64_t items, int wgs, int slabs, int64_t tile) {
  return items < PJ_ITEMS_32 ? project_shares_of<unsigned>((unsigned)items, (unsigned)wgs, (unsigned)slabs, (unsigned)tile)
                             : project_shares_of<int64_t>(items, wgs, slabs, tile);
}

// Order in which the shares are dealt out to the eight compute dies (workgroup b runs on die b mod 8): by the begin of the share modulo
// `period`, in eight consecutive runs, or by number if not `sorted`.  The begins are built up by additions and the sort is one pass over
// 256 buckets (exact up to a period of 256, a finer order is of no use): with two 64-bit divisions a share and a comparison sort this
// was 9.0 us of host time for 512 shares, now 1.7, twice in a step.
// long_first: a die takes those of its run that are an item longer first.  Two workgroups of the reconstruction share a CU, the j-th of a die and the
// one that is as many further on as it has CUs; in the order of the run, with one and a half items to a share, they were two long ones or two short
// ones (us, before and after: 16384 x 768 of rank 256 19.3 and 18.3, 12608 x 768 15.1 and 13.9, of rank 64 9.1 and 8.4, 8192 x 1088 of rank 256 18.3 and 16.6).
static inline void project_share_order(int64_t items, int wgs, int64_t period, bool sorted, unsigned short* share_of, bool long_first = false) {
  unsigned char bucket[PJ_MAX_WGS];
  bool longer[PJ_MAX_WGS];
  unsigned short order[PJ_MAX_WGS];
  int start[257] = {0};
  int shift = 0;
  while (((period - 1) >> shift) > 255) ++shift;
  const int64_t step = items / wgs, rem = items % wgs, step_in = step % period;
  int64_t key = 0, cut = 0;                      // floor(items w / wgs) mod period, and what the floor has cut off, times wgs
  for (int w = 0; w < wgs; ++w) {
    bucket[w] = sorted ? (unsigned char)(key >> shift) : 0;
    ++start[bucket[w] + 1];
    key += step_in;
    cut += rem;
    longer[w] = long_first && cut >= wgs;
    if (cut >= wgs) { cut -= wgs; ++key; }
    if (key >= period) key -= period;
  }
  for (int i = 0; i < 256; ++i) start[i + 1] += start[i];
  for (int w = 0; w < wgs; ++w) order[start[bucket[w]]++] = (unsigned short)w;
  for (int die = 0, at = 0; die < 8; ++die) {
    const int end = at + (wgs - die + 7) / 8;
    int first = 0;
    for (int i = at; i < end; ++i) first += longer[order[i]];
    for (int pos[2] = {first, 0}; at < end; ++at) share_of[die + 8 * pos[longer[order[at]]]++] = order[at];     // (the others after the longer ones)
  }
}

// Few slabs and tiles of 64 rows: whether a workgroup takes a whole output tile, which then goes straight to V, instead of a share of
// four slabs whose partial tiles a launch adds up.  That launch and the stores it reads take about as long as two to three
// slabs more in a row, the most where there are many tiles (four slabs or fewer are one share either way).  Whole compress of
// rank 64, us, by shares and straight: 320 rows x 128 40.8 and 40.4, x 8192 51.0 and 47.2; 384 x 128 41.6 and 42.0, x 256 43.8 and 42.3; 448 x
// 256 43.2 and 43.7, x 512 45.7 and 45.0, x 8192 52.2 and 49.5; 512 x 256 43.0 and 44.2, x 2048 47.2 and 48.3, x 8192 51.0 and
// 50.1 (rank 16 35.6 and 36.0).  U^T G of the LoRA gradient at 512 rows, ranks 64 (one tile) 24.4 and 26.3, 256 (four) 37.6 and 39.2.
static inline bool project_goes_direct(int64_t slabs, int64_t tiles) {
  return slabs <= (tiles > 3 ? 7 : (tiles > 1 ? 6 : 5));
}
