// Which workgroup of the one-vector step's dot and update passes takes which
// row tile (512 rows) and launch position.  Plain integers, so that the host
// and a CPU test use the kernels' own map.
#pragma once

#include <cstddef>

#ifdef __HIPCC__
#define SGN_MAP_FN __host__ __device__ inline
#else
#define SGN_MAP_FN inline
#endif

// Workgroup i runs on XCD i mod 8.  The dot and update passes give the rows of
// tile t (512 rows) to XCD t mod 8, so the columns that the dot pass reads
// into an XCD's 4 MB of L2 are still there for the update pass, and the other
// way round, as far as they fit (the L2 keeps its contents from one kernel to
// the next: 32 MB read twice by the same XCDs take no longer than an empty
// kernel, read by other XCDs 5.8 us).  A launch of few tiles would leave some
// XCDs with a tile more than others, so where the shares would differ by more
// than an eighth launch position z counts its tiles on from z ntiles (elsewhere
// the slots share the Schur rows).  The update walks its tiles from the last to
// the first: what the dot pass read last is then still in the L2 and in the 256
// MB of the Infinity Cache, and so for the next dot pass.
// Dot and update of a step, tiles of both upwards / update downwards: 1764
// sites x 12 slots, FP64, 100 columns 182 / 160 us, 250 columns 399 / 375; 8^4
// x 6, FP32, 150 columns 168 / 137; 8^4 x 1, FP64, 50 columns 28.5 / 25.6;
// 12^4 x 8, FP32, 100 + 100 columns 995 / 955.
constexpr int kXcds = 8;
constexpr int kTileRows = 512;

// Lattices of so few tiles that an XCD would be idle or hold a quarter more
// than its share deal the workgroups of every tile out over all XCDs instead
// (and launch none for tiles that are not there).  By XCD / dealt out (the
// former kernels), FP64, us: 64 sites x 32 slots, 20 columns 27.1 / 13.5 (19.1);
// 380 x 4, 420 columns 58.0 / 51.0 (50.1); 450 x 4, 580 columns 90.0 / 78.5
// (77.8); 720 x 4, 420 columns 93.6 / 85.7 (84.0), 120 columns 33.7 / 34.2
// (34.9); 720 x 8, 300 columns 121 / 114 (120).  14 and 20 tiles are faster by
// XCD: 560 x 8, 580 columns 1.14 times the former kernels' speed, dealt out 1.12;
// 850 x 8, 60 columns 1.18 and 1.12.
// Up to eight tiles the rows count, as the last tile may hold few of them: 300
// sites (seven tiles and 16 rows) x 32, 150 columns 12.6 / 11.7 ms an apply
// (12.3).
SGN_MAP_FN bool dealt_out(int ntiles, int rows) {
  if (ntiles <= kXcds) return rows + rows / 8 < kXcds * kTileRows;
  return ntiles < 3 * kXcds && kXcds * ((ntiles + kXcds - 1) / kXcds) > ntiles + ntiles / 4;
}

SGN_MAP_FN int rotate_tile(int t, int z, int ntiles) {
  const bool uneven = kXcds * ((ntiles + kXcds - 1) / kXcds) > ntiles + ntiles / 8;
  return uneven ? (t & ~(kXcds - 1)) | ((t - z * ntiles) & (kXcds - 1)) : t;
}

// i -> (tile t, index in [0, per) with position z = in mod nb): false for the
// padding.  BY_XCD: dealt out on no lattice (the parts of the dot pass are the
// XCDs').
template <bool DOWN, bool BY_XCD>
SGN_MAP_FN bool tile_of(unsigned i, unsigned per, unsigned nb, int ntiles, int rows, int& t, int& z, int& in) {
  const bool dealt = !BY_XCD && dealt_out(ntiles, rows);
  const unsigned l = dealt ? i : i / kXcds, up = l / per, k = l - up * per;
  in = (int)(k / nb);
  z = (int)(k - (unsigned)in * nb);
  if (dealt) {
    t = DOWN ? ntiles - 1 - (int)up : (int)up;
    return true;
  }
  const unsigned q = DOWN ? (unsigned)(ntiles - 1) / kXcds - up : up;
  t = rotate_tile((int)(q * kXcds + i % kXcds), z, ntiles);
  return t < ntiles;
}

// workgroups of a launch
inline size_t tile_grid(size_t per, int ntiles, int rows, bool by_xcd) {
  if (!by_xcd && dealt_out(ntiles, rows)) return per * ntiles;
  return (size_t)kXcds * per * ((ntiles + kXcds - 1) / kXcds);
}
