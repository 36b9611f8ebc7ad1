// Which tile of a problem a block works on, in the launches of the matrix kernel and of expand + depthwise.
// Hardware block b runs on XCD b % 8.  A launch is rows of 8 blocks; each XCD takes an eighth of every problem's tiles,
// consecutive ones, so that tiles which read the same activations share an L2, and works through the problems in turn.  One range of consecutive tiles per XCD over all problems of a mixed
// call, as before, left the XCD with the widest subnets' tiles with 1.2 to 1.75 times the mean's work in the 3x3 layers:
// 64 requests over sixteen ResNet-shaped subnets 2211 -> 2109 us; a lone request of the largest subnet, whose few tiles
// used to fill up the first XCDs, 490 -> 476.
// An XCD's blocks without a tile come last.  With rows for every problem they lay in between, and as blocks go to the
// shader engines in turn, some engines got one block more than they have CUs while a CU elsewhere stood idle: the three
// projections of 14 sequences, 252 tiles of one block a CU, took 19 us instead of 13; 14 sequences 969 -> 880 us, 64 mixed
// requests 2087 -> 1948.
#pragma once

#if defined(__HIPCC__)
#define SNA_HD __host__ __device__ __forceinline__
#else
#define SNA_HD inline
#endif

namespace sna {

constexpr int kXcds = 8;
SNA_HD int tile_rows(int tiles) { return (tiles + kXcds - 1) / kXcds; }

// The first tile of XCD x's share of a problem.  tile_start, the rows of 8 that the problems before it would fill, only
// decides which XCDs take one tile more than the others, differently for the problems of a launch.
SNA_HD int first_tile(int tiles, int tile_start, int x) { return (x * tiles + (tile_start & (kXcds - 1))) >> 3; }

// The tile that block b works on in a launch of one problem, or -1.
SNA_HD int tile_of_block(int tiles, int tile_start, int b) {
  const int x = b & (kXcds - 1), t = first_tile(tiles, tile_start, x) + (b >> 3);
  return t < first_tile(tiles, tile_start, x + 1) ? t : -1;
}

// Problem and tile of block b, tile -1 if it has none.
struct TilePlace { int problem, tile; };
template <class Args>
SNA_HD TilePlace place_of_block(const Args& a, int b) {
  const int x = b & (kXcds - 1);
  int j = b >> 3;
  for (int g = 0; g < a.n; ++g) {
    const int tiles = a.p[g].tiles, start = a.p[g].tile_start;
    const int lo = first_tile(tiles, start, x), count = first_tile(tiles, start, x + 1) - lo;
    if (j < count) return {g, lo + j};
    j -= count;
  }
  return {0, -1};
}

// Blocks of a launch: 8 for every tile of the XCD that has most.
template <class Args>
inline int launch_blocks(const Args& a) {
  int most = 0;
  for (int x = 0; x < kXcds; ++x) {
    int count = 0;
    for (int g = 0; g < a.n; ++g) count += first_tile(a.p[g].tiles, a.p[g].tile_start, x + 1) - first_tile(a.p[g].tiles, a.p[g].tile_start, x);
    most = count > most ? count : most;
  }
  return most * kXcds;
}

}  // namespace sna
