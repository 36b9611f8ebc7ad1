// Which tile of a problem a block works on, in the launches of the matrix kernel and of expand + depthwise.
// Hardware block b runs on XCD b % 8.  A launch is rows of 8 blocks, and every problem of it has rows of its own:
// ceil(tiles / 8) from tile_start on, in which each XCD takes an eighth of the problem's tiles, consecutive ones, so that
// tiles which read the same activations share an L2.  One range of consecutive tiles per XCD over all problems of a mixed
// call, as before, left the XCD with the widest subnets' tiles with 1.2 to 1.75 times the mean's work in the 3x3 layers:
// 64 requests over sixteen ResNet-shaped subnets 2211 -> 2109 us; a lone request of the largest subnet, whose few tiles
// used to fill up the first XCDs, 490 -> 476.
#pragma once

#if defined(__HIPCC__)
#define SNA_HD __host__ __device__ __forceinline__
#else
#define SNA_HD inline
#endif

namespace sna {

constexpr int kXcds = 8;
SNA_HD int tile_rows(int tiles) { return (tiles + kXcds - 1) / kXcds; }

// The tile that block b works on in a problem of `tiles` tiles whose rows begin at tile_start, or -1.  `phase` only decides
// which XCDs take one tile more than the others, differently for the problems of a launch.
SNA_HD int tile_of_block(int tiles, int tile_start, int b) {
  const int x = b & (kXcds - 1), phase = tile_start & (kXcds - 1);
  const int lo = (x * tiles + phase) >> 3, hi = ((x + 1) * tiles + phase) >> 3;
  const int t = lo + (b >> 3) - tile_start;
  return t < hi ? t : -1;
}

}  // namespace sna
