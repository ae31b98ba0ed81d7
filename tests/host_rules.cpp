// The tile arithmetic of the region launch (csrc/lbm_internal.h), built for the host.
#include "lbm_internal.h"

using namespace lbmk;

// The first work-group of a launch over ntx x nty tiles (frame: of its frame only) whose tile is not
// the one a division gives, -1 when all are right.
extern "C" long long first_wrong_tile(int ntx, int nty, int frame, int pery, int perx) {
  if (!frame) {
    const uint32_t divisor = tile_divisor(ntx);
    for (long long b = 0; b < (long long)ntx * nty; ++b) {
      const TileIndex t = region_tile((int)b, ntx, divisor);
      if (t.by != b / ntx || t.bx != b % ntx) return b;
    }
    return -1;
  }
  const int rows = pery ? 0 : 2 * ntx, grid = rows + (perx ? 0 : 2 * (nty - (pery ? 0 : 2)));
  for (int b = 0; b < grid; ++b) {
    const TileIndex t = frame_tile(b, ntx, nty - 1, pery != 0);
    const int q = b - rows;
    const int by = q < 0 ? (b / ntx ? nty - 1 : 0) : (pery ? 0 : 1) + q / 2;
    const int bx = q < 0 ? b % ntx : (q % 2 ? ntx - 1 : 0);
    if (t.bx != bx || t.by != by) return b;
  }
  return -1;
}

extern "C" int divides_exactly(long long tiles, int ntx) { return tile_divisor_exact(tiles, ntx); }
