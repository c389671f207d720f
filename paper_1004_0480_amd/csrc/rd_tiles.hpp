// rd_tiles.hpp -- the tile of a workgroup of the register marches.
#pragma once

#ifdef __HIPCC__
#define RD_TILES_FN __host__ __device__ __forceinline__
#else
#define RD_TILES_FN inline
#endif

namespace rdk {

// Workgroup b's tile of tiles_x * tiles_y * chunks: x first, then y, then the z
// chunk, or (zfast: a plan's order 1) the z chunk first.
struct MarchTile { int x, y, z; };
RD_TILES_FN MarchTile march_tile(int b, int tiles_x, int tiles_y, int chunks, bool zfast) {
    const int n0 = zfast ? chunks : tiles_x, n1 = zfast ? tiles_x : tiles_y;
    const int r = b / n0, i0 = b - r * n0, i2 = r / n1, i1 = r - i2 * n1;
    return zfast ? MarchTile{i1, i2, i0} : MarchTile{i0, i1, i2};
}

}  // namespace rdk
