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
    MarchTile t;
    if (zfast) {
        t.z = b % chunks;
        b /= chunks;
        t.x = b % tiles_x;
        t.y = b / tiles_x;
    } else {
        t.x = b % tiles_x;
        b /= tiles_x;
        t.y = b % tiles_y;
        t.z = b / tiles_y;
    }
    return t;
}

}  // namespace rdk
