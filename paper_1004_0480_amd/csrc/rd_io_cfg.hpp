// rd_io_cfg.hpp -- how the layout conversions (rd_io.hpp) are split into
// workgroups: host arithmetic alone, shared with the kernels.
#pragma once

#include <algorithm>
#include <cstdint>

namespace rdk {

constexpr int IO_DEPTH = 4;                       // units of four cells a thread has in flight
constexpr int IO_CELLS = 256 * 4;                 // cells of a workgroup's turn at depth 1
constexpr int IO_MAX_BLOCKS = (1 << 24) - 1;      // a launch holds fewer than 2^32 threads, 256 a workgroup

// Workgroups of a conversion: runs of whole rows, 4096 cells each (four units
// of four cells per thread), fewer where that would not give each CU several
// workgroups; a row longer than that is split into equal parts, so that fields
// of few long rows fill the chip as well (one row of 2^24 FP32 cells, written:
// 5.87 ms by one workgroup per row, 21 us by parts).
struct RowRuns {
    long long rows;
    int run, parts;      // rows of a workgroup, workgroups of a row (one of the two is 1)
    unsigned blocks;
    bool deep;           // more than one turn at depth 1
};
inline RowRuns row_runs(int64_t nx, int64_t rows) {
    const int64_t cells = std::min<int64_t>(IO_DEPTH * IO_CELLS, std::max<int64_t>(IO_CELLS, nx * rows / 2048));
    const int64_t row = (nx + 3) / 4 * 4;
    // (longer runs where the count of workgroups would not fit a launch)
    const int64_t run = std::max<int64_t>({1, cells / row, (rows + IO_MAX_BLOCKS - 1) / IO_MAX_BLOCKS});
    const int64_t parts = run > 1 ? 1 : std::min<int64_t>((row + cells - 1) / cells, IO_MAX_BLOCKS / rows);
    return RowRuns{(long long)rows, int(run), int(parts), unsigned((rows + run - 1) / run * parts),
                   run * ((row + parts - 1) / parts) > IO_CELLS};
}

}  // namespace rdk
