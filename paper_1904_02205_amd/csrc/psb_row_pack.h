// How the row packing of a first layer (TransposeJob) is cut into tiles.  No HIP types, so that it can be tested without a GPU.
#pragma once
#include <stdint.h>

#include <algorithm>

namespace psb {

constexpr int kRowPackOutputs = 256;         // packed pixels of a tile: one per thread
constexpr int kRowPackLds = 12288;           // bytes of its image rows in LDS

// A tile is `rows` whole rows of packed pixels, or (rows = 1) one of the `segments` of a row, `outputs` pixels each.  Its part of an
// image row lies in LDS with the channels of a pixel next to each other: columns first .. first + cols - 1, row_bytes from one row
// to the next, so that a packed pixel is 32 consecutive bytes from stride_w * C times its number in the segment on.  The last word
// that it reads starts up to 32 bytes behind that.
struct RowPackTiles { int outputs, segments, rows, cols, row_bytes; };

inline RowPackTiles row_pack_tiles(int64_t n_rows, int OW, int stride_w, int C, int KW)
{
    const int64_t step = (int64_t)stride_w * C;                  // bytes between the packed pixels of a row
    RowPackTiles t;
    const int most = (int)std::min<int64_t>(std::min(OW, kRowPackOutputs), 1 + (kRowPackLds - 36) / step);
    t.segments = (OW + most - 1) / most;
    t.outputs = (OW + t.segments - 1) / t.segments;
    const int64_t last = (t.outputs - 1) * step;
    t.cols = (int)((int64_t)(t.outputs - 1) * stride_w) + KW;
    t.row_bytes = (int)((last + 36 + 3) / 4 * 4);
    t.rows = t.segments > 1 ? 1 : (int)std::min<int64_t>(n_rows, std::min(kRowPackOutputs / t.outputs, kRowPackLds / t.row_bytes));
    return t;
}

}  // namespace psb
