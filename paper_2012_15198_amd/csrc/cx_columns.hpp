// Which columns a lane touches in a tile that a segment boundary or the row end crosses (a boundary tile).
// Plain C++ with no device intrinsics, so that the same text runs inside the kernels (the including file
// defines CX_SCHED_FN as __device__ __forceinline__) and in a host test.
//
// Columns [P, ld) of a row are never read, and the last row's storage may end at column P.  A slice that hangs
// over the row end can therefore not be loaded where it stands, and column by column its loads would cost the
// wavefront memory latencies of their own on every row.  So a lane's slices slide: they start the few columns
// earlier that make the one at the row end stop at P, and columns that belong to another lane's slice are masked off.
//   one slice per lane:  the lane whose slice is cut slides; needs P >= one slice;
//   more per lane:       all lanes of the tile slide, so that the slices stay gapless; needs P >= one tile.
// The host chooses the shape accordingly (rows shorter than a tile take one slice per lane, rows shorter than a
// slice the short-row kernels, which load column by column).
#ifndef CX_COLUMNS_HPP
#define CX_COLUMNS_HPP
#include <cstdint>

#ifndef CX_SCHED_FN
#define CX_SCHED_FN inline
#endif

// By how many columns the slices of the lane slide whose first slice stands at column `place` of the tile at c0.
CX_SCHED_FN int row_end_slide(int64_t P, int64_t c0, int64_t place, int slices_per_lane, int tile_cols, int slice_cols)
{
    if (c0 + tile_cols <= P) return 0;
    if (slices_per_lane > 1) return static_cast<int>(-P & (slice_cols - 1));
    const int64_t over = place + slice_cols - P;
    return over > 0 && over < slice_cols ? static_cast<int>(over) : 0;
}

// Bit q: column first + q lies in [b, e).
CX_SCHED_FN unsigned slice_mask(int64_t first, int slice_cols, int64_t b, int64_t e)
{
    unsigned mask = 0;
#pragma unroll
    for (int q = 0; q < slice_cols; ++q)
        if (first + q >= b && first + q < e) mask |= 1u << q;
    return mask;
}

// Where the lane's wanted columns of a piece [b, e) begin: a single slice that slid leaves to the lane before it
// the columns that stand in that one's slice.
CX_SCHED_FN int64_t wanted_from(int64_t b, int64_t place, int slices_per_lane)
{
    return slices_per_lane == 1 && place > b ? place : b;
}

#endif  // CX_COLUMNS_HPP
