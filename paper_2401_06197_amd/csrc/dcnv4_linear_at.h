// Where the linear kernels' loads and stores lie (plain functions, so that they can be walked over on the CPU).
//
// The kernel that keeps x: a load has a vector and a scalar byte offset, and the range check that makes it read zero is
// documented for the vector offset alone.  So what lies past an end -- of K, of a layer's rows, of the last pass -- has the
// vector offset `outside`, or a descriptor of no bytes, and no scalar offset; everything else lies inside the tensor with both.
// The tiles: vector offsets only.  Rows past the last are the last one once more, units past the end of K have the bit
// `outside` (2^31, past any descriptor).
#pragma once

struct LinAt {
    int v, s;
};

// Unit tid % 16 of row n0 + 16 * i + tid / 16 of a layer's weights.  nout is a multiple of 32:
// the 16 rows of a unit are all there or all past the last one, which is the same for all threads, as is the scalar offset
// (so the choice takes scalar instructions only: in the vector offset it cost the fp16 layers 1 to 2 %).
struct LinWeightAt {
    LinAt at;
    unsigned bytes;      // of the descriptor
};
constexpr LinWeightAt lin_weight_at(int tid, int i, int n0, int nout, int kbytes, int outside)
{
    const int row = n0 + 16 * i, u = (tid & 15) * 16;
    const bool in = n0 + 16 * (i & ~1) < nout;             // (32 rows at a time)
    return {{u < kbytes ? (tid >> 4) * kbytes + u : outside, in ? row * kbytes : 0}, in ? (unsigned)nout * (unsigned)kbytes : 0u};
}

// Byte column `col` of a pixel row, counted from the row's first byte: rows (shift 0), or planes of 2^shift bytes that lie
// plane_stride apart: column c lies in plane c >> shift, at c & (2^shift - 1) of the pixel's piece there.
constexpr int lin_plane_at(int col, int plane_shift, int plane_stride)
{
    return plane_shift == 0 ? col : (col >> plane_shift) * plane_stride + (col & ((1 << plane_shift) - 1));
}

// The 32-byte group at byte column col (the same for all lanes) of the pixel row that starts at xo.
constexpr LinAt lin_x_at(int xo, int col, int kbytes, int plane_shift, int plane_stride, int outside)
{
    if (col >= kbytes)
        return {outside, 0};
    return {xo, lin_plane_at(col, plane_shift, plane_stride)};
}

// The tiles.  A row or the last one:
constexpr int lin_row(int row, int rows)
{
    return row < rows - 1 ? row : rows - 1;
}
// Byte column `col` of pixel px, of x and of a layer's results: rows, or planes of image img (of hw pixels).
constexpr int lin_pixel_at(int px, int row_bytes, int col)
{
    return px * row_bytes + col;
}
constexpr int lin_pixel_in_planes_at(int px, int img, int hw, int row_bytes, int col, int plane_shift)
{
    return img * hw * row_bytes + ((px - img * hw) << plane_shift) + lin_plane_at(col, plane_shift, hw << plane_shift);
}
// What is to be added to the place of unit `unit` of K's first step for step t, and `outside` where that unit is past the end.
// (Steps of 64 or 128 bytes and planes of 32 to 128: neither crosses the other in part, so the two parts of a column add up.)
constexpr unsigned lin_step_at(int t, int step, int plane_shift, int plane_stride)
{
    return (unsigned)lin_plane_at(t * step, plane_shift, plane_stride);
}
constexpr unsigned lin_past(int t, int step, int unit, int kbytes, int outside)
{
    return t * step + unit * 16 < kbytes ? 0u : (unsigned)outside;
}
