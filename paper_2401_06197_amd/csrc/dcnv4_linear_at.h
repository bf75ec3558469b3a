// Where the linear kernel's loads lie (plain functions, so that they can be walked over on the CPU).
//
// A load has a vector and a scalar byte offset, and the range check that makes it read zero is documented for the vector
// offset alone.  So what lies past an end -- of K, of a layer's rows, of the last pass -- has the vector offset
// `outside` and no scalar one; everything else lies inside the tensor with both.
#pragma once

struct LinAt {
    int v, s;
};

// Unit tid % 16 of row n0 + 16 * i + tid / 16 of a layer's weights, K bytes from kbase on.  nout is a multiple of 32:
// a unit's 16 rows are all there or all past the last one, so the scalar offset is the same for all threads.
constexpr LinAt lin_weight_at(int tid, int i, int n0, int kbase, int nout, int kbytes, int outside)
{
    const int row = n0 + 16 * i, u = (tid & 15) * 16;
    return {row < nout && kbase + u < kbytes ? (tid >> 4) * kbytes + u : outside, row < nout ? row * kbytes + kbase : 0};
}

// The 32-byte group at byte column col (the same for all lanes) of the pixel row that starts at xo.  Plane-major x: column c
// lies in plane c >> shift, at c & (2^shift - 1) of the pixel's piece there.
constexpr LinAt lin_x_at(int xo, int col, int kbytes, int plane_shift, int plane_stride, int outside)
{
    if (col >= kbytes)
        return {outside, 0};
    return {xo, plane_shift == 0 ? col : (col >> plane_shift) * plane_stride + (col & ((1 << plane_shift) - 1))};
}
