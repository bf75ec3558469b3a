// Where the linear kernel's loads lie (plain functions, so that they can be walked over on the CPU).
//
// A load has a vector and a scalar byte offset, and the range check that makes it read zero is documented for the vector
// offset alone.  So what lies past an end -- of K, of a layer's rows, of the last pass -- has the vector offset
// `outside`, or a descriptor of no bytes, and no scalar offset; everything else lies inside the tensor with both.
#pragma once

struct LinAt {
    int v, s;
};

// Unit tid % 16 of row n0 + 16 * i + tid / 16 of a layer's weights, K bytes from kbase on.  nout is a multiple of 32:
// the 16 rows of a unit are all there or all past the last one, which is the same for all threads, as is the scalar offset
// (so the choice takes scalar instructions only: in the vector offset it cost the fp16 layers 1 to 2 %).
struct LinWeightAt {
    LinAt at;
    unsigned bytes;      // of the descriptor
};
constexpr LinWeightAt lin_weight_at(int tid, int i, int n0, int kbase, int nout, int kbytes, int outside)
{
    const int row = n0 + 16 * i, u = (tid & 15) * 16;
    const bool in = n0 + 16 * (i & ~1) < nout;             // (32 rows at a time)
    return {{kbase + u < kbytes ? (tid >> 4) * kbytes + u : outside, in ? row * kbytes + kbase : 0},
            in ? (unsigned)nout * (unsigned)kbytes : 0u};
}

// The 32-byte group at byte column col (the same for all lanes) of the pixel row that starts at xo.  Plane-major x: column c
// lies in plane c >> shift, at c & (2^shift - 1) of the pixel's piece there.
constexpr LinAt lin_x_at(int xo, int col, int kbytes, int plane_shift, int plane_stride, int outside)
{
    if (col >= kbytes)
        return {outside, 0};
    return {xo, plane_shift == 0 ? col : (col >> plane_shift) * plane_stride + (col & ((1 << plane_shift) - 1))};
}

// Byte column `col` of a pixel row, counted from the row's first byte: rows (shift 0), or planes of 2^shift bytes that lie
// plane_stride apart.
constexpr int lin_plane_at(int col, int plane_shift, int plane_stride)
{
    return plane_shift == 0 ? col : (col >> plane_shift) * plane_stride + (col & ((1 << plane_shift) - 1));
}
