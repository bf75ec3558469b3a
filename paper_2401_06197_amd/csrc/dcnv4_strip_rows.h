// Which rows of its window a batch of the strip kernel reaches (plain functions, so that the order in which rows come and
// go can be walked over on the CPU).  P points to the plan; tr is an output row of the tile, oh0 the tile's first one.
//
// A workgroup's rows are numbered through: row r of the window of its s-th tile is virtual row s*VR + r, and lies in slot
// (virtual row mod ring).  The rows asked for so far are a count that only grows, and a batch's last row is never before its
// tile's first one, however far above the image (padding) its window lies: a count below zero would ask for rows that are in
// no tile, in slots that rows of the same round have.
#pragma once

template <class P> constexpr int strip_row_want(P p, int oh0) { return oh0 * p->sh - p->ph - p->halo_r; }
template <class P> constexpr int strip_row_end(P p, int oh0)
{
    return ((oh0 + p->R < p->Ho ? oh0 + p->R : p->Ho) - 1) * p->sh - p->ph + 2 * p->dh + p->halo_r + 2;
}
// first row and number of rows of a tile's window, clipped to the image plus a two-pixel border
template <class P> constexpr int strip_row_from(P p, int oh0)
{
    return strip_row_want(p, oh0) > -2 ? strip_row_want(p, oh0) : -2;
}
template <class P> constexpr int strip_rows(P p, int oh0)
{
    const int end = strip_row_end(p, oh0), n = (end < p->H + 2 ? end : p->H + 2) - strip_row_from(p, oh0);
    return n > 0 ? n : 0;
}
// virtual rows that a batch can reach within the halo: the first, by its first pixel's row, and the last, by its last one's
template <class P> constexpr int strip_first_row(P p, int s, int oh0, int tr)
{
    const int r = strip_row_want(p, oh0 + tr) - strip_row_from(p, oh0), n = strip_rows(p, oh0);
    return s * p->VR + (r < 0 ? 0 : r < n ? r : n);
}
template <class P> constexpr int strip_last_row(P p, int s, int oh0, int tr)
{
    const int r = (oh0 + tr) * p->sh - p->ph + 2 * p->dh + p->halo_r + 1 - strip_row_from(p, oh0), n = strip_rows(p, oh0);
    return s * p->VR + (r < -1 ? -1 : r < n - 1 ? r : n - 1);
}
// rows asked for before the first round
constexpr int strip_asked_first(int last_row, int ring, int total)
{
    const int f = last_row + 1 < ring ? last_row + 1 : ring;
    return f < total ? f : total;
}
// ... and by the end of a round: up to the last row of the batches after it, as far as the ring can take them while this
// round's first row is in use; never fewer than before, and at most a ring of rows more
constexpr int strip_wanted(int last_row_next, int first_row, int ring, int total)
{
    const int f = last_row_next + 1 < first_row + ring ? last_row_next + 1 : first_row + ring;
    return f < total ? f : total;
}
constexpr int strip_asked(int wanted, int before, int ring)
{
    const int f = wanted < before + ring ? wanted : before + ring;
    return f > before ? f : before;
}
