// Tile choice of the rectangle kernels (a plain function, so that it can be compared with trying every tile, on the CPU).
#pragma once

// Tile choice for the LDS-staged forward: full-width row bands when a band with a useful
// number of rows fits the LDS budget, otherwise split the columns too.  Returns false when
// no tile with at least as many output rows/cols as the halo fits (the rectangle would be
// mostly halo); the caller then uses the direct kernel.
//   waves, lds_bytes   of a workgroup (without its per-wave slices); nbuf rectangles of pixels of pb bytes
//   accum              the rectangle is an accumulator, with a dword more per pixel; tiles of up to max_px output pixels
//   zero_pixels        staged pixels of zeros beyond a row's
template <class Problem, class Out>
bool tile_choice(const Problem &q, int waves, int halo, int lds_bytes, int nbuf, int pb, bool accum, int max_px, int zero_pixels,
                 int chan_slices, int cus, Out *out, double *cost_out)
{
    const int need = halo > 4 ? halo : 4;
    // Cost of a candidate (column splits kq, band height R), in units of one round (= every wave
    // of a workgroup doing one batch of 64 output pixels): a tile of B batches takes ceil(B / waves)
    // rounds plus about four for the switch (barrier, drained pipeline; measured; six with a single
    // buffer, whose refill is not hidden), and a workgroup
    // works through ceil(tiles / CUs) tiles -- so few, huge tiles that leave CUs idle lose against
    // more, smaller ones.
    double best_cost = 1e30;
    bool found = false;
    int splits_tried = 0;
    for (int kq = 1; kq <= q.Wo && splits_tried < 12; ++kq) {
        const int Q = (q.Wo + kq - 1) / kq;
        if (kq > 1 && Q == (q.Wo + kq - 2) / (kq - 1))
            continue;                        // same tile width as the previous split count
        long long cols = (long long)(Q - 1) * q.sw + 2LL * q.dw + 2LL * halo + 2;
        if (cols > q.W + 4) cols = q.W + 4;
        // the rectangle buffers (each a multiple of 1 KiB) share what the slices leave, after
        // a block of zeros (pitch + 2 pixels) or one more dword per rectangle pixel (the bound words of the grad_x accumulator)
        const long long zero_bytes = accum ? 16 : ((cols + zero_pixels) * pb + 15) & ~15LL;
        const long long budget_px =
            ((((long long)lds_bytes - zero_bytes) * pb / (pb + (accum ? 4 : 0)) / nbuf) & ~1023LL) / pb;
        if (budget_px < 64)
            continue;
        const long long rows_max = budget_px / cols;
        long long Rmax = (rows_max - 2LL * q.dh - 2LL * halo - 2) / q.sh + 1;
        if (rows_max >= q.H + 4) Rmax = q.Ho;               // the whole (clipped) height fits
        if (Rmax > q.Ho) Rmax = q.Ho;
        if (Rmax < 1 || (Rmax < need && Rmax < q.Ho) || (Q < need && Q < q.Wo))
            continue;
        const long long Rlow = Rmax < need ? Rmax : need;
        if (accum && Rmax * Q > max_px) {        // (the bound words must not wrap)
            Rmax = max_px / Q;
            if (Rmax < Rlow)
                continue;
        }
        ++splits_tried;
        const int tiles_q = (q.Wo + Q - 1) / Q;
        const int px_round = 64 * waves, top = (int)Rmax, low = (int)Rlow;
        const double change = nbuf == 1 && !accum ? 6.0 : 4.0;
        // Band heights from the highest down, those that cut the image into the same number of bands together: none of them
        // takes fewer rounds than all rows in one piece, so most numbers of bands are dropped by one comparison, and all
        // further ones once an even share of the rounds and switches is no better (the choice is that of trying every height:
        // 1 image of 200x200, 4 groups of 8: 75 us of host time for the whole forward call that way, 6.5 like this)
        const int least = (q.Ho * Q + px_round - 1) / px_round;
        const double even = (double)q.N * q.G * chan_slices * tiles_q / cus * (1.0 - 1e-12);
        for (int R = top; R >= low;) {
            const int bands = (q.Ho + R - 1) / R, same = (q.Ho + bands - 1) / bands, last = same > low ? same : low;
            if (even * (least + change * bands) >= best_cost)
                break;
            const long long tiles = (long long)q.N * q.G * chan_slices * bands * tiles_q;
            const double share = tiles < (1LL << 31) ? (double)(((unsigned)tiles + (unsigned)cus - 1u) / (unsigned)cus) : (double)((tiles + cus - 1) / cus);
            auto cost_of = [&](int rounds) { return share * (tiles_q * (rounds + change * bands) / (double)(bands * tiles_q)); };
            for (; R >= last && cost_of(least) < best_cost - 1e-9; --R) {
                const int rounds = (bands - 1) * ((R * Q + px_round - 1) / px_round) +
                                   ((q.Ho - (bands - 1) * R) * Q + px_round - 1) / px_round;
                const double cost = cost_of(rounds);
                if (cost < best_cost - 1e-9) {
                    best_cost = cost;
                    found = true;
                    long long rows = (R - 1) * (long long)q.sh + 2LL * q.dh + 2LL * halo + 2;
                    if (rows > q.H + 4) rows = q.H + 4;
                    out->R = R;
                    out->Q = Q;
                    out->halo = halo;
                    out->pitch = (int)cols;
                    out->tiles_q = tiles_q;
                    out->tiles_per_img = bands * tiles_q;
                    out->xtile_bytes = (int)((rows * cols * pb + 1023) & ~1023LL);
                }
            }
            R = last - 1;
        }
    }
    if (cost_out)
        *cost_out = best_cost;
    return found;
}
