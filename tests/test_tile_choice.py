"""The rectangle kernels' tile choice against trying every tile, on the CPU: the header is compiled by itself, with no GPU."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2401_06197_amd", "csrc")

COMPARE = r"""
#include <cstdio>
#include <random>
#include "dcnv4_tile_choice.h"
struct Problem {
    int N, H, W, G, Ho, Wo, sh, sw, ph, pw, dh, dw;
};
struct Tile {
    int R, Q, halo, pitch, tiles_q, tiles_per_img, xtile_bytes;
    bool operator==(const Tile &o) const
    {
        return R == o.R && Q == o.Q && halo == o.halo && pitch == o.pitch && tiles_q == o.tiles_q && tiles_per_img == o.tiles_per_img &&
               xtile_bytes == o.xtile_bytes;
    }
};
// every height of every split, from the highest down; a later one only where it is better
static bool every_tile(const Problem &q, int waves, int halo, int lds, int nbuf, int pb, bool accum, int max_px, int zeros, int slices,
                       int cus, Tile *out, double *cost_out)
{
    const int need = halo > 4 ? halo : 4;
    double best = 1e30;
    int tried = 0;
    for (int kq = 1; kq <= q.Wo && tried < 12; ++kq) {
        const int Q = (q.Wo + kq - 1) / kq;
        if (kq > 1 && Q == (q.Wo + kq - 2) / (kq - 1)) continue;
        long long cols = (Q - 1LL) * q.sw + 2LL * q.dw + 2LL * halo + 2;
        if (cols > q.W + 4) cols = q.W + 4;
        const long long zero = accum ? 16 : ((cols + zeros) * pb + 15) & ~15LL;
        const long long budget = ((((long long)lds - zero) * pb / (pb + (accum ? 4 : 0)) / nbuf) & ~1023LL) / pb;
        if (budget < 64) continue;
        long long top = (budget / cols - 2LL * q.dh - 2LL * halo - 2) / q.sh + 1;
        if (budget / cols >= q.H + 4) top = q.Ho;
        if (top > q.Ho) top = q.Ho;
        if (top < 1 || (top < need && top < q.Ho) || (Q < need && Q < q.Wo)) continue;
        const long long low = top < need ? top : need;
        if (accum && top * Q > max_px) {
            top = max_px / Q;
            if (top < low) continue;
        }
        ++tried;
        const long long tiles_q = (q.Wo + Q - 1) / Q;
        for (long long R = top; R >= low; --R) {
            const long long bands = (q.Ho + R - 1) / R, last = q.Ho - (bands - 1) * R;
            const long long full = (R * Q + 63) / 64, part = (last * Q + 63) / 64;
            const double img = tiles_q * ((bands - 1) * (double)((full + waves - 1) / waves) + (double)((part + waves - 1) / waves) +
                                          (nbuf == 1 && !accum ? 6.0 : 4.0) * bands);
            const long long tiles = (long long)q.N * q.G * slices * bands * tiles_q;
            const double cost = (double)((tiles + cus - 1) / cus) * (img / (double)(bands * tiles_q));
            if (cost < best - 1e-9) {
                best = cost;
                long long rows = (R - 1) * q.sh + 2LL * q.dh + 2LL * halo + 2;
                if (rows > q.H + 4) rows = q.H + 4;
                *out = {(int)R, Q, halo, (int)cols, (int)tiles_q, (int)(bands * tiles_q), (int)((rows * cols * pb + 1023) & ~1023LL)};
            }
        }
    }
    *cost_out = best;
    return best < 1e30;
}
int main()
{
    std::mt19937 g(5);
    auto in = [&](int lo, int hi) { return lo + (int)(g() % (unsigned)(hi - lo + 1)); };
    auto of = [&](std::initializer_list<int> l) { return l.begin()[g() % l.size()]; };
    int found = 0;
    for (int i = 0; i < 30000; ++i) {
        const int most = i % 5 ? 70 : 500;
        Problem q = {of({1, 2, 3, 8, 64, 1000}), in(1, most), in(1, most), of({1, 2, 3, 8, 33}), 0, 0, of({1, 1, 1, 2, 3}), of({1, 1, 2}),
                     of({0, 1, 2, 9, 40}), of({0, 1, 5}), of({1, 1, 2, 7}), of({1, 1, 3})};
        if (q.H + 2 * q.ph < 2 * q.dh + 1 || q.W + 2 * q.pw < 2 * q.dw + 1) continue;
        q.Ho = (q.H + 2 * q.ph - 2 * q.dh - 1) / q.sh + 1;
        q.Wo = (q.W + 2 * q.pw - 2 * q.dw - 1) / q.sw + 1;
        const bool accum = in(0, 3) == 0;
        const int waves = of({1, 2, 4, 8, 12}), halo = in(1, 9), lds = 1024 * of({8, 16, 40, 100, 158, 160}), nbuf = accum ? 1 : in(1, 2);
        const int pb = of({16, 32, 64, 128}), slices = of({1, 1, 2, 4}), cus = of({256, 256, 304, 38}), max_px = of({29000, 500});
        Tile a{}, b{};
        double ca, cb;
        const bool fa = tile_choice(q, waves, halo, lds, nbuf, pb, accum, max_px, 2, slices, cus, &a, &ca);
        const bool fb = every_tile(q, waves, halo, lds, nbuf, pb, accum, max_px, 2, slices, cus, &b, &cb);
        if (fa != fb || (fa && (!(a == b) || ca != cb)))
            return printf("case %d: %d %d, %d x %d (%g) and %d x %d (%g)\n", i, fa, fb, a.R, a.Q, ca, b.R, b.Q, cb), 1;
        found += fa;
    }
    return found > 10000 ? 0 : 2;
}
"""


def test_tile_choice_is_that_of_trying_every_tile(tmp_path):
    (tmp_path / "compare.cpp").write_text(COMPARE)
    exe = str(tmp_path / "compare")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, "-o", exe, str(tmp_path / "compare.cpp")], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert res.returncode == 0, res.stdout
