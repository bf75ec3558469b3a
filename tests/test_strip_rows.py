"""Which rows the strip kernel asks for, round by round, walked over on the CPU: the header is compiled by itself, with no
GPU."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2401_06197_amd", "csrc")

WALK = r"""
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include <vector>
#include "dcnv4_strip_rows.h"
struct Plan {
    int H, Ho, sh, ph, dh, R, Q, halo_r, VR, B;
};
static int min(int a, int b) { return a < b ? a : b; }
static int max(int a, int b) { return a > b ? a : b; }
static void fail(const char *what, const Plan &p, int ring, int waves, int bands, int t, int a, int b)
{
    printf("%s: H %d Ho %d stride %d pad %d dilation %d R %d Q %d halo %d ring %d waves %d bands %d round %d: %d %d\n", what, p.H,
           p.Ho, p.sh, p.ph, p.dh, p.R, p.Q, p.halo_r, ring, waves, bands, t, a, b);
    exit(1);
}
// the rows that the workgroup with tiles first, first + step, ... asks for, as the kernel counts them
static void walk(const Plan &p, int ring, int waves, int bands, int first, int step, int S)
{
    const int NB = S * p.B, total = S * p.VR, rounds = (NB + waves - 1) / waves;
    ring = min(ring, total);
    auto oh0 = [&](int s) { return (first + s * step) % bands * p.R; };
    auto first_row = [&](int gb) {
        const int s = gb / p.B;
        return strip_first_row(&p, s, oh0(s), (gb - s * p.B) * 64 / p.Q);
    };
    auto last_row = [&](int gb) {
        const int s = gb / p.B;
        return strip_last_row(&p, s, oh0(s), min((gb - s * p.B) * 64 + 63, p.R * p.Q - 1) / p.Q);
    };
    auto asked = [&](int t, int from, int to) {
        if (from < 0 || to < from || to > total || to - from > ring)    // (so that every row asked for has a slot of its own)
            fail("rows asked for", p, ring, waves, bands, t, from, to);
    };
    int F = strip_asked_first(last_row(min(waves, NB) - 1), ring, total);
    asked(0, 0, F);
    for (int t = 0; t < rounds; ++t) {
        // with slots for all rows, every row that this round's batches can reach has been asked for
        const int reach = last_row(min((t + 1) * waves, NB) - 1) + 1;
        if (F < reach && ring == total)
            fail("rows missing", p, ring, waves, bands, t, F, reach);
        for (int gb = t * waves; gb < min((t + 1) * waves, NB); ++gb) {
            const int s = gb / p.B;
            if (first_row(gb) < s * p.VR || last_row(gb) < s * p.VR - 1 || last_row(gb) >= (s + 1) * p.VR || strip_rows(&p, oh0(s)) > p.VR)
                fail("rows of another tile", p, ring, waves, bands, t, first_row(gb), last_row(gb));
        }
        if (t + 1 == rounds)
            break;
        const int next = strip_asked(strip_wanted(last_row(min((t + 2) * waves, NB) - 1), first_row(t * waves), ring, total), F, ring);
        asked(t, F, next);
        // rows that this round's first batch can reach stay
        if (next - ring > first_row(t * waves))
            fail("row replaced in use", p, ring, waves, bands, t, next, first_row(t * waves));
        F = next;
    }
}
int main()
{
    for (int H : {1, 7, 20, 35, 67})
        for (int ph : {0, 1, 2, 6, 9, 14, 29, 39, 60, 150})
            for (int sh : {1, 2, 3})
                for (int dh : {1, 2, 9})
                    for (int halo : {1, 4, 12}) {
                        const int span = H + 2 * ph - 2 * dh - 1;
                        if (span < 0)
                            continue;
                        Plan p = {H, span / sh + 1, sh, ph, dh, 0, 0, halo, 0, 0};
                        for (int bands : {1, 2, 5}) {
                            p.R = (p.Ho + bands - 1) / bands;
                            const int nb = (p.Ho + p.R - 1) / p.R;
                            for (int Q : {3, 28, 51, 130}) {
                                p.Q = Q;
                                p.B = (p.R * Q + 63) / 64;
                                p.VR = min((p.R - 1) * sh + 2 * dh + 2 * halo + 2, H + 4);
                                for (int ring : {4, 11, 37, 150, 1 << 20})
                                    for (int waves : {8, 12})
                                        for (int step : {1, 2, 32})
                                            walk(p, ring, waves, nb, step == 1 ? nb - 1 : 0, step, 5);
                            }
                        }
                    }
    return 0;
}
"""


def test_rows_asked_for_lie_in_the_tiles_and_have_slots_of_their_own(tmp_path):
    (tmp_path / "walk.cpp").write_text(WALK)
    exe = str(tmp_path / "walk")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, "-o", exe, str(tmp_path / "walk.cpp")], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert res.returncode == 0, res.stdout
