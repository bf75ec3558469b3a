"""Where the linear kernels' loads and stores lie, walked over on the CPU: the header is compiled by itself, with no GPU."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2401_06197_amd", "csrc")

WALK = r"""
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include "dcnv4_linear_at.h"
constexpr int kOutside = (int)0x80000000u;
static void check(const LinAt &at, long long bytes, const char *what, int a, int b, int c, int d)
{
    // outside by the vector offset alone, or all 16 bytes inside
    const bool ok = at.v == kOutside ? at.s >= 0 && at.s < bytes : at.v >= 0 && at.s >= 0 && (long long)at.v + at.s + 16 <= bytes;
    if (!ok) {
        printf("%s %d %d %d %d: v %d s %d of %lld\n", what, a, b, c, d, at.v, at.s, bytes);
        exit(1);
    }
}
// The tiles: every unit of every step, steps and rows past the end included, of rows and of planes; and every unit of the results.
static int tiles()
{
    for (int step : {64, 128})
        for (int kbytes = 32; kbytes <= 1056; kbytes += kbytes < 320 ? 32 : 96)
            for (int shift : {0, 5, 6, 7})
                for (int hw : {1, 5, 33}) {
                    if (shift && kbytes % (1 << shift)) continue;
                    const int images = 3, P = images * hw;
                    const long long bytes = (long long)P * kbytes;
                    auto place = [&](int px, int col) {                 // by definition
                        const int img = px / hw, at = px % hw;
                        return shift == 0 ? px * kbytes + col
                                          : img * hw * kbytes + ((col >> shift) * hw + at) * (1 << shift) + col % (1 << shift);
                    };
                    for (int row = 0; row < P + 70; row += row + 2 < P ? 1 : 13)
                        for (int unit = 0; unit < step / 16; ++unit)
                            for (int t = 0; t < kbytes / step + 5; ++t) {
                                const int px = lin_row(row, P), col = t * step + unit * 16;
                                const int first = shift == 0 ? lin_pixel_at(px, kbytes, unit * 16)
                                                             : lin_pixel_in_planes_at(px, px / hw, hw, kbytes, unit * 16, shift);
                                const unsigned at = ((unsigned)first + lin_step_at(t, step, shift, hw << shift)) | lin_past(t, step, unit, kbytes, kOutside);
                                if (px != (row < P ? row : P - 1)) return printf("row %d of %d: %d\n", row, P, px), 1;
                                if (col >= kbytes ? at < 0x80000000u : (long long)at + 16 > bytes || (int)at != place(px, col))
                                    return printf("tile: step %d K %d shift %d hw %d row %d unit %d t %d: %u\n", step, kbytes, shift, hw, row, unit, t, at), 1;
                            }
                    for (int px = 0; px < P; ++px)
                        for (int col = 0; col < kbytes; col += 16) {
                            const int at = shift == 0 ? lin_pixel_at(px, kbytes, col) : lin_pixel_in_planes_at(px, px / hw, hw, kbytes, col, shift);
                            if (at != place(px, col) || at < 0 || at + 16 > bytes) return printf("result\n"), 1;
                        }
                }
    return 0;
}
int main()
{
    const int nouts[] = {32, 64, 96, 128, 160, 320, 512};
    for (int kbytes = 32; kbytes <= 256; kbytes += 32)
        for (int nout : nouts) {
            const int nblocks = (nout + 127) / 128;
            for (int pass = 0; pass < 2 * nblocks + 2; ++pass)          // (the pass after the last one included)
                for (int i = 0; i < 8; ++i) {
                    int s = 0;
                    for (int tid = 0; tid < 256; ++tid) {
                        const LinWeightAt w = lin_weight_at(tid, i, pass * 128, nout, kbytes, kOutside);
                        LinAt at = w.at;
                        if (w.bytes != 0 && w.bytes != (unsigned)nout * kbytes) return printf("descriptor\n"), 1;
                        if (w.bytes == 0) {                             // all outside, then, with no scalar offset
                            if (at.s != 0) return printf("scalar offset with an empty descriptor\n"), 1;
                            at.v = kOutside;
                        }
                        check(at, (long long)nout * kbytes, "weights", kbytes, nout, pass, i);
                        if (tid == 0) s = at.s;
                        if (at.s != s) return printf("scalar offset differs between threads\n"), 1;
                        const int row = pass * 128 + 16 * i + tid / 16, col = tid % 16 * 16;
                        const bool in = row < nout && col < kbytes;
                        if (in != (at.v != kOutside) || (in && at.v + at.s != row * kbytes + col))
                            return printf("wrong place\n"), 1;
                    }
                }
        }
    for (int P = 1; P <= 37; P += 12)                                   // one image of P pixels
        for (int kbytes = 32; kbytes <= 1024; kbytes += 32)
            for (int shift : {0, 5, 6, 7}) {
                if (shift && kbytes % (1 << shift)) continue;
                for (int px = 0; px <= P; ++px)
                    for (int half = 0; half < 2; ++half)
                        for (int col = 0; col < kbytes + 512; col += 32) {
                            const int xo = px == P ? kOutside : (shift ? px << shift : px * kbytes) + half * 16;
                            const LinAt at = lin_x_at(xo, col, kbytes, shift, P << shift, kOutside);
                            check(at, (long long)P * kbytes, "x", P, kbytes, shift, col);
                            const int c = col + half * 16;
                            const int want = !shift ? px * kbytes + c : (c >> shift) * (P << shift) + (px << shift) + (c & ((1 << shift) - 1));
                            if (col < kbytes && px < P && at.v + at.s != want) return printf("wrong place in x\n"), 1;
                            if ((col >= kbytes || px == P) != (at.v == kOutside)) return printf("x past the end\n"), 1;
                        }
            }
    return tiles();
}
"""


def test_every_load_is_inside_its_tensor_or_outside_by_its_vector_offset(tmp_path):
    (tmp_path / "walk.cpp").write_text(WALK)
    exe = str(tmp_path / "walk")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", exe, str(tmp_path / "walk.cpp")], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert res.returncode == 0, res.stdout
