"""Where the linear kernel's loads lie, walked over on the CPU: the header is compiled by itself, with no GPU."""
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
int main()
{
    const int nouts[] = {32, 64, 96, 128, 160, 320, 512};
    for (int kbytes = 32; kbytes <= 4096; kbytes += kbytes < 640 ? 32 : 416)
        for (int nout : nouts) {
            const int nblocks = (nout + 127) / 128, nchunks = (kbytes + 255) / 256;
            for (int pass = 0; pass < 2 * nblocks + 2; ++pass)          // (the step after the last one included)
                for (int ch = 0; ch < nchunks; ++ch)
                    for (int i = 0; i < 8; ++i) {
                        int s = 0;
                        for (int tid = 0; tid < 256; ++tid) {
                            const LinWeightAt w = lin_weight_at(tid, i, pass * 128, ch * 256, nout, kbytes, kOutside);
                            LinAt at = w.at;
                            if (w.bytes != 0 && w.bytes != (unsigned)nout * kbytes) return printf("descriptor\n"), 1;
                            if (w.bytes == 0) {                         // all outside, then, with no scalar offset
                                if (at.s != 0) return printf("scalar offset with an empty descriptor\n"), 1;
                                at.v = kOutside;
                            }
                            check(at, (long long)nout * kbytes, "weights", kbytes, nout, pass, i);
                            if (tid == 0) s = at.s;
                            if (at.s != s) return printf("scalar offset differs between threads\n"), 1;
                            const int row = pass * 128 + 16 * i + tid / 16, col = ch * 256 + tid % 16 * 16;
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
    return 0;
}
"""


def test_every_load_is_inside_its_tensor_or_outside_by_its_vector_offset(tmp_path):
    (tmp_path / "walk.cpp").write_text(WALK)
    exe = str(tmp_path / "walk")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", exe, str(tmp_path / "walk.cpp")], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert res.returncode == 0, res.stdout
