"""The linear layers' tile choice against measured times, on the CPU: the header is compiled by itself, with no GPU."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2401_06197_amd", "csrc")

# fp32 layers: pixels, K, output channels; us by tile (128x128, 64x64, 256x256, 128x256) and by the kernel before the tiles
# (medians over three to five turns of graph replays, all of a layer's variants in turn)
MEASURED = [(200704, 128, 256, (109.5, 130.2, 118.4, 131.8), 106.2), (400413, 96, 128, (95.3, 119.5, 161.3, 128.3), 101.5),
            (339006, 128, 160, (161.6, 160.3, 162.2, 180.4), 151.6), (400000, 128, 96, (108.0, 126.0, 178.3, 132.8), 109.9),
            (221965, 128, 128, (60.3, 69.5, 100.6, 71.0), 61.9), (88622, 64, 352, (45.0, 51.1, 55.8, 54.0), 46.5),
            (158242, 32, 160, (35.2, 31.2, 38.6, 39.0), 32.8), (12544, 512, 1024, (90.2, 97.5, 76.6, 83.4), 96.9),
            (12544, 512, 512, (48.1, 54.9, 63.8, 43.2), 50.6), (200704, 64, 192, (61.7, 56.9, 77.3, 73.6), 58.6),
            (6272, 512, 512, (30.8, 32.7, 63.1, 38.6), 36.5), (1000, 320, 320, (19.3, 10.1, 41.0, 24.2), 23.2),
            (67200, 320, 320, (110.1, 104.9, 145.4, 118.2), 107.6)]

PICK = r"""
#include <cstdio>
#include "dcnv4_linear_choice.h"
int main()
{
    int f16, P, kbytes, nseg, nout[2];
    while (scanf("%d %d %d %d %d %d", &f16, &P, &kbytes, &nseg, nout, nout + 1) == 6)      // (no output channels: P is the tile asked for)
        printf("%d\n", nout[0] ? linear_tile_choice(P, kbytes, nout, nseg, f16 != 0, 256) : linear_tile_asked(P, kbytes, f16 != 0));
    return 0;
}
"""


def picks(tmp_path, calls):
    (tmp_path / "pick.cpp").write_text(PICK)
    exe = str(tmp_path / "pick")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", exe, str(tmp_path / "pick.cpp")], check=True)
    text = "".join(f"{int(f16)} {P} {kbytes} {len(nout)} {nout[0]} {nout[1] if len(nout) > 1 else 0}\n" for f16, P, kbytes, nout in calls)
    return [int(v) for v in subprocess.run([exe], input=text, capture_output=True, text=True, timeout=60, check=True).stdout.split()]


def test_fp32_layers_take_a_tile_near_the_best_one_and_near_the_former_kernel(tmp_path):
    for (P, K, O, times, former), tile in zip(MEASURED, picks(tmp_path, [(False, P, 4 * K, [O]) for P, K, O, _, _ in MEASURED])):
        us = times[tile - 1]
        assert us <= 1.06 * min(times), (P, K, O, tile, us, times)
        assert us <= 1.07 * former, (P, K, O, tile, us, former)


def test_fp16_layers_and_pairs_of_layers(tmp_path):
    """K in one chunk: 64x64 tiles for few pixels, else the kernel that reads x once; longer K by the estimates; two layers' channels count together."""
    assert picks(tmp_path, [(True, 200704, 256, [128]), (True, 196, 256, [64]), (True, 1000, 2048, [1024]), (True, 12544, 1024, [1024]),
                            (True, 12544, 1024, [512, 512]), (False, 12544, 2048, [1024]), (False, 12544, 2048, [512, 512])]) == [5, 2, 2, 3, 3, 3, 3]


def test_tiles_asked_for_that_a_type_or_k_does_not_have_are_128x128(tmp_path):
    asked = [(f16, tile, kbytes, [0]) for f16, kbytes in ((False, 256), (True, 256), (True, 272)) for tile in (1, 2, 3, 4, 5)]
    assert picks(tmp_path, asked) == [1, 2, 3, 4, 1, 1, 2, 3, 1, 5, 1, 2, 3, 1, 1]
