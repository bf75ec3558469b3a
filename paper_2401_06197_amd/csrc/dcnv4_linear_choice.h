// Tile choice of the linear layers (a plain function, so that it can be held against measured times on the CPU).
#pragma once
#include <math.h>

// Tiles of the linear layers: channels x pixels.
constexpr int kLinChunk = 256;         // bytes of K that the kernel of one chunk takes at most (16 units of 16 bytes)
enum { kLinear128x128 = 1, kLinear64x64 = 2, kLinear256x256 = 3, kLinear128x256 = 4, kLinearInOneChunk = 5 };

// The tile that an option asks for; in place of one that the type, or K, does not have: 128x128.
inline int linear_tile_asked(int shape, int kbytes, bool f16)
{
    const bool there = f16 ? shape != kLinear128x256 && (shape != kLinearInOneChunk || kbytes <= kLinChunk) : shape != kLinearInOneChunk;
    return there ? shape : kLinear128x128;
}

// The tile with the lowest estimated time (us).  A compute unit works through its share of the tiles one after the other or,
// `slots` of them, side by side, where half the difference between the fullest unit and the mean is felt, and a part (`gen`) of
// the idle slots of the last round.  A tile takes `step` for 128 (fp16) or 64 (fp32) bytes of K, a lone one `alone` at least, and
// `fixed` for its first loads and its results; the layer takes `memory` of the time its tensors need at 5.5 TB/s, and `once`.
//
// fp32: fitted to 770 layers (49 to 400000 pixels, K 32 to 1024, 32 to 1440 channels): estimates within 3 to 6 % (rms); the choice
// costs 0.3 % on average and more than 5 % in 14 of them (without `memory`, `gen` and `once`: 2 to 4 % in large layers with K in a few
// steps, where the tensors' time is not hidden: 200704 pixels, 128 -> 256: 131 us in 128x256 tiles, 110 in 128x128; 400413, 96 -> 128:
// 128 and 95).  12544 pixels, 512 -> 1024: 92 (128x128), 101 (64x64), 75 (256x256), 86 (128x256); 512 -> 512: 48, 56, 64, 44.5.
// fp16: ten to twenty layers, and of 400 others the choice costs more than 5 % in 4: 12544 pixels, 512 -> 1024: 24, 34, 21.8;
// 512 -> 512: 13.5, 19.2, 18.5; 1000 pixels, 1024 -> 1024: 13.9, 7.9, 27.
inline int linear_tile_choice(int P, int kbytes, const int *nout, int nseg, bool f16, int cus)
{
    struct Tile {
        int shape, run, waves_out, pixels, slots;
        float step, fixed, alone, memory, once, gen;
    };
    static const Tile f16_tiles[] = {{kLinear128x128, 64, 2, 128, 2, .55f, 1.9f, .55f, 0.f, 0.f, 0.f},
                                     {kLinear64x64, 32, 2, 64, 2, .17f, 1.2f, .25f, 0.f, 0.f, 0.f},
                                     {kLinear256x256, 64, 4, 256, 1, 1.15f, 8.6f, 1.15f, 0.f, 0.f, 0.f}};
    static const Tile f32_tiles[] = {{kLinear128x128, 64, 2, 128, 2, .63f, 1.06f, .71f, .39f, 4.f, .3f},
                                     {kLinear64x64, 32, 2, 64, 5, .23f, .31f, .34f, .32f, 2.8f, .08f},
                                     {kLinear256x256, 64, 4, 256, 1, 1.73f, 4.7f, 1.73f, .68f, 1.9f, 0.f},
                                     {kLinear128x256, 64, 2, 256, 1, .99f, 3.9f, .99f, .58f, 1.2f, 0.f}};
    const Tile *tiles = f16 ? f16_tiles : f32_tiles;
    const int count = f16 ? 3 : 4;
    const float steps = (float)((kbytes + (f16 ? 127 : 63)) / (f16 ? 128 : 64));
    float row_bytes = (float)kbytes;
    for (int k = 0; k < nseg; ++k)
        row_bytes += (float)nout[k] * (f16 ? 2.f : 4.f);
    const float tensors = (float)P * row_bytes / 5.5e6f;
    int best = 0;
    float best_us = 0.f, small = 0.f;
    for (int i = 0; i < count; ++i) {
        const Tile &t = tiles[i];
        int runs = 0;
        for (int k = 0; k < nseg; ++k)
            runs += (nout[k] + t.run - 1) / t.run;
        const float n = (float)((runs + t.waves_out - 1) / t.waves_out) * (float)((P + t.pixels - 1) / t.pixels) / (float)cus;
        const float full = ceilf(n), rounds = n > (float)t.slots ? (float)t.slots * ceilf(n / (float)t.slots) : full;
        const float even = t.slots > 1 && n > 1.f ? .5f * (n + full) : full, share = even + t.gen * (rounds - even);
        const float us = steps * (t.step * share > t.alone ? t.step * share : t.alone) + t.fixed * share + t.memory * tensors + t.once;
        if (t.shape == kLinear64x64)
            small = n;
        if (best == 0 || us < best_us) {
            best = t.shape;
            best_us = us;
        }
    }
    // K in one chunk, fp16: 64x64 tiles up to two a compute unit (3136 pixels, 128 -> 256: 3.8 us, 5.1 in one chunk; 12544 pixels:
    // 7.6 and 6.8)
    if (f16 && kbytes <= kLinChunk)
        return small <= 2.f ? kLinear64x64 : kLinearInOneChunk;
    return best;
}
