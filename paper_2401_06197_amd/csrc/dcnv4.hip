// DCNv4 spatial aggregation for MI355X (gfx950): kernels and the C ABI of include/dcnv4.h.
//
// Operator: paper Sec. 3.1, Eq. 1-2 without the softmax.  Work organisation follows the
// idea of Sec. 3.2 (one thread serves a run of channels of one group at one output pixel,
// so one offset/mask read and one set of bilinear coefficients is shared, and the channel
// run is moved with 128-bit memory instructions); everything below that idea is laid out
// for CDNA4: wave64, raw buffer loads whose hardware range check supplies the zero for
// rows outside the image, offset/mask tiles staged through LDS with 128-bit coalesced
// loads, tiles handed to XCDs in contiguous bands so that neighbouring outputs share an L2.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <type_traits>

#include "dcnv4.h"

namespace {

constexpr int kThreads = 256;
constexpr int kTaps = 9;
constexpr int kXcds = 8;
// Word 3 of a gfx9-family raw buffer descriptor: 32-bit data format, no swizzle, no stride.
constexpr int kRsrcWord3 = 0x00020000;
// A byte offset no descriptor of ours reaches (images are validated below 2^31 bytes):
// loads through it return zero, atomics through it are dropped.
constexpr int kOutside = (int)0x80000000u;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef __amdgpu_buffer_rsrc_t rsrc_t;

// n / d for 0 <= n < 2^31 as mulhi + add + shift (d >= 1), constants made on the host.
struct FastDiv {
    unsigned mul, shift;
};

__device__ __forceinline__ int fdiv(int n, FastDiv f)
{
    return (int)((__umulhi((unsigned)n, f.mul) + (unsigned)n) >> f.shift);
}

typedef const __attribute__((address_space(4))) FastDiv ArgDiv;        // in the kernel's arguments
__device__ __forceinline__ int arg_div(int n, ArgDiv &f)
{
    return fdiv(n, FastDiv{f.mul, f.shift});
}
__device__ __forceinline__ int arg_div(int n, const FastDiv &f) { return fdiv(n, f); }

struct Geo {
    int H, W, Ho, Wo, G;
    int sh, sw, ph, pw, dh, dw;
    float scale;        // offset_scale
    float dmax;         // scaled offsets are clamped to [-dmax, dmax]; beyond that every corner is outside
    int pgi;            // (pixel, group) pairs per image = Ho*Wo*G
    int tiles_per_image, ntiles, tiles_per_xcd, remap;
    FastDiv div_g, div_wo, div_tpi;
    int x_img_bytes;    // H*W*C*sizeof(T)
    int y_img_bytes;    // Ho*Wo*C*sizeof(T)
    int row_bytes;      // W*C*sizeof(T)
    int pix_bytes;      // C*sizeof(T)
};

__device__ __forceinline__ rsrc_t make_rsrc(const void *base, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, kRsrcWord3);
}

// blockIdx -> tile.  Hardware deals consecutive workgroups to the 8 XCDs in turn; with the
// remap XCD i works through tiles [i*tiles_per_xcd, (i+1)*tiles_per_xcd) in order, so the
// tiles in flight on one XCD are spatial neighbours and their input pixels hit that XCD's L2.
__device__ __forceinline__ int tile_of_block(const Geo &p)
{
    const int b = blockIdx.x;
    return p.remap ? (b & (kXcds - 1)) * p.tiles_per_xcd + (b >> 3) : b;
}

// Copy `bytes` of a tensor region starting at byte `start` (of `base`, 16-byte aligned) into
// LDS, beginning at the 16-byte boundary below `start`; returns how many bytes of lead-in
// precede the region in LDS.  All global reads are aligned 128-bit loads whose dwords are
// range-checked one by one against a descriptor that ends exactly at the region's end, so
// nothing past the tensor is touched.  A region of 2-byte elements can end in the middle of a
// dword; the hardware zeroes that whole dword, so the thread that holds it fetches the last
// element again with a 16-bit load.
template <int CAP_BYTES, int ELEM_BYTES>
__device__ __forceinline__ int stage_region(char *lds, const char *base, long long start, int bytes)
{
    const long long aligned = start & ~15LL;
    const int delta = (int)(start - aligned);
    const int total = delta + bytes;                       // < CAP_BYTES by construction
    const rsrc_t r = make_rsrc(base + aligned, (unsigned)total);
#pragma unroll
    for (int o = 0; o < CAP_BYTES; o += kThreads * 16) {
        const int off = o + (int)threadIdx.x * 16;
        if (off < total) {
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
            *reinterpret_cast<u32x4 *>(lds + off) = v;
            if (ELEM_BYTES == 2 && (total & 2) && off + 16 >= total) {
                const unsigned short tail = __builtin_amdgcn_raw_buffer_load_b16(r, total - 2, 0, 0);
                *reinterpret_cast<unsigned short *>(lds + total - 2) = tail;
            }
        }
    }
    return delta;
}

template <typename T, int CPT> struct Vec;          // CPT channels of one pixel in registers
template <int CPT> struct Vec<_Float16, CPT> {
    static constexpr int kRegs = CPT / 8;
    f16x8 v[kRegs];
    __device__ __forceinline__ void load(rsrc_t r, int off)
    {
#pragma unroll
        for (int i = 0; i < kRegs; ++i)
            v[i] = __builtin_bit_cast(f16x8, __builtin_amdgcn_raw_buffer_load_b128(r, off + 16 * i, 0, 0));
    }
    __device__ __forceinline__ float get(int c) const { return (float)v[c / 8][c % 8]; }
};
template <int CPT> struct Vec<float, CPT> {
    static constexpr int kRegs = CPT / 4;
    f32x4 v[kRegs];
    __device__ __forceinline__ void load(rsrc_t r, int off)
    {
#pragma unroll
        for (int i = 0; i < kRegs; ++i)
            v[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off + 16 * i, 0, 0));
    }
    __device__ __forceinline__ float get(int c) const { return v[c / 4][c % 4]; }
};
template <> struct Vec<float, 2> {              // narrow runs: the backward's lane-per-channel layouts
    float v[2];
    __device__ __forceinline__ void load(rsrc_t r, int off)
    {
        // two dword loads (the 64-bit raw buffer load builtin of this compiler fetches one dword only)
        v[0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
        v[1] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off + 4, 0, 0));
    }
    __device__ __forceinline__ float get(int c) const { return v[c]; }
};
template <> struct Vec<float, 1> {
    float v;
    __device__ __forceinline__ void load(rsrc_t r, int off)
    {
        v = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
    }
    __device__ __forceinline__ float get(int) const { return v; }
};

template <int CPT>
__device__ __forceinline__ void store_run(rsrc_t r, int off, const float (&a)[CPT], _Float16 *)
{
#pragma unroll
    for (int i = 0; i < CPT / 8; ++i) {
        f16x8 h;
#pragma unroll
        for (int c = 0; c < 8; ++c)
            h[c] = (_Float16)a[8 * i + c];                 // round to nearest even, once
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, h), r, off + 16 * i, 0, 0);
    }
}
template <int CPT>
__device__ __forceinline__ void store_run(rsrc_t r, int off, const float (&a)[CPT], float *)
{
#pragma unroll
    for (int i = 0; i < CPT / 4; ++i) {
        f32x4 f = {a[4 * i], a[4 * i + 1], a[4 * i + 2], a[4 * i + 3]};
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, f), r, off + 16 * i, 0, 0);
    }
}

// One tap's sampling geometry: fractional parts, the byte offsets of the 4 neighbours inside
// the image's descriptor (kOutside where the column is outside; rows outside fall out of the
// descriptor's range by themselves) -- Eq. 1's x_g(p0 + p_k + dp_gk).
struct Tap {
    float lh, lw;
    int o00, o01, o10, o11;
};

// Byte offsets of the 4 neighbours of a sampling position given as whole-pixel window origin
// (base_h, base_w) plus the already scaled displacement (dy, dx).
__device__ __forceinline__ Tap tap_offsets(float dy, float dx, int base_h, int base_w, int chan_bytes, float dmax,
                                           int W, int row_bytes, int pix_bytes)
{
    // The whole-pixel part of the sampling position is kept in integers and only the scaled
    // offset goes through fp32, so the fractional parts carry no error from the magnitude of
    // the pixel coordinate.  Beyond +-dmax every neighbour is outside, so clamping changes nothing.
    dy = __builtin_fminf(__builtin_fmaxf(dy, -dmax), dmax);
    dx = __builtin_fminf(__builtin_fmaxf(dx, -dmax), dmax);
    const float fy = __builtin_floorf(dy), fx = __builtin_floorf(dx);
    Tap t;
    t.lh = dy - fy;
    t.lw = dx - fx;
    const int h0 = base_h + (int)fy, w0 = base_w + (int)fx;
    const int o = h0 * row_bytes + w0 * pix_bytes + chan_bytes;
    const bool in0 = (unsigned)w0 < (unsigned)W, in1 = (unsigned)(w0 + 1) < (unsigned)W;
    t.o00 = in0 ? o : kOutside;
    t.o10 = in0 ? o + row_bytes : kOutside;
    t.o01 = in1 ? o + pix_bytes : kOutside;
    t.o11 = in1 ? o + row_bytes + pix_bytes : kOutside;
    return t;
}

__device__ __forceinline__ Tap tap_geometry(float dY, float dX, int base_h, int base_w, int chan_bytes,
                                            const Geo &p)
{
    return tap_offsets(p.scale * dY, p.scale * dX, base_h, base_w, chan_bytes, p.dmax, p.W, p.row_bytes,
                       p.pix_bytes);
}

__device__ __forceinline__ int cvt_floor_i32(float v)
{
    int r;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(v));       // floor, saturating, NaN -> 0
    return r;
}

__device__ __forceinline__ int cvt_round_i32(float v)      // floor(v + 0.5), saturating
{
    int r;
    asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}

__device__ __forceinline__ int med3i(int v, int lo, int hi)     // clamp to [lo, hi] in one instruction
{
    int r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(v), "v"(lo), "v"(hi));
    return r;
}

// channel c of a 16-byte unit, widened to fp32
template <typename T> __device__ __forceinline__ float unit_get(const u32x4 &v, int c);
template <> __device__ __forceinline__ float unit_get<_Float16>(const u32x4 &v, int c)
{
    return (float)__builtin_bit_cast(f16x8, v)[c];
}
template <> __device__ __forceinline__ float unit_get<float>(const u32x4 &v, int c)
{
    return __builtin_bit_cast(f32x4, v)[c];
}

// store one 16-byte unit of results (8 fp16 or 4 fp32 values, one rounding to nearest even)
template <typename T> __device__ __forceinline__ void store_unit(rsrc_t r, int off, const float *a);
template <> __device__ __forceinline__ void store_unit<_Float16>(rsrc_t r, int off, const float *a)
{
    f16x8 h;
#pragma unroll
    for (int c = 0; c < 8; ++c)
        h[c] = (_Float16)a[c];
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, h), r, off, 0, 0);
}
template <> __device__ __forceinline__ void store_unit<float>(rsrc_t r, int off, const float *a)
{
    f32x4 f = {a[0], a[1], a[2], a[3]};
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, f), r, off, 0, 0);
}

// Shared per-thread decode: which (pixel, group, channel run) this thread serves.
struct Item {
    int n, pg0, npg;          // image, first (pixel,group) of the tile, pairs in the tile
    int pgl, sub;             // pair inside the tile, channel run inside the group
    int pix, g, oh, ow;
    bool active;
};

template <int TPG>
__device__ __forceinline__ Item decode_item(const Geo &p, int tile)
{
    constexpr int PGB = kThreads / TPG;
    Item it;
    it.n = fdiv(tile, p.div_tpi);
    it.pg0 = (tile - it.n * p.tiles_per_image) * PGB;
    it.npg = min(PGB, p.pgi - it.pg0);
    it.pgl = (int)threadIdx.x / TPG;
    it.sub = (int)threadIdx.x % TPG;
    it.active = it.pgl < it.npg;
    const int pg = it.pg0 + min(it.pgl, it.npg - 1);
    it.pix = fdiv(pg, p.div_g);
    it.g = pg - it.pix * p.G;
    it.oh = fdiv(it.pix, p.div_wo);
    it.ow = it.pix - it.oh * p.Wo;
    return it;
}

}  // namespace

// ------------------------------------------------------------------------------------------
// Forward (Eq. 1-2): thread = (output pixel, group, run of CPT channels).
// ------------------------------------------------------------------------------------------
template <typename T, int CG, int CPT, int KH = 3, int KW = 3>
__global__ __launch_bounds__(kThreads) void dcnv4_fwd_kernel(const T *__restrict__ x, const T *__restrict__ offset,
                                                             const T *__restrict__ mask, T *__restrict__ y, Geo p)
{
    constexpr int TPG = CG / CPT;
    constexpr int KT = KH * KW;                 // sampling points of the window
    constexpr int PGB = kThreads / TPG;
    constexpr int OFF_CAP = PGB * 2 * KT * (int)sizeof(T) + 16;
    constexpr int MSK_CAP = PGB * KT * (int)sizeof(T) + 16;
    __shared__ __attribute__((aligned(16))) char s_off[OFF_CAP];
    __shared__ __attribute__((aligned(16))) char s_msk[MSK_CAP];

    const int tile = tile_of_block(p);
    if (tile >= p.ntiles)
        return;
    const Item it = decode_item<TPG>(p, tile);

    const long long pg_first = (long long)it.n * p.pgi + it.pg0;
    const int d_off = stage_region<OFF_CAP, (int)sizeof(T)>(s_off, (const char *)offset, pg_first * (2 * KT * (int)sizeof(T)),
                                            it.npg * 2 * KT * (int)sizeof(T));
    const int d_msk = stage_region<MSK_CAP, (int)sizeof(T)>(s_msk, (const char *)mask, pg_first * (KT * (int)sizeof(T)),
                                            it.npg * KT * (int)sizeof(T));
    __syncthreads();
    if (!it.active)
        return;

    const T *my_off = reinterpret_cast<const T *>(s_off + d_off) + it.pgl * 2 * KT;
    const T *my_msk = reinterpret_cast<const T *>(s_msk + d_msk) + it.pgl * KT;
    const rsrc_t rx = make_rsrc((const char *)x + (long long)it.n * p.x_img_bytes, (unsigned)p.x_img_bytes);
    const int chan_bytes = (it.g * CG + it.sub * CPT) * (int)sizeof(T);
    const int bh = it.oh * p.sh - p.ph, bw = it.ow * p.sw - p.pw;

    float acc[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c)
        acc[c] = 0.f;

#pragma unroll
    for (int j = 0; j < KW; ++j) {
#pragma unroll
        for (int i = 0; i < KH; ++i) {
            const int k = j * KH + i;
            const float off_y = (float)my_off[2 * k + 1], off_x = (float)my_off[2 * k];
            Tap t = tap_geometry(off_y, off_x, bh + i * p.dh, bw + j * p.dw, chan_bytes, p);
            // fp16 groups of 64, which come here and go through rectangles: an infinite offset has no fractional part there either
            // (NaN, not a clamped one's; the host keeps finite products finite)
            if constexpr (sizeof(T) == 2 && CG == 64 && KH == 3) {
                t.lh = __builtin_amdgcn_fractf(p.scale * off_y);
                t.lw = __builtin_amdgcn_fractf(p.scale * off_x);
            }
            Vec<T, CPT> v00, v01, v10, v11;
            v00.load(rx, t.o00);
            v01.load(rx, t.o01);
            v10.load(rx, t.o10);
            v11.load(rx, t.o11);
            const float m = (float)my_msk[k];
            const float mh0 = m * (1.f - t.lh), mh1 = m * t.lh;
            const float w00 = mh0 * (1.f - t.lw), w01 = mh0 * t.lw, w10 = mh1 * (1.f - t.lw), w11 = mh1 * t.lw;
#pragma unroll
            for (int c = 0; c < CPT; ++c) {
                float a = acc[c];
                a = __builtin_fmaf(v00.get(c), w00, a);
                a = __builtin_fmaf(v01.get(c), w01, a);
                a = __builtin_fmaf(v10.get(c), w10, a);
                a = __builtin_fmaf(v11.get(c), w11, a);
                acc[c] = a;
            }
        }
    }

    const rsrc_t ry = make_rsrc((char *)y + (long long)it.n * p.y_img_bytes, (unsigned)p.y_img_bytes);
    store_run<CPT>(ry, it.pix * p.pix_bytes + chan_bytes, acc, (T *)nullptr);
}

#include "dcnv4_tile_choice.h"
#include "dcnv4_tiled.inc"
#include "dcnv4_gradx.inc"
#include "dcnv4_ring.inc"
#include "dcnv4_strip.inc"
#include "dcnv4_linear_choice.h"
#include "dcnv4_linear.inc"
#include "dcnv4_linear_tile.inc"

// ------------------------------------------------------------------------------------------
// Backward (chain rule on Eq. 1), fp32, in one pass with grad_x added straight to memory; used
// where the LDS-staged kernels do not apply (groups wider than 16 channels, tiny images).  A group
// is spread over TPG lanes of CPT channels each -- by default one channel per lane, so that a
// wave's atomic instruction covers a few whole cache lines; the L2 atomic units then sustain about
// eight times the rate they reach when every lane adds to a line of its own.  The lanes' partial
// sums for grad_offset/grad_mask are combined with DPP exchanges inside a 16-lane row (plus one
// swizzle for 32 lanes).
// grad_offset / grad_mask leave through the same LDS tile the inputs came in by.
// ------------------------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v)
{
    const int o = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false);
    return v + __builtin_bit_cast(float, o);
}

template <int TPG>
__device__ __forceinline__ float group_sum(float v)
{
    if (TPG >= 2) v = dpp_add<0xB1>(v);      // quad_perm [1,0,3,2]
    if (TPG >= 4) v = dpp_add<0x4E>(v);      // quad_perm [2,3,0,1]
    if (TPG >= 8) v = dpp_add<0x141>(v);     // row_half_mirror
    if (TPG >= 16) v = dpp_add<0x140>(v);    // row_mirror
    if (TPG >= 32)                           // the other 16-lane row of the 32-lane half: swizzle, lane ^ 16
        v += __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), 0x401F));
    return v;
}

template <int CG, int CPT, int KH = 3, int KW = 3>
__global__ __launch_bounds__(kThreads) void dcnv4_bwd_kernel(const float *__restrict__ x,
                                                             const float *__restrict__ offset,
                                                             const float *__restrict__ mask,
                                                             const float *__restrict__ grad_y,
                                                             float *__restrict__ grad_x,
                                                             float *__restrict__ grad_offset,
                                                             float *__restrict__ grad_mask, Geo p)
{
    typedef float T;
    constexpr int TPG = CG / CPT;
    constexpr int KT = KH * KW;
    constexpr int PGB = kThreads / TPG;
    constexpr int OFF_CAP = PGB * 2 * KT * (int)sizeof(T) + 16;
    constexpr int MSK_CAP = PGB * KT * (int)sizeof(T) + 16;
    __shared__ __attribute__((aligned(16))) char s_off[OFF_CAP];
    __shared__ __attribute__((aligned(16))) char s_msk[MSK_CAP];

    const int tile = tile_of_block(p);
    if (tile >= p.ntiles)
        return;
    const Item it = decode_item<TPG>(p, tile);

    const long long pg_first = (long long)it.n * p.pgi + it.pg0;
    const int d_off = stage_region<OFF_CAP, (int)sizeof(T)>(s_off, (const char *)offset, pg_first * (2 * KT * (int)sizeof(T)),
                                            it.npg * 2 * KT * (int)sizeof(T));
    const int d_msk = stage_region<MSK_CAP, (int)sizeof(T)>(s_msk, (const char *)mask, pg_first * (KT * (int)sizeof(T)),
                                            it.npg * KT * (int)sizeof(T));
    __syncthreads();

    T *tile_off = reinterpret_cast<T *>(s_off + d_off);
    T *tile_msk = reinterpret_cast<T *>(s_msk + d_msk);
    if (it.active) {
        T *my_off = tile_off + it.pgl * 2 * KT;
        T *my_msk = tile_msk + it.pgl * KT;
        const rsrc_t rx = make_rsrc((const char *)x + (long long)it.n * p.x_img_bytes, (unsigned)p.x_img_bytes);
        const rsrc_t rgx = make_rsrc((char *)grad_x + (long long)it.n * p.x_img_bytes, (unsigned)p.x_img_bytes);
        const rsrc_t rgy =
            make_rsrc((const char *)grad_y + (long long)it.n * p.y_img_bytes, (unsigned)p.y_img_bytes);
        const int chan_bytes = (it.g * CG + it.sub * CPT) * (int)sizeof(T);
        const int bh = it.oh * p.sh - p.ph, bw = it.ow * p.sw - p.pw;

        Vec<T, CPT> gy;
        gy.load(rgy, it.pix * p.pix_bytes + chan_bytes);

#pragma unroll
        for (int j = 0; j < KW; ++j) {
#pragma unroll
            for (int i = 0; i < KH; ++i) {
                const int k = j * KH + i;
                const Tap t = tap_geometry(my_off[2 * k + 1], my_off[2 * k], bh + i * p.dh, bw + j * p.dw,
                                           chan_bytes, p);
                Vec<T, CPT> v00, v01, v10, v11;
                v00.load(rx, t.o00);
                v01.load(rx, t.o01);
                v10.load(rx, t.o10);
                v11.load(rx, t.o11);
                const float m = my_msk[k];
                const float hh = 1.f - t.lh, hw = 1.f - t.lw;
                // grad_x: m * corner weight * gy, dropped by the descriptor where the corner is outside
                const float w00 = m * hh * hw, w01 = m * hh * t.lw, w10 = m * t.lh * hw, w11 = m * t.lh * t.lw;
                float d00 = 0.f, d01 = 0.f, d10 = 0.f, d11 = 0.f;
#pragma unroll
                for (int c = 0; c < CPT; ++c) {
                    const float g = gy.get(c);
                    d00 = __builtin_fmaf(g, v00.get(c), d00);
                    d01 = __builtin_fmaf(g, v01.get(c), d01);
                    d10 = __builtin_fmaf(g, v10.get(c), d10);
                    d11 = __builtin_fmaf(g, v11.get(c), d11);
                    __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(w00 * g, rgx, t.o00 + 4 * c, 0, 0);
                    __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(w01 * g, rgx, t.o01 + 4 * c, 0, 0);
                    __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(w10 * g, rgx, t.o10 + 4 * c, 0, 0);
                    __builtin_amdgcn_raw_ptr_buffer_atomic_fadd_f32(w11 * g, rgx, t.o11 + 4 * c, 0, 0);
                }
                d00 = group_sum<TPG>(d00);
                d01 = group_sum<TPG>(d01);
                d10 = group_sum<TPG>(d10);
                d11 = group_sum<TPG>(d11);
                // grad_mask = sum_c gy*S;  grad_offset = scale * m * sum_c gy * dS/d(wx, hy)
                const float gm = hh * (hw * d00 + t.lw * d01) + t.lh * (hw * d10 + t.lw * d11);
                const float gdy = p.scale * m * (hw * (d10 - d00) + t.lw * (d11 - d01));
                const float gdx = p.scale * m * (hh * (d01 - d00) + t.lh * (d11 - d10));
                if (it.sub == 0) {                       // after every lane of the pair has read tap k
                    my_off[2 * k] = gdx;
                    my_off[2 * k + 1] = gdy;
                    my_msk[k] = gm;
                }
            }
        }
    }
    __syncthreads();
    float *go = grad_offset + pg_first * (2 * KT);
    float *gm = grad_mask + pg_first * KT;
    for (int e = threadIdx.x; e < it.npg * 2 * KT; e += kThreads)
        go[e] = tile_off[e];
    for (int e = threadIdx.x; e < it.npg * KT; e += kThreads)
        gm[e] = tile_msk[e];
}

// Zero-fill of `bytes` bytes (a multiple of 4) at a 16-byte aligned address: 128-bit stores, then the
// last few dwords one by one.  A kernel rather than a memset node, so that a call can be captured
// into a graph.
__global__ __launch_bounds__(kThreads) void dcnv4_zero_kernel(u32x4 *__restrict__ dst, long long bytes)
{
    const long long n16 = bytes / 16;
    const u32x4 z = {0u, 0u, 0u, 0u};
    for (long long i = (long long)blockIdx.x * kThreads + threadIdx.x; i < n16; i += (long long)gridDim.x * kThreads)
        dst[i] = z;
    const int tail = (int)((bytes - n16 * 16) / 4);
    if (blockIdx.x == 0 && (int)threadIdx.x < tail)
        reinterpret_cast<unsigned *>(dst + n16)[threadIdx.x] = 0u;
}

// ------------------------------------------------------------------------------------------
// Host side: validation, launch geometry, dispatch.
// ------------------------------------------------------------------------------------------
namespace {

// Test and benchmark switches (dcnv4_set_option): they force a path or a tile shape so that every
// kernel can be checked on every shape; 0 = the library's own choice.  Not meant for applications.
struct Options {
    int fwd_path = 0;      // 1 direct global gather, 2 rectangle staged in LDS, 3 ring of record rows in LDS
    int bwd_path = 0;      // 1 direct (global atomics), 2 LDS-staged (two passes)
    int fwd_cpt = 0;       // channels per lane of the direct forward (8 or 16)
    int bwd_cpt = 0;       // channels per lane of the direct backward (1, 2, 4, 8, 16)
    int xcd_remap = 1;     // consecutive tiles go to one XCD (0: plain block order)
    int halo = 0;          // displacement in pixels (rows, for the ring) the staged window allows for
    int lds_kb = 0;        // LDS budget per workgroup of the staged kernels (8..160)
    int fwd_threads = 0;   // workgroup size of the staged forward kernels (64, 128, 256, 512, 640, 768)
    int wg_per_cu = 0;     // persistent workgroups per compute unit of the rectangle kernels (1..32)
    int fwd_single = 0;    // rectangle buffers of the staged gather kernels: 1 always two, 2 always one
    int gx_threads = 0;    // workgroup size of the grad_x kernel (256, 512, 768)
    int gx_own = 0;        // grad_x kernel, an (image, channel run) to one workgroup: 1 always, 2 never
    int gom_coop = 0;      // 1: the fp32 grad_offset/grad_mask pass goes through LDS slices even for whole groups
    int fwd_strip = 0;     // forward and grad_offset/grad_mask out of a rolling window of rows: 1 wherever it applies, 2 never
    int linear_tile = 0;   // tile of the linear layers (linear_tile_choice)
    int module_rows = 0;   // 1: the module keeps its tensors channel-last between the layers (default: plane-major)
} g_opt;

char g_last_kernel[2][128];

FastDiv make_div(unsigned d)
{
    unsigned s = 0;
    while ((1ull << s) < d)
        ++s;
    FastDiv f;
    f.shift = s;
    f.mul = (unsigned)(((1ull << 32) * ((1ull << s) - d)) / d + 1);
    return f;
}

int esize(int dtype) { return dtype == DCNV4_F16 ? 2 : 4; }

struct Problem {
    int N, H, W, G, Cg, Ho, Wo;
    int kh, kw;     // window: 3x3 everywhere; 1x1 and 5x5 through the direct kernels only
    int sh, sw, ph, pw, dh, dw;
    float scale;
    int dtype;
    int merged;     // offsets and mask values share one buffer of 32 values per (pixel, group)
    int softmax;    // the mask tensor holds logits, normalised over the 9 taps inside the kernels
};

int validate(const Problem &q, int kh, int kw, const void *const *ptrs, int nptrs)
{
    for (int i = 0; i < nptrs; ++i)
        if (!ptrs[i])
            return DCNV4_ERR_NULL;
    if (q.N < 1 || q.H < 1 || q.W < 1 || q.G < 1 || q.Cg < 1 || kh < 1 || kw < 1 || q.sh < 1 || q.sw < 1 ||
        q.ph < 0 || q.pw < 0 || q.dh < 1 || q.dw < 1)
        return DCNV4_ERR_SHAPE;
    if (q.Ho < 1 || q.Wo < 1)
        return DCNV4_ERR_SHAPE;
    if (kh != kw || (kh != 1 && kh != 3 && kh != 5))
        return DCNV4_ERR_UNSUPPORTED;
    if (q.dtype != DCNV4_F32 && q.dtype != DCNV4_F16)
        return DCNV4_ERR_UNSUPPORTED;
    if (q.Cg != 8 && q.Cg != 16 && q.Cg != 32 && q.Cg != 64)
        return DCNV4_ERR_UNSUPPORTED;
    if (!(q.scale == q.scale) || q.scale > 3.0e38f || q.scale < -3.0e38f)
        return DCNV4_ERR_UNSUPPORTED;
    for (int i = 0; i < nptrs; ++i)
        if (reinterpret_cast<uintptr_t>(ptrs[i]) & 15u)
            return DCNV4_ERR_ALIGN;
    return DCNV4_OK;
}

// Fills the kernel's geometry block; returns DCNV4_ERR_UNSUPPORTED when 32-bit byte offsets
// inside one image could overflow.
int make_geo(const Problem &q, int tpg, Geo *out)
{
    Geo p;
    memset(&p, 0, sizeof(p));
    const long long es = esize(q.dtype), C = (long long)q.G * q.Cg;
    p.H = q.H; p.W = q.W; p.Ho = q.Ho; p.Wo = q.Wo; p.G = q.G;
    p.sh = q.sh; p.sw = q.sw; p.ph = q.ph; p.pw = q.pw; p.dh = q.dh; p.dw = q.dw;
    p.scale = q.scale;
    // window origin of any tap lies in [-pad, (out-1)*stride - pad + (k-1)*dil]
    const long long bh = (long long)(q.Ho - 1) * q.sh + (long long)(q.kh - 1) * q.dh + q.ph;
    const long long bw = (long long)(q.Wo - 1) * q.sw + (long long)(q.kw - 1) * q.dw + q.pw;
    const long long reach = (q.H > q.W ? q.H : q.W) + (bh > bw ? bh : bw) + 4;
    if (reach >= (1 << 22))
        return DCNV4_ERR_UNSUPPORTED;
    p.dmax = (float)reach;
    // |row| <= 2*reach+1, |col| <= 2*reach+1 after clamping: the byte offset must fit in int32
    const long long worst = (2 * reach + 2) * ((long long)q.W + 1) * C * es + (2 * reach + 2) * C * es;
    const long long ximg = (long long)q.H * q.W * C * es, yimg = (long long)q.Ho * q.Wo * C * es;
    if (worst >= (1LL << 31) || ximg >= (1LL << 31) || yimg >= (1LL << 31))
        return DCNV4_ERR_UNSUPPORTED;
    const long long pgi = (long long)q.Ho * q.Wo * q.G;
    const int pgb = kThreads / tpg;
    const long long tpi = (pgi + pgb - 1) / pgb;
    const long long ntiles = tpi * q.N;
    if (pgi >= (1LL << 31) || ntiles >= (1LL << 30))
        return DCNV4_ERR_UNSUPPORTED;
    p.pgi = (int)pgi;
    p.tiles_per_image = (int)tpi;
    p.ntiles = (int)ntiles;
    p.tiles_per_xcd = (int)((ntiles + kXcds - 1) / kXcds);
    p.remap = g_opt.xcd_remap;
    p.div_g = make_div((unsigned)q.G);
    p.div_wo = make_div((unsigned)q.Wo);
    p.div_tpi = make_div((unsigned)tpi);
    p.x_img_bytes = (int)ximg;
    p.y_img_bytes = (int)yimg;
    p.row_bytes = (int)(q.W * C * es);
    p.pix_bytes = (int)(C * es);
    *out = p;
    return DCNV4_OK;
}

unsigned grid_of(const Geo &p) { return (unsigned)(p.remap ? p.tiles_per_xcd * kXcds : p.ntiles); }

// Eight channels per lane in the direct forward: 16-byte (fp16) or 32-byte (fp32) runs, so that
// neighbouring lanes share cache lines.
constexpr int kDefaultFwdCpt = 8;
// One or two channels per lane: a wave's atomic instruction then covers a few whole cache lines
// (16 lanes x 4 or 8 bytes per pixel) instead of 64 different ones, and the L2 atomic rate follows.
int default_bwd_cpt(int Cg) { return Cg <= 32 ? 1 : Cg / 32; }

int pick_fwd_cpt(int Cg)
{
    int c = g_opt.fwd_cpt ? g_opt.fwd_cpt : kDefaultFwdCpt;
    if (c > Cg) c = Cg;
    if (Cg / c > 8) c = Cg / 8;        // at most 8 lanes per group
    return c;
}
int pick_bwd_cpt(int Cg)
{
    int c = g_opt.bwd_cpt ? g_opt.bwd_cpt : default_bwd_cpt(Cg);
    if (c > Cg) c = Cg;
    if (Cg / c > 32) c = Cg / 32;      // the lane reduction spans at most two 16-lane rows
    return c;
}

template <typename T, int CG, int CPT, int KS = 3>
int launch_fwd(const void *x, const void *off, const void *msk, void *y, const Problem &q, hipStream_t s)
{
    Geo p;
    int rc = make_geo(q, CG / CPT, &p);
    if (rc)
        return rc;
    // (products of finite fp16 offsets stay finite; past this scale the smallest offset but zero is outside the image all the same)
    if (sizeof(T) == 2 && CG == 64 && KS == 3)
        p.scale = fminf(fmaxf(p.scale, -5e33f), 5e33f);
    hipLaunchKernelGGL((dcnv4_fwd_kernel<T, CG, CPT, KS, KS>), dim3(grid_of(p)), dim3(kThreads), 0, s, (const T *)x,
                       (const T *)off, (const T *)msk, (T *)y, p);
    if (KS == 3)
        snprintf(g_last_kernel[0], sizeof(g_last_kernel[0]), "dcnv4_fwd_kernel<%s, %d, %d>",
                 sizeof(T) == 2 ? "_Float16" : "float", CG, CPT);
    else
        snprintf(g_last_kernel[0], sizeof(g_last_kernel[0]), "dcnv4_fwd_kernel<%s, %d, %d, %d, %d>",
                 sizeof(T) == 2 ? "_Float16" : "float", CG, CPT, KS, KS);
    return hipGetLastError() == hipSuccess ? DCNV4_OK : DCNV4_ERR_LAUNCH;
}

// Windows other than 3x3 (1x1, 5x5): the direct kernel, eight channels per lane.  A 5x5 window keeps
// 75 values per (pixel, group) in the kernel's static LDS tiles, which fit for groups of 16 channels
// or more (128 pairs per workgroup).
template <typename T, int KS>
int dispatch_fwd_window(const void *x, const void *off, const void *msk, void *y, const Problem &q, hipStream_t s)
{
    switch (q.Cg) {
    case 8:
        if constexpr (KS <= 3)
            return launch_fwd<T, 8, 8, KS>(x, off, msk, y, q, s);
        return DCNV4_ERR_UNSUPPORTED;
    case 16: return launch_fwd<T, 16, 8, KS>(x, off, msk, y, q, s);
    case 32: return launch_fwd<T, 32, 8, KS>(x, off, msk, y, q, s);
    case 64: return launch_fwd<T, 64, 8, KS>(x, off, msk, y, q, s);
    }
    return DCNV4_ERR_UNSUPPORTED;
}

template <typename T, int CG>
int dispatch_fwd_cpt(int cpt, const void *x, const void *off, const void *msk, void *y, const Problem &q,
                     hipStream_t s)
{
    if constexpr (CG >= 16) {
        if (cpt == 16) return launch_fwd<T, CG, 16>(x, off, msk, y, q, s);
    }
    if constexpr (CG <= 64) {
        if (cpt == 8) return launch_fwd<T, CG, 8>(x, off, msk, y, q, s);
    }
    return DCNV4_ERR_UNSUPPORTED;
}


// (pitch + 2) staged pixels of zeros follow the slices; the chooser reserves room for the widest pitch
constexpr int kTiledZeroPixelsExtra = 2;
constexpr int kDefaultHalo = 6;
constexpr int kDefaultHaloGradX = 4;
constexpr int kStripMinHalo = 4, kStripMaxHalo = 12;
constexpr int kDefaultLdsKb = 158;
constexpr int kMaxLdsBytes = 160 * 1024;

// Per-device caches (compute-unit count, dynamic-LDS grants) are indexed by the HIP device number.
constexpr int kMaxDevices = 64;
int current_device()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
        return -1;
    return dev;
}

// Number of compute units of the current device (persistent kernels launch one workgroup each).
int device_cus()
{
    static int cus[kMaxDevices];
    const int dev = current_device();
    if (dev < 0)
        return 0;
    if (cus[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < kXcds)
            return 0;
        cus[dev] = n;
    }
    return cus[dev];
}

// Lets `kern` use `lds` bytes of dynamic LDS on the current device (asked for once per device and size).
bool grant_lds(const void *kern, int lds, int (&granted)[kMaxDevices])
{
    if (lds <= 64 * 1024)
        return true;
    const int dev = current_device();
    if (dev < 0)
        return false;
    if (lds > granted[dev]) {
        if (hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
            return false;
        granted[dev] = lds;
    }
    return true;
}

bool choose_tile(const Problem &q, int threads, int halo, int lds_bytes, int nbuf, int pb, bool accum, bool with_slices,
                 int chan_slices, TGeo *out, double *cost_out = nullptr)
{
    // per-wave LDS slices for the 27 offset/mask values of 64 pixels (grad_offset/grad_mask pass only)
    const int slices = with_slices ? (threads / 64) * 64 * 27 * esize(q.dtype) : 0;
    int cus = device_cus();
    if (cus <= 0) cus = 256;                 // no device in this process (host-only checks): assume a full MI355X
    return tile_choice(q, threads / 64, halo, lds_bytes - slices, nbuf, pb, accum, kFixMaxTilePixels, kTiledZeroPixelsExtra, chan_slices,
                       cus, out, cost_out);
}

// `mode`: kTiledGradX has a single LDS rectangle of Cg + 1 dwords per pixel (fixed-point sums and a bound word);
// kTiledGradOM additionally keeps per-wave slices for the offset/mask values.
int make_tgeo(const Problem &q, int threads, int mode, TGeo *out, int cg_kernel = 0, int want_nbuf = 0)
{
    const bool gradx = mode == kTiledGradX, with_slices = mode == kTiledGradOM;
    // a group wider than the kernel's channel run is cut into slices that are tiles of their own
    const int cgk = cg_kernel ? cg_kernel : q.Cg;
    // (the grad_offset/grad_mask pass can combine slices only in fp32, where it adds them up atomically)
    if (q.Cg % cgk != 0 || (with_slices && cgk != q.Cg && q.dtype != DCNV4_F32))
        return DCNV4_ERR_UNSUPPORTED;
    const int chan_slices = q.Cg / cgk;
    Geo base;
    int rc = make_geo(q, 1, &base);          // shares the 32-bit offset validation
    if (rc)
        return rc;
    TGeo p;
    memset(&p, 0, sizeof(p));
    // the grad_x kernel sends far samples straight to memory without waiting for them, so it can
    // afford a tighter rectangle (taller tiles, fewer flushes)
    const int halo = g_opt.halo ? g_opt.halo : (gradx ? kDefaultHaloGradX : kDefaultHalo);
    int lds = (g_opt.lds_kb ? g_opt.lds_kb : kDefaultLdsKb) * 1024;
    if (lds > kMaxLdsBytes) lds = kMaxLdsBytes;
    const int pb = cgk * esize(q.dtype);
    if (gradx) {
        if (!choose_tile(q, threads, halo, lds, 1, cgk * 4, true, false, chan_slices, &p))
            return DCNV4_ERR_UNSUPPORTED;
        p.nbuf = 1;
    } else {
        // Two buffers overlap the copy of the next tile with the work on this one; one buffer holds a
        // rectangle twice as big (taller bands, fewer tile switches, less halo).  Take the cheaper one
        // by the chooser's own estimate.
        TGeo one;
        memset(&one, 0, sizeof(one));
        double cost2 = 0, cost1 = 0;
        const int pick = g_opt.fwd_single ? g_opt.fwd_single : want_nbuf == 1 ? 2 : want_nbuf == 2 ? 1 : 0;
        const bool ok2 = pick != 2 && choose_tile(q, threads, halo, lds, 2, pb, false, with_slices, chan_slices, &p, &cost2);
        const bool ok1 = pick != 1 && choose_tile(q, threads, halo, lds, 1, pb, false, with_slices, chan_slices, &one, &cost1);
        if (!ok2 && !ok1)
            return DCNV4_ERR_UNSUPPORTED;
        if (!ok2 || (ok1 && cost1 < cost2)) {
            p = one;
            p.nbuf = 1;
        } else {
            p.nbuf = 2;
        }
    }
    const long long es = esize(q.dtype);
    const long long pgi = (long long)q.Ho * q.Wo * q.G;
    if (pgi >= 0x1000000)                    // offset/mask byte offsets inside one image stay in int32
        return DCNV4_ERR_UNSUPPORTED;
    p.H = q.H; p.W = q.W; p.Ho = q.Ho; p.Wo = q.Wo; p.G = q.G;
    p.sh = q.sh; p.sw = q.sw; p.ph = q.ph; p.pw = q.pw; p.dh = q.dh; p.dw = q.dw;
    p.scale = q.scale;
    p.dmax = base.dmax;
    const long long nblocks = (long long)q.N * p.tiles_per_img * q.G * chan_slices;
    if (nblocks >= (1LL << 30))
        return DCNV4_ERR_UNSUPPORTED;
    p.nblocks = (int)nblocks;
    p.blocks_per_xcd = (int)((nblocks + kXcds - 1) / kXcds);
    p.remap = g_opt.xcd_remap;
    p.blocked = 0;                          // (contiguous runs per wave leave waves without work when a tile has few batches)
    p.div_g = make_div((unsigned)q.G);
    p.div_s = make_div((unsigned)chan_slices);
    p.slices = chan_slices;
    p.group_bytes = q.Cg * esize(q.dtype);
    p.div_tpi = make_div((unsigned)p.tiles_per_img);
    p.div_tq = make_div((unsigned)p.tiles_q);
    p.div_q = make_div((unsigned)p.Q);
    p.div_pitch = make_div((unsigned)p.pitch);
    p.x_img_bytes = base.x_img_bytes;
    p.y_img_bytes = base.y_img_bytes;
    p.row_bytes = base.row_bytes;
    p.pix_bytes = base.pix_bytes;
    p.softmax = q.softmax;
    p.og_bytes = (int)((q.merged ? 32 : 18) * es);
    p.mg_bytes = (int)((q.merged ? 32 : 9) * es);
    // (idle lanes point at (pixel, group) number 2^24 of the image, which has to lie past its end)
    if (pgi * p.og_bytes >= (1LL << 31) || pgi >= (1LL << 24))
        return DCNV4_ERR_UNSUPPORTED;
    p.off_img_bytes = (int)(pgi * p.og_bytes);
    p.msk_img_bytes = (int)(pgi * p.mg_bytes);
    p.off_ext_bytes = (int)((pgi - 1) * p.og_bytes + 18 * es);
    p.msk_ext_bytes = (int)((pgi - 1) * p.mg_bytes + 9 * es);
    *out = p;
    return DCNV4_OK;
}

// A launch of the LDS-staged kernel in one of its modes, in two steps: prepare_tiled does everything
// that can refuse (tile choice, LDS size, LDS grant, device query) and launches nothing; run_tiled
// launches what was prepared.  `which` = 0 forward, 1 backward (for the kernel-name record).
struct TiledLaunch {
    TGeoClear p;
    int lds;
    unsigned grid;
};

template <typename T, int CG, int THREADS, int MODE>
int finish_tiled(const TGeo &p, bool any_tile_size, int want_per_cu, TiledLaunch *out)
{
    constexpr bool kGradX = MODE == kTiledGradX;
    // a tile of one or two 64-pixel batches leaves most of the workgroup's waves idle and pays the
    // tile switch for almost no work: such images are left to the direct kernel unless forced
    if (!any_tile_size && p.R * p.Q < 128)
        return DCNV4_ERR_UNSUPPORTED;
    const int px_bytes = kGradX ? CG * 4 : CG * (int)sizeof(T);
    const int tail = kGradX ? (p.xtile_bytes / px_bytes) * 4 + 16 : ((p.pitch + kTiledZeroPixelsExtra) * px_bytes + 15) & ~15;
    const int slices = MODE == kTiledGradOM ? (THREADS / 64) * 64 * 27 * (int)sizeof(T) : 0;     // (not kTiledGradOMDirect)
    const int lds = p.nbuf * p.xtile_bytes + slices + tail;
    if (lds > kMaxLdsBytes)
        return DCNV4_ERR_UNSUPPORTED;
    static int granted[kMaxDevices];         // largest dynamic-LDS size already requested for this kernel, per device
    if (!grant_lds(reinterpret_cast<const void *>(dcnv4_tiled_kernel<T, CG, THREADS, MODE>), lds, granted))
        return DCNV4_ERR_LAUNCH;
    // persistent workgroups: one per compute unit (or fewer when there are fewer tiles)
    const int cus = device_cus();
    if (cus <= 0)
        return DCNV4_ERR_LAUNCH;
    // several persistent workgroups per compute unit when their LDS and registers fit: their tile
    // switches (barrier, drained pipeline) then overlap with each other's work
    int per_cu = g_opt.wg_per_cu ? g_opt.wg_per_cu : want_per_cu ? want_per_cu : (MODE != kTiledFwd || CG * sizeof(T) >= 64 ? 1 : THREADS == 256 ? 2 : THREADS == 64 ? 16 : 1);
    while (per_cu > 1 && (per_cu * lds > kMaxLdsBytes || per_cu * THREADS > 2048))
        --per_cu;
    const int slots = cus * per_cu;
    unsigned grid;
    if (p.remap) {
        const int per = slots / kXcds < p.blocks_per_xcd ? slots / kXcds : p.blocks_per_xcd;
        grid = (unsigned)(per * kXcds);
    } else {
        grid = (unsigned)(slots < p.nblocks ? slots : p.nblocks);
    }
    memset(&out->p, 0, sizeof(out->p));
    static_cast<TGeo &>(out->p) = p;
    out->lds = lds;
    out->grid = grid;
    return DCNV4_OK;
}

template <typename T, int CG, int THREADS, int MODE>
int prepare_tiled(const Problem &q, bool any_tile_size, int want_nbuf, int want_per_cu, TiledLaunch *out)
{
    TGeo p;
    const int rc = make_tgeo(q, THREADS, MODE, &p, CG, want_nbuf);
    return rc ? rc : finish_tiled<T, CG, THREADS, MODE>(p, any_tile_size, want_per_cu, out);
}

template <typename T, int CG, int THREADS, int MODE>
int run_tiled(const TiledLaunch &l, const void *x, const void *off, const void *msk, const void *gy, void *o1, void *o2,
              hipStream_t s, int which)
{
    hipLaunchKernelGGL((dcnv4_tiled_kernel<T, CG, THREADS, MODE>), dim3(l.grid), dim3(THREADS), l.lds, s, (const T *)x,
                       (const T *)off, (const T *)msk, (const T *)gy, (T *)o1, (T *)o2,
                       static_cast<const TArgs<MODE> &>(l.p));
    snprintf(g_last_kernel[which], sizeof(g_last_kernel[which]), "dcnv4_tiled_kernel<%s, %d, %d, %d>",
             sizeof(T) == 2 ? "_Float16" : "float", CG, THREADS, MODE);
    return hipGetLastError() == hipSuccess ? DCNV4_OK : DCNV4_ERR_LAUNCH;
}

// The forward through rectangles, ready to be launched: the choice between it and the strips looks at its tile.
struct RectForward {
    TiledLaunch l;
    int (*run)(const TiledLaunch &, const void *, const void *, const void *, const void *, void *, void *, hipStream_t, int);
    int waves;
    bool many;               // several workgroups on a compute unit
};

template <typename T, int CG, int THREADS>
int finish_fwd_tiled(const TGeo &p, bool any_tile_size, int want_per_cu, RectForward *out)
{
    out->run = run_tiled<T, CG, THREADS, kTiledFwd>;
    out->waves = THREADS / 64;
    out->many = THREADS == 64 || want_per_cu > 1;
    return finish_tiled<T, CG, THREADS, kTiledFwd>(p, any_tile_size, want_per_cu, &out->l);
}

template <typename T, int CG, int THREADS>
int prepare_fwd_tiled(const Problem &q, RectForward *out)
{
    TGeo p;
    const int rc = make_tgeo(q, THREADS, kTiledFwd, &p, CG);
    return rc ? rc : finish_fwd_tiled<T, CG, THREADS>(p, g_opt.fwd_path == 2 || q.merged || q.softmax, 0, out);
}

// The tiled kernel keeps Cg fp32 accumulators and 4*Cg input values per lane, so it is built
// for staged pixels of up to 64 bytes.
template <typename T, int CG>
int choose_fwd_tiled(const Problem &q, RectForward *out)
{
    if constexpr (CG * sizeof(T) <= 64 && CG * sizeof(T) >= 16) {
        if constexpr (CG * sizeof(T) == 64) {
            // 64-byte pixels: eight waves still fit the register file (no LDS slices, no exchange registers)
            if (g_opt.fwd_threads == 64)
                return prepare_fwd_tiled<T, CG, 64>(q, out);
            if (g_opt.fwd_threads == 256)
                return prepare_fwd_tiled<T, CG, 256>(q, out);
            // Whole images of a few batches leave waves of eight idle, and nothing runs beside a refill.  More of them than
            // compute units go to smaller workgroups with one rectangle each: two of four waves a unit, eight of one wave
            // where an image is one or two batches.  us, 64 images: fp32 14x14x512, 16 groups 44 -> 34; 20x20x256 35 -> 30;
            // 28x28x256 57 (strips) -> 52, on inputs in no cache 58.8 -> 56.9; fp16 28x28x256, 8 groups 40.5 (strips) -> 34.4; merged fp32
            // 7x7x1024 60 -> 18, fp16 41 -> 13.  (With fewer images: 8 of 28x28x256, 13.3 in eight waves and 15.7 like this.  In place of
            // rectangles of eight waves 0.70 to 0.96 times as long; in place of strips, 69 random calls, 0.94 times on average, 6 of
            // them 2 to 9 % longer: 227 of 15x26, 8 groups of 32, fp16 65 -> 71.)
            const long long px = (long long)q.Ho * q.Wo, tiles = (long long)q.N * q.G * (q.Cg / CG);
            const int cus = device_cus();
            if (g_opt.fwd_threads == 0 && g_opt.fwd_path != 1 && cus > 0 && tiles > cus && px <= 16 * 64) {
                TGeo whole;
                if (px <= 128) {
                    // Two separate tensors: the direct kernel (fp16: 64 x 8x11x512 13.3 and 14.8), in fp32 until it has so many
                    // workgroups to a unit; one-wave workgroups pay for idle lanes, and in groups of 32 and 64 they read the offsets
                    // again for every slice.  us by the direct kernel and here: 9x9x512, 32 groups, 9 images 5.5 and 9.6, 24: 10.6 and
                    // 10.9, 64: 26 and 18; 7x7x1024, 32 groups, 33 images 11.8 and 13.0, 64: 19 and 17; 282 of 1x1x512, 32 groups 3.9 and
                    // 23.  (Of 400 calls 143 come here, two of them 4 % slower; all take 0.91 times as long as by the
                    // direct kernel.  128 pixels: rectangles of eight waves otherwise, 8x16x512, 32 groups, 22 images 15.1 and 11.5.)
                    const long long b = (px + 63) / 64;
                    const double fill = (double)px / (double)(64 * b), direct = (double)q.N * (double)((px * q.G * q.Cg + 2047) / 2048) / cus;
                    const double least = q.Cg > 16 ? 3.6 / (fill * fill) : b > 1 ? 2.0 : fill < 0.83 ? 0.7 / (fill * fill) : 1.0;
                    // (more padding, dilations: more taps outside, which cost the direct kernel less)
                    const bool plain = q.sh == 1 && q.sw == 1 && q.dh == 1 && q.dw == 1 && q.ph <= 1 && q.pw <= 1;
                    const bool fewer = px == 128 || (plain && px >= (b > 1 ? 72 : 40) && direct > least);
                    if ((q.merged || q.softmax || (sizeof(T) == 4 && fewer)) && make_tgeo(q, 64, kTiledFwd, &whole, CG, 1) == DCNV4_OK &&
                        whole.tiles_per_img == 1) {
                        // Where fewer than seven of them fit a unit (strides, dilations): three at least, and two batches an image only
                        // with tiles enough to overlap, since one wave fills a large rectangle slowly.  us in eight waves and here: 4x29
                        // outputs at stride 3, 28 images of 16 groups of 16, fp32 15.5 and 29.7 (one fits); 23x5 at stride 2, 110 of 4 groups of
                        // 32 19.9 and 22.7 (three fit, 3.4 tiles a unit); 10x3 at stride 3, 522 of 4 groups of 32, fp16 49.7 and 18.8 (five).
                        const int rc = finish_fwd_tiled<T, CG, 64>(whole, true, 8, out);
                        const int fit = rc == DCNV4_OK ? kMaxLdsBytes / out->l.lds : 8;
                        if (fit >= 7 || (fit >= 3 && tiles > (b == 1 ? 1LL : fit == 3 ? 4LL : 2LL) * cus))
                            return rc;
                    }
                } else if (make_tgeo(q, 256, kTiledFwd, &whole, CG, 1) == DCNV4_OK && whole.tiles_per_img == 1 &&
                           finish_fwd_tiled<T, CG, 256>(whole, true, 2, out) == DCNV4_OK && 2 * out->l.lds <= kMaxLdsBytes) {
                    // (a last round of four with one wave in it, many times over, is dearer than strips: 30 x 24x24x1024 fp32,
                    // 32 groups, 9 batches an image: 82.5 and 78.5; 64 x 17x19x256, 6 batches: 27.3 and 29.6)
                    const long long batches = (px + 63) / 64, rounds = (tiles + 2 * cus - 1) / (2 * cus) * ((batches + 3) / 4);
                    if (tiles < 6LL * cus || (double)(tiles * batches) >= 0.72 * 8 * (double)(rounds * cus))
                        return DCNV4_OK;
                }
            }
            return prepare_fwd_tiled<T, CG, 512>(q, out);
        }
        if (g_opt.fwd_threads == 256)
            return prepare_fwd_tiled<T, CG, 256>(q, out);
        if constexpr (CG * sizeof(T) < 64) {
            // Small whole-image tiles: several four-wave workgroups per compute unit, whose tile
            // switches overlap with each other's work, beat one big workgroup.
            if (g_opt.fwd_threads == 64)
                return prepare_fwd_tiled<T, CG, 64>(q, out);
            if (g_opt.fwd_threads == 128)
                return prepare_fwd_tiled<T, CG, 128>(q, out);
            if (g_opt.fwd_threads == 768)
                return prepare_fwd_tiled<T, CG, 768>(q, out);
            const long long px = (long long)q.Ho * q.Wo;
            if (g_opt.fwd_threads == 0 && g_opt.fwd_path != 1 && px <= 128) {
                // An image of one or two batches: one-wave workgroups, eight to a compute unit, so that
                // no wave idles while another works (beats the direct kernel on 7x7 maps).
                TGeo tiny;
                if (make_tgeo(q, 64, kTiledFwd, &tiny, CG) == DCNV4_OK && tiny.tiles_per_img == 1)
                    return finish_fwd_tiled<T, CG, 64>(tiny, true, 0, out);
            }
            if (g_opt.fwd_threads == 0 && px <= 16 * 64) {
                TGeo whole;
                // (one rectangle buffer each: with several workgroups on the unit, one computes while
                // another refills, and the halved LDS lets three of them in)
                if (make_tgeo(q, 256, kTiledFwd, &whole, CG, 1) == DCNV4_OK && whole.tiles_per_img == 1)
                    return finish_fwd_tiled<T, CG, 256>(whole, g_opt.fwd_path == 2 || q.merged || q.softmax, 3, out);
            }
            if (g_opt.fwd_threads == 512)
                return prepare_fwd_tiled<T, CG, 512>(q, out);
            // pixels of up to 32 bytes leave room for twelve waves in the register file (measured: 2-5 %
            // over eight)
            return prepare_fwd_tiled<T, CG, 768>(q, out);
        } else {
            return DCNV4_ERR_UNSUPPORTED;
        }
    }
    return DCNV4_ERR_UNSUPPORTED;
}

// fp16 groups of 64 on small maps, more of them than half the compute units: the direct kernel where rectangles would go through
// them in slices (64 images, us: 14x14x512 18 and 24, 20x20x256 19 and 22; 29 random calls 0.46 to 0.91 times as long), and, up to
// so many batches a unit, where strips would.  Direct kernel against strips, on inputs in no cache: 17 to 26 batches 0.83 to 1.10
// times as long, 31 to 41 1.06 to 1.23 times (219 of 17x22, 4 groups: 71 us and 58); on the same inputs again and again 17 to 45
// batches 0.74 to 1.03 times (most on maps below 200 pixels), 45 to 77 batches 0.94 to 1.13 times.
bool few_wide_batches(const Problem &q)
{
    const long long px = (long long)q.Ho * q.Wo;
    return (long long)q.N * q.G * 2 * ((px + 63) / 64) < (px < 200 ? 45LL : 30LL) * device_cus();
}
template <typename T> bool direct_for_wide_groups(const Problem &q)
{
    return sizeof(T) == 2 && q.Cg == 64 && (long long)q.Ho * q.Wo <= 512 && q.sh == 1 && q.sw == 1 && 2LL * q.N * q.G > device_cus() &&
           !q.merged && !q.softmax && g_opt.fwd_path == 0 && g_opt.fwd_strip == 0 && g_opt.fwd_threads == 0;
}

template <typename T>
int choose_fwd_tiled_cg(const Problem &q, RectForward *out)
{
    constexpr int kWidest = 64 / (int)sizeof(T);     // channels of a 64-byte pixel: the widest run a lane keeps
    switch (q.Cg) {
    case 8: return choose_fwd_tiled<T, 8>(q, out);
    case 16: return choose_fwd_tiled<T, 16>(q, out);
    case 32:
    case 64:
        // wider groups go through in slices of 64 bytes (same offsets and mask, own channels)
        if constexpr (sizeof(T) == 2) {
            // (rectangles that the strips are compared with: not launched themselves)
            if (direct_for_wide_groups<T>(q))
                return few_wide_batches(q) ? DCNV4_ERR_UNSUPPORTED : prepare_fwd_tiled<T, kWidest, 512>(q, out);
        }
        if (q.Cg <= kWidest)
            return choose_fwd_tiled<T, 32>(q, out);
        return choose_fwd_tiled<T, kWidest>(q, out);
    }
    return DCNV4_ERR_UNSUPPORTED;
}

// ---- forward out of a ring of record rows (fp16, 16 channels per group, full-width tiles) ----
// Chooses how many record rows the LDS ring holds and the row halo: a host-side walk over the
// rounds of one workgroup (same arithmetic as the kernel's) finds the largest halo, up to 8 rows,
// for which the rows of two consecutive rounds always fit the ring, and checks that one round can
// stage the rows the next one adds.  Returns DCNV4_ERR_UNSUPPORTED where the kernel does not apply.
int make_rgeo(const Problem &q, int waves, int grid_wgs, RGeo *out)
{
    if (q.dtype != DCNV4_F16 || q.Cg != 16)
        return DCNV4_ERR_UNSUPPORTED;
    Geo base;
    int rc = make_geo(q, 1, &base);
    if (rc)
        return rc;
    RGeo p;
    memset(&p, 0, sizeof(p));
    const long long C = (long long)q.G * q.Cg;
    const long long xbytes = (long long)q.N * q.H * q.W * C * 2;
    const long long pgi = (long long)q.Ho * q.Wo * q.G;
    if (xbytes >= (1LL << 31) || pgi >= 0x1000000 || (long long)q.N * q.G >= (1LL << 24))
        return DCNV4_ERR_UNSUPPORTED;
    p.H = q.H; p.W = q.W; p.Ho = q.Ho; p.Wo = q.Wo; p.G = q.G;
    p.sh = q.sh; p.sw = q.sw; p.ph = q.ph; p.pw = q.pw; p.dh = q.dh; p.dw = q.dw;
    p.scale = q.scale;
    p.dmax = base.dmax;
    p.pitch = q.W + 4;
    p.VR = q.H + 3;
    p.npx = q.Ho * q.Wo;
    p.B = (p.npx + 63) / 64;
    const int lds_budget = (g_opt.lds_kb ? g_opt.lds_kb : 160) * 1024 - 128;
    p.ring = lds_budget / (p.pitch * kRingRecBytes);
    p.ntiles = q.N * q.G;
    p.tiles_per_xcd = (p.ntiles + kXcds - 1) / kXcds;
    p.remap = g_opt.xcd_remap;
    p.cbn = (p.pitch + 31) / 32;
    p.max_groups_round = kRingMaxTasks * ring_staging_waves(waves) / p.cbn;
    if (p.ring < 2 * kRingTaskRows || p.max_groups_round < 1)
        return DCNV4_ERR_UNSUPPORTED;
    // tiles the busiest workgroup walks
    int S;
    if (p.remap) {
        const int per = grid_wgs / kXcds;
        S = (p.tiles_per_xcd + per - 1) / per;
    } else {
        S = (p.ntiles + grid_wgs - 1) / grid_wgs;
    }
    const int RK = kRingTaskRows;
    if (p.ring > (S * p.VR + RK - 1) / RK * RK)
        p.ring = (S * p.VR + RK - 1) / RK * RK;      // no use for more rows than the workgroup ever stages
    const int NB = S * p.B;
    auto need = [&](int gb, int hr, int *lo, int *hi) {
        const int s = gb / p.B, b = gb - s * p.B;
        const int q0 = b * 64, q1 = q0 + 63 < p.npx - 1 ? q0 + 63 : p.npx - 1;
        const int oa = q0 / p.Wo, ob = q1 / p.Wo;
        int l = oa * p.sh - p.ph - hr, h = ob * p.sh - p.ph + 2 * p.dh + hr;
        l = l < -2 ? -2 : l > p.H ? p.H : l;
        h = h > p.H ? p.H : h < -2 ? -2 : h;
        *lo = s * p.VR + 2 + l;
        *hi = s * p.VR + 2 + h;
    };
    const int rounds = (NB + waves - 1) / waves;
    const int sim_rounds = rounds < 4096 ? rounds : 4096;
    int best = -1;
    const int hr_cap = g_opt.halo ? g_opt.halo : 8;
    for (int hr = hr_cap; hr >= 2 && best < 0; --hr) {
        bool ok = true;
        for (int t = 0; t < sim_rounds && ok; ++t) {
            int lo_first, hi_dummy, lo_dummy, hi_next, hi_this;
            need(t * waves, hr, &lo_first, &hi_dummy);
            const int last_this = (t + 1) * waves < NB ? (t + 1) * waves - 1 : NB - 1;
            const int last_next = (t + 2) * waves < NB ? (t + 2) * waves - 1 : NB - 1;
            need(last_this, hr, &lo_dummy, &hi_this);
            need(last_next, hr, &lo_dummy, &hi_next);
            const int g_this = (hi_this + RK) / RK, g_next = (hi_next + RK) / RK;    // row groups staged by then
            if (g_next * RK > lo_first + p.ring)
                ok = false;                                   // two rounds' rows do not fit
            if (t == 0 && g_this * RK > p.ring)
                ok = false;
            if (g_next - g_this > p.max_groups_round)
                ok = false;                                   // one round cannot stage the next one's rows
        }
        if (ok)
            best = hr;
    }
    if (best < 0)
        return DCNV4_ERR_UNSUPPORTED;
    p.hr = best;
    p.div_g = make_div((unsigned)q.G);
    p.div_wo = make_div((unsigned)q.Wo);
    p.div_cbn = make_div((unsigned)p.cbn);
    p.div_vr = make_div((unsigned)p.VR);
    p.div_ring = make_div((unsigned)p.ring);
    p.div_b = make_div((unsigned)p.B);
    p.x_bytes = (int)xbytes;
    p.x_img_bytes = base.x_img_bytes;
    p.y_img_bytes = base.y_img_bytes;
    p.row_bytes = base.row_bytes;
    p.pix_bytes = base.pix_bytes;
    p.og_bytes = q.merged ? 64 : 36;
    p.mg_bytes = q.merged ? 64 : 18;
    p.off_img_bytes = (int)(pgi * p.og_bytes);
    p.msk_img_bytes = (int)(pgi * p.mg_bytes);
    p.off_ext_bytes = (int)((pgi - 1) * p.og_bytes + 36);
    p.msk_ext_bytes = (int)((pgi - 1) * p.mg_bytes + 18);
    *out = p;
    return DCNV4_OK;
}

template <int WAVES, bool SOFTMAX = false>
int launch_ring_fwd(const void *x, const void *off, const void *msk, void *y, const Problem &q, hipStream_t s)
{
    const int cus = device_cus();
    if (cus <= 0)
        return DCNV4_ERR_LAUNCH;
    const long long ntiles = (long long)q.N * q.G;
    const long long tiles_per_xcd = (ntiles + kXcds - 1) / kXcds;
    unsigned grid;
    if (g_opt.xcd_remap) {
        const long long per = cus / kXcds < tiles_per_xcd ? cus / kXcds : tiles_per_xcd;
        grid = (unsigned)(per * kXcds);
    } else {
        grid = (unsigned)(cus < ntiles ? cus : ntiles);
    }
    RGeo p;
    int rc = make_rgeo(q, WAVES, (int)grid, &p);
    if (rc)
        return rc;
    const int lds = p.ring * p.pitch * kRingRecBytes + 128;
    if (lds > kMaxLdsBytes)
        return DCNV4_ERR_UNSUPPORTED;
    auto kern = dcnv4_ring_fwd_kernel<WAVES, SOFTMAX>;
    static int granted[kMaxDevices];
    if (!grant_lds(reinterpret_cast<const void *>(kern), lds, granted))
        return DCNV4_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(WAVES * 64), lds, s, (const _Float16 *)x, (const _Float16 *)off,
                       (const _Float16 *)msk, (_Float16 *)y, p);
    snprintf(g_last_kernel[0], sizeof(g_last_kernel[0]), SOFTMAX ? "dcnv4_ring_fwd_kernel<%d, softmax>" : "dcnv4_ring_fwd_kernel<%d>", WAVES);
    return hipGetLastError() == hipSuccess ? DCNV4_OK : DCNV4_ERR_LAUNCH;
}

int dispatch_ring_fwd(const void *x, const void *off, const void *msk, void *y, const Problem &q, hipStream_t s)
{
    // eight waves: two per SIMD, 256 registers each (four waves on request, for tests)
    if (q.softmax)
        return g_opt.fwd_threads == 256 ? launch_ring_fwd<4, true>(x, off, msk, y, q, s) : launch_ring_fwd<8, true>(x, off, msk, y, q, s);
    if (g_opt.fwd_threads == 256)
        return launch_ring_fwd<4>(x, off, msk, y, q, s);
    return launch_ring_fwd<8>(x, off, msk, y, q, s);
}

// ---- forward out of a rolling window of rows (any type and group width) ----
constexpr int kStripRow = 1024;              // LDS bytes that one staging instruction fills

struct StripLaunch {
    SGeo p;
    int lds;
    unsigned grid;
    long long busiest;                       // batches of the busiest workgroup
};

// The forward's time through rectangles and through strips (us), for calls of more than two batches of 64 pixels to a compute
// unit: by the busiest unit's rounds (a batch to each wave), whole and in fractions, its staged LDS bytes, its tiles, and the
// mean rounds of all units.  Fitted to graph replays of 5800 random calls of both kernels (stride 1; maps of 7x7 to 200x360, up
// to 64 groups, offsets of 1, 2 and 4 pixels): either within 7 to 13 % (one standard deviation), their ratio within 6 to 8 %,
// most of it by the offsets' size, which the host does not know.
struct ForwardTimes {
    float rect_rounds, rect_staged, rect_tiles, rect_mean, rect_once;
    float strip_whole, strip_rounds, strip_staged, strip_near, strip_mean, strip_once;
};
ForwardTimes forward_times(int dtype, int pb)
{
    if (pb == 64)
        return dtype == DCNV4_F32 ? ForwardTimes{3.82f, 1.51f, 1.58f, 3.00f, 5.92f, 2.73f, 3.07f, 1.37f, 0.08f, 1.24f, 8.72f}
                                  : ForwardTimes{5.27f, 1.17f, 2.13f, 2.77f, 6.47f, 3.38f, 3.50f, 0.93f, 0.08f, 1.17f, 10.72f};
    if (pb == 32)
        return dtype == DCNV4_F32 ? ForwardTimes{5.12f, 0.07f, 1.44f, 6.23f, -14.23f, 1.69f, 1.56f, 1.49f, 0.15f, 6.69f, -7.56f}
                                  : ForwardTimes{4.21f, 1.82f, 1.05f, 3.17f, 2.80f, 2.31f, 3.51f, 0.84f, 0.16f, 2.10f, 6.93f};
    return ForwardTimes{3.80f, 0.00f, 0.88f, 1.98f, 2.89f, 2.78f, 0.00f, 1.36f, 0.00f, 2.67f, 6.29f};
}
// The same once more where strips have become faster since, fitted to 13 thousand random calls in which both kernels launch
// (16 batches of 64-byte pixels a unit and more, 24 of narrower ones): 64-byte pixels by the times at offsets of 4 pixels, which cost
// strips most, others by the mean over 1, 2 and 4.  Their ratio within 6, 4 and 6 %.  `strip_near` counts columns too.
ForwardTimes strip_times_now(int pb)
{
    if (pb == 64)
        return ForwardTimes{2.93f, 3.35f, 1.11f, 4.37f, 3.09f, 3.29f, 2.53f, 1.54f, 0.49f, 1.59f, 7.33f};
    if (pb == 32)
        return ForwardTimes{4.17f, 4.75f, -0.29f, 6.10f, -4.30f, 2.03f, 1.98f, 2.38f, 0.31f, 5.94f, -0.83f};
    return ForwardTimes{2.83f, 6.89f, -0.27f, 3.38f, 0.74f, 1.59f, -0.23f, 1.87f, 0.21f, 5.49f, 2.79f};
}
bool strips_win(const Problem &q, const TGeo &r, int rect_waves, const SGeo &p, int waves, long long busiest, int pb, long long batches, int cus)
{
    const float mean = (float)batches / (float)(cus * waves);
    const float tiles = (float)((r.nblocks + cus - 1) / cus), rounds = (float)((r.R * r.Q + 63) / 64) / rect_waves;
    const int near_r = p.halo_r < 7 ? 7 - p.halo_r : 0, near_c = p.tiles_q > 1 && p.halo_c < 7 ? 7 - p.halo_c : 0;
    const float staged = (float)((p.ntiles + cus - 1) / cus) * (float)p.VR * (float)p.row_lds * (1.f / 65536);
    auto rect = [&](const ForwardTimes &t) {
        return tiles * (t.rect_rounds * rounds + t.rect_staged * (float)r.xtile_bytes * (1.f / 65536) + t.rect_tiles) +
               t.rect_mean * mean + t.rect_once;
    };
    auto strip = [&](const ForwardTimes &t, int near) {
        return t.strip_whole * (float)((busiest + waves - 1) / waves) + (t.strip_rounds + t.strip_near * (float)near) * (float)busiest / waves +
               t.strip_staged * staged + t.strip_mean * mean + t.strip_once;
    };
    // A margin for windows that allow for small displacements: offsets of 4 pixels cost the strips most there (64-byte pixels in
    // fp32, allowing for 4: 6 % faster than rectangles at offsets of 1 and 2 pixels, 7 % slower at 4).  Over a thousand other
    // calls for which this picks strips: 9 % faster on average, 6 % of the calls slower by 5 % or more.
    const ForwardTimes t = forward_times(q.dtype, pb);
    if (strip(t, near_r) * (1.f + 0.02f * (float)(near_r > near_c ? near_r : near_c)) < rect(t))
        return true;
    // And what the strips' present times add to that, by a margin of the fit's error, so that a call is hardly ever slower than
    // through its rectangles: of those 13 thousand calls 1331 come here, at offsets of 1, 2 and 4 pixels 0.91, 0.91 and 0.94 times as
    // long, 77 of them more than 3 % longer at one of the three.  (A factor of 0.89 on the first estimate: 2469 calls, 0.93, 0.94 and
    // 1.00 times as long, and 768 of them 3 to 32 % longer.)  fp32, offsets of 1, 2 and 4 pixels: 5 x 74x116x256, 8 groups, stays with
    // rectangles (65, 66 and 67 us; strips 61, 63 and 71).
    // Not with strides, which are not among them (fp16 1 x 155x271x360, 45 groups, stride 2: rectangles 38 us, strips 50).
    if ((q.dtype != DCNV4_F32 && pb != 16) || q.sh > 1 || q.sw > 1)
        return false;
    const ForwardTimes now = strip_times_now(pb);
    return strip(now, near_r + near_c) < (pb == 64 ? 0.95f : 0.94f) * rect(now);
}

// Chooses strips of columns, bands of rows, the window's rows and the displacement it allows for, by the batches that
// the busiest workgroup works through.  `rect`: what the forward's rectangles would launch, if there are any.
int make_sgeo(const Problem &q, int cg_kernel, int waves, StripLaunch *out, const RectForward *rect, bool gom = false, int slices_lds = 0)
{
    const long long es = esize(q.dtype), pb = cg_kernel * es, pgi = (long long)q.Ho * q.Wo * q.G;
    if (q.Cg % cg_kernel != 0)
        return DCNV4_ERR_UNSUPPORTED;
    const int cus = device_cus(), slices = q.Cg / cg_kernel;
    const long long batches = (long long)q.N * q.G * slices * (((long long)q.Ho * q.Wo + 63) / 64);
    // The forward: for two batches to a compute unit or less of maps that are not tiny, since bands are cut finer than rectangles
    // (1 of 40x47, 16 groups of 8, fp32: 12.3 us by rectangles, 8.2 by strips; 16 of 14x14, 16 groups of 16: 8.6 and 10.3), at
    // stride 1 (at 2 a window holds four times the pixels: 2 of 64x98, 7 groups of 32, fp16: 12.6 and 16.0); and by both kernels'
    // estimates where there are batches to stream, two rounds of eight waves or of twelve (narrow pixels, 24 to 48 batches a unit:
    // 372 random calls that the first estimate takes there 0.81, 0.81 and 0.85 times as long at offsets of 1, 2 and 4 pixels, four
    // of them more than 3 % longer, at 4).  In between, where several small workgroups share a unit and where narrow pixels lie
    // side by side in memory (one group: 5 % faster over 86 calls), rectangles.  (Strips in place of several small workgroups, 3256
    // random calls: below 64 batches a unit 1.02 to 1.05 times as long, above 0.96 to 0.98: the line could lie there.)
    const bool few = !gom && batches <= 2LL * cus && (long long)q.Ho * q.Wo >= (pb == 64 ? 400 : 700);
    // The grad_offset/grad_mask pass from a quarter of a batch on (1 image of 28x28, 8 groups, fp32: 21.2 us by rectangles, 18.6
    // by strips, with grad_x; 1 of 14x14, 4 groups: 16.3 and 16.5).
    if (cus > 0 && g_opt.fwd_strip != 1) {
        if (gom ? batches * 4 < cus : !few && batches < (pb == 64 ? 16LL : 24LL) * cus)
            return DCNV4_ERR_UNSUPPORTED;
        if (!gom && ((few && (q.sh > 1 || q.sw > 1) && pb > 16) || (!few && q.G == 1 && pb < 64) || (rect != nullptr && rect->many)))
            return DCNV4_ERR_UNSUPPORTED;
    }
    // (what no kernel takes is refused before the device is asked for: the answer does not depend on there being one)
    Geo base;
    int rc = make_geo(q, 1, &base);
    if (rc)
        return rc;
    if (cus <= 0)
        return DCNV4_ERR_LAUNCH;
    SGeo p;
    memset(&p, 0, sizeof(p));
    p.og_bytes = (int)((q.merged ? 32 : 18) * es);
    p.mg_bytes = (int)((q.merged ? 32 : 9) * es);
    // offsets whose product with the scale is past fp32 (fp16 ones with a scale of 5e33 or more: rectangles)
    const float scale = q.scale < 0.f ? -q.scale : q.scale;
    if (es == 2 && scale > 5e33f)
        return DCNV4_ERR_UNSUPPORTED;
    p.off_max = es == 4 && scale > 1.f ? 3.4e38f / scale : 0.f;
    // (whole tensors behind one descriptor each)
    const long long xbytes = (long long)q.N * base.x_img_bytes, ybytes = (long long)q.N * base.y_img_bytes;
    if (xbytes >= (1LL << 31) || ybytes >= (1LL << 31) || q.N * pgi * p.og_bytes >= (1LL << 31) || q.Ho >= (1 << 15) || q.Wo >= (1 << 15))
        return DCNV4_ERR_UNSUPPORTED;
    p.slices = slices;
    int lds = (g_opt.lds_kb ? g_opt.lds_kb : kMaxLdsBytes / 1024) * 1024;
    if (lds > kMaxLdsBytes) lds = kMaxLdsBytes;
    lds -= slices_lds;
    const int halo_lo = g_opt.halo ? g_opt.halo : kStripMinHalo, halo_hi = g_opt.halo ? g_opt.halo : kStripMaxHalo;
    auto cols_of = [&](int Q, int h) {
        const int c = (Q - 1) * q.sw + 2 * q.dw + 2 * h + 2;
        return c < q.W + 4 ? c : q.W + 4;
    };
    auto rows_of = [&](int R, int h) {
        const int r = (R - 1) * q.sh + 2 * q.dh + 2 * h + 2;
        return r < q.H + 4 ? r : q.H + 4;
    };
    double best = 1e30;
    int splits = 0;
    for (int kq = 1; kq <= q.Wo && splits < 6; ++kq) {
        const int Q = (q.Wo + kq - 1) / kq;
        if (kq > 1 && Q == (q.Wo + kq - 2) / (kq - 1))
            continue;
        const int tiles_q = (q.Wo + Q - 1) / Q;
        int row = 0;
        bool any = false;
        for (int hc = halo_lo; hc <= (g_opt.halo ? halo_lo : 8); hc += 2) {
            const int row_hc = (cols_of(Q, hc) * (int)pb + kStripRow - 1) / kStripRow * kStripRow;
            const int ring = (lds - row_hc - 2 * (int)pb) / row_hc - 1;
            if (row_hc == row || ring < 4)
                continue;
            row = row_hc;
            any = true;
            int hcm = hc;
            while (hcm < halo_hi && cols_of(Q, hcm + 1) * (int)pb <= row)
                ++hcm;
            for (int bands = 1; bands <= q.Ho && bands <= 16; ++bands) {
                const int R = (q.Ho + bands - 1) / bands;
                if (bands > 1 && R == (q.Ho + bands - 2) / (bands - 1))
                    continue;
                const int nb = (q.Ho + R - 1) / R;
                const long long tiles = (long long)q.N * q.G * p.slices * nb * tiles_q;
                if (tiles >= (1LL << 24) || (long long)R * Q >= (1LL << 24))
                    break;
                const int S = ((int)tiles + cus - 1) / cus, B = (R * Q + 63) / 64;
                if ((long long)S * B >= (1LL << 24))
                    continue;
                // virtual rows that two consecutive rounds can reach: a run of output rows, and what changes of tile add
                // (a change of image in a run of several rounds is rare and adds little: left out)
                const int px = 2 * waves * 64, run = ((px + Q - 2) / Q) * q.sh + 2 * q.dh + 2;
                const int changes = S == 1 ? 0 : B < 2 * waves ? (2 * waves - 2) / B + (nb > 1 ? 1 : 0) : nb > 1 ? 1 : 0;
                auto span = [&](int h) {
                    const int change = nb > 1 ? 2 * q.dh + 2 * h + 2 - q.sh : 2 * q.dh + 5 - 2 * q.ph - q.sh;
                    const long long most = run + 2 * h + (long long)changes * (change > 0 ? change : 0), all = (long long)S * rows_of(R, h);
                    return most < all ? most : all;
                };
                if (span(halo_lo) > ring)
                    continue;
                int hr = halo_lo;
                while (hr < halo_hi && span(hr + 1) <= ring)
                    ++hr;
                const double staged = (double)(row / pb) * rows_of(R, hr) / ((double)R * Q);
                // taps that leave the window (on one side of a strip that has neighbours on both, on average)
                auto leave = [&](int h) { return (h < 6 ? 0.04 * (6 - h) : 0.0) + (h < 8 ? 0.015 * (8 - h) : 0.0); };
                const double far = g_opt.halo ? 0.0 : leave(hr) + (tiles_q > 1 ? leave(hcm) * 32.0 / Q : 0.0);
                const double cost = ((double)S * B / waves + 0.5) * (1.0 + (pb < 64 ? 0.05 : 0.1) * staged + far) + 1.0;
                if (cost < best - 1e-9) {
                    best = cost;
                    p.R = R;
                    p.Q = Q;
                    p.halo_r = hr;
                    p.halo_c = hcm;
                    p.row_lds = row;
                    p.VR = rows_of(R, hr);
                    p.B = B;
                    p.ring = (long long)ring < (long long)S * p.VR ? ring : S * p.VR;
                    p.tiles_q = tiles_q;
                    p.tiles_per_img = nb * tiles_q;
                    p.ntiles = (int)tiles;
                    out->busiest = (long long)S * B;
                }
            }
        }
        splits += any;
    }
    if (best >= 1e30 || (long long)p.ntiles * p.VR >= (1LL << 30))
        return DCNV4_ERR_UNSUPPORTED;
    if (g_opt.fwd_strip != 1 && !gom && !few && rect != nullptr &&
        !strips_win(q, rect->l.p, rect->waves, p, waves, out->busiest, (int)pb, batches, cus))
        return DCNV4_ERR_UNSUPPORTED;
    p.H = q.H; p.W = q.W; p.Ho = q.Ho; p.Wo = q.Wo; p.G = q.G;
    p.sh = q.sh; p.sw = q.sw; p.ph = q.ph; p.pw = q.pw; p.dh = q.dh; p.dw = q.dw;
    p.scale = q.scale;
    p.dmax = base.dmax;
    p.softmax = q.softmax;
    p.cpr = p.row_lds / kStripRow;
    p.tiles_per_xcd = (p.ntiles + kXcds - 1) / kXcds;
    p.remap = g_opt.xcd_remap;
    p.div_g = make_div((unsigned)q.G);
    p.div_s = make_div((unsigned)p.slices);
    p.div_tpi = make_div((unsigned)p.tiles_per_img);
    p.div_tq = make_div((unsigned)p.tiles_q);
    p.div_q = make_div((unsigned)p.Q);
    p.div_vr = make_div((unsigned)p.VR);
    p.div_b = make_div((unsigned)p.B);
    p.div_ring = make_div((unsigned)p.ring);
    p.div_cpr = make_div((unsigned)p.cpr);
    p.group_bytes = (int)(q.Cg * es);
    p.x_img_bytes = base.x_img_bytes;
    p.row_bytes = base.row_bytes;
    p.pix_bytes = base.pix_bytes;
    p.x_bytes = (int)xbytes;
    p.y_bytes = (int)ybytes;
    p.off_bytes = (int)((q.N * pgi - 1) * p.og_bytes + 18 * es);
    p.msk_bytes = (int)(((q.N * pgi - 1) * p.mg_bytes + 9 * es + 3) & ~3LL);
    out->p = p;
    out->lds = (p.ring + 2) * p.row_lds + (int)(2 * pb) + slices_lds;
    if (p.remap) {
        const int per = cus / kXcds < p.tiles_per_xcd ? cus / kXcds : p.tiles_per_xcd;
        out->grid = (unsigned)(per * kXcds);
    } else {
        out->grid = (unsigned)(cus < p.ntiles ? cus : p.ntiles);
    }
    return DCNV4_OK;
}

// in two steps, as prepare_tiled and run_tiled
template <typename T, int CG, int WAVES, int GOM>
int prepare_strip(const Problem &q, StripLaunch *l, const RectForward *rect = nullptr)
{
    const int rc = make_sgeo(q, CG, WAVES, l, rect, GOM != 0, GOM == 1 && sizeof(T) == 2 ? WAVES * 64 * 27 * 2 : 0);
    if (rc)
        return rc;
    static int granted[kMaxDevices];
    return grant_lds(reinterpret_cast<const void *>(dcnv4_strip_kernel<T, CG, WAVES, GOM>), l->lds, granted) ? DCNV4_OK : DCNV4_ERR_LAUNCH;
}

template <typename T, int CG, int WAVES, int GOM>
int run_strip(const StripLaunch &l, const void *x, const void *off, const void *msk, const void *gy, void *o1, void *o2, hipStream_t s)
{
    hipLaunchKernelGGL((dcnv4_strip_kernel<T, CG, WAVES, GOM>), dim3(l.grid), dim3(WAVES * 64), l.lds, s, (const T *)x, (const T *)off,
                       (const T *)msk, (const T *)gy, (T *)o1, (T *)o2, l.p);
    snprintf(g_last_kernel[GOM != 0], sizeof(g_last_kernel[GOM != 0]), "dcnv4_strip_kernel<%s, %d, %d, %d>",
             sizeof(T) == 2 ? "_Float16" : "float", CG, WAVES, GOM);
    return hipGetLastError() == hipSuccess ? DCNV4_OK : DCNV4_ERR_LAUNCH;
}

template <typename T, int CG, int WAVES>
int launch_strip(const void *x, const void *off, const void *msk, void *y, const Problem &q, const RectForward *rect, hipStream_t s)
{
    StripLaunch l;
    const int rc = prepare_strip<T, CG, WAVES, 0>(q, &l, rect);
    return rc ? rc : run_strip<T, CG, WAVES, 0>(l, x, off, msk, nullptr, y, nullptr, s);
}

// a lane keeps up to 64 bytes of a pixel (wider groups in slices); twelve waves fit the registers with up to 32
template <typename T>
int dispatch_strip(const void *x, const void *off, const void *msk, void *y, const Problem &q, const RectForward *rect, hipStream_t s)
{
    constexpr int kWidest = 64 / (int)sizeof(T);
    if (q.Cg >= kWidest)
        return launch_strip<T, kWidest, 8>(x, off, msk, y, q, rect, s);
    if constexpr (sizeof(T) == 2) {
        if (q.Cg == 16)
            return launch_strip<T, 16, 12>(x, off, msk, y, q, rect, s);
    }
    return launch_strip<T, 8, 12>(x, off, msk, y, q, rect, s);
}

// fp16, 16 channels per group: where the ring kernel (dot products of fp16 pairs) is the better one.  It takes whole images,
// so with few (image, group) pairs compute units stay idle, and on wide maps its window is too low: 1 image of 128x128, 16
// groups: 217 us by the ring, 21 by rectangles; 10 of 75x101, 8 groups: 106, by strips 37.  Where it fills the chip a batch
// costs it 0.77 us, the others about 1 (16 of 28x28, 16 groups: 15.4 and 17.1; 5 of 40x40, 44 groups: 23.1 and 23.4; 16 of
// 40x47, 8 groups: 23.9 and 20.9).  Past 80 wide it was the faster in none of 36 calls that fill the chip (32 of 56x84, 8 groups:
// 60 us and 58; of 56x104: 111 and 67).  Of 300 random calls that this keeps from the ring, 10 would be 5 % or more faster by it,
// and it is 1.7 times slower on average.
bool ring_first(const Problem &q)
{
    const long long tiles = (long long)q.N * q.G, B = ((long long)q.Ho * q.Wo + 63) / 64;
    const int cus = device_cus();
    if (cus <= 0 || q.Cg != 16 || B <= 12)
        return true;
    const double share = (double)((tiles + cus - 1) / cus * B), mean = (double)(tiles * B) / cus;
    return q.W <= 80 && 0.77 * share <= mean + 4.0;
}

template <typename T>
int dispatch_fwd(const void *x, const void *off, const void *msk, void *y, const Problem &q, hipStream_t s)
{
    if (q.kh != 3) {
        if (q.merged || q.softmax || g_opt.fwd_path >= 2)
            return DCNV4_ERR_UNSUPPORTED;
        return q.kh == 1 ? dispatch_fwd_window<T, 1>(x, off, msk, y, q, s) : dispatch_fwd_window<T, 5>(x, off, msk, y, q, s);
    }
    // (maps of a few batches per image leave most of a ring workgroup idle: the rectangle kernels,
    // with several small workgroups per compute unit, are faster there -- measured at 14x14 and 7x7)
    if (sizeof(T) == 2 && (g_opt.fwd_path == 3 || (g_opt.fwd_path == 0 && g_opt.fwd_strip != 1 && q.Ho * q.Wo >= 512 && (g_opt.fwd_strip == 2 || ring_first(q))))) {
        const int rc = dispatch_ring_fwd(x, off, msk, y, q, s);
        if (rc != DCNV4_ERR_UNSUPPORTED || g_opt.fwd_path == 3)
            return rc;
    }
    if (g_opt.fwd_path == 3)
        return DCNV4_ERR_UNSUPPORTED;
    if (g_opt.fwd_path != 1) {
        RectForward rect;
        const int rc = choose_fwd_tiled_cg<T>(q, &rect);
        if (rc != DCNV4_OK && rc != DCNV4_ERR_UNSUPPORTED)
            return rc;
        // (two separate tensors without a useful rectangle go to the direct kernel, strips or not: 1 of 36x48, 1 group of 64,
        // stride 2, fp16: 5.7 us, by strips 11.2)
        if (g_opt.fwd_path == 0 && g_opt.fwd_strip != 2 && (rc == DCNV4_OK || q.merged || q.softmax || g_opt.fwd_strip == 1)) {
            const int rs = dispatch_strip<T>(x, off, msk, y, q, rc == DCNV4_OK ? &rect : nullptr, s);
            if (rs != DCNV4_ERR_UNSUPPORTED || g_opt.fwd_strip == 1)
                return rs;
        }
        if (rc == DCNV4_OK && !direct_for_wide_groups<T>(q))
            return rect.run(rect.l, x, off, msk, nullptr, y, nullptr, s, 0);
        if (g_opt.fwd_path == 2)
            return rc;
        // (no useful rectangle: the ring after all, where it was passed over)
        if (sizeof(T) == 2 && g_opt.fwd_path == 0 && q.Ho * q.Wo >= 512) {
            const int rr = dispatch_ring_fwd(x, off, msk, y, q, s);
            if (rr != DCNV4_ERR_UNSUPPORTED)
                return rr;
        }
    }
    if (q.merged || q.softmax)               // (the direct kernels read two separate tensors and take m as given)
        return DCNV4_ERR_UNSUPPORTED;
    const int cpt = pick_fwd_cpt(q.Cg);
    switch (q.Cg) {
    case 8: return dispatch_fwd_cpt<T, 8>(cpt, x, off, msk, y, q, s);
    case 16: return dispatch_fwd_cpt<T, 16>(cpt, x, off, msk, y, q, s);
    case 32: return dispatch_fwd_cpt<T, 32>(cpt, x, off, msk, y, q, s);
    case 64: return dispatch_fwd_cpt<T, 64>(cpt, x, off, msk, y, q, s);
    }
    return DCNV4_ERR_UNSUPPORTED;
}

template <int CG, int CPT, int KS = 3>
int launch_bwd(const void *x, const void *off, const void *msk, const void *gy, void *gx, void *go, void *gm,
               const Problem &q, hipStream_t s)
{
    Geo p;
    int rc = make_geo(q, CG / CPT, &p);
    if (rc)
        return rc;
    const long long zbytes = (long long)q.N * p.x_img_bytes;
    long long zb = (zbytes / 16 + kThreads - 1) / kThreads;
    if (zb > 8192) zb = 8192;
    hipLaunchKernelGGL(dcnv4_zero_kernel, dim3((unsigned)zb), dim3(kThreads), 0, s, (u32x4 *)gx, zbytes);
    hipLaunchKernelGGL((dcnv4_bwd_kernel<CG, CPT, KS, KS>), dim3(grid_of(p)), dim3(kThreads), 0, s, (const float *)x,
                       (const float *)off, (const float *)msk, (const float *)gy, (float *)gx, (float *)go,
                       (float *)gm, p);
    if (KS == 3)
        snprintf(g_last_kernel[1], sizeof(g_last_kernel[1]), "dcnv4_bwd_kernel<%d, %d>", CG, CPT);
    else
        snprintf(g_last_kernel[1], sizeof(g_last_kernel[1]), "dcnv4_bwd_kernel<%d, %d, %d, %d>", CG, CPT, KS, KS);
    return hipGetLastError() == hipSuccess ? DCNV4_OK : DCNV4_ERR_LAUNCH;
}

template <int CG>
int dispatch_bwd_cpt(int cpt, const void *x, const void *off, const void *msk, const void *gy, void *gx, void *go,
                     void *gm, const Problem &q, hipStream_t s)
{
    if constexpr (CG >= 16) {
        if (cpt == 16) return launch_bwd<CG, 16>(x, off, msk, gy, gx, go, gm, q, s);
    }
    if (cpt == 8) return launch_bwd<CG, 8>(x, off, msk, gy, gx, go, gm, q, s);
    if constexpr (CG <= 64) {
        if (cpt == 4) return launch_bwd<CG, 4>(x, off, msk, gy, gx, go, gm, q, s);
    }
    if constexpr (CG <= 64) {
        if (cpt == 2) return launch_bwd<CG, 2>(x, off, msk, gy, gx, go, gm, q, s);
    }
    if constexpr (CG <= 32) {
        if (cpt == 1) return launch_bwd<CG, 1>(x, off, msk, gy, gx, go, gm, q, s);
    }
    return DCNV4_ERR_UNSUPPORTED;
}

// ---- grad_x through dcnv4_gradx_kernel ----------------------------------------------------------
constexpr int kMaxHaloGradX = 8;

struct GxLaunch {
    GxGeo p;
    int lds;
    unsigned grid;
    int waves;
};

// Clocks of the kernel in tiles of R x Q outputs with so many cells, `tiles_img` an image: handed out one by one, their sums
// added atomically, or (owned) all tiles of an (image, channel run) to one workgroup, which stores them.  The wave with the
// most units of 16 pixels takes a time per batch of up to four for the evaluation and per unit for the adds; it waits for most
// of that, so other waves of its SIMD add less than as much again.  Then the flush, which the workgroups of a compute unit
// share.  (Fitted to 230 kernels of 20 calls, 7 to 1200 us: 13 % rms; the tile it takes for each call is within 7 % of its
// best measured one.)
double gx_time(const Problem &q, int waves, int per_cu, int slices, int cus, int R, int Q, long long tiles_img, long long cells, bool owned)
{
    auto ceil_div = [](long long a, long long b) { return (a + b - 1) / b; };
    const int units = (int)ceil_div(R * ceil_div(Q, 4), 4), most = (units + waves - 1) / waves;
    const long long slots = (long long)cus * per_cu, planes = (long long)q.N * q.G * slices, blocks = owned ? planes : planes * tiles_img;
    const double resident = blocks < slots ? (double)ceil_div(blocks, cus) : (double)per_cu;
    const double simd = resident * (waves < units ? waves : units) / 4.0;
    const double flush = (owned ? 4.3 : q.dtype == DCNV4_F32 ? 10.8 : 8.3) * resident * (double)cells;
    return (double)(ceil_div(blocks, slots) * (owned ? tiles_img : 1)) * ((1800.0 * ((most + 3) / 4) + 960.0 * most) * (simd + 4.5) + flush);
}

struct GxTile {
    int R, Q, pitch, tiles_q, tiles_per_img;
    int waves, per_cu, lds;
    double cost;
};

// Rows (columns) the largest rectangle of a split into parts of `len` outputs can have; `border`: cells kept
// outside the image on each side.  Columns need one more cell unless every tile goes from border to border.
long long gx_extent(int out, int len, int size, int s, int pad, int dil, int h, int border, bool columns)
{
    const long long parts = ((long long)out + len - 1) / len, span = (long long)(len - 1) * s + 2LL * dil + 2LL * h + 2;
    if (parts > 8)                                     // (many parts: those inside are not clipped)
        return (span < size + 2 * border ? span : size + 2 * border) + (columns ? 1 : 0);
    long long most = 0;
    for (long long k = 0; k < parts; ++k) {
        const long long o0 = k * len, n = out - o0 < len ? out - o0 : len;
        const long long want = o0 * s - pad - h, end = (o0 + n - 1) * s - pad + 2LL * dil + h + 2;
        const long long lo = want > -border ? want : -border, hi = end < size + border ? end : size + border;
        const long long e = (hi - lo > 0 ? hi - lo : 0) + (columns && !(want <= -border && end >= size + border) ? 1 : 0);
        if (e > most) most = e;
    }
    return most;
}
int gx_max_cells(int lds_bytes) { return (lds_bytes - kGxCell - 16) / (kGxCell + 4) - 2; }

// Tile choice: output rows per band x columns per tile whose cells fit the LDS, by an estimate of the time (in
// clocks) of the busiest compute unit, `per_cu` workgroups of `waves` waves on each; for tiles handed out one by one and for
// owned planes in one search (either may be null), each kept where it is better than what is there.
void choose_gx_tiles(const Problem &q, int waves, int per_cu, int halo, int lds_bytes, int slices, int cus, GxTile *any, GxTile *own)
{
    const int max_cells = gx_max_cells(lds_bytes);
    auto ceil_div = [](long long a, long long b) { return (a + b - 1) / b; };
    // the band heights, with their rectangles' rows
    struct {
        int R;
        long long rows;
    } heights[128];
    int nheights = 0;
    for (int bands = 1; bands <= q.Ho && bands <= 256 && nheights < 128; bands += bands < 32 ? 1 : bands / 16) {
        const int R = (int)ceil_div(q.Ho, bands);
        if (nheights == 0 || R != heights[nheights - 1].R)
            heights[nheights++] = {R, gx_extent(q.Ho, R, q.H, q.sh, q.ph, q.dh, halo, 2, false)};
    }
    int splits = 0;
    for (int kq = 1; kq <= q.Wo && splits < 12; ++kq) {
        const int Q = (int)ceil_div(q.Wo, kq);
        if (kq > 1 && Q == (int)ceil_div(q.Wo, kq - 1))
            continue;
        const long long cols = gx_extent(q.Wo, Q, q.W, q.sw, q.pw, q.dw, halo, 1, true);
        if (cols < 1 || cols > max_cells)
            continue;
        const int tiles_q = (int)ceil_div(q.Wo, Q);
        bool fits = false;
        for (int h = 0; h < nheights; ++h) {
            const int R = heights[h].R;
            const long long rows = heights[h].rows;
            if (rows * cols > max_cells || (long long)R * Q > kFixMaxTilePixels)     // (the bound words must not wrap)
                continue;
            fits = true;
            const int bands = (int)ceil_div(q.Ho, R);
            auto keep = [&](GxTile *t, double cost) {
                if (cost < t->cost)
                    *t = {R, Q, (int)cols, tiles_q, bands * tiles_q, waves, per_cu, lds_bytes, cost};
            };
            if (own != nullptr)
                keep(own, gx_time(q, waves, per_cu, slices, cus, R, Q, (long long)bands * tiles_q, rows * cols, true));
            if (any != nullptr) {
                // the wave with the most units of 16 pixels: per batch of up to four of them the evaluation, per unit the
                // adds, shared with the other waves of its SIMD; then the flush, which the workgroups of a unit share as
                // well, and the drained pipeline at the tile's end
                const long long tiles = (long long)q.N * q.G * slices * bands * tiles_q;
                const int units = (int)ceil_div(R * ceil_div(Q, 4), 4), most = (units + waves - 1) / waves;
                const long long slots = (long long)cus * per_cu;
                const double resident = tiles < slots ? (double)ceil_div(tiles, cus) : (double)per_cu;
                const double simd = resident * (waves < units ? waves : units) / 4.0;
                const double batches = (simd > 1.0 ? simd : 1.0) * (2900.0 * ((most + 3) / 4) + 1200.0 * most);
                keep(any, (double)ceil_div(tiles, slots) * (batches + 9.0 * resident * (double)(rows * cols) + 5000.0));
            }
        }
        if (fits)
            ++splits;
    }
}

// A tile into the geometry; what is left of the LDS allows for larger displacements.
void set_gx_tile(const Problem &q, const GxTile &t, int halo, int max_halo, GxGeo *p)
{
    p->R = t.R;
    p->Q = t.Q;
    p->pitch = t.pitch;
    p->tiles_q = t.tiles_q;
    p->tiles_per_img = t.tiles_per_img;
    p->halo = halo;
    for (int h = halo; h <= max_halo; ++h) {
        const long long rows = gx_extent(q.Ho, t.R, q.H, q.sh, q.ph, q.dh, h, 2, false);
        const long long cols = gx_extent(q.Wo, t.Q, q.W, q.sw, q.pw, q.dw, h, 1, true);
        if (rows * cols > gx_max_cells(t.lds))
            break;
        p->halo = h;
        p->pitch = (int)cols;
        // (at least a row: taps that stay out of the cells book on the corners of cell 0)
        p->cells = (int)((rows > 1 ? rows : 1) * cols) + 2;
    }
}

// Tiles, workgroup and ownership of a call; false where no tile fits.
bool choose_gx(const Problem &q, int slices, int cus, GxGeo *p, GxTile *pick)
{
    const int halo = g_opt.halo ? g_opt.halo : kDefaultHaloGradX, max_halo = g_opt.halo ? halo : kMaxHaloGradX;
    // Twelve waves per compute unit either way, in one workgroup or, where that makes small tiles, in three, whose
    // flushes and tile switches overlap and whose waves get whole batches (14x14x512, 32 groups, batch 64, fp32: 106 us
    // in one, 59 in three; two of six waves do not fit a unit's SIMDs together: 28x28x256 fp16 115 -> 150)
    struct {
        int waves, per_cu;
    } shapes[3] = {{12, 1}, {4, 3}, {1, 12}};
    const int nshapes = g_opt.gx_threads ? 1 : 3;
    if (g_opt.gx_threads)
        shapes[0].waves = g_opt.gx_threads / 64;
    const long long planes = (long long)q.N * q.G * slices;
    const bool may_own = g_opt.gx_own == 0 && planes >= cus;
    GxTile any = {}, own = {};
    any.cost = own.cost = 1e30;
    for (int i = 0; i < nshapes; ++i) {
        // (one wave: maps of one or two batches, many of them)
        const bool one_wave = shapes[i].waves == 1;
        if (one_wave && (!may_own || (long long)q.Ho * q.Wo > 128))
            continue;
        const int lds = (g_opt.lds_kb ? g_opt.lds_kb * 1024 : kMaxLdsBytes) / shapes[i].per_cu & ~1023;
        choose_gx_tiles(q, shapes[i].waves, shapes[i].per_cu, halo, lds, slices, cus, one_wave ? nullptr : &any, may_own ? &own : nullptr);
    }
    if (any.waves == 0)
        return false;
    set_gx_tile(q, any, halo, max_halo, p);
    *pick = any;
    p->owned = 0;
    // An (image, channel run) to one workgroup, which then stores its sums instead of adding them atomically, where that is
    // faster in these tiles, or clearly so in others.
    if (g_opt.gx_own == 1) {
        p->owned = p->tiles_per_img;
    } else if (may_own) {
        auto now = [&](bool owned) { return gx_time(q, any.waves, any.per_cu, slices, cus, p->R, p->Q, p->tiles_per_img, p->cells, owned); };
        const double one_by_one = now(false), owned = now(true);
        if (own.cost < 0.85 * (owned < one_by_one ? owned : one_by_one)) {
            set_gx_tile(q, own, halo, max_halo, p);
            *pick = own;
            p->owned = p->tiles_per_img;
        } else if (owned < one_by_one) {
            p->owned = p->tiles_per_img;
        }
    }
    return true;
}

template <typename T>
int prepare_gx(const Problem &q, GxLaunch *out)
{
    if (q.Cg % kGxChan != 0 || q.softmax)
        return DCNV4_ERR_UNSUPPORTED;
    Geo base;
    int rc = make_geo(q, 1, &base);
    if (rc)
        return rc;
    const long long es = (long long)sizeof(T), pgi = (long long)q.Ho * q.Wo * q.G, lim24 = 1LL << 23;
    GxGeo p;
    memset(&p, 0, sizeof(p));
    p.og_bytes = (int)((q.merged ? 32 : 18) * es);
    p.mg_bytes = (int)((q.merged ? 32 : 9) * es);
    // 24-bit multiplications of pixel numbers, strides and positions
    if (pgi >= 0x1000000 || pgi * p.og_bytes >= (1LL << 31) || base.pix_bytes >= lim24 || q.Ho >= lim24 || q.Wo >= lim24 ||
        q.sh >= lim24 || q.sw >= lim24)
        return DCNV4_ERR_UNSUPPORTED;
    const int cus = device_cus();
    if (cus <= 0)
        return DCNV4_ERR_LAUNCH;
    p.slices = q.Cg / kGxChan;
    GxTile pick;
    if (!choose_gx(q, p.slices, cus, &p, &pick))
        return DCNV4_ERR_UNSUPPORTED;
    const long long planes = (long long)q.N * q.G * p.slices;
    // Its stores are the first ones where its bands leave no row or column of the image out; grad_x needs no clearing then
    // (103 MB of zeros: 16 us).
    const long long reach = 2LL * q.dh + p.halo + 2;
    p.fresh = p.owned != 0 && p.tiles_q == 1 && (q.Ho - 1LL) * q.sh - q.ph + reach >= q.H && (q.Wo - 1LL) * q.sw - q.pw + reach >= q.W &&
              q.sh <= reach + p.halo;
    const long long tiles = planes * p.tiles_per_img;
    if (tiles >= (1LL << 30))
        return DCNV4_ERR_UNSUPPORTED;
    const int slots = cus * pick.per_cu;
    const long long nblocks = p.owned ? planes : tiles;
    p.Wo = q.Wo; p.Ho = q.Ho; p.G = q.G; p.H = q.H; p.W = q.W;
    p.sh = q.sh; p.sw = q.sw; p.ph = q.ph; p.pw = q.pw; p.dh = q.dh; p.dw = q.dw;
    p.scale = q.scale;
    p.dmax = base.dmax;
    p.bound_bytes = (p.cells * 4 + kGxCell - 1) / kGxCell * kGxCell;
    p.quads_row = (p.Q + 3) / 4;
    p.div_quads = make_div((unsigned)p.quads_row);
    p.nblocks = (int)nblocks;
    p.blocks_per_xcd = (int)((nblocks + kXcds - 1) / kXcds);
    p.remap = g_opt.xcd_remap;
    p.div_g = make_div((unsigned)q.G);
    p.div_s = make_div((unsigned)p.slices);
    p.div_tpi = make_div((unsigned)p.tiles_per_img);
    p.div_tq = make_div((unsigned)p.tiles_q);
    p.div_pitch = make_div((unsigned)p.pitch);
    p.group_bytes = (int)(q.Cg * es);
    p.pix_bytes = base.pix_bytes;
    p.row_bytes = base.row_bytes;
    p.x_img_bytes = base.x_img_bytes;
    p.y_img_bytes = base.y_img_bytes;
    p.off_img_bytes = (int)(pgi * p.og_bytes);
    p.msk_img_bytes = (int)(pgi * p.mg_bytes);
    p.off_ext_bytes = (int)((pgi - 1) * p.og_bytes + 18 * es);
    p.msk_ext_bytes = (int)((pgi - 1) * p.mg_bytes + 9 * es);
    out->p = p;
    out->lds = p.bound_bytes + p.cells * kGxCell + 16;
    out->waves = pick.waves;
    static int granted[4][kMaxDevices];
    const void *kern = pick.waves == 12  ? reinterpret_cast<const void *>(dcnv4_gradx_kernel<T, 12>)
                       : pick.waves == 8 ? reinterpret_cast<const void *>(dcnv4_gradx_kernel<T, 8>)
                       : pick.waves == 4 ? reinterpret_cast<const void *>(dcnv4_gradx_kernel<T, 4>)
                                         : reinterpret_cast<const void *>(dcnv4_gradx_kernel<T, 1>);
    if (!grant_lds(kern, out->lds, granted[pick.waves / 4]))
        return DCNV4_ERR_LAUNCH;
    if (p.remap) {
        const int per = slots / kXcds < p.blocks_per_xcd ? slots / kXcds : p.blocks_per_xcd;
        out->grid = (unsigned)(per * kXcds);
    } else {
        out->grid = (unsigned)(slots < p.nblocks ? slots : p.nblocks);
    }
    return DCNV4_OK;
}

template <typename T>
int run_gx(const GxLaunch &l, const void *off, const void *msk, const void *gy, void *gx, hipStream_t s)
{
    auto kern = l.waves == 12  ? dcnv4_gradx_kernel<T, 12>
                : l.waves == 8 ? dcnv4_gradx_kernel<T, 8>
                : l.waves == 4 ? dcnv4_gradx_kernel<T, 4>
                               : dcnv4_gradx_kernel<T, 1>;
    hipLaunchKernelGGL(kern, dim3(l.grid), dim3((unsigned)l.waves * 64), l.lds, s, (const T *)off, (const T *)msk, (const T *)gy,
                       (T *)gx, l.p);
    const size_t had = strlen(g_last_kernel[1]);             // (the grad_offset/grad_mask pass, launched just before)
    snprintf(g_last_kernel[1] + had, sizeof(g_last_kernel[1]) - had, " + %sdcnv4_gradx_kernel<%s, %d>",
             l.p.fresh ? "(owned, uncleared) " : l.p.owned ? "(owned) " : "", sizeof(T) == 2 ? "_Float16" : "float", l.waves);
    return hipGetLastError() == hipSuccess ? DCNV4_OK : DCNV4_ERR_LAUNCH;
}

// Backward through the LDS-staged kernels: the grad_offset/grad_mask pass (gathers, like the forward;
// it clears grad_x on its way) and the grad_x pass (LDS-private accumulation, one flush per
// tile).  Both passes are prepared -- everything that can refuse -- before anything is launched,
// so a call that returns an error has written nothing.
template <typename T, int CG>
int launch_bwd_tiled(const void *x, const void *off, const void *msk, const void *gy, void *gx, void *go, void *gm,
                     const Problem &q, hipStream_t s)
{
    // the gather pass keeps 4*Cg inputs and gy per lane: eight waves fit the register file with pixels of up to
    // 32 bytes, four with 64-byte pixels
    constexpr int THREADS = CG * sizeof(T) >= 64 ? 256 : 512;
    // CG is the kernels' channel run; a wider group (q.Cg) goes through as q.Cg / CG slices whose
    // grad_offset/grad_mask parts are added up in zero-filled outputs
    const bool sliced = q.Cg != CG;
    // whole fp32 groups: the lanes read and write their own pixels' values, no LDS slices, eight waves
    bool gom_direct = false;
    if constexpr (sizeof(T) == 4)
        gom_direct = !sliced && g_opt.gom_coop == 0;
    // (for fp16 there is no other backward, so the tile-size heuristic does not apply)
    const bool any_size = g_opt.bwd_path == 2 || sizeof(T) == 2 || q.merged || q.softmax;
    // the grad_x pass: twelve waves keep the LDS busiest (measured)
    const int gxt = g_opt.gx_threads ? g_opt.gx_threads : 768;
    TiledLaunch l_gom, l_gx;
    // The grad_offset/grad_mask pass out of a rolling window of rows where that applies (whole groups), else out of
    // rectangles.  fp32 calls on two separate tensors: at stride 1 (58 calls at stride 2: 1.4 % slower on average, 18 of them by
    // 3 % or more), and those without a useful rectangle stay with the direct kernel all the same: its sums of grad_x are fp32
    // (4 images of 48x46, 4 groups, stride 2: error 7e-8 of grad_x, 2e-7 through the fixed-point sums).
    constexpr int kGomWaves = CG * sizeof(T) >= 32 ? 8 : 12;
    StripLaunch l_strip;
    // More images of one or two batches than compute units (those that no strip takes): one-wave workgroups, where one of eight
    // waves had work (64 x 7x7x1024 fp16, 64 groups: kernel 82 -> 20 us).
    bool one_wave = false;
    auto rectangles = [&]() {
        if constexpr (sizeof(T) == 2) {
            one_wave = g_opt.bwd_path == 0 && (long long)q.Ho * q.Wo <= 128 && (long long)q.N * q.G > device_cus() &&
                       prepare_tiled<T, CG, 64, kTiledGradOM>(q, true, 1, CG * sizeof(T) >= 64 ? 4 : 8, &l_gom) == DCNV4_OK &&
                       l_gom.p.tiles_per_img == 1;
            if (one_wave)
                return (int)DCNV4_OK;
        }
        if constexpr (sizeof(T) == 4) {
            if (gom_direct)
                return prepare_tiled<T, CG, 512, kTiledGradOMDirect>(q, any_size, 0, 0, &l_gom);
        }
        return prepare_tiled<T, CG, THREADS, kTiledGradOM>(q, any_size, 0, 0, &l_gom);
    };
    const bool free_choice = any_size || g_opt.fwd_strip == 1;
    int rc = free_choice ? DCNV4_ERR_UNSUPPORTED : rectangles();
    if (rc != DCNV4_OK && !free_choice)
        return rc;
    const bool strip = !sliced && !q.softmax && (free_choice || (q.sh == 1 && q.sw == 1)) && g_opt.bwd_path == 0 && g_opt.fwd_strip != 2 &&
                       g_opt.gom_coop == 0 &&
                       (q.merged ? prepare_strip<T, CG, kGomWaves, 2>(q, &l_strip) : prepare_strip<T, CG, kGomWaves, 1>(q, &l_strip)) == DCNV4_OK;
    if (!strip && free_choice)
        rc = rectangles();
    if (!strip && rc != DCNV4_OK)
        return rc;
    GxLaunch l_gx16;
    rc = prepare_gx<T>(q, &l_gx16);
    if (rc != DCNV4_OK && rc != DCNV4_ERR_UNSUPPORTED)
        return rc;
    // (groups of 8 channels and the softmax form stay with the accumulation by lanes = pixels)
    const bool use_gx16 = rc == DCNV4_OK;
    if (!use_gx16)
        rc = gxt == 768   ? prepare_tiled<T, CG, 768, kTiledGradX>(q, any_size, 0, 0, &l_gx)
             : gxt == 512 ? prepare_tiled<T, CG, 512, kTiledGradX>(q, any_size, 0, 0, &l_gx)
                          : prepare_tiled<T, CG, 256, kTiledGradX>(q, any_size, 0, 0, &l_gx);
    if (rc)
        return rc;
    auto zero = [&](void *ptr, long long bytes) {
        long long zb = (bytes / 16 + kThreads - 1) / kThreads;
        if (zb > 8192) zb = 8192;
        if (zb < 1) zb = 1;
        hipLaunchKernelGGL(dcnv4_zero_kernel, dim3((unsigned)zb), dim3(kThreads), 0, s, (u32x4 *)ptr, bytes);
    };
    // grad_x: by the grad_offset/grad_mask pass on the way, in whole 16-byte units (its pixels have 16 bytes or more);
    // 32-bit unit numbers
    const long long gx_bytes = (long long)q.N * q.H * q.W * q.G * q.Cg * (long long)sizeof(T), gx_units = gx_bytes / 16;
    const long long parts = strip ? (long long)l_strip.p.ntiles * l_strip.p.B : l_gom.p.nblocks, share = (gx_units + parts - 1) / parts;
    u32x4 *cleared = gx_units + share < (1LL << 31) && (parts + 1) * share < (1LL << 32) ? (u32x4 *)gx : nullptr;
    if (use_gx16 && l_gx16.p.fresh)
        cleared = nullptr;
    else if (cleared == nullptr)
        zero(gx, gx_bytes);
    if (strip) {
        l_strip.p.zero = cleared;
        l_strip.p.zero_units = (unsigned)gx_units;
        l_strip.p.zero_per_batch = (unsigned)share;
    } else {
        l_gom.p.zero = cleared;
        l_gom.p.zero_units = (unsigned)gx_units;
        l_gom.p.zero_per_tile = (unsigned)share;
    }
    const long long pairs = (long long)q.N * q.Ho * q.Wo * q.G * (long long)sizeof(T);
    if (q.merged && !strip) {                                   // (strips write whole records)
        zero(go, 32 * pairs);                                   // one buffer: gradients and padding
    } else if (sliced) {
        zero(go, 18 * pairs);
        zero(gm, 9 * pairs);
    }
    if (strip) {
        rc = q.merged ? run_strip<T, CG, kGomWaves, 2>(l_strip, x, off, msk, gy, go, gm, s)
                      : run_strip<T, CG, kGomWaves, 1>(l_strip, x, off, msk, gy, go, gm, s);
    } else if constexpr (sizeof(T) == 4) {
        rc = gom_direct ? run_tiled<T, CG, 512, kTiledGradOMDirect>(l_gom, x, off, msk, gy, go, gm, s, 1)
                        : run_tiled<T, CG, THREADS, kTiledGradOM>(l_gom, x, off, msk, gy, go, gm, s, 1);
    } else {
        rc = one_wave ? run_tiled<T, CG, 64, kTiledGradOM>(l_gom, x, off, msk, gy, go, gm, s, 1)
                      : run_tiled<T, CG, THREADS, kTiledGradOM>(l_gom, x, off, msk, gy, go, gm, s, 1);
    }
    if (rc == DCNV4_OK && use_gx16)
        return run_gx<T>(l_gx16, off, msk, gy, gx, s);
    if (rc == DCNV4_OK)
        rc = gxt == 768   ? run_tiled<T, CG, 768, kTiledGradX>(l_gx, x, off, msk, gy, gx, nullptr, s, 1)
             : gxt == 512 ? run_tiled<T, CG, 512, kTiledGradX>(l_gx, x, off, msk, gy, gx, nullptr, s, 1)
                          : run_tiled<T, CG, 256, kTiledGradX>(l_gx, x, off, msk, gy, gx, nullptr, s, 1);
    return rc;
}

int fill_problem(Problem *q, int N, int H, int W, int G, int Cg, int kh, int kw, int sh, int sw, int ph, int pw,
                 int dh, int dw, float scale, int dtype)
{
    q->N = N; q->H = H; q->W = W; q->G = G; q->Cg = Cg;
    q->kh = kh; q->kw = kw;
    q->sh = sh; q->sw = sw; q->ph = ph; q->pw = pw; q->dh = dh; q->dw = dw;
    q->scale = scale; q->dtype = dtype;
    q->merged = 0;
    q->softmax = 0;
    q->Ho = q->Wo = 0;
    if (H < 1 || W < 1 || kh < 1 || kw < 1 || sh < 1 || sw < 1 || ph < 0 || pw < 0 || dh < 1 || dw < 1)
        return DCNV4_ERR_SHAPE;
    return dcnv4_output_hw(H, W, kh, kw, sh, sw, ph, pw, dh, dw, &q->Ho, &q->Wo);
}

}  // namespace

namespace {

template <typename T, int WR, int WC, int WM, int WN, int STAGES> int launch_linear_tile(const void *x, const LinGeo &g, hipStream_t s)
{
    GemmGeo q;
    constexpr int RUN = 32 * WM, BN = WC * 32 * WN, STEP = sizeof(T) == 2 ? 128 : 64;
    q.lin = g;
    q.steps = (g.kbytes + STEP - 1) / STEP;
    q.runs0 = (g.seg[0].nout + RUN - 1) / RUN;
    q.runs = q.runs0 + (g.nseg > 1 ? (g.seg[1].nout + RUN - 1) / RUN : 0);
    q.out_tiles = (q.runs + WR - 1) / WR;
    q.tiles = q.out_tiles * ((g.P + BN - 1) / BN);
    q.tiles_per_xcd = (q.tiles + kXcds - 1) / kXcds;
    q.div_out = make_div((unsigned)q.out_tiles);
    hipLaunchKernelGGL((dcnv4_linear_tile_kernel<T, WR, WC, WM, WN, STAGES>), dim3((unsigned)(q.tiles_per_xcd * kXcds)), dim3(WR * WC * 64), 0, s,
                       (const T *)x, q);
    return hipGetLastError() == hipSuccess ? DCNV4_OK : DCNV4_ERR_LAUNCH;
}

template <typename T> int launch_linear_shape(int shape, const void *x, const LinGeo &g, hipStream_t s)
{
    constexpr bool f16 = sizeof(T) == 2;
    if (shape == kLinear64x64)
        return launch_linear_tile<T, 2, 2, 1, 1, 4>(x, g, s);
    if (shape == kLinear256x256)
        return launch_linear_tile<T, 4, 2, 2, 4, 2>(x, g, s);
    if constexpr (!f16)
        if (shape == kLinear128x256)
            return launch_linear_tile<T, 2, 4, 2, 2, 2>(x, g, s);
    return launch_linear_tile<T, 2, 2, 2, 2, 2>(x, g, s);
}

int pick_linear_tile(const LinGeo &g, int dtype)
{
    const int nout[kLinMaxSeg] = {g.seg[0].nout, g.nseg > 1 ? g.seg[1].nout : 0};
    return linear_tile_choice(g.P, g.kbytes, nout, g.nseg, dtype == DCNV4_F16, device_cus());
}

}  // namespace

extern "C" {

int dcnv4_output_hw(int H, int W, int kernel_h, int kernel_w, int stride_h, int stride_w, int pad_h, int pad_w,
                    int dil_h, int dil_w, int *H_out, int *W_out)
{
    if (!H_out || !W_out)
        return DCNV4_ERR_NULL;
    if (H < 1 || W < 1 || kernel_h < 1 || kernel_w < 1 || stride_h < 1 || stride_w < 1 || pad_h < 0 || pad_w < 0 ||
        dil_h < 1 || dil_w < 1)
        return DCNV4_ERR_SHAPE;
    const long long eh = (long long)H + 2LL * pad_h - (long long)dil_h * (kernel_h - 1) - 1;
    const long long ew = (long long)W + 2LL * pad_w - (long long)dil_w * (kernel_w - 1) - 1;
    if (eh < 0 || ew < 0)
        return DCNV4_ERR_SHAPE;
    *H_out = (int)(eh / stride_h + 1);
    *W_out = (int)(ew / stride_w + 1);
    return DCNV4_OK;
}

namespace {

int forward_impl(const void *x, const void *offset, const void *mask, void *y, int N, int H, int W, int G, int Cg,
                 int kernel_h, int kernel_w, int stride_h, int stride_w, int pad_h, int pad_w, int dil_h, int dil_w,
                 float offset_scale, int dtype, void *stream, bool merged, bool softmax = false)
{
    const void *ptrs[4] = {x, offset, y, mask};
    for (int i = 0; i < (merged ? 3 : 4); ++i)
        if (!ptrs[i])
            return DCNV4_ERR_NULL;
    Problem q;
    int rc = fill_problem(&q, N, H, W, G, Cg, kernel_h, kernel_w, stride_h, stride_w, pad_h, pad_w, dil_h, dil_w,
                          offset_scale, dtype);
    if (rc)
        return rc;
    rc = validate(q, kernel_h, kernel_w, ptrs, merged ? 3 : 4);
    if (rc)
        return rc;
    q.softmax = softmax;
    if (merged) {
        // the mask values follow the 18 offsets of their (pixel, group) in the same buffer
        q.merged = 1;
        mask = (const char *)offset + 18 * esize(dtype);
    }
    hipStream_t s = (hipStream_t)stream;
    return dtype == DCNV4_F16 ? dispatch_fwd<_Float16>(x, offset, mask, y, q, s)
                              : dispatch_fwd<float>(x, offset, mask, y, q, s);
}

int backward_impl(const void *x, const void *offset, const void *mask, const void *grad_y, void *grad_x,
                  void *grad_offset, void *grad_mask, int N, int H, int W, int G, int Cg, int kernel_h,
                  int kernel_w, int stride_h, int stride_w, int pad_h, int pad_w, int dil_h, int dil_w,
                  float offset_scale, int dtype, void *stream, bool merged, bool softmax = false)
{
    const void *ptrs[7] = {x, offset, grad_y, grad_x, grad_offset, mask, grad_mask};
    for (int i = 0; i < (merged ? 5 : 7); ++i)
        if (!ptrs[i])
            return DCNV4_ERR_NULL;
    Problem q;
    int rc = fill_problem(&q, N, H, W, G, Cg, kernel_h, kernel_w, stride_h, stride_w, pad_h, pad_w, dil_h, dil_w,
                          offset_scale, dtype);
    if (rc)
        return rc;
    rc = validate(q, kernel_h, kernel_w, ptrs, merged ? 5 : 7);
    if (rc)
        return rc;
    q.softmax = softmax;
    if (merged) {
        q.merged = 1;
        mask = (const char *)offset + 18 * esize(dtype);
        grad_mask = (char *)grad_offset + 18 * esize(dtype);
    }
    hipStream_t s = (hipStream_t)stream;
    if (kernel_h != 3) {
        // 1x1 and 5x5 windows: the direct fp32 kernel, one channel per lane (two for groups of 64)
        if (merged || softmax || dtype != DCNV4_F32 || g_opt.bwd_path == 2)
            return DCNV4_ERR_UNSUPPORTED;
        if (kernel_h == 1) {
            switch (Cg) {
            case 8: return launch_bwd<8, 1, 1>(x, offset, mask, grad_y, grad_x, grad_offset, grad_mask, q, s);
            case 16: return launch_bwd<16, 1, 1>(x, offset, mask, grad_y, grad_x, grad_offset, grad_mask, q, s);
            case 32: return launch_bwd<32, 1, 1>(x, offset, mask, grad_y, grad_x, grad_offset, grad_mask, q, s);
            case 64: return launch_bwd<64, 2, 1>(x, offset, mask, grad_y, grad_x, grad_offset, grad_mask, q, s);
            }
        } else {
            switch (Cg) {
            case 8: return launch_bwd<8, 1, 5>(x, offset, mask, grad_y, grad_x, grad_offset, grad_mask, q, s);
            case 16: return launch_bwd<16, 1, 5>(x, offset, mask, grad_y, grad_x, grad_offset, grad_mask, q, s);
            case 32: return launch_bwd<32, 1, 5>(x, offset, mask, grad_y, grad_x, grad_offset, grad_mask, q, s);
            case 64: return launch_bwd<64, 2, 5>(x, offset, mask, grad_y, grad_x, grad_offset, grad_mask, q, s);
            }
        }
        return DCNV4_ERR_UNSUPPORTED;
    }
    if (dtype == DCNV4_F16) {
        // fp16 storage, fp32 arithmetic; only the LDS-staged kernels exist for it (Cg 8, 16 or 32)
        if (g_opt.bwd_path == 1)
            return DCNV4_ERR_UNSUPPORTED;
        if (Cg == 8)
            return launch_bwd_tiled<_Float16, 8>(x, offset, mask, grad_y, grad_x, grad_offset, grad_mask, q, s);
        if (Cg == 16)
            return launch_bwd_tiled<_Float16, 16>(x, offset, mask, grad_y, grad_x, grad_offset, grad_mask, q, s);
        if (Cg == 32)                                  // 64-byte pixels, like fp32 groups of 16
            return launch_bwd_tiled<_Float16, 32>(x, offset, mask, grad_y, grad_x, grad_offset, grad_mask, q, s);
        return DCNV4_ERR_UNSUPPORTED;
    }
    if (g_opt.bwd_path != 1 || merged || softmax) {
        rc = DCNV4_ERR_UNSUPPORTED;
        if (Cg == 8)
            rc = launch_bwd_tiled<float, 8>(x, offset, mask, grad_y, grad_x, grad_offset, grad_mask, q, s);
        else if (Cg == 16 || Cg == 32 || Cg == 64)     // wider groups: 64-byte channel slices
            rc = launch_bwd_tiled<float, 16>(x, offset, mask, grad_y, grad_x, grad_offset, grad_mask, q, s);
        if (rc != DCNV4_ERR_UNSUPPORTED || g_opt.bwd_path == 2 || merged || softmax)
            return rc;
    }
    const int cpt = pick_bwd_cpt(Cg);
    switch (Cg) {
    case 8: return dispatch_bwd_cpt<8>(cpt, x, offset, mask, grad_y, grad_x, grad_offset, grad_mask, q, s);
    case 16: return dispatch_bwd_cpt<16>(cpt, x, offset, mask, grad_y, grad_x, grad_offset, grad_mask, q, s);
    case 32: return dispatch_bwd_cpt<32>(cpt, x, offset, mask, grad_y, grad_x, grad_offset, grad_mask, q, s);
    case 64: return dispatch_bwd_cpt<64>(cpt, x, offset, mask, grad_y, grad_x, grad_offset, grad_mask, q, s);
    }
    return DCNV4_ERR_UNSUPPORTED;
}

// ---- the module's linear layers ----------------------------------------------------------------
// One layer of the linear kernel's work list, checked: K * element size a multiple of 32 bytes (one
// MFMA group), nout a multiple of 32 (one MFMA block), 32-bit byte offsets inside every tensor.
int add_linear_segment(LinGeo *g, long long P, int K, int dtype, const void *w, const void *b, void *y, int nout,
                       int plane_shift = 0)
{
    if (!w || !y)
        return DCNV4_ERR_NULL;
    if (nout < 1)
        return DCNV4_ERR_SHAPE;
    const long long es = esize(dtype);
    if (nout % 32 || (long long)nout * K * es >= (1LL << 31) || P * nout * es >= (1LL << 31) || g->nseg >= kLinMaxSeg)
        return DCNV4_ERR_UNSUPPORTED;
    if ((reinterpret_cast<uintptr_t>(w) & 15u) || (reinterpret_cast<uintptr_t>(y) & 15u) ||
        (reinterpret_cast<uintptr_t>(b) & (uintptr_t)(es - 1)))
        return DCNV4_ERR_ALIGN;
    LinSeg &sg = g->seg[g->nseg++];
    sg.w = w; sg.b = b; sg.y = y; sg.nout = nout;
    sg.plane_shift = plane_shift;
    sg.nblocks = (nout + kLinBlock - 1) / kLinBlock;
    return DCNV4_OK;
}

int begin_linear(LinGeo *g, const void *x, long long P, int K, int dtype)
{
    memset(g, 0, sizeof(*g));
    if (!x)
        return DCNV4_ERR_NULL;
    if (P < 1 || K < 1)
        return DCNV4_ERR_SHAPE;
    if (dtype != DCNV4_F32 && dtype != DCNV4_F16)
        return DCNV4_ERR_UNSUPPORTED;
    const long long kbytes = (long long)K * esize(dtype);
    if (kbytes % 32 || P * kbytes >= (1LL << 31))
        return DCNV4_ERR_UNSUPPORTED;
    if (reinterpret_cast<uintptr_t>(x) & 15u)
        return DCNV4_ERR_ALIGN;
    g->P = (int)P;
    g->kbytes = (int)kbytes;
    return DCNV4_OK;
}

int launch_linear(const void *x, const LinGeo &g, int dtype, hipStream_t s)
{
    const int shape = g_opt.linear_tile != 0 ? linear_tile_asked(g_opt.linear_tile, g.kbytes, dtype == DCNV4_F16) : pick_linear_tile(g, dtype);
    if (shape != kLinearInOneChunk)
        return dtype == DCNV4_F16 ? launch_linear_shape<_Float16>(shape, x, g, s) : launch_linear_shape<float>(shape, x, g, s);
    const int tiles = (g.P + kLinPixels - 1) / kLinPixels;
    // maps of few pixels and many channels: the passes over blocks of output channels are spread over
    // workgroups as well, until there are about two workgroups per compute unit
    int npass = 0;
    for (int i = 0; i < g.nseg; ++i)
        npass += g.seg[i].nblocks;
    const int want = 2 * device_cus();
    int split = (want + tiles - 1) / tiles;
    if (split > npass) split = npass;
    if (split < 1) split = 1;
    hipLaunchKernelGGL(dcnv4_linear_kernel, dim3((unsigned)tiles, (unsigned)split), dim3(256), 0, s, (const _Float16 *)x, g);
    return hipGetLastError() == hipSuccess ? DCNV4_OK : DCNV4_ERR_LAUNCH;
}

int launch_depthwise(const void *x, const void *w, const void *b, void *y, int N, int H, int W, int C, int dtype,
                     hipStream_t s)
{
    if (!x || !w || !y)
        return DCNV4_ERR_NULL;
    if (N < 1 || H < 1 || W < 1 || C < 1)
        return DCNV4_ERR_SHAPE;
    if (dtype != DCNV4_F32 && dtype != DCNV4_F16)
        return DCNV4_ERR_UNSUPPORTED;
    const long long es = esize(dtype), pix_bytes = (long long)C * es;
    const long long bytes = (long long)N * H * W * pix_bytes;
    if (pix_bytes % 16 || bytes >= (1LL << 31))
        return DCNV4_ERR_UNSUPPORTED;
    if ((reinterpret_cast<uintptr_t>(x) & 15u) || (reinterpret_cast<uintptr_t>(w) & 15u) ||
        (reinterpret_cast<uintptr_t>(y) & 15u) || (reinterpret_cast<uintptr_t>(b) & 15u))
        return DCNV4_ERR_ALIGN;
    DwGeo g;
    g.H = H; g.W = W;
    g.units = (int)(pix_bytes / 16);
    g.total = (int)(bytes / 16);
    g.row_bytes = (int)(W * pix_bytes);
    g.pix_bytes = (int)pix_bytes;
    g.div_units = make_div((unsigned)g.units);
    g.div_w = make_div((unsigned)W);
    g.div_h = make_div((unsigned)H);
    const unsigned grid = (unsigned)((g.total + 255) / 256);
    if (dtype == DCNV4_F16)
        hipLaunchKernelGGL(dcnv4_depthwise3x3_kernel<_Float16>, dim3(grid), dim3(256), 0, s, (const _Float16 *)x,
                           (const _Float16 *)w, (const _Float16 *)b, (_Float16 *)y, g);
    else
        hipLaunchKernelGGL(dcnv4_depthwise3x3_kernel<float>, dim3(grid), dim3(256), 0, s, (const float *)x,
                           (const float *)w, (const float *)b, (float *)y, g);
    return hipGetLastError() == hipSuccess ? DCNV4_OK : DCNV4_ERR_LAUNCH;
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

}  // namespace

int dcnv4_forward(const void *x, const void *offset, const void *mask, void *y, int N, int H, int W, int G, int Cg,
                  int kernel_h, int kernel_w, int stride_h, int stride_w, int pad_h, int pad_w, int dil_h, int dil_w,
                  float offset_scale, int dtype, void *stream)
{
    return forward_impl(x, offset, mask, y, N, H, W, G, Cg, kernel_h, kernel_w, stride_h, stride_w, pad_h, pad_w, dil_h,
                        dil_w, offset_scale, dtype, stream, false);
}

int dcnv4_forward_merged(const void *x, const void *offset_mask, void *y, int N, int H, int W, int G, int Cg,
                         int kernel_h, int kernel_w, int stride_h, int stride_w, int pad_h, int pad_w, int dil_h,
                         int dil_w, float offset_scale, int dtype, void *stream)
{
    return forward_impl(x, offset_mask, nullptr, y, N, H, W, G, Cg, kernel_h, kernel_w, stride_h, stride_w, pad_h, pad_w,
                        dil_h, dil_w, offset_scale, dtype, stream, true);
}

int dcnv4_backward(const void *x, const void *offset, const void *mask, const void *grad_y, void *grad_x,
                   void *grad_offset, void *grad_mask, int N, int H, int W, int G, int Cg, int kernel_h,
                   int kernel_w, int stride_h, int stride_w, int pad_h, int pad_w, int dil_h, int dil_w,
                   float offset_scale, int dtype, void *stream)
{
    return backward_impl(x, offset, mask, grad_y, grad_x, grad_offset, grad_mask, N, H, W, G, Cg, kernel_h, kernel_w,
                         stride_h, stride_w, pad_h, pad_w, dil_h, dil_w, offset_scale, dtype, stream, false);
}

int dcnv4_forward_softmax(const void *x, const void *offset, const void *mask_logits, void *y, int N, int H, int W,
                          int G, int Cg, int kernel_h, int kernel_w, int stride_h, int stride_w, int pad_h, int pad_w,
                          int dil_h, int dil_w, float offset_scale, int dtype, void *stream)
{
    return forward_impl(x, offset, mask_logits, y, N, H, W, G, Cg, kernel_h, kernel_w, stride_h, stride_w, pad_h, pad_w,
                        dil_h, dil_w, offset_scale, dtype, stream, false, true);
}

int dcnv4_backward_softmax(const void *x, const void *offset, const void *mask_logits, const void *grad_y,
                           void *grad_x, void *grad_offset, void *grad_mask_logits, int N, int H, int W, int G,
                           int Cg, int kernel_h, int kernel_w, int stride_h, int stride_w, int pad_h, int pad_w,
                           int dil_h, int dil_w, float offset_scale, int dtype, void *stream)
{
    return backward_impl(x, offset, mask_logits, grad_y, grad_x, grad_offset, grad_mask_logits, N, H, W, G, Cg, kernel_h,
                         kernel_w, stride_h, stride_w, pad_h, pad_w, dil_h, dil_w, offset_scale, dtype, stream, false,
                         true);
}

int dcnv4_backward_merged(const void *x, const void *offset_mask, const void *grad_y, void *grad_x,
                          void *grad_offset_mask, int N, int H, int W, int G, int Cg, int kernel_h, int kernel_w,
                          int stride_h, int stride_w, int pad_h, int pad_w, int dil_h, int dil_w, float offset_scale,
                          int dtype, void *stream)
{
    return backward_impl(x, offset_mask, nullptr, grad_y, grad_x, grad_offset_mask, nullptr, N, H, W, G, Cg, kernel_h,
                         kernel_w, stride_h, stride_w, pad_h, pad_w, dil_h, dil_w, offset_scale, dtype, stream, true);
}

long long dcnv4_forward_algorithmic_bytes(int N, int H, int W, int G, int Cg, int H_out, int W_out, int dtype)
{
    const long long es = esize(dtype), C = (long long)G * Cg;
    const long long P = (long long)N * H_out * W_out;
    return es * ((long long)N * H * W * C + P * C + P * G * 27);
}

long long dcnv4_backward_algorithmic_bytes(int N, int H, int W, int G, int Cg, int H_out, int W_out, int dtype)
{
    const long long es = esize(dtype), C = (long long)G * Cg;
    const long long P = (long long)N * H_out * W_out;
    return es * (2 * (long long)N * H * W * C + P * C + 2 * P * G * 27);
}

long long dcnv4_forward_merged_algorithmic_bytes(int N, int H, int W, int G, int Cg, int H_out, int W_out, int dtype)
{
    const long long es = esize(dtype), C = (long long)G * Cg;
    const long long P = (long long)N * H_out * W_out;
    return es * ((long long)N * H * W * C + P * C + P * G * 32);
}

long long dcnv4_backward_merged_algorithmic_bytes(int N, int H, int W, int G, int Cg, int H_out, int W_out, int dtype)
{
    const long long es = esize(dtype), C = (long long)G * Cg;
    const long long P = (long long)N * H_out * W_out;
    return es * (2 * (long long)N * H * W * C + P * C + 2 * P * G * 32);
}

int dcnv4_linear(const void *x, const void *w, const void *b, void *y, long long P, int K, int Nout, int dtype,
                 void *stream)
{
    LinGeo g;
    int rc = begin_linear(&g, x, P, K, dtype);
    if (rc)
        return rc;
    rc = add_linear_segment(&g, P, K, dtype, w, b, y, Nout);
    if (rc)
        return rc;
    return launch_linear(x, g, dtype, (hipStream_t)stream);
}

int dcnv4_depthwise3x3(const void *x, const void *w, const void *b, void *y, int N, int H, int W, int C, int dtype,
                       void *stream)
{
    return launch_depthwise(x, w, b, y, N, H, W, C, dtype, (hipStream_t)stream);
}

long long dcnv4_module_workspace_bytes(int N, int H, int W, int G, int Cg, int dtype, int lightweight, int depthwise)
{
    if (N < 1 || H < 1 || W < 1 || G < 1 || Cg < 1 || (dtype != DCNV4_F32 && dtype != DCNV4_F16))
        return -1;
    const long long P = (long long)N * H * W, es = esize(dtype), C = (long long)G * Cg;
    const long long om = (long long)align256((size_t)(P * G * 32 * es)), act = (long long)align256((size_t)(P * C * es));
    return om + (lightweight ? 0 : 2 * act) + (depthwise ? act : 0);
}

namespace {

// Built-in workspace of dcnv4_module_forward_static: one copy per GPU, held until the process ends.
constexpr long long kScratchBytes = 32ll << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

// Device address of `scratch` on the current device (the array's name is only a host-side stand-in:
// every GPU has its own copy at its own address), looked up once per device; null on failure.
void *scratch_address()
{
    static void *ptr[kMaxDevices];
    const int dev = current_device();
    if (dev < 0)
        return nullptr;
    if (!ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess)
            return nullptr;
        ptr[dev] = p;
    }
    return ptr[dev];
}

int module_forward_impl(const void *x, const void *w_in, const void *b_in, const void *w_dw, const void *b_dw,
                        const void *w_om, const void *b_om, const void *w_out, const void *b_out, void *workspace,
                        long long workspace_bytes, void *y, int N, int H, int W, int G, int Cg, int kernel_h,
                        int kernel_w, int stride_h, int stride_w, int pad_h, int pad_w, int dil_h, int dil_w,
                        float offset_scale, int dtype, void *stream)
{
    if (!x || !w_om || !workspace || !y)
        return DCNV4_ERR_NULL;
    if ((w_in == nullptr) != (w_out == nullptr))        // the two projections come together (or not at all)
        return DCNV4_ERR_NULL;
    const bool light = w_in == nullptr, dw = w_dw != nullptr;
    Problem q;
    int rc = fill_problem(&q, N, H, W, G, Cg, kernel_h, kernel_w, stride_h, stride_w, pad_h, pad_w, dil_h, dil_w,
                          offset_scale, dtype);
    if (rc)
        return rc;
    const void *ptrs[3] = {x, workspace, y};
    rc = validate(q, kernel_h, kernel_w, ptrs, 3);
    if (rc)
        return rc;
    // the merged layer predicts one set of offsets per INPUT pixel: the window must keep the map's size
    if (q.Ho != H || q.Wo != W || kernel_h != 3)
        return DCNV4_ERR_UNSUPPORTED;
    const long long need = dcnv4_module_workspace_bytes(N, H, W, G, Cg, dtype, light ? 1 : 0, dw ? 1 : 0);
    if (workspace_bytes < need)
        return DCNV4_ERR_SHAPE;
    const long long P = (long long)N * H * W, es = esize(dtype);
    const int C = G * Cg;
    const size_t act = align256((size_t)(P * C * es));
    char *om = (char *)workspace;
    char *next = om + align256((size_t)(P * G * 32 * es));
    char *value = nullptr, *y_op = nullptr, *x_dw = nullptr;
    if (!light) {
        value = next;
        y_op = next + act;
        next += 2 * act;
    }
    if (dw)
        x_dw = next;
    // Between its layers the full module keeps value, offsets/scalars and the operator's output plane-major,
    // [image][group][pixel][channels of the group]: the operator then sees N*G images of ONE group whose
    // pixels are whole, contiguous pieces (a workgroup of its kernels reads full cache lines instead of a
    // quarter of each), and the linear layers write and read 1 KB runs.  (Not the lightweight variant, whose
    // value tensor is the caller's channel-last x; not groups whose bytes are no power of two in 32..128.)
    int vshift = 0;
    for (int sft = 5; sft <= 7; ++sft)
        if ((long long)Cg * es == (1LL << sft))
            vshift = sft;
    const bool planar = !light && vshift != 0 && g_opt.module_rows == 0;
    const int oshift = planar ? (es == 2 ? 6 : 7) : 0;            // 32 entries per (pixel, group)
    if (!planar)
        vshift = 0;
    // Everything that can refuse is checked before the first launch.  Without the depthwise convolution
    // both layers that read x are one launch; with it the offset/scalar layer reads the convolved map.
    LinGeo first, second, last;
    const bool fused = !dw && !light;
    rc = begin_linear(&first, x, P, C, dtype);
    if (!rc && !light)
        rc = add_linear_segment(&first, P, C, dtype, w_in, b_in, value, C, vshift);
    if (!rc && (fused || light) && !dw)
        rc = add_linear_segment(&first, P, C, dtype, w_om, b_om, om, G * 32, oshift);
    first.hw = H * W;
    first.div_hw = make_div((unsigned)(H * W));
    if (!rc && dw) {
        rc = begin_linear(&second, x_dw, P, C, dtype);
        if (!rc)
            rc = add_linear_segment(&second, P, C, dtype, w_om, b_om, om, G * 32, oshift);
        second.hw = H * W;
        second.div_hw = make_div((unsigned)(H * W));
        if (!rc && ((reinterpret_cast<uintptr_t>(w_dw) & 15u) || (reinterpret_cast<uintptr_t>(b_dw) & 15u)))
            rc = DCNV4_ERR_ALIGN;
        if (!rc && (P * C * es >= (1LL << 31) || (C * es) % 16))
            rc = DCNV4_ERR_UNSUPPORTED;
    }
    if (!rc && !light) {
        rc = begin_linear(&last, y_op, P, C, dtype);
        if (!rc)
            rc = add_linear_segment(&last, P, C, dtype, w_out, b_out, y, C);
        last.hw = H * W;
        last.div_hw = make_div((unsigned)(H * W));
        last.in_plane_shift = vshift;
    }
    if (rc)
        return rc;
    hipStream_t s = (hipStream_t)stream;
    if (first.nseg > 0) {
        rc = launch_linear(x, first, dtype, s);
        if (rc)
            return rc;
    }
    if (dw) {
        rc = launch_depthwise(x, w_dw, b_dw, x_dw, N, H, W, C, dtype, s);
        if (rc)
            return rc;
        rc = launch_linear(x_dw, second, dtype, s);
        if (rc)
            return rc;
    }
    if (planar)
        rc = forward_impl(value, om, nullptr, y_op, N * G, H, W, 1, Cg, kernel_h, kernel_w, stride_h, stride_w, pad_h, pad_w,
                          dil_h, dil_w, offset_scale, dtype, stream, true);
    else
        rc = forward_impl(light ? x : (const void *)value, om, nullptr, light ? y : (void *)y_op, N, H, W, G, Cg, kernel_h,
                          kernel_w, stride_h, stride_w, pad_h, pad_w, dil_h, dil_w, offset_scale, dtype, stream, true);
    if (rc || light)
        return rc;
    return launch_linear(y_op, last, dtype, s);
}

}  // namespace

int dcnv4_module_forward(const void *x, const void *w_in, const void *b_in, const void *w_dw, const void *b_dw,
                         const void *w_om, const void *b_om, const void *w_out, const void *b_out, void *workspace,
                         long long workspace_bytes, void *y, int N, int H, int W, int G, int Cg, int kernel_h,
                         int kernel_w, int stride_h, int stride_w, int pad_h, int pad_w, int dil_h, int dil_w,
                         float offset_scale, int dtype, void *stream)
{
    return module_forward_impl(x, w_in, b_in, w_dw, b_dw, w_om, b_om, w_out, b_out, workspace, workspace_bytes, y, N, H, W,
                               G, Cg, kernel_h, kernel_w, stride_h, stride_w, pad_h, pad_w, dil_h, dil_w, offset_scale,
                               dtype, stream);
}

long long dcnv4_module_static_workspace_limit(void) { return kScratchBytes; }

int dcnv4_module_forward_static(const void *x, const void *w_in, const void *b_in, const void *w_dw, const void *b_dw,
                                const void *w_om, const void *b_om, const void *w_out, const void *b_out, void *y,
                                int N, int H, int W, int G, int Cg, int kernel_h, int kernel_w, int stride_h,
                                int stride_w, int pad_h, int pad_w, int dil_h, int dil_w, float offset_scale, int dtype,
                                void *stream)
{
    if (!x || !w_om || !y)
        return DCNV4_ERR_NULL;
    if ((w_in == nullptr) != (w_out == nullptr))
        return DCNV4_ERR_NULL;
    const long long need = dcnv4_module_workspace_bytes(N, H, W, G, Cg, dtype, w_in == nullptr, w_dw != nullptr);
    if (need < 0)
        return (dtype != DCNV4_F32 && dtype != DCNV4_F16) ? DCNV4_ERR_UNSUPPORTED : DCNV4_ERR_SHAPE;
    if (need > kScratchBytes)
        return DCNV4_ERR_TOO_LARGE;
    void *ws = scratch_address();
    if (!ws)
        return DCNV4_ERR_LAUNCH;
    return module_forward_impl(x, w_in, b_in, w_dw, b_dw, w_om, b_om, w_out, b_out, ws, kScratchBytes, y, N, H, W, G, Cg,
                               kernel_h, kernel_w, stride_h, stride_w, pad_h, pad_w, dil_h, dil_w, offset_scale, dtype,
                               stream);
}

int dcnv4_set_option(const char *key, int value)
{
    if (!key)
        return DCNV4_ERR_NULL;
    if (!strcmp(key, "reset")) {             // every switch back to the library's own choice
        g_opt = Options();
        return DCNV4_OK;
    }
    if (!strcmp(key, "fwd_cpt") && (value == 0 || value == 8 || value == 16)) {
        g_opt.fwd_cpt = value;
        return DCNV4_OK;
    }
    if (!strcmp(key, "bwd_cpt") && (value == 0 || value == 1 || value == 2 || value == 4 || value == 8 || value == 16)) {
        g_opt.bwd_cpt = value;
        return DCNV4_OK;
    }
    if (!strcmp(key, "xcd_remap") && (value == 0 || value == 1)) {
        g_opt.xcd_remap = value;
        return DCNV4_OK;
    }
    if (!strcmp(key, "fwd_path") && value >= 0 && value <= 3) {
        g_opt.fwd_path = value;
        return DCNV4_OK;
    }
    if (!strcmp(key, "fwd_strip") && value >= 0 && value <= 2) {
        g_opt.fwd_strip = value;
        return DCNV4_OK;
    }
    if (!strcmp(key, "gx_threads") && (value == 0 || value == 256 || value == 512 || value == 768)) {
        g_opt.gx_threads = value;
        return DCNV4_OK;
    }
    if (!strcmp(key, "gx_own") && value >= 0 && value <= 2) {
        g_opt.gx_own = value;
        return DCNV4_OK;
    }
    if (!strcmp(key, "fwd_single") && value >= 0 && value <= 2) {
        g_opt.fwd_single = value;
        return DCNV4_OK;
    }
    if (!strcmp(key, "linear_tile") && value >= 0 && value <= 5) {
        g_opt.linear_tile = value;
        return DCNV4_OK;
    }
    if (!strcmp(key, "module_rows") && (value == 0 || value == 1)) {
        g_opt.module_rows = value;
        return DCNV4_OK;
    }
    if (!strcmp(key, "gom_coop") && (value == 0 || value == 1)) {
        g_opt.gom_coop = value;
        return DCNV4_OK;
    }
    if (!strcmp(key, "wg_per_cu") && value >= 0 && value <= 32) {
        g_opt.wg_per_cu = value;
        return DCNV4_OK;
    }
    if (!strcmp(key, "bwd_path") && value >= 0 && value <= 2) {
        g_opt.bwd_path = value;
        return DCNV4_OK;
    }
    if (!strcmp(key, "halo") && value >= 0 && value <= 64) {
        g_opt.halo = value;
        return DCNV4_OK;
    }
    if (!strcmp(key, "lds_kb") && (value == 0 || (value >= 8 && value <= 160))) {
        g_opt.lds_kb = value;
        return DCNV4_OK;
    }
    if (!strcmp(key, "fwd_threads") && (value == 0 || value == 64 || value == 128 || value == 256 || value == 512 || value == 640 || value == 768)) {
        g_opt.fwd_threads = value;
        return DCNV4_OK;
    }
    return DCNV4_ERR_UNSUPPORTED;
}

const char *dcnv4_last_kernel_name(int backward)
{
    const char *n = g_last_kernel[backward ? 1 : 0];
    return n[0] ? n : nullptr;
}

const char *dcnv4_status_string(int status)
{
    switch (status) {
    case DCNV4_OK: return "ok";
    case DCNV4_ERR_NULL: return "null pointer";
    case DCNV4_ERR_SHAPE: return "bad shape: a size is non-positive or the window does not fit";
    case DCNV4_ERR_UNSUPPORTED: return "unsupported kernel size, group width, dtype, option or tensor size";
    case DCNV4_ERR_ALIGN: return "tensor pointer not 16-byte aligned";
    case DCNV4_ERR_LAUNCH: return "HIP launch failed";
    case DCNV4_ERR_TOO_LARGE: return "the call needs more workspace than the built-in scratch buffer holds";
    }
    return "unknown status";
}

}  // extern "C"
