// fp16 / bf16 windowed convolution for small grids (Sec. III-C, III-D): few
// output pixels, long windows (single images and small batches).
//
// What bounds such a layer is not a rate but the length of one workgroup:
// with 64 x 128 tiles a 14 x 14 layer with 256 channels is eight workgroups
// that each walk the whole window.  Here a tile is small (32 or 64 channels x
// 16 to 64 pixels) and the waves of a workgroup split the window's taps:
// wave w takes the 32-tap steps w, w + NW, w + 2*NW, ..., with no barrier
// between them, and the waves' fp32 sums are added through LDS at the end in
// wave order (a fixed order, so results are reproducible).
//
// Operands go from global memory straight to registers, in the lane layout
// of v_mfma_f32_16x16x32 (lane l: row or column l % 16, taps 8*(l/16) .. +7):
//   * windows: one 16-byte load per lane and 16 pixels, aligned or not;
//   * filter: read from the caller's [K_h][K_w][C_i][C_o] filter, which saves
//     the pack (a launch of 4-8 us, as long as the convolution itself here).
//     A lane reads F consecutive channels of each of its 8 taps and
//     transposes them in registers: lane row m of matrix i is channel F*m+i,
//     so each lane ends with 4*F consecutive output channels.
// Taps past K (the last step) are cleared in both operands, so a value of
// the next window that is not finite never meets a product.
#include "common.hpp"
#include "mfma16.hpp"

#include <string.h>

namespace im2win {
namespace {

struct DirArgs {
    const uint16_t *ws;    // window tensor
    const uint16_t *filt;  // the caller's filter, window tap k at row (u*K_w + v)*C_i + r
    uint16_t *out;
    uint32_t P, K, Co, Wo, L, Ci, Kh, Kw;
    WinCols wc;
    TileGrid tg;
    uint32_t swap;         // tg.x counts channel tiles, tg.y pixel tiles
    FastDiv div_Wo, div_khci, div_ci;
};

template <int F_, int NB_, int NW_, int U_>
struct DirCfg {
    static constexpr int F = F_;    // channels per lane (2 or 4)
    static constexpr int NB = NB_;  // 16-pixel blocks per tile
    static constexpr int NW = NW_;  // waves, each a share of the taps
    static constexpr int U = U_;    // steps per batch; two batches in flight
    static constexpr int NT = 64 * NW;
    static constexpr int BM = 16 * F, BN = 16 * NB;
    static constexpr int ITEMS = NB * F * 64;  // 4-channel pieces of the output tile
    static_assert(F == 2 || F == 4, "4- or 8-byte filter loads");
    static_assert(NW * ITEMS * 16 <= 160 * 1024, "the waves' sums fit in LDS");
};

// One step (32 taps) of a wave: the lane's 8 taps of F channels (tap e in
// dwords e*F/2 ..) and of NB pixels.
template <class C>
struct DirStep {
    uint32_t x[8 * C::F / 2];
    u32x4 w[C::NB];
};

// AL8: C_i is a multiple of 8, so the 8 taps of a lane are consecutive rows
// of the filter and windows start on 16-byte boundaries.
template <class C, class E, bool AL8>
struct DirWave {
    typedef typename E::v8 v8;
    const char *wsb, *fb;
    uint32_t woff[C::NB];  // byte offset of each pixel's window
    uint32_t cofs, cshift; // byte offset of the lane's channels in a filter row, shift of an odd last channel
    uint32_t g, nst;
    f32x4_acc acc[C::F][C::NB];

    __device__ inline uint32_t filter_row(uint32_t k, const DirArgs &a, uint32_t &v, uint32_t &u, uint32_t &r) const
    {
        v = fdiv(k, a.div_khci);
        const uint32_t rem = k - v * (a.Kh * a.Ci);
        u = fdiv(rem, a.div_ci);
        r = rem - u * a.Ci;
        return (u * a.Kw + v) * a.Ci + r;
    }

    __device__ inline void ld_filter(uint32_t *x, uint32_t row, const DirArgs &a) const
    {
        const char *src = fb + (row * a.Co * 2u + cofs);
        __builtin_memcpy(x, src, 2 * C::F);
    }

    __device__ inline void load(DirStep<C> &s, uint32_t st, const DirArgs &a) const
    {
        const uint32_t kg = st * 32 + 8 * g;
#pragma unroll
        for (int j = 0; j < C::NB; ++j) {
            // taps past K: at most 62 bytes past the window, inside the pad
            const char *src = wsb + (woff[j] + 2u * kg);
            if (AL8)
                s.w[j] = *reinterpret_cast<const u32x4 *>(src);
            else
                __builtin_memcpy(&s.w[j], src, 16);
        }
        uint32_t v, u, r;
        if (AL8) {
            const uint32_t row = filter_row(kg < a.K ? kg : a.K - 8, a, v, u, r);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                ld_filter(&s.x[e * C::F / 2], row + e, a);
        } else {
            uint32_t k = kg < a.K ? kg : a.K - 1;
            uint32_t row = filter_row(k, a, v, u, r);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                ld_filter(&s.x[e * C::F / 2], row, a);
                if (k + 1 < a.K) {  // taps past K re-read the last row
                    ++k;
                    ++row;
                    if (++r == a.Ci) {
                        r = 0;
                        row += (a.Kw - 1) * a.Ci;
                        if (++u == a.Kh) {
                            u = 0;
                            ++v;
                            row = v * a.Ci;
                        }
                    }
                }
            }
        }
    }

    __device__ inline void compute(DirStep<C> &s, uint32_t st, const DirArgs &a)
    {
        if (st * 32 + 32 > a.K) {  // the last step: clear the taps past K
            const uint32_t kg = st * 32 + 8 * g;
            const uint32_t n = kg < a.K ? a.K - kg : 0u;
#pragma unroll
            for (uint32_t e = 0; e < 8; ++e)
#pragma unroll
                for (int d = 0; d < C::F / 2; ++d)
                    s.x[e * C::F / 2 + d] = e < n ? s.x[e * C::F / 2 + d] : 0u;
#pragma unroll
            for (int j = 0; j < C::NB; ++j)
#pragma unroll
                for (uint32_t d = 0; d < 4; ++d)
                    s.w[j][d] &= (2 * d < n ? 0xffffu : 0u) | (2 * d + 1 < n ? 0xffff0000u : 0u);
        }
        v8 af[C::F];
#pragma unroll
        for (int i = 0; i < C::F; ++i) {
            u32x4 t;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                uint32_t lo = s.x[(2 * d) * C::F / 2 + i / 2], hi = s.x[(2 * d + 1) * C::F / 2 + i / 2];
                if (C::F == 2) {
                    lo >>= cshift;
                    hi >>= cshift;
                }
                t[d] = __builtin_amdgcn_perm(hi, lo, i % 2 ? 0x07060302u : 0x05040100u);
            }
            af[i] = __builtin_bit_cast(v8, t);
        }
#pragma unroll
        for (int j = 0; j < C::NB; ++j) {
            const v8 bf = __builtin_bit_cast(v8, s.w[j]);
#pragma unroll
            for (int i = 0; i < C::F; ++i)
                acc[i][j] = E::mfma16(af[i], bf, acc[i][j]);
        }
    }

    __device__ inline void load_batch(DirStep<C> (&b)[C::U], uint32_t st, const DirArgs &a) const
    {
#pragma unroll
        for (int t = 0; t < C::U; ++t)
            if (st + C::NW * t < nst)
                load(b[t], st + C::NW * t, a);
    }

    __device__ inline void compute_batch(DirStep<C> (&b)[C::U], uint32_t st, const DirArgs &a)
    {
#pragma unroll
        for (int t = 0; t < C::U; ++t)
            if (st + C::NW * t < nst)
                compute(b[t], st + C::NW * t, a);
    }
};

template <class C, class E, bool AL8>
__global__ __launch_bounds__(C::NT) void conv_fp16_direct(DirArgs a)
{
    __shared__ __attribute__((aligned(16))) float4 part[C::NW][C::NB * C::F][64];

    DirWave<C, E, AL8> w;
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t tx, ty;
    a.tg.tile(tx, ty);
    const uint32_t p0 = (a.swap ? ty : tx) * C::BN, ch0 = (a.swap ? tx : ty) * C::BM;
    const uint32_t q0 = fdiv(p0, a.div_Wo);
    const uint32_t c16 = lane & 15;
    w.wsb = reinterpret_cast<const char *>(a.ws + (uint64_t)q0 * a.L);
    w.fb = reinterpret_cast<const char *>(a.filt);
    w.g = lane >> 4;
    w.nst = (a.K + 31) / 32;
#pragma unroll
    for (int j = 0; j < C::NB; ++j) {
        // a pixel past the last one repeats it (its sums are not stored)
        const uint32_t p = p0 + 16 * j + c16 < a.P ? p0 + 16 * j + c16 : a.P - 1;
        const uint32_t q = fdiv(p, a.div_Wo);
        w.woff[j] = ((q - q0) * a.L + a.wc.start(p - q * a.Wo)) * 2u;
    }
    // Channels past C_o read the row's last F (their sums are not stored);
    // with an odd C_o the last channel is the upper half of that read.
    const uint32_t ch = ch0 + C::F * c16, last = a.Co - C::F;
    w.cofs = (ch < last ? ch : last) * 2u;
    w.cshift = C::F == 2 && ch == last + 1 ? 16u : 0u;
#pragma unroll
    for (int i = 0; i < C::F; ++i)
#pragma unroll
        for (int j = 0; j < C::NB; ++j)
            w.acc[i][j] = f32x4_acc{0.f, 0.f, 0.f, 0.f};

    // two batches of U steps: one in flight while the other is multiplied
    constexpr uint32_t B = C::NW * C::U;
    DirStep<C> b0[C::U], b1[C::U];
    w.load_batch(b0, wave, a);
    for (uint32_t st = wave; st < w.nst; st += 2 * B) {
        w.load_batch(b1, st + B, a);
        w.compute_batch(b0, st, a);
        w.load_batch(b0, st + 2 * B, a);
        w.compute_batch(b1, st + B, a);
    }

    // Lane (pixel c16 of block j): element e of matrix i is channel
    // ch0 + 4*F*g + F*e + i; piece c of the lane's 4*F channels is 4 of them.
#pragma unroll
    for (int j = 0; j < C::NB; ++j)
#pragma unroll
        for (int c = 0; c < C::F; ++c) {
            float v[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int idx = 4 * c + t;
                v[t] = w.acc[idx % C::F][j][idx / C::F];
            }
            part[wave][j * C::F + c][lane] = make_float4(v[0], v[1], v[2], v[3]);
        }
    __syncthreads();
    for (uint32_t it = tid; it < (uint32_t)C::ITEMS; it += C::NT) {
        const uint32_t l = it & 63, jc = it >> 6, j = jc / C::F, c = jc % C::F;
        const uint32_t p = p0 + 16 * j + (l & 15), cc = ch0 + 4 * C::F * (l >> 4) + 4 * c;
        if (p >= a.P || cc >= a.Co)
            continue;
        float4 s = part[0][jc][l];
#pragma unroll
        for (int z = 1; z < C::NW; ++z) {
            const float4 v = part[z][jc][l];
            s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
        }
        const uint32_t h[4] = {E::bits(s.x), E::bits(s.y), E::bits(s.z), E::bits(s.w)};
        uint16_t *o = a.out + (uint64_t)p * a.Co + cc;
        if ((a.Co & 3) == 0) {
            *reinterpret_cast<uint2 *>(o) = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
        } else {
#pragma unroll
            for (uint32_t e = 0; e < 4; ++e)
                if (cc + e < a.Co)
                    o[e] = (uint16_t)h[e];
        }
    }
}

struct DirVariant {
    const char *name;
    const void *f[2][2];  // [bf16][C_i a multiple of 8]
    int bm, bn, nt, fch;
    int cost;             // nanoseconds per 32-tap step of a workgroup alone on its CU
};

template <int F, int NB, int NW, int U>
DirVariant dir_variant(const char *name, int cost)
{
    using C = DirCfg<F, NB, NW, U>;
    return DirVariant{
        name,
        {{(const void *)&conv_fp16_direct<C, F16Op, false>, (const void *)&conv_fp16_direct<C, F16Op, true>},
         {(const void *)&conv_fp16_direct<C, BF16Op, false>, (const void *)&conv_fp16_direct<C, BF16Op, true>}},
        C::BM, C::BN, C::NT, F, cost};
}

const DirVariant *dir_variants(int *n)
{
    // name: channels x pixels per tile, waves.  The cost is the slope of the
    // measured times over K (3x3 C=512 against C=256, one workgroup per CU);
    // 3.5 us come on top for the launch, the first loads and the final sum.
    // Sixteen waves measured within 3 % of eight.
    static const DirVariant v[] = {
        dir_variant<2, 1, 8, 4>("c32p16w8", 42),
        dir_variant<2, 2, 8, 4>("c32p32w8", 69),
        dir_variant<4, 2, 8, 3>("c64p32w8", 115),
        dir_variant<4, 4, 8, 2>("c64p64w8", 178),
        // two workgroups per CU
        dir_variant<4, 4, 4, 2>("c64p64w4", 178),
    };
    *n = (int)(sizeof v / sizeof v[0]);
    return v;
}

}  // namespace

int direct_find(const char *name)
{
    int n;
    const DirVariant *v = dir_variants(&n);
    for (int t = 0; t < n; ++t)
        if (strcmp(name, v[t].name) == 0)
            return t;
    return -1;
}

const char *direct_name(int v)
{
    int n;
    return dir_variants(&n)[v].name;
}

bool direct_fits(const Shape &sh, int pick)
{
    int n;
    const DirVariant *v = dir_variants(&n);
    if (pick < 0 || pick >= n || sh.Co < 2 || (v[pick].fch == 4 && sh.Co % 4 != 0))
        return false;
    // window offsets inside a tile (its strips, one window) and filter
    // offsets need 31 bits; the latter hold with the packed filter's bound
    const int64_t strips = (v[pick].bn - 1) / sh.Wo + 2;
    return (strips * sh.L + 64) * 2 < (int64_t)kMaxRecords && sh.K * sh.Co * 2 < (int64_t)kMaxRecords;
}

// Small grids, measured against the kernels that run otherwise (conv call
// with its filter pack, GPU time, us):
//   C_i % 8 == 0 (column-staged and row-per-pixel kernels): ahead while one
//   64 x 64 tile per CU covers the output, 256 tiles:
//     3x3 C=256 at 14x14, 1 / 8 / 28 images     6.7 / 12.0 / 16.7 vs 19.3 / 20.6 / 20.8
//     3x3 C=512 at 7x7, 1 / 8 / 24 images       9.5 / 14.1 / 29.4 vs 27.6 / 30.7 / 31.0
//     3x3 C=64 at 56x56, 1 / 5 images           4.7 / 7.4 vs 9.9 / 10.1
//     1x1 C=1024 at 14x14, 1 / 5 images         5.9 / 10.0 vs 12.2 / 14.1
//   and behind from there on (3x3 C=512 at 7x7, 48 images: 53 vs 32; 3x3
//   C=64 at 56x56, 8 images: 10.9 vs 10.4; 1x1 C=1024, 9 images: 16.3 vs 15.0).
//   Other C_i (segment- and register-staged kernels): ahead up to 1.5 tiles
//   per CU (3x5 36 -> 100, 7 / 16 images 5.5 / 6.7 vs 27.6 / 27.2; 3x3 217 ->
//   63 at 28x28, 4 images 15.3 vs 86; 7x7 3 -> 64, one 224x224 image 5.2 vs
//   9.1), even or behind from about 650 tiles (3x3 21 -> 120 14.1 vs 13.0;
//   3x3 217 -> 256 62 vs 58).  Windows of at most two steps (K <= 64) stay with
//   the kernels that hold a short window in registers or LDS: there are no
//   taps to split.
// 3x3 layers of up to 64 input and 65 to 128 output channels gain as much: 0.32
// to 0.43 of the column-staged kernel's time up to 4000 pixels, 0.53 at 8000
// (3x3 64 -> 104 at 32x32, 2 images, 11.0 -> 4.3 us).
int direct_default(const Shape &sh)
{
    constexpr int64_t kCUs = 256;
    const bool aligned = sh.Ci % 8 == 0;
    if (!aligned && sh.K <= 64)
        return -1;
    int n, best = -1;
    int64_t best_cost = 0, best_rounds = 0;
    const DirVariant *v = dir_variants(&n);
    for (int t = 0; t < n; ++t) {
        if (!direct_fits(sh, t))
            continue;
        const int64_t tiles = ((sh.P + v[t].bn - 1) / v[t].bn) * ((sh.Co + v[t].bm - 1) / v[t].bm);
        const int64_t rounds = (tiles + kCUs - 1) / kCUs;
        if (v[t].nt == 256 ? rounds != 2 || aligned : rounds > 2)
            continue;
        const int64_t cost = rounds * v[t].cost;
        if (best < 0 || cost < best_cost) {
            best = t;
            best_cost = cost;
            best_rounds = rounds;
        }
    }
    if (best < 0)
        return -1;
    // With long windows the row kernel's 64 x 64 tile with four slots is
    // ahead where this one would use as large a tile (3x3 C=512 at 7x7, 24
    // images: 24.1 vs 29.3 us; 3x3 C=256 at 14x14, 12 images: 14.8 vs 16.4;
    // 1x1 1024 -> 256 at 14x14, 16 images: 10.3 vs 9.8), and with longer ones
    // where two rounds of this one's would run (7x7 stride 2 208 -> 344, 1458
    // pixels: 40.0 vs 59.6 us; over 24 layers even at 2000 taps, 0.92 of the
    // time at 3000, 0.81 at 6000, 0.68 from 8192 on; not two of its smallest
    // tile, 7x7 stride 2 112 -> 224, 1156 pixels, 20.5 vs 24.7).  Where another kernel
    // would run instead, up to 64 channels and on the column-staged one's
    // layers, this one stays ahead (3x3 400 -> 4, 10830 pixels: 16.2 vs 29.9;
    // 7x7 136 -> 72, 4800 pixels, 32.2 vs 47.2).
    if (aligned && sh.K >= 1536 && v[best].bm == 64 && v[best].bn == 64)
        return -1;
    if (aligned && sh.K >= 2560 && best_rounds > 1 && v[best].bn > 16 && sh.Co > 64 && col_default(sh) < 0)
        return -1;
    // the largest tile the layer's channels allow decides whether the grid is small
    const int64_t big = sh.Co % 4 == 0 ? 64 : 32;
    const int64_t tiles = ((sh.P + big - 1) / big) * ((sh.Co + big - 1) / big);
    return tiles <= (aligned ? kCUs : kCUs * 3 / 2) ? best : -1;
}

hipError_t launch_conv_fp16_direct(const Shape &sh, int plan, const Tuning &t, const void *ws, const uint16_t *filt,
                                   uint16_t *out, hipStream_t st, Op16 op)
{
    int n;
    const DirVariant &v = dir_variants(&n)[plan];
    DirArgs a;
    a.ws = static_cast<const uint16_t *>(ws);
    a.filt = filt;
    a.out = out;
    a.P = (uint32_t)sh.P; a.K = (uint32_t)sh.K; a.Co = (uint32_t)sh.Co; a.Wo = (uint32_t)sh.Wo;
    a.L = (uint32_t)sh.L; a.Ci = (uint32_t)sh.Ci; a.Kh = (uint32_t)sh.Kh; a.Kw = (uint32_t)sh.Kw;
    a.wc = make_wincols(sh);
    a.div_Wo = make_fastdiv(a.Wo);
    a.div_khci = make_fastdiv(a.Kh * a.Ci);
    a.div_ci = make_fastdiv(a.Ci);
    const int64_t gx = (sh.P + v.bn - 1) / v.bn, gy = (sh.Co + v.bm - 1) / v.bm;
    if (gx * gy > 0x7fffffff)
        return hipErrorInvalidValue;
    // Each XCD's L2 holds what its run of tiles reads: the tiles that share
    // the larger operand follow one another, so that operand is fetched by
    // one XCD and only the smaller one by all.
    a.swap = sh.K * sh.Co > sh.win_elems ? 1u : 0u;
    a.tg = a.swap ? make_tilegrid(gy, gx, t.tile_linear) : make_tilegrid(gx, gy, t.tile_linear);
    void *args[] = {&a};
    return hipLaunchKernel(v.f[op == Op16::BF16][sh.Ci % 8 == 0], dim3((uint32_t)(gx * gy)), dim3(v.nt), args, 0, st);
}

}  // namespace im2win
