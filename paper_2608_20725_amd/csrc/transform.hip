// im2win transform (Sec. III-B, Eq. 2) for gfx950.
//
//   W[i][m][k*K_h + u][r] = I[i][m*s + u][k][r]
//
// Pure copy, HBM-bound: every byte of the window tensor is written once; the
// K_h/s-fold re-reads of input rows are served by L2 and the Infinity Cache.
// Three kernels:
//   * vec:    C_i*elt is a multiple of 16 bytes.  A thread copies whole
//             16-byte granules; a workgroup covers a contiguous run of the
//             window tensor (possibly across strips), so the stores of a wave
//             are one contiguous 1 KiB run, in an XCD-aware block order.
//   * pieces: any other C_i, undilated: a workgroup reads the input rows of
//             a piece of the window tensor in their own order and puts the
//             piece together in LDS.
//   * pieces3: smaller 3-channel layers, undilated and unpadded (16-bit with
//             K_h <= 3): the gather below with one load per 3-channel pixel.
//   * gather: the rest (dilated layers, smaller ones).  A thread assembles
//             one 16-byte granule of the flat window tensor element by
//             element; granules may straddle strips.
// All zero the pad bytes that follow the window tensor.
//
// Zero padding of the input (not in the paper's layers) is folded in: the
// window tensor is that of the input surrounded by ph zero rows and pw zero
// columns on each side, and positions outside the stored input are written
// as zeros; the padded input itself is never built.
#include "common.hpp"

#include <stdlib.h>
#include <string.h>

namespace im2win {
namespace {

constexpr int kThreads = 256;
constexpr int kGranPerThread = 4;

struct TArgs {
    const char *in;
    char *ws;
    uint32_t Ci, Hi, Wi, Kh, s, Ho;  // Hi x Wi: the stored (unpadded) input
    uint32_t Wp, ph, pw;             // padded width Wi + 2*pw; zero rows / columns per side
    uint32_t d, Wq, cols;            // dilation; strip columns per residue group; d*Wq columns
    uint32_t L;              // strip length (elements)
    uint32_t strips;
    uint32_t gran_per_strip; // vec: 16-byte granules per strip
    uint64_t win_elems;
    uint64_t win_bytes, pad_end;
    uint64_t grans;          // gather: 16-byte granules of the window tensor
    uint64_t in_pixels;      // pieces3: pixels of the input (N * H_i * W_i)
    uint32_t cu;             // pieces: units per pixel
    uint32_t spb, segs, cpb; // pieces: strips per block; pieces per strip, columns per piece
    uint32_t xcd_order;      // vec, pieces: 1 = XCD-aware block order, 0 = linear (ablation)
    FastDiv div_Ci, div_Kh, div_Wi, div_Ho, div_L, div_gps, div_Wq, div_cu;
};

// Padded-input column held by strip column position k: k itself, or with
// dilation d (columns grouped by residue mod d, Wq per group) column
// (k mod Wq)*d + floor(k/Wq); positions past the padded width are filler and
// map to columns >= Wp, outside the stored input like the right-hand padding.
__device__ inline uint32_t strip_col(uint32_t k, const TArgs &a)
{
    if (a.d == 1)
        return k;
    const uint32_t g = fdiv(k, a.div_Wq);
    return (k - g * a.Wq) * a.d + g;
}

__device__ inline void zero_pad(const TArgs &a)
{
    // [win_bytes, pad_end) holds at most 256 + 255 + 15 bytes
    for (uint64_t b = a.win_bytes + threadIdx.x; b < a.pad_end; b += blockDim.x)
        a.ws[b] = 0;
}

// XCD-aware block order: the hardware deals the blocks of a launch to the 8
// XCDs round-robin (block b to XCD b % 8), and each XCD has its own L2.  Block
// b works on logical block xcd_block(b), so that every XCD walks one
// contiguous run of the window tensor: strips that share input rows are then
// copied by the same XCD at about the same time and the re-reads hit its L2.
// A bijection on [0, nb).
__device__ inline uint32_t xcd_block(uint32_t b, uint32_t nb)
{
    const uint32_t x = b % 8, j = b / 8;
    const uint32_t per = nb / 8, rem = nb % 8;
    return x * per + (x < rem ? x : rem) + j;
}

template <int ELT>
__global__ __launch_bounds__(kThreads) void transform_vec(TArgs a)
{
    constexpr uint32_t V = 16 / ELT;  // elements per granule
    if (blockIdx.x == 0)
        zero_pad(a);
    // granules of the whole window tensor, numbered strip by strip
    // (granule counts fit 32 bits: transform_range_ok)
    const uint32_t lb = a.xcd_order ? xcd_block(blockIdx.x, gridDim.x) : blockIdx.x;
    const uint32_t gb = lb * (kThreads * kGranPerThread);
#pragma unroll
    for (int t = 0; t < kGranPerThread; ++t) {
        const uint32_t g = gb + t * kThreads + threadIdx.x;
        if (g < a.grans) {
            const uint32_t q = fdiv(g, a.div_gps);  // strip
            const uint32_t pos = (g - q * a.gran_per_strip) * V;
            const uint32_t i = fdiv(q, a.div_Ho);
            const uint32_t m = q - i * a.Ho;
            const uint32_t seg = fdiv(pos, a.div_Ci);  // k*K_h + u
            const uint32_t r = pos - seg * a.Ci;
            const uint32_t k = fdiv(seg, a.div_Kh);
            const uint32_t u = seg - k * a.Kh;
            // a granule lies inside one (column, row) piece of C_i elements:
            // all of it is padding or none
            const int32_t h = (int32_t)(m * a.s + u * a.d) - (int32_t)a.ph;
            const int32_t w = (int32_t)strip_col(k, a) - (int32_t)a.pw;
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (h >= 0 && h < (int32_t)a.Hi && w >= 0 && w < (int32_t)a.Wi) {
                const uint64_t src = (((uint64_t)i * a.Hi + (uint32_t)h) * a.Wi + (uint32_t)w) * a.Ci + r;
                v = *reinterpret_cast<const uint4 *>(a.in + src * ELT);
            }
            *reinterpret_cast<uint4 *>(a.ws + (uint64_t)g * 16) = v;
        }
    }
}

// Strips of any other C_i, undilated: what bounds the element gather below is
// not memory but the order of its reads, a granule's elements lying in up to
// eight input rows, and the index arithmetic of every element.  Here a
// workgroup owns a contiguous piece of the window tensor of at most 16 KiB
// (some columns of a strip, or a few whole strips), reads the input rows it
// comes from in their own order, places each element in LDS where the window
// tensor has it, and copies the piece out as 16-byte granules.  A row's
// position (image, strip, filter row) is the same for a whole wave, so a lane
// adds little more than one LDS address per element.  Measured (us, 128
// images unless said, element gather -> pieces): fp16 11x11 stride 4 at
// 227x227 65 -> 26.4 (5.5 TB/s), 7x7 stride 2 80 -> 34, 3x3 at 224x224 64 ->
// 24.5; fp32 7x7 stride 2 pad 3 at 224x224, 32 images, 27.4 -> 18.6 (4.8
// TB/s), 11x11 74 -> 58; fp16 3x3 52 channels at 81x81, 92 images, 108 -> 38;
// and against the one-load-per-pixel gather it replaces, fp32 3x3 at 224x224
// 67 -> 60.
//
// The row is read as units of UB = 2, 4 or 8 bytes, the largest that divides
// a pixel's C_i*elt bytes, V consecutive units per lane and load: 16 bytes (8
// with 2-byte units), one unit for rows too short to fill a wave that way, or
// one or two 3-channel pixels, which need no carry into the next column:
// three 4-byte units, or six 2-byte ones, whose two pixels leave as one dword
// and one half each.  Two pixels a lane against one, its three halves stored
// one by one, took the 16-bit times above from 40, 47.5 and 41 us (LDS writes
// and address arithmetic bound them), 7x7 stride 2 pad 3, 32 images, 18.4 ->
// 12.5; with the input from HBM and a conv between, 11x11 52 -> 40, transform
// and conv together 104 -> 93, 7x7 147 -> 131, 3x3 199 -> 181.  Two such
// loads in flight need rows of more than 64 pairs to be of use: with one,
// 32-wide images 8.3 -> 6.9, one 224-wide image cut into short pieces 4.17 ->
// 3.94.  Padding rows and columns are the zeros the piece starts with.
template <int UB>
struct UnitOf;
template <>
struct UnitOf<2> { typedef uint16_t type; };
template <>
struct UnitOf<4> { typedef uint32_t type; };
template <>
struct UnitOf<8> { typedef uint64_t type; };

constexpr uint32_t kPieceBytes = 16384;

// U: loads in flight per lane
template <int UB, int V, int U = 4>
__global__ __launch_bounds__(kThreads) void transform_pieces(TArgs a)
{
    typedef typename UnitOf<UB>::type unit;
    __shared__ uint4 buf[kPieceBytes / 16 + 2];
    char *lds = reinterpret_cast<char *>(buf);

    if (blockIdx.x == 0)
        zero_pad(a);
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t b = a.xcd_order ? xcd_block(blockIdx.x, gridDim.x) : blockIdx.x;
    const uint32_t sb = b / a.segs, seg = b - sb * a.segs;
    const uint32_t q0 = sb * a.spb;                                      // first strip
    const uint32_t ns = a.strips - q0 < a.spb ? a.strips - q0 : a.spb;   // strips (1 if a strip is split)
    const uint32_t k0 = seg * a.cpb;                                     // first column
    const uint32_t k1 = a.Wp - k0 < a.cpb ? a.Wp : k0 + a.cpb;
    const uint32_t cu = a.cu, colu = a.Kh * cu;                          // units per pixel and per column
    const uint32_t stripu = a.Wp * colu;                                 // units per strip
    const uint64_t first = ((uint64_t)q0 * stripu + (uint64_t)k0 * colu) * UB;  // byte offset of the piece
    const uint32_t len = (ns > 1 ? ns * stripu : (k1 - k0) * colu) * UB;
    const uint32_t lead = (uint32_t)first & 15u;                         // its offset in its first granule

    if (a.ph | a.pw) {
        for (uint32_t g = threadIdx.x; g < kPieceBytes / 16 + 2; g += kThreads)
            buf[g] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
    }
    // stored columns among k0 .. k1-1
    const uint32_t v0 = k0 > a.pw ? k0 : a.pw, v1 = k1 < a.pw + a.Wi ? k1 : a.pw + a.Wi;
    const uint32_t rows = v0 < v1 ? ns * a.Kh : 0u, n = v0 < v1 ? (v1 - v0) * cu : 0u;
    for (uint32_t rr = wave; rr < rows; rr += kThreads / 64) {
        const uint32_t st = fdiv(rr, a.div_Kh), u = rr - st * a.Kh;
        const uint32_t q = q0 + st, i = fdiv(q, a.div_Ho), m = q - i * a.Ho;
        const int32_t h = (int32_t)(m * a.s + u) - (int32_t)a.ph;
        if (h < 0 || h >= (int32_t)a.Hi)
            continue;
        const char *src = a.in + (((uint64_t)i * a.Hi + (uint32_t)h) * a.Wi + (v0 - a.pw)) * cu * UB;
        char *dst = lds + lead + (st * stripu + ((v0 - k0) * a.Kh + u) * cu) * UB;
        if constexpr (UB == 2 && V == 6) {
            // columns k (even), k + 1 of a lane: whether their six bytes each
            // start on a 4-byte boundary of LDS is the same for the whole wave
            const uint32_t np = (v1 - v0) / 2, o0 = lead + (st * stripu + ((v0 - k0) * a.Kh + u) * 3) * 2;
            const bool a0 = (o0 & 2) == 0, a1 = ((o0 + colu * 2) & 2) == 0;
            for (uint32_t x = lane; x < np; x += 64 * U) {
                uint32_t el[U][3];
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    // lanes past the row repeat its last pair
                    const uint32_t p = x + 64 * t < np ? x + 64 * t : np - 1;
                    __builtin_memcpy(el[t], src + p * 12u, 12);
                }
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    const uint32_t p = x + 64 * t < np ? x + 64 * t : np - 1;
                    char *o = dst + p * (colu * 4), *e = o + colu * 2;
                    if (a0) {
                        *reinterpret_cast<uint32_t *>(o) = el[t][0];
                        *reinterpret_cast<uint16_t *>(o + 4) = (uint16_t)el[t][1];
                    } else {
                        *reinterpret_cast<uint16_t *>(o) = (uint16_t)el[t][0];
                        *reinterpret_cast<uint32_t *>(o + 2) = __builtin_amdgcn_alignbyte(el[t][1], el[t][0], 2);
                    }
                    if (a1) {
                        *reinterpret_cast<uint32_t *>(e) = __builtin_amdgcn_alignbyte(el[t][2], el[t][1], 2);
                        *reinterpret_cast<uint16_t *>(e + 4) = (uint16_t)(el[t][2] >> 16);
                    } else {
                        *reinterpret_cast<uint16_t *>(e) = (uint16_t)(el[t][1] >> 16);
                        *reinterpret_cast<uint32_t *>(e + 2) = el[t][2];
                    }
                }
            }
            // the last column of an odd number
            if (((v1 - v0) & 1) && lane < 3) {
                unit el;
                __builtin_memcpy(&el, src + (np * 6 + lane) * UB, UB);
                *reinterpret_cast<unit *>(dst + (2 * np * colu + lane) * UB) = el;
            }
        } else if constexpr (V == 3) {
            const uint32_t nk = v1 - v0;
            for (uint32_t x = lane; x < nk; x += 64 * U) {
                unit el[U][3];
#pragma unroll
                for (int t = 0; t < U; ++t)
                    if (x + 64 * t < nk)
                        __builtin_memcpy(el[t], src + (x + 64 * t) * 12u, 12);
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    const uint32_t k = x + 64 * t;
                    if (k >= nk)
                        continue;
                    unit *o = reinterpret_cast<unit *>(dst + k * (colu * UB));
                    o[0] = el[t][0];
                    o[1] = el[t][1];
                    o[2] = el[t][2];
                }
            }
        } else {
            // whole groups of V units, then the row's last n % V
            for (uint32_t x = lane * V; x + V <= n; x += 64 * V * U) {
                unit el[U][V];
#pragma unroll
                for (int t = 0; t < U; ++t)
                    if (x + 64 * V * t + V <= n)
                        __builtin_memcpy(el[t], src + (x + 64 * V * t) * UB, V * UB);
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    const uint32_t xt = x + 64 * V * t;
                    if (xt + V > n)
                        continue;
                    const uint32_t k = fdiv(xt, a.div_cu);
                    uint32_t r = xt - k * cu, o = (k * colu + r) * UB;
#pragma unroll
                    for (int e = 0; e < V; ++e) {
                        *reinterpret_cast<unit *>(dst + o) = el[t][e];
                        const bool wrap = ++r == cu;  // into the next column
                        o += wrap ? UB + (colu - cu) * UB : UB;
                        r = wrap ? 0u : r;
                    }
                }
            }
            const uint32_t xt = n - n % V + lane;
            if (V > 1 && xt < n) {
                unit el;
                __builtin_memcpy(&el, src + xt * UB, UB);
                const uint32_t k = fdiv(xt, a.div_cu);
                *reinterpret_cast<unit *>(dst + (k * colu + (xt - k * cu)) * UB) = el;
            }
        }
    }
    __syncthreads();
    // whole granules, and the elements of the first and last one that this
    // piece shares with its neighbours
    char *out = a.ws + (first - lead);
    for (uint32_t g = threadIdx.x; 16 * g < lead + len; g += kThreads) {
        if (16 * g >= lead && 16 * g + 16 <= lead + len) {
            *reinterpret_cast<uint4 *>(out + 16 * (uint64_t)g) = buf[g];
        } else {
            for (uint32_t o = 16 * g; o < 16 * g + 16; o += UB)
                if (o >= lead && o < lead + len)
                    *reinterpret_cast<unit *>(out + o) = *reinterpret_cast<const unit *>(lds + o);
        }
    }
}

template <int ELT>
__device__ inline void store_elem(uint32_t *w, int e, uint32_t bits)
{
    if (ELT == 4) {
        w[e] = bits;
    } else {
        const int d = e >> 1;
        w[d] = (e & 1) ? (w[d] & 0xffffu) | (bits << 16) : (w[d] & 0xffff0000u) | (bits & 0xffffu);
    }
}

// The gather of the 3-channel layers with one load per piece: a 16-byte
// granule of the window tensor (8 fp16 or 4 fp32 elements) spans at most 4
// (fp16) or 2 (fp32) pieces, a piece being the 3 channels of one input pixel
// (one column of one filter row of one strip).  Each piece is read with one
// load, 8 bytes for fp16 (6 used) and 12 for fp32, instead of one load per
// element; the granule is assembled in registers and stored whole, so a
// wave's stores stay one contiguous 1 KiB run.  An 8-byte fp16 read would
// reach 2 bytes past the last pixel of the input: that piece is read as 4 + 2
// bytes.  For window tensors too small for transform_pieces: against the
// element gather, us, fp32 7x7 at 74x74, 20 images (8.1 MB), 4.7 and 5.5; fp16
// 3x3 at 36x41, 51 images (1.2 MB), 3.5 and 4.0.
template <int ELT>
__global__ __launch_bounds__(kThreads) void transform_pieces3(TArgs a)
{
    constexpr uint32_t V = 16 / ELT;                // elements per granule
    constexpr int NP = ELT == 2 ? 4 : 2;            // pieces a granule can touch
    const uint64_t g = (uint64_t)blockIdx.x * kThreads + threadIdx.x;
    if (blockIdx.x == 0)
        zero_pad(a);
    if (g >= a.grans)
        return;
    // first element of this granule (win_elems < 2^32, checked on the host)
    const uint32_t e0 = (uint32_t)(g * V);
    uint32_t q = fdiv(e0, a.div_L);
    const uint32_t pos = e0 - q * a.L;
    uint32_t seg = fdiv(pos, a.div_Ci);              // k*K_h + u of the first piece
    const uint32_t r0 = pos - seg * 3;               // its first channel used
    const uint32_t segs = a.L / 3;                   // pieces per strip (W_i * K_h)
    uint32_t el[NP * 3];                             // the pieces' elements (ELT bytes each)
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        el[3 * j] = el[3 * j + 1] = el[3 * j + 2] = 0u;
        // piece j holds granule elements 3j - r0 .. 3j - r0 + 2
        if (3 * j >= (int)(r0 + V) || (uint64_t)e0 + 3 * j - r0 >= a.win_elems)
            continue;
        if (seg == segs) {  // into the next strip
            seg = 0;
            ++q;
        }
        const uint32_t k = fdiv(seg, a.div_Kh), u = seg - k * a.Kh;
        const uint32_t i = fdiv(q, a.div_Ho), m = q - i * a.Ho;
        const uint64_t px = ((uint64_t)i * a.Hi + m * a.s + u) * a.Wi + k;  // input pixel
        const char *src = a.in + px * (3 * ELT);
        if (ELT == 4) {
            uint32_t v[3];
            __builtin_memcpy(v, src, 12);
            el[3 * j] = v[0]; el[3 * j + 1] = v[1]; el[3 * j + 2] = v[2];
        } else {
            uint64_t v;  // one 8-byte load (the last pixel: 4 + 2 bytes)
            if (px + 1 < a.in_pixels) {
                __builtin_memcpy(&v, src, 8);
            } else {
                uint32_t lo;
                uint16_t hi;
                __builtin_memcpy(&lo, src, 4);
                __builtin_memcpy(&hi, src + 4, 2);
                v = lo | ((uint64_t)hi << 32);
            }
            el[3 * j] = (uint32_t)v & 0xffffu;
            el[3 * j + 1] = (uint32_t)(v >> 16) & 0xffffu;
            el[3 * j + 2] = (uint32_t)(v >> 32) & 0xffffu;
        }
        ++seg;
    }
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (uint32_t t = 0; t < V; ++t) {
        // element t of the granule is element r0 + t of the pieces' run
        // (r0 < 3)
        const uint32_t bits = r0 == 0 ? el[t] : r0 == 1 ? el[t + 1] : el[t + 2];
        store_elem<ELT>(w, (int)t, bits);
    }
    // bytes past the window tensor are inside the zero pad: zeros are written
    *reinterpret_cast<uint4 *>(a.ws + g * 16) = make_uint4(w[0], w[1], w[2], w[3]);
}

template <int ELT>
__global__ __launch_bounds__(kThreads) void transform_gather(TArgs a)
{
    constexpr uint32_t V = 16 / ELT;
    const uint64_t g = (uint64_t)blockIdx.x * kThreads + threadIdx.x;
    if (blockIdx.x == 0)
        zero_pad(a);
    if (g >= a.grans)
        return;
    // first element of this granule; win_elems < 2^32 is checked on the host
    uint32_t e = (uint32_t)(g * V);
    uint32_t q = fdiv(e, a.div_L);
    uint32_t pos = e - q * a.L;
    uint32_t seg = fdiv(pos, a.div_Ci);
    uint32_t r = pos - seg * a.Ci;
    uint32_t k = fdiv(seg, a.div_Kh);
    uint32_t u = seg - k * a.Kh;
    uint32_t i = fdiv(q, a.div_Ho);
    uint32_t m = q - i * a.Ho;
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (uint32_t t = 0; t < V; ++t) {
        if ((uint64_t)e + t < a.win_elems) {
            const int32_t hh = (int32_t)(m * a.s + u * a.d) - (int32_t)a.ph;
            const int32_t ww = (int32_t)strip_col(k, a) - (int32_t)a.pw;
            uint32_t bits = 0;
            if (hh >= 0 && hh < (int32_t)a.Hi && ww >= 0 && ww < (int32_t)a.Wi) {
                const uint64_t src = (((uint64_t)i * a.Hi + (uint32_t)hh) * a.Wi + (uint32_t)ww) * a.Ci + r;
                if (ELT == 4)
                    bits = reinterpret_cast<const uint32_t *>(a.in)[src];
                else
                    bits = reinterpret_cast<const uint16_t *>(a.in)[src];
            }
            store_elem<ELT>(w, (int)t, bits);
            // advance (r, u, k, m, i) to the next window-tensor element
            if (++r == a.Ci) {
                r = 0;
                if (++u == a.Kh) {
                    u = 0;
                    if (++k == a.cols) {
                        k = 0;
                        if (++m == a.Ho) {
                            m = 0;
                            ++i;
                        }
                    }
                }
            }
        }
    }
    // bytes past the window tensor are inside the zero pad: zeros are written
    *reinterpret_cast<uint4 *>(a.ws + g * 16) = make_uint4(w[0], w[1], w[2], w[3]);
}

}  // namespace

bool transform_range_ok(const Shape &sh)
{
    if ((sh.Ci * sh.elt) % 16 == 0)  // granule indices fit 32 bits
        return (uint64_t)sh.win_bytes / 16 + kThreads * kGranPerThread < (1ull << 32);
    return (uint64_t)sh.win_elems + 16 < (1ull << 32);
}

namespace {

// How transform_pieces divides a layer's window tensor.
struct PieceGrid {
    int64_t cpb, spb, segs;  // columns and strips per piece, pieces per strip
    int64_t blocks;
    int64_t ub, cu;          // bytes of a unit, units per pixel
};

PieceGrid piece_grid(const Shape &sh)
{
    PieceGrid g;
    const int64_t colb = sh.Kh * sh.Ci * sh.elt, pxb = sh.Ci * sh.elt;
    // pieces of at most 16 KiB (eight blocks per CU), smaller ones while there
    // is less than one per CU (512 or 1024 pieces of one image's split strips
    // measured up to 1.1 us slower).  Whole strips share a piece only beyond
    // four pieces per CU: each strip adds K_h rows to what the piece's four
    // waves read one after another (fp16 padded 3x3 at 110x15, 3 channels, 110
    // images: 31 strips a piece 20.7 us, 11 strips 11.1, the element gather 4.8).
    const int64_t most = kPieceBytes / colb, want = 256, shared = 1024;
    g.cpb = sh.Wi < most ? sh.Wi : most;
    g.spb = 1;
    if (g.cpb < sh.Wi || sh.strips < want) {
        int64_t segs = (sh.Wi + g.cpb - 1) / g.cpb;
        if (sh.strips * segs < want)
            segs = (want + sh.strips - 1) / sh.strips;
        g.cpb = (sh.Wi + segs - 1) / segs;
        g.cpb = g.cpb < 4 ? (sh.Wi < 4 ? sh.Wi : 4) : g.cpb;
        g.cpb = g.cpb < most ? g.cpb : most;
    } else {
        g.spb = kPieceBytes / (sh.Wi * colb);
        const int64_t lim = sh.strips / shared;
        g.spb = g.spb < lim ? g.spb : lim;
        g.spb = g.spb < 1 ? 1 : g.spb;
    }
    g.segs = (sh.Wi + g.cpb - 1) / g.cpb;
    g.blocks = (sh.strips + g.spb - 1) / g.spb * g.segs;
    g.ub = pxb % 8 == 0 ? 8 : pxb % 4 == 0 && sh.Ci != 3 ? 4 : sh.elt;
    g.cu = pxb / g.ub;
    return g;
}

// Where transform_pieces is ahead of the gathers, fitted to 4000 layers (GPU
// time).  What it costs is the rows its waves read one after another: a piece
// of r rows takes r/4 passes of about half a microsecond, and 2048 pieces are
// resident at once, so the window tensor has to be large enough for its
// passes.  Against the gathers (us):
//   fp32 from 10 MiB, 5 MiB a pass: 3x3 23 channels at 57x62, 11.7 MiB in one
//   pass, 6.3 and 6.9; 7x7 padded 3 channels at 45x45, 116 images, 16.3 MiB in
//   seven, 10.3 and 7.9.
//   16-bit from 512 KiB, 1.5 MiB a pass (2 MiB with 3 channels): 3x3 at
//   107x107, 7.5 MiB in three, 7.1 and 7.5; 3x3 padded stride 2 at 126x31, 126
//   images, 4.2 MiB in six, 8.8 and 5.4.  More than 3 channels in one pass
//   always pay, and so do two passes of up to 512 pieces, which do not wait for
//   one another (5x5 stride 2 54 channels at 32x32, 1.2 MiB, 3.4 and 3.9; 3
//   channels at 66x66, 0.6 MiB, 3.4 and 4.0), unless the rows are long runs of
//   2-byte units (5x5 209 channels at 10x10, 1.7 MiB: 4.7 and 3.8).
//   One-row filters, which the gather reads in input order, 16-bit from 4 MiB
//   (6 MiB with 2-byte units) and more than 3 channels: 1x1 stride 2 68
//   channels, 7.6 MiB, 4.9 and 6.8; 299 channels, 4.0 MiB, 7.2 and 4.8.
// One and two channels stay with the gather (5x5 one channel, 32 MB: 11.3 vs 8.9).
bool pieces_pay(const Shape &sh, const PieceGrid &g)
{
    constexpr int64_t kMiB = 1 << 20, kResident = 2048;
    if (sh.Ci <= (sh.Kh > 1 ? 2 : 3))
        return false;
    const int64_t per = (g.spb * sh.Kh + 3) / 4, win = sh.win_bytes;
    const double passes = (double)per * (g.blocks > kResident ? (double)g.blocks / kResident : 1.);
    if (sh.elt == 4)
        return win >= 10 * kMiB && win >= 5. * kMiB * passes;
    if (sh.Kh == 1)
        return win >= (g.ub == 2 ? 6 : 4) * kMiB;
    const bool short_rows = g.ub > 2 || g.cpb * g.cu <= 768;
    if (win >= kMiB / 2 && short_rows && ((per <= 2 && g.blocks <= 512) || (passes == 1. && sh.Ci > 3)))
        return true;
    return win >= (sh.Ci == 3 ? 2. : 1.5) * kMiB * passes;
}

}  // namespace

hipError_t launch_transform(const Shape &sh, const void *in, void *ws, hipStream_t st, const Tuning &t,
                            const Pad *pad)
{
    TArgs a;
    a.in = static_cast<const char *>(in);
    a.ws = static_cast<char *>(ws);
    a.Ci = (uint32_t)sh.Ci;
    a.Wp = (uint32_t)sh.Wi;
    if (pad) {
        a.Hi = (uint32_t)pad->Hi; a.Wi = (uint32_t)pad->Wi;
        a.ph = (uint32_t)pad->ph; a.pw = (uint32_t)pad->pw;
    } else {
        a.Hi = (uint32_t)sh.Hi; a.Wi = (uint32_t)sh.Wi;
        a.ph = 0; a.pw = 0;
    }
    a.Kh = (uint32_t)sh.Kh; a.s = (uint32_t)sh.s; a.Ho = (uint32_t)sh.Ho;
    a.L = (uint32_t)sh.L;
    a.strips = (uint32_t)sh.strips;
    a.win_elems = (uint64_t)sh.win_elems;
    a.win_bytes = (uint64_t)sh.win_bytes;
    a.pad_end = (uint64_t)sh.pad_end;
    a.div_Ci = make_fastdiv((uint32_t)sh.Ci);
    a.div_Kh = make_fastdiv((uint32_t)sh.Kh);
    a.div_Wi = make_fastdiv((uint32_t)sh.Wi);
    a.div_Ho = make_fastdiv((uint32_t)sh.Ho);
    a.div_L = make_fastdiv((uint32_t)sh.L);
    a.d = (uint32_t)sh.d;
    a.Wq = (uint32_t)sh.Wq;
    a.cols = (uint32_t)sh.cols;
    a.div_Wq = make_fastdiv((uint32_t)sh.Wq);
    // IM2WIN_TRANSFORM_ORDER=linear deals blocks in launch order (to measure
    // what the XCD-aware order gains)
    a.xcd_order = t.transform_linear ? 0u : 1u;
    void *args[] = {&a};
    const bool vec = (sh.Ci * sh.elt) % 16 == 0;
    if (vec) {
        a.gran_per_strip = (uint32_t)(sh.L * sh.elt / 16);
        a.div_gps = make_fastdiv(a.gran_per_strip);
        a.grans = (uint64_t)sh.win_bytes / 16;
        const uint64_t per_block = kThreads * kGranPerThread;
        const uint64_t blocks = (a.grans + per_block - 1) / per_block;
        if (blocks > 0x7fffffffull)
            return hipErrorInvalidValue;
        const void *f = sh.elt == 4 ? (const void *)&transform_vec<4> : (const void *)&transform_vec<2>;
        return hipLaunchKernel(f, dim3((uint32_t)blocks), dim3(kThreads), args, 0, st);
    }
    a.gran_per_strip = 0;
    a.grans = ((uint64_t)sh.win_bytes + 15) / 16;
    const uint64_t blocks = (a.grans + kThreads - 1) / kThreads;
    if (blocks > 0x7fffffffull)
        return hipErrorInvalidValue;
    // pieces: undilated layers whose columns leave room for two in a piece,
    // where it pays (pieces_pay).  IM2WIN_TRANSFORM_KERNEL=pieces takes it
    // wherever it can run, =gather nowhere.
    const int64_t colb = sh.Kh * sh.Ci * sh.elt;
    if (sh.d == 1 && 2 * colb <= kPieceBytes && !t.transform_gather) {
        const PieceGrid pg = piece_grid(sh);
        if ((t.transform_pieces || pieces_pay(sh, pg)) && pg.blocks <= 0x7fffffff) {
            a.cpb = (uint32_t)pg.cpb;
            a.spb = (uint32_t)pg.spb;
            a.segs = (uint32_t)pg.segs;
            a.cu = (uint32_t)pg.cu;
            a.div_cu = make_fastdiv(a.cu);
            const bool narrow = pg.cpb * pg.cu <= 256;  // one unit per lane, U times, covers a row
            const void *f =
                sh.Ci == 3   ? (sh.elt == 4     ? (const void *)&transform_pieces<4, 3>
                                : pg.cpb <= 128 ? (const void *)&transform_pieces<2, 6, 1>
                                                : (const void *)&transform_pieces<2, 6, 2>)
                : pg.ub == 8 ? (narrow ? (const void *)&transform_pieces<8, 1> : (const void *)&transform_pieces<8, 2>)
                : pg.ub == 4 ? (narrow ? (const void *)&transform_pieces<4, 1> : (const void *)&transform_pieces<4, 4>)
                             : (narrow ? (const void *)&transform_pieces<2, 1> : (const void *)&transform_pieces<2, 4>);
            return hipLaunchKernel(f, dim3((uint32_t)pg.blocks), dim3(kThreads), args, 0, st);
        }
    }
    // pieces3: 16-bit only with filters of up to 3 rows (a granule's pixels
    // otherwise come from up to four input rows: 11x11 even with the gather)
    if (sh.Ci == 3 && sh.d == 1 && a.ph == 0 && a.pw == 0 && !t.transform_gather && !t.transform_pieces &&
        (sh.elt == 4 || sh.Kh <= 3)) {
        a.in_pixels = (uint64_t)sh.N * a.Hi * a.Wi;
        const void *f = sh.elt == 4 ? (const void *)&transform_pieces3<4> : (const void *)&transform_pieces3<2>;
        return hipLaunchKernel(f, dim3((uint32_t)blocks), dim3(kThreads), args, 0, st);
    }
    // gather: element indices fit 32 bits (transform_range_ok)
    const void *f = sh.elt == 4 ? (const void *)&transform_gather<4> : (const void *)&transform_gather<2>;
    return hipLaunchKernel(f, dim3((uint32_t)blocks), dim3(kThreads), args, 0, st);
}

}  // namespace im2win
