// fp32 windowed convolution on the gfx950 matrix cores (an alternate fp32
// path beside the vector-ALU one; Sec. III-C, Eq. 3 computed as the product
// of Alg. 1).
//
// The output is D[j][p] = sum_k F'[j][k] * Wn[p][k] (M = C_o, N = pixels,
// K = K_h*K_w*C_i) in fp32 with v_mfma_f32_32x32x2_f32: fp32 operands, fp32
// accumulation.  Everything around the multiply follows the row-per-pixel
// fp16 kernel: a stage is 32 taps (128 bytes) of the workgroup's BM filter
// rows and BN window rows, fetched with buffer_load ... lds into a ring of
// NS slots, rows XOR-swizzled in 16-byte chunks.
//
// Operands: one 16-byte LDS read gives a lane four consecutive taps of its
// row.  For the 8 taps of chunk pair (2g, 2g+1), lanes 0-31 read chunk 2g and
// lanes 32-63 chunk 2g+1, and MFMA t (t < 4) takes element t of each: it sums
// taps 8g+t and 8g+4+t.  A and B use the same assignment, so the four MFMAs
// cover the eight taps exactly once; only the order of the fp32 additions
// differs from a tap-by-tap sum.
//
// Windows must start on 16-byte boundaries and hold whole 16-byte chunks
// (C_i a multiple of 4); the launcher sends other layers to the vector-ALU
// kernels.
#include "common.hpp"

#include <stdlib.h>
#include <string.h>

namespace im2win {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void *lds_ptr;

constexpr int BK = 32;  // taps per stage (128-byte rows)

struct M32Args {
    const float *ws;      // window tensor
    const float *packed;  // [K_pad/32][C_o_pad][32]
    float *out;
    uint64_t win_bytes;
    uint32_t pk_bytes;
    uint32_t P, K, K_pad, Co, Co_pad, Wo, L;
    WinCols wc;
    TileGrid tg;          // pixel x channel tiles of the 1-D launch
    FastDiv div_Wo;
    TapOrder to;          // order of the 32-tap stages
};

// Filter repack: element (tile, j, t) = F'[j][tile*32 + t] with
// F'[j][(v*K_h + u)*C_i + r] = F[u][v][r][j] (window tap order), zero for
// j >= C_o or a tap past K.  One thread per 16-byte granule.
struct P32Args {
    const float *filt;
    float *packed;
    uint64_t grans;
    uint32_t K, Co, Co_pad, Ci, Kh, Kw;
};

__global__ __launch_bounds__(256) void pack_filter_fp32_mfma(P32Args a)
{
    for (uint64_t g = (uint64_t)blockIdx.x * 256 + threadIdx.x; g < a.grans; g += (uint64_t)gridDim.x * 256) {
        const uint64_t e0 = g * 4;
        const uint32_t t0 = (uint32_t)(e0 % BK);
        const uint64_t q = e0 / BK;
        const uint32_t j = (uint32_t)(q % a.Co_pad);
        const uint32_t tile = (uint32_t)(q / a.Co_pad);
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t k = tile * BK + t0 + e;
            float x = 0.f;
            if (j < a.Co && k < a.K) {
                const uint32_t khci = a.Kh * a.Ci;
                const uint32_t fv = k / khci, rem = k % khci;
                const uint32_t u = rem / a.Ci, r = rem % a.Ci;
                x = a.filt[(((uint64_t)u * a.Kw + fv) * a.Ci + r) * a.Co + j];
            }
            v[e] = x;
        }
        *reinterpret_cast<float4 *>(a.packed + g * 4) = make_float4(v[0], v[1], v[2], v[3]);
    }
}

// KS: the waves of a tile split the taps of every stage (each takes one of the
// four chunk pairs, and their sums are added through LDS at the end).
template <int WM_, int WN_, int WGM_, int WGN_, int NS_, int KS_ = 1>
struct MCfg {
    static constexpr int WM = WM_, WN = WN_, WGM = WGM_, WGN = WGN_, NS = NS_, KS = KS_;
    static_assert(KS == 1 || KS == BK / 8, "one chunk pair per wave, or all");
    static constexpr int NW = WGM * WGN * KS, NT = 64 * NW;
    static constexpr int BM = 32 * WM * WGM;     // channels per workgroup
    static constexpr int BN = 32 * WN * WGN;     // pixels per workgroup
    static constexpr int ROWS = BM + BN;
    static constexpr int STAGE = ROWS * 128;     // bytes per stage
    static constexpr int BLOCKS = ROWS / 8;      // 1 KiB (8-row) blocks per stage
    static_assert(BLOCKS % NW == 0, "blocks split evenly over the waves");
    static constexpr int I = BLOCKS / NW;        // loads per wave per stage
    static_assert(NS >= 2 && NS <= 4, "ring depth");
    static_assert((NS - 2) * I <= 63, "vmcnt range");
    static constexpr int PART = WM * WN * 4096;  // bytes of a wave's sums
    static constexpr int PPS = STAGE / PART;     // such parts per slot
    static_assert(KS == 1 || (WGM * WGN == 1 && NS * PPS >= KS), "the waves' sums fit the ring");
};

template <int VM>
__device__ inline void wait_vmcnt()
{
    __builtin_amdgcn_s_waitcnt((VM & 15) | ((VM >> 4) << 14) | (7 << 4) | (15 << 8));
}

// 16-byte chunk c of row r sits in slot c ^ rsw(r): the 16 lanes that read
// one chunk of 16 consecutive rows touch 16 different slots of the 64 banks.
__device__ inline uint32_t rsw(uint32_t r) { return (r ^ (r >> 3)) & 7u; }

template <class C>
struct MTile {
    __amdgpu_buffer_rsrc_t rf, rw;
    uint32_t voff[C::I];    // byte offset of this lane's chunk at tap 0 (kOOB: no pixel)
    uint32_t vtap[C::I];    // first tap of this lane's chunk within a stage
    uint32_t wave, lane, K, nst, apitch, arow, brow;
    TapOrder to;
    floatx16 acc[C::WM][C::WN];

    // Stage s >= nst loads nothing (zero-filled).
    __device__ inline void issue(uint32_t st, char *slot)
    {
        // first tap of the stage (column order only when every stage is
        // whole), which is filter tile k0 / 32
        const uint32_t k0 = to.map(st * BK), fadd = k0 / BK * apitch;
        const bool past = st >= nst;
#pragma unroll
        for (int j = 0; j < C::I; ++j) {
            const uint32_t b = wave + C::NW * j;
            const bool filt = b < (uint32_t)C::BM / 8;
            uint32_t off = voff[j] + (filt ? fadd : 4u * k0);
            if (past || (!filt && k0 + vtap[j] >= K))
                off = kOOB;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(filt ? rf : rw, (lds_ptr)(slot + 1024 * b), 16, off, 0, 0, 0);
        }
    }

    __device__ inline void frags(const char *slot, int g, floatx4 (&af)[C::WM], floatx4 (&bf)[C::WN])
    {
        const uint32_t ch = 2 * g + (lane >> 5);
#pragma unroll
        for (int i = 0; i < C::WM; ++i) {
            const uint32_t r = arow + 32 * i;
            af[i] = *reinterpret_cast<const floatx4 *>(slot + r * 128 + 16u * (ch ^ rsw(r)));
        }
#pragma unroll
        for (int j = 0; j < C::WN; ++j) {
            const uint32_t r = brow + 32 * j;
            bf[j] = *reinterpret_cast<const floatx4 *>(slot + r * 128 + 16u * (ch ^ rsw(r)));
        }
    }

    // The four chunk pairs of a stage; the next pair's operands are read
    // before the current pair's 4*WM*WN matrix operations.
    __device__ inline void compute(const char *slot)
    {
        floatx4 af[2][C::WM], bf[2][C::WN];
        if constexpr (C::KS > 1) {
            frags(slot, (int)wave, af[0], bf[0]);
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < C::WM; ++i)
#pragma unroll
                    for (int j = 0; j < C::WN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[0][i][t], bf[0][j][t], acc[i][j], 0, 0, 0);
            return;
        }
        frags(slot, 0, af[0], bf[0]);
#pragma unroll
        for (int g = 0; g < BK / 8; ++g) {
            if (g + 1 < BK / 8)
                frags(slot, g + 1, af[(g + 1) & 1], bf[(g + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < C::WM; ++i)
#pragma unroll
                    for (int j = 0; j < C::WN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[g & 1][i][t], bf[g & 1][j][t],
                                                                         acc[i][j], 0, 0, 0);
        }
    }

    // Ring slots are separate LDS arrays named at compile time, so reading
    // the current slot does not wait for the loads landing in the next.
    template <int N>
    __device__ inline void step(uint32_t st, char (&cur)[N], char (&next)[N])
    {
        wait_vmcnt<(C::NS - 2) * C::I>();
        ring_barrier();
        issue(st + C::NS - 1, next);
        if (st < nst)
            compute(cur);
    }
};

template <class C>
__global__ __launch_bounds__(C::NT) void conv_fp32_mfma(M32Args a)
{
    constexpr int S2 = C::NS > 2 ? C::STAGE : 1024, S3 = C::NS > 3 ? C::STAGE : 1024;
    __shared__ __attribute__((aligned(1024))) char r0[C::STAGE];
    __shared__ __attribute__((aligned(1024))) char r1[C::STAGE];
    __shared__ __attribute__((aligned(1024))) char r2[S2];
    __shared__ __attribute__((aligned(1024))) char r3[S3];
    // Window offsets of the tile's pixels, in the slot that is loaded last (the
    // first load into it follows a barrier that follows every read of them):
    // an array of its own would take the 64 x 256 tile past half of the
    // 160 KiB LDS, one workgroup per CU instead of two (7x7 C=64 stride 2 at
    // 224x224, 128 images: 5123 -> 4791 us together with the column order of
    // launch_conv_fp32_mfma and the tile that mfma32_default takes).
    uint32_t *const rowoff = reinterpret_cast<uint32_t *>(C::NS > 3 ? r3 : C::NS > 2 ? r2 : r1);

    MTile<C> w;
    const uint32_t tid = threadIdx.x;
    w.lane = tid & 63;
    w.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    __builtin_assume(w.wave < (uint32_t)C::NW);
    w.K = a.K;
    w.to = a.to;
    w.nst = a.K_pad / BK;
    const uint32_t wt = C::KS > 1 ? 0u : w.wave;  // with the taps split, every wave has the whole tile
    const uint32_t wm = wt / C::WGN, wn = wt % C::WGN;
    uint32_t tx, ty;
    a.tg.tile(tx, ty);
    const uint32_t p0 = tx * C::BN;
    const uint32_t ch0 = ty * C::BM;

    // windows from the strip of p0 on; the packed filter from row ch0 of tile 0
    const uint32_t q0 = fdiv(p0, a.div_Wo);
    const uint64_t tb = (uint64_t)q0 * a.L;
    const uint64_t left = a.win_bytes - tb * 4;
    w.rw = make_rsrc(a.ws + tb, (uint32_t)(left < kMaxRecords ? left : kMaxRecords));
    w.rf = make_rsrc(a.packed + (uint64_t)ch0 * BK, a.pk_bytes - ch0 * (uint32_t)BK * 4u);
    w.apitch = a.Co_pad * (uint32_t)BK * 4u;
    for (uint32_t t = tid; t < (uint32_t)C::BN; t += C::NT) {
        const uint32_t p = p0 + t;
        uint32_t off = 0;
        if (p < a.P) {
            const uint32_t q = fdiv(p, a.div_Wo);
            off = (q - q0) * a.L + a.wc.start(p - q * a.Wo);
        }
        rowoff[t] = off;
    }
    __syncthreads();

    // Lane L of a load fills LDS slot L & 7 of row 8*block + L/8 with chunk
    // (L & 7) ^ rsw(row) of that row (rows counted from the first filter row).
    const uint32_t rib = w.lane >> 3, slot = w.lane & 7;
#pragma unroll
    for (int j = 0; j < C::I; ++j) {
        const uint32_t b = w.wave + C::NW * j;
        if (b < (uint32_t)C::BM / 8) {
            const uint32_t row = 8 * b + rib;
            const uint32_t c = slot ^ rsw(row);
            w.voff[j] = row * (uint32_t)BK * 4u + 16u * c;
            w.vtap[j] = 4 * c;
        } else {
            const uint32_t row = 8 * (b - C::BM / 8) + rib;
            const uint32_t c = slot ^ rsw(C::BM + row);
            w.voff[j] = (p0 + row < a.P) ? rowoff[row] * 4u + 16u * c : kOOB;
            w.vtap[j] = 4 * c;
        }
    }
    w.arow = wm * 32 * C::WM + (w.lane & 31);
    w.brow = C::BM + wn * 32 * C::WN + (w.lane & 31);
#pragma unroll
    for (int i = 0; i < C::WM; ++i)
#pragma unroll
        for (int j = 0; j < C::WN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                w.acc[i][j][e] = 0.f;

    w.issue(0, r0);
    if constexpr (C::NS == 2) {
        for (uint32_t st = 0; st < w.nst; st += 2) {
            w.step(st, r0, r1);
            w.step(st + 1, r1, r0);
        }
    } else if constexpr (C::NS == 3) {
        w.issue(1, r1);
        for (uint32_t st = 0; st < w.nst; st += 3) {
            w.step(st, r0, r2);
            w.step(st + 1, r1, r0);
            w.step(st + 2, r2, r1);
        }
    } else {
        w.issue(1, r1);
        w.issue(2, r2);
        for (uint32_t st = 0; st < w.nst; st += 4) {
            w.step(st, r0, r3);
            w.step(st + 1, r1, r0);
            w.step(st + 2, r2, r1);
            w.step(st + 3, r3, r2);
        }
    }
    wait_vmcnt<0>();  // no load may still be writing LDS when the workgroup ends

    if constexpr (C::KS > 1) {
        // the waves' sums as 16-byte quads [block][quad][lane], PPS parts per
        // ring slot; wave q then adds quad q of every block in wave order and
        // stores it
        __syncthreads();
        auto part = [&](uint32_t k) {
            const uint32_t s = k / C::PPS;
            char *slot = s == 0 ? r0 : s == 1 ? r1 : r2;
            if constexpr (C::NS > 3)
                slot = s == 3 ? r3 : slot;
            return reinterpret_cast<float4 *>(slot + k % C::PPS * C::PART);
        };
        float4 *mine = part(w.wave);
#pragma unroll
        for (int i = 0; i < C::WM; ++i)
#pragma unroll
            for (int j = 0; j < C::WN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    mine[((i * C::WN + j) * 4 + q) * 64 + w.lane] =
                        make_float4(w.acc[i][j][4 * q], w.acc[i][j][4 * q + 1], w.acc[i][j][4 * q + 2],
                                    w.acc[i][j][4 * q + 3]);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < C::WM; ++i)
#pragma unroll
            for (int j = 0; j < C::WN; ++j) {
                const uint32_t at = ((i * C::WN + j) * 4 + w.wave) * 64 + w.lane;
                float4 s = part(0)[at];
#pragma unroll
                for (uint32_t k = 1; k < 4; ++k) {
                    const float4 v = part(k)[at];
                    s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
                }
                const uint32_t p = p0 + 32 * j + (w.lane & 31), c = ch0 + 32 * i + 8 * w.wave + 4 * (w.lane >> 5);
                if (p >= a.P)
                    continue;
                float *o = a.out + (uint64_t)p * a.Co + c;
                if (c + 3 < a.Co && (a.Co & 3) == 0) {
                    *reinterpret_cast<float4 *>(o) = s;
                } else {
                    const float v[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (c + e < a.Co)
                            o[e] = v[e];
                }
            }
        return;
    }

    // Lane holds pixel pb + 32*j + (lane & 31) and, for accumulator element e
    // of block (i, j), channel cb + 32*i + 8*(e/4) + 4*(lane/32) + e%4: four
    // consecutive channels per 16-byte store.
    const uint32_t pb = p0 + wn * 32 * C::WN, cb = ch0 + wm * 32 * C::WM;
#pragma unroll
    for (int j = 0; j < C::WN; ++j) {
        const uint32_t p = pb + 32 * j + (w.lane & 31);
        if (p >= a.P)
            continue;
        float *o = a.out + (uint64_t)p * a.Co;
#pragma unroll
        for (int i = 0; i < C::WM; ++i) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const uint32_t c = cb + 32 * i + 8 * g + 4 * (w.lane >> 5);
                const floatx16 &v = w.acc[i][j];
                if (c + 3 < a.Co && (a.Co & 3) == 0) {
                    *reinterpret_cast<float4 *>(o + c) =
                        make_float4(v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (c + e < a.Co)
                            o[c + e] = v[4 * g + e];
                }
            }
        }
    }
}

struct MVariant {
    const char *name;
    const void *f;
    int bm, bn, nt;
    int weight;  // time of a sum beside the 128 x 128 tile's, percent
    int few;     // tiles up to which a CU's loads stay uncovered, and what that costs, percent
    int alone;
    int start;   // what a tile costs before its first tap, in taps (windows shorter than kShortTaps)
};

constexpr int64_t kShortTaps = 128;

template <int WM, int WN, int WGM, int WGN, int NS, int KS = 1>
MVariant m_variant(const char *name, int weight, int few = 256, int alone = 106, int start = 0)
{
    using C = MCfg<WM, WN, WGM, WGN, NS, KS>;
    return MVariant{name, (const void *)&conv_fp32_mfma<C>, C::BM, C::BN, C::NT, weight, few, alone, start};
}

const MVariant *m_variants(int *n)
{
    // channels x pixels per workgroup, ring slots.  Weights: 3x3 64 -> 128 at
    // 112x112 (6050 tiles of 128 x 128: 1826 us; 64-row tiles 1880, 32 x 128
    // 1977, 32 x 256 2031), the tap-split ones against those at even balance.
    // One workgroup per CU leaves its barriers and load waits uncovered (1x1 140
    // -> 313 at 18x18, 15 images: 190 tiles 17.7 us, 380 half as large 16.2),
    // and the two-slot tap-split tile wants more than two (392 tiles 36.3
    // against 33.2 with four slots, 1520 14.7 against 15.9).
    static const MVariant v[] = {
        m_variant<2, 2, 2, 2, 2>("c128p128s2", 100),
        m_variant<2, 2, 1, 4, 2>("c64p256s2", 103),
        m_variant<1, 2, 1, 4, 2>("c32p256s2", 111),
        // smaller tiles for layers with few output pixels
        m_variant<1, 2, 2, 2, 2>("c64p128s2", 103),
        m_variant<1, 1, 1, 4, 2>("c32p128s2", 108),
        // the taps of a stage split over four waves (small grids)
        m_variant<1, 1, 1, 1, 4, 4>("c32p32s4t4", 116, 256, 106, 30),
        m_variant<1, 1, 1, 1, 2, 4>("c32p32s2t4", 114, 512, 112, 20),
        m_variant<2, 1, 1, 1, 4, 4>("c64p32s4t4", 111, 256, 106, 30),
    };
    *n = (int)(sizeof v / sizeof v[0]);
    return v;
}

int64_t co_pad_mfma(int64_t Co) { return round_up(Co, 128); }
int64_t k_pad_mfma(int64_t K) { return round_up(K, BK); }

}  // namespace

bool fp32_mfma_ok(const Shape &sh)
{
    // whole 16-byte chunks per window, 31-bit offsets into the packed filter,
    // and every window byte offset of a 256-pixel tile (its strips plus one
    // window) below the out-of-range marker
    const int64_t strips_per_tile = (256 - 1) / sh.Wo + 2;
    return sh.Ci % 4 == 0 && co_pad_mfma(sh.Co) * k_pad_mfma(sh.K) * 4 < (int64_t)kMaxRecords &&
           (strips_per_tile * sh.L + k_pad_mfma(sh.K)) * 4 < (int64_t)kOOB;
}

int64_t fp32_mfma_packed_bytes(const Shape &sh) { return co_pad_mfma(sh.Co) * k_pad_mfma(sh.K) * 4; }

int mfma32_find(const char *name)
{
    int n;
    const MVariant *v = m_variants(&n);
    for (int t = 0; t < n; ++t)
        if (strcmp(name, v[t].name) == 0)
            return t;
    return -1;
}

const char *mfma32_name(int v)
{
    int n;
    return m_variants(&n)[v].name;
}

int mfma32_default(const Shape &sh)
{
    int n;
    const MVariant *v = m_variants(&n);
    // The matrix cores bound these tiles, and a CU's workgroups share them:
    // the time is that of the CU with the most tiles, ceil(tiles / 256) tiles
    // of bm x bn sums, times what the tile's operand reads cost beside a 128 x
    // 128 one's.  Against the largest tile with two workgroups per CU: 3x3
    // C=512 at 14x14 (576 / 2304 tiles) 848 -> 713 us, 3x3 C=256 at 14x14 226
    // -> 207, 1x1 C=1024 at 14x14 457 -> 437.  The tiles whose waves split the
    // taps fill the chip with the fewest pixels and come within 11 to 16 % of
    // the large ones at even balance (3x3 C=256 at 14x14, one image 55.6 ->
    // 24.9, 128 images 207 -> 191; 3x3 C=512 at 7x7, 128 images, 170 -> 157;
    // 5x5 40 -> 88 at 42x42, 3 images, 28.4 -> 17.5), but their first loads and
    // the sum over the waves are not repaid by a short window: `start` taps,
    // less of them the longer it is (1x1 16 -> 88, 29547 pixels: 11.7 us with
    // c32p32s2t4 against 9.3 with c32p128s2; 1x1 8 -> 288, 2880 pixels, 7.6
    // against 6.8).  Fitted to 2500 layers, of which 13 ran over a tenth slower
    // than with the largest tile of two workgroups per CU, and one does now.
    const int64_t k = k_pad_mfma(sh.K), lack = k < kShortTaps ? kShortTaps - k : 0;
    int best = 0;
    double least = -1.;
    for (int i = 0; i < n; ++i) {
        const int64_t tiles = ((sh.P + v[i].bn - 1) / v[i].bn) * ((sh.Co + v[i].bm - 1) / v[i].bm);
        const int64_t alone = tiles <= v[i].few ? v[i].alone : 100;
        const int64_t sums = (tiles + 255) / 256 * v[i].bm * v[i].bn;
        const double cost = (double)(sums * v[i].weight * alone) * (double)(k * kShortTaps + v[i].start * lack);
        if (least < 0. || cost < least) {
            best = i;
            least = cost;
        }
    }
    return best;
}

hipError_t launch_conv_fp32_mfma(const Shape &sh, const Plan32 &plan, const Tuning &t, const float *filt,
                                 void *packed, float *out, const void *ws, hipStream_t st)
{
    P32Args p;
    p.filt = filt;
    p.packed = static_cast<float *>(packed);
    p.K = (uint32_t)sh.K;
    p.Co = (uint32_t)sh.Co;
    p.Co_pad = (uint32_t)co_pad_mfma(sh.Co);
    p.Ci = (uint32_t)sh.Ci; p.Kh = (uint32_t)sh.Kh; p.Kw = (uint32_t)sh.Kw;
    p.grans = (uint64_t)p.Co_pad * k_pad_mfma(sh.K) / 4;
    uint64_t blocks = (p.grans + 255) / 256;
    if (blocks > 65536)
        blocks = 65536;
    void *pargs[] = {&p};
    hipError_t e = hipLaunchKernel((const void *)&pack_filter_fp32_mfma, dim3((uint32_t)blocks), dim3(256), pargs,
                                   0, st);
    if (e != hipSuccess)
        return e;

    int n;
    const MVariant *v = m_variants(&n);
    const int pick = plan.v;
    M32Args a;
    a.ws = static_cast<const float *>(ws);
    a.packed = p.packed;
    a.out = out;
    a.win_bytes = (uint64_t)sh.win_bytes;
    a.pk_bytes = (uint32_t)fp32_mfma_packed_bytes(sh);
    a.P = (uint32_t)sh.P; a.K = (uint32_t)sh.K; a.K_pad = (uint32_t)k_pad_mfma(sh.K);
    a.Co = (uint32_t)sh.Co; a.Co_pad = p.Co_pad;
    a.Wo = (uint32_t)sh.Wo; a.L = (uint32_t)sh.L;
    a.wc = make_wincols(sh);
    a.div_Wo = make_fastdiv((uint32_t)sh.Wo);
    // Column order where windows overlap with a stride: 7x7 stride 2 C=64 at
    // 224x224 is bound by re-reading its windows in linear order (64 x 256
    // tiles 5410 us against 4970, the default 64 x 128 ones 5264 against 4791
    // to 4960).  At stride 1 linear order is ahead: 3x3 C=64 at 56x56 253
    // against 266, 3x3 C=512 at 7x7 177 against 192, 3x3 64 -> 128 at 112x112
    // 1770 against 1800.
    const bool linear = t.tap_order == Tuning::kDefault ? sh.s == 1 || sh.Kw <= sh.s : t.tap_order == Tuning::kLinear;
    a.to = make_taporder(sh.Kw, sh.Kh, sh.Ci, (uint32_t)BK, linear, sh.s);
    const int64_t gx = (sh.P + v[pick].bn - 1) / v[pick].bn, gy = (sh.Co + v[pick].bm - 1) / v[pick].bm;
    if (gx * gy > 0x7fffffff)
        return hipErrorInvalidValue;
    a.tg = make_tilegrid(gx, gy, t.tile_linear);
    void *args[] = {&a};
    return hipLaunchKernel(v[pick].f, dim3((uint32_t)(gx * gy)), dim3(v[pick].nt), args, 0, st);
}

}  // namespace im2win
