// fp16 windowed convolution on the matrix cores for windows that are not
// 16-byte aligned (C_i*2 not a multiple of 16, e.g. the 3-channel stem
// layers), staged by strip segment (Sec. III-B..D, Eq. 3, Alg. 1).
//
// The windows of consecutive output columns of one strip are overlapping
// spans of that strip, S = s*K_h*C_i elements apart.  A tile of BN
// consecutive pixels touches at most RMAX strips; for each strip it needs one
// contiguous segment, from the first pixel's window start to the last
// pixel's window start + K_pad.  The kernel loads each segment once, as
// 16-byte granules from the granule that holds its first element
// (buffer_load ... lds: aligned loads, no element loads), keeps all of them in
// LDS for the whole K loop, and reads every pixel's MFMA operand from there at
// its own (2-byte aligned) offset.  The filter, packed stage-major (64-tap
// tiles of C_o_pad contiguous rows), streams through a two-slot ring.
//
// Taps past K: the filter rows are zero there, and the window values past a
// pixel's K taps (which belong to the next pixel) are cleared in registers,
// so they add exactly 0 and a non-finite neighbour cannot leak in.
#include "common.hpp"
#include "epilogue16.hpp"

#include <atomic>
#include <type_traits>

#include <stdlib.h>
#include <string.h>

namespace im2win {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void *lds_ptr;

constexpr int BK = 64;  // taps per filter stage

struct SegArgs {
    const uint16_t *ws;
    const uint16_t *packed;
    uint16_t *out;
    uint64_t pad_end;  // window tensor bytes plus the transform's zero pad
    uint32_t pk_bytes;
    uint32_t P, K, K_pad, Co, Co_pad, Wo, L, S;
    FastDiv div_Wo;
};

template <int WM_, int WN_, int WGM_, int WGN_, int GMAX_, int RMAX_>
struct SegCfg {
    static constexpr int WM = WM_, WN = WN_, WGM = WGM_, WGN = WGN_;
    static constexpr int NW = WGM * WGN, NT = 64 * NW;
    static constexpr int BM = 32 * WM * WGM, BN = 32 * WN * WGN;
    static constexpr int GMAX = GMAX_;  // 16-byte granules of window segments a tile may need
    static constexpr int RMAX = RMAX_;  // strips a tile may touch
    static constexpr bool SERIAL = false;  // see Serialized
    static constexpr int ASTAGE = BM * 128;        // filter rows of one stage
    static constexpr int IA = BM / 8 / NW;         // filter loads per wave per stage
    static constexpr int IBMAX = GMAX / 64 / NW;   // segment loads per wave, at most
    static_assert(BM % (8 * NW) == 0, "filter blocks split evenly over the waves");
    static_assert(GMAX % (64 * NW) == 0, "segment blocks split evenly over the waves");
    static_assert(GMAX * 16 >= BM * BN * 2, "the epilogue tile fits the segment area");
    static_assert(RMAX >= 2 && RMAX <= 64 && (RMAX & (RMAX - 1)) == 0, "one lane per strip, scanned in log2 steps");
};

// The same tile with the filter ring serialized: a stage's filter loads are
// issued only after every wave has finished with the previous stage, so no
// load is in flight while LDS is read.  Same sums in the same order; a check
// variant for the ring's waits and barriers.
template <class Base>
struct Serialized : Base {
    static constexpr bool SERIAL = true;
};

__device__ inline uint32_t rsw(uint32_t r) { return (r ^ (r >> 3)) & 7u; }

template <int VM>
__device__ inline void wait_vmcnt()
{
    __builtin_amdgcn_s_waitcnt((VM & 15) | ((VM >> 4) << 14) | (7 << 4) | (15 << 8));
}

// E: the operand type (F16Op or BF16Op).
template <class C, class E>
struct SegTile {
    typedef typename E::v8 v8;
    __amdgpu_buffer_rsrc_t rf;
    uint32_t aoff[C::IA];  // filter byte offset at stage 0
    uint32_t bb[C::WN];    // LDS byte offset of each of this lane's pixels' window
    uint32_t wave, lane, wm, wn, K, nst, apitch;
    floatx16 acc[C::WM][C::WN];

    __device__ inline void issue_a(uint32_t st, char *slot)
    {
#pragma unroll
        for (int i = 0; i < C::IA; ++i) {
            const uint32_t b = wave + C::NW * i;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rf, (lds_ptr)(slot + 1024 * b), 16, aoff[i] + st * apitch,
                                                     0, 0, 0);
        }
    }

    // 16 bytes of LDS from a 2-byte-aligned offset.  An unaligned ds_read_b128
    // stalls the LDS pipe (~11 cycles per read measured on the 3-channel
    // stem); three aligned 8-byte reads of the span and a byte-align of each
    // dword in registers give the same bytes.
    __device__ static inline void read16(const char *lds, uint32_t o, v8 &dst)
    {
        const uint32_t base = o & ~7u, sh = o & 7u;
        const uint2 a0 = *reinterpret_cast<const uint2 *>(lds + base);
        const uint2 a1 = *reinterpret_cast<const uint2 *>(lds + base + 8);
        const uint2 a2 = *reinterpret_cast<const uint2 *>(lds + base + 16);
        const uint32_t w[6] = {a0.x, a0.y, a1.x, a1.y, a2.x, a2.y};
        const bool hi4 = sh >= 4;
        const uint32_t b = sh & 3u;
        uint32_t out[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t lo = hi4 ? w[i + 1] : w[i], hi = hi4 ? w[i + 2] : w[i + 1];
            out[i] = __builtin_amdgcn_alignbyte(hi, lo, b);
        }
        __builtin_memcpy(&dst, out, 16);
    }

    __device__ inline void compute(uint32_t st, const char *aslot, const char *seg)
    {
        const bool tail = st * BK + BK > K;
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            const uint32_t ch = 2 * ks + (lane >> 5);
            const uint32_t k = st * BK + 8 * ch;  // first of this lane's 8 taps
            v8 af[C::WM], bf[C::WN];
#pragma unroll
            for (int i = 0; i < C::WM; ++i) {
                const uint32_t r = wm * 32 * C::WM + 32 * i + (lane & 31);
                af[i] = *reinterpret_cast<const v8 *>(aslot + r * 128 + 16u * (ch ^ rsw(r)));
            }
#pragma unroll
            for (int j = 0; j < C::WN; ++j) {
                read16(seg, bb[j] + 2 * k, bf[j]);  // a window starts at any element
                if (tail) {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (k + e >= K)
                            bf[j][e] = (typename E::elem)0.f;
                }
            }
#pragma unroll
            for (int i = 0; i < C::WM; ++i)
#pragma unroll
                for (int j = 0; j < C::WN; ++j)
                    acc[i][j] = E::mfma(af[i], bf[j], acc[i][j]);
        }
    }
};

template <class C, class E>
__global__ __launch_bounds__(C::NT) void conv_fp16_seg(SegArgs a)
{
    __shared__ __attribute__((aligned(1024))) char r0[C::ASTAGE];
    __shared__ __attribute__((aligned(1024))) char r1[C::ASTAGE];
    // 16 bytes of slack: a fragment read spans up to 8 bytes past its 16
    __shared__ __attribute__((aligned(1024))) char seg[C::GMAX * 16 + 16];

    SegTile<C, E> w;
    const uint32_t tid = threadIdx.x;
    w.lane = tid & 63;
    w.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    __builtin_assume(w.wave < (uint32_t)C::NW);
    w.wm = w.wave / C::WGN;
    w.wn = w.wave % C::WGN;
    w.K = a.K;
    w.nst = a.K_pad / BK;
    const uint32_t p0 = blockIdx.x * C::BN;
    const uint32_t ch0 = blockIdx.y * C::BM;
    const uint32_t q0 = fdiv(p0, a.div_Wo);
    const uint32_t plast = (p0 + C::BN < a.P ? p0 + C::BN : a.P) - 1;

    // Segments: one per strip q0 + t the tile touches (t < RMAX), measured in
    // elements from the start of strip q0 and begun at the granule holding
    // the first pixel's window start; their granules are laid out one after
    // another in `seg`.  Every wave builds the table itself, lane t holding
    // strip t: cnt = its granules, gb = granules of the strips before it, and
    // rel = (first element of its segment) - 8*gb, so that element e of strip
    // run t sits at LDS element e - rel.
    uint32_t cnt = 0, rel = 0;
    if (w.lane < (uint32_t)C::RMAX) {
        const uint32_t q = q0 + w.lane;
        const uint32_t pf = q * a.Wo > p0 ? q * a.Wo : p0;  // first pixel of the tile in strip q
        const uint32_t pe = (q + 1) * a.Wo - 1 < plast ? (q + 1) * a.Wo - 1 : plast;
        if (pf <= pe) {
            const uint32_t s0 = w.lane * a.L + (pf - q * a.Wo) * a.S;
            const uint32_t s1 = w.lane * a.L + (pe - q * a.Wo) * a.S + a.K_pad;
            rel = s0 & ~7u;
            cnt = (s1 - rel + 7) / 8;
        }
    }
    uint32_t inc = cnt;  // inclusive prefix sum over the lanes
#pragma unroll
    for (int d = 1; d < C::RMAX; d <<= 1) {
        const uint32_t v = __shfl_up(inc, d, 64);
        if (w.lane >= (uint32_t)d)
            inc += v;
    }
    rel -= 8 * (inc - cnt);  // unsigned wrap-around is intended
    const uint32_t G = __builtin_amdgcn_readlane(inc, C::RMAX - 1);
    uint32_t gb[C::RMAX];  // first granule of each strip run (wave-uniform)
#pragma unroll
    for (int t = 0; t < C::RMAX; ++t)
        gb[t] = __builtin_amdgcn_readlane(inc - cnt, t);

    const uint64_t tb = (uint64_t)q0 * a.L;
    // granules reach up to 7 elements past a window's end: the zero pad
    // after the window tensor keeps them inside the workspace
    const uint64_t left = a.pad_end - tb * 2;
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(a.ws + tb, (uint32_t)(left < kMaxRecords ? left : kMaxRecords));
    w.rf = make_rsrc(a.packed + (uint64_t)ch0 * BK, a.pk_bytes - ch0 * (uint32_t)BK * 2u);
    w.apitch = a.Co_pad * (uint32_t)BK * 2u;

    // Segment loads: instruction i of this wave fills granules
    // 64*(wave + NW*i) .. +63; those past G read nothing (zero fill).
#pragma unroll
    for (int i = 0; i < C::IBMAX; ++i) {
        const uint32_t blk = w.wave + C::NW * i;
        if (blk * 64 >= G)
            break;  // uniform: the wave's remaining blocks are all past G
        const uint32_t g = blk * 64 + w.lane;
        uint32_t r = 0;
#pragma unroll
        for (int t = 1; t < C::RMAX; ++t)
            r += g >= gb[t] ? 1u : 0u;
        const uint32_t rl = __shfl(rel, (int)r, 64);
        const uint32_t off = g < G ? (rl + 8 * g) * 2u : kOOB;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_ptr)(seg + 1024 * blk), 16, off, 0, 0, 0);
    }
    // filter loads: lane -> row 8*blk + lane/8, 16-byte chunk (lane%8)^rsw(row)
#pragma unroll
    for (int i = 0; i < C::IA; ++i) {
        const uint32_t blk = w.wave + C::NW * i;
        const uint32_t row = 8 * blk + w.lane / 8;
        const uint32_t c = (w.lane % 8) ^ rsw(row);
        w.aoff[i] = (row * (uint32_t)BK + 8 * c) * 2u;
    }
    // this lane's pixels: LDS offset of the window start
#pragma unroll
    for (int j = 0; j < C::WN; ++j) {
        const uint32_t p = p0 + w.wn * 32 * C::WN + 32 * j + (w.lane & 31);
        // a pixel past P reads from granule 0 (its result is never stored)
        const bool live = p < a.P;
        const uint32_t q = live ? fdiv(p, a.div_Wo) : q0;
        const uint32_t r = q - q0;
        const uint32_t rl = __shfl(rel, (int)r, 64);
        const uint32_t el = r * a.L + (p - q * a.Wo) * a.S;
        w.bb[j] = live ? (el - rl) * 2u : 0u;
    }
#pragma unroll
    for (int i = 0; i < C::WM; ++i)
#pragma unroll
        for (int j = 0; j < C::WN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                w.acc[i][j][e] = 0.f;

    w.issue_a(0, r0);
    // two-slot filter ring: wait for stage st (and, at st = 0, the
    // segments), then load stage st+1 into the other slot, then multiply
    if constexpr (C::SERIAL) {
        for (uint32_t st = 0; st < w.nst; st += 2) {
            wait_vmcnt<0>();
            ring_barrier();
            w.compute(st, r0, seg);
            ring_barrier();
            if (st + 1 < w.nst) {
                w.issue_a(st + 1, r1);
                wait_vmcnt<0>();
                ring_barrier();
                w.compute(st + 1, r1, seg);
                ring_barrier();
                if (st + 2 < w.nst)
                    w.issue_a(st + 2, r0);
            }
        }
    } else {
        for (uint32_t st = 0; st < w.nst; st += 2) {
            wait_vmcnt<0>();
            ring_barrier();
            if (st + 1 < w.nst)
                w.issue_a(st + 1, r1);
            w.compute(st, r0, seg);
            if (st + 1 < w.nst) {
                wait_vmcnt<0>();
                ring_barrier();
                if (st + 2 < w.nst)
                    w.issue_a(st + 2, r0);
                w.compute(st + 1, r1, seg);
            }
        }
    }
    wait_vmcnt<0>();

    store_tile_lds<E, C::WM, C::WN, C::WGM, C::WGN>(w.acc, seg, a.out, a.P, a.Co, p0, ch0, w.wm, w.wn, w.lane,
                                                 tid);
}

struct SegVariant {
    const char *name;
    const void *f[2];  // fp16 and bf16 operands
    int bm, bn, gmax, rmax, nt;
};

template <int WM, int WN, int WGM, int WGN, int GMAX, int RMAX, bool SERIAL = false>
SegVariant seg_variant(const char *name)
{
    using B = SegCfg<WM, WN, WGM, WGN, GMAX, RMAX>;
    using C = typename std::conditional<SERIAL, Serialized<B>, B>::type;
    return SegVariant{name, {(const void *)&conv_fp16_seg<C, F16Op>, (const void *)&conv_fp16_seg<C, BF16Op>}, C::BM,
                      C::BN, GMAX, RMAX, C::NT};
}

const SegVariant *seg_variants(int *n)
{
    // name: channels x pixels per tile
    static const SegVariant v[] = {
        seg_variant<2, 2, 1, 4, 2560, 16>("s64p256"),
        seg_variant<3, 1, 1, 4, 2560, 16>("s96p128"),
        seg_variant<2, 2, 2, 2, 2560, 16>("s128p128"),
        // a 16 KiB segment area (more workgroups per CU) for short windows
        seg_variant<2, 1, 1, 4, 1024, 16>("s64p128g1024"),
        // serialized filter ring (check variant)
        seg_variant<2, 2, 1, 4, 2560, 16, true>("s64p256-serial"),
    };
    *n = (int)(sizeof v / sizeof v[0]);
    return v;
}

// Granules a tile of bn consecutive pixels needs at most.  A tile split into
// `runs` strip runs of c_1 + ... + c_runs = bn pixels needs, per run,
// (c - 1)*S + K_pad elements from a start rounded down by at most 7, i.e. at
// most ((c - 1)*S + K_pad + 14) / 8 granules; summed over the runs that is at
// most ((bn - runs)*S + runs*(K_pad + 14)) / 8.  The number of runs can be
// anything from 1 to runs_max, so the bound takes the largest.
int64_t seg_granules_needed(const Shape &sh, int bn, int64_t runs_max)
{
    int64_t worst = 0;
    for (int64_t runs = 1; runs <= runs_max && runs <= bn; ++runs) {
        const int64_t g = ((bn - runs) * sh.S + runs * (sh.K_pad + 14)) / 8;
        worst = g > worst ? g : worst;
    }
    return worst;
}

// ---------------------------------------------------------------------------
// The same strips, one wave at a time, with the filter kept in LDS.
//
// What bound the tiles above on the large stems is not the matrix cores (17 %
// busy on 11x11 stride 4) but their phases: every 128-pixel tile waits for its
// segments, streams the whole filter from L2 (74 KB beside 34 KB of windows)
// between barriers, and stores.  Here a persistent workgroup keeps the filter
// of its channels in LDS for good (transposed once from the caller's filter,
// so nothing is packed), and each of its eight waves works alone on blocks of
// 32 consecutive pixels of one strip: its segment is one span, loaded
// unaligned into registers a block ahead and written to the wave's LDS area,
// so that the span's first element is 16-byte aligned there.  Pixel n then
// starts 2*n*S bytes in, and its operand is read in AL-byte pieces, AL = 8, 4
// or 2 the largest that divides 2*S.  No barrier after the filter is loaded.
struct SegWArgs {
    const uint16_t *ws, *filt;
    uint16_t *out;
    uint32_t K, Co, Wo, Ci, Kh, Kw, S;
    uint64_t L;
    uint32_t nblk, wps;      // 32-pixel blocks in all and per strip
    uint32_t nks, pitch;     // 16-tap steps; bytes of a filter row in LDS (an odd number of 16-byte chunks)
    uint32_t segb;           // bytes of a wave's area
    FastDiv div_wps, div_khci, div_ci;
};

constexpr int kSegWWaves = 8;

// NG: 16-byte granules of a segment per lane; WPE: waves per SIMD the
// registers are held to.
template <class E, int WM, int NG, int AL, int WPE>
__global__ __launch_bounds__(64 * kSegWWaves, WPE) void conv_fp16_segw(SegWArgs a)
{
    typedef typename E::v8 v8;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t ch0 = blockIdx.y * (32 * WM);
    char *const area = smem + 32 * WM * a.pitch + wave * a.segb;

    uint32_t blk = blockIdx.x * kSegWWaves + wave;
    const uint32_t step = gridDim.x * kSegWWaves;
    u32x4 pre[NG];
    // granules of block b's span, from its first element (2-byte aligned) to
    // its last pixel's last step: at most 45 bytes past the last window
    auto load = [&](uint32_t b) {
        const uint32_t q = fdiv(b, a.div_wps), n0 = (b - q * a.wps) * 32;
        const uint32_t npx = a.Wo - n0 < 32 ? a.Wo - n0 : 32;
        const char *src = reinterpret_cast<const char *>(a.ws + (uint64_t)q * a.L + (uint64_t)n0 * a.S);
        const uint32_t need = ((npx - 1) * a.S + 16 * a.nks) * 2;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const uint32_t off = (g * 64 + lane) * 16;
            if (off < need)
                __builtin_memcpy(&pre[g], src + off, 16);
        }
    };
    if (blk < a.nblk)
        load(blk);

    // filter: row j, tap k at smem + j*pitch + 2*k; a thread moves 8 taps of a
    // channel pair.  Zero past K and past C_o.
    const uint32_t units = 16 * WM * a.nks * 2;
    for (uint32_t t = tid; t < units; t += 64 * kSegWWaves) {
        const uint32_t k8 = t / (16 * WM), cp = t - k8 * (16 * WM);
        const uint32_t ch = ch0 + 2 * cp;
        uint32_t k = 8 * k8, x[8];
        uint32_t v = fdiv(k, a.div_khci), rem = k - v * (a.Kh * a.Ci);
        uint32_t u = fdiv(rem, a.div_ci), r = rem - u * a.Ci;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            x[e] = 0u;
            if (k < a.K && ch < a.Co) {
                const uint16_t *src = a.filt + ((uint64_t)(u * a.Kw + v) * a.Ci + r) * a.Co + ch;
                if (ch + 1 < a.Co)
                    __builtin_memcpy(&x[e], src, 4);
                else
                    x[e] = *src;
            }
            ++k;
            if (++r == a.Ci) {
                r = 0;
                if (++u == a.Kh) {
                    u = 0;
                    ++v;
                }
            }
        }
        u32x4 lo, hi;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            lo[d] = __builtin_amdgcn_perm(x[2 * d + 1], x[2 * d], 0x05040100u);
            hi[d] = __builtin_amdgcn_perm(x[2 * d + 1], x[2 * d], 0x07060302u);
        }
        *reinterpret_cast<u32x4 *>(smem + (2 * cp) * a.pitch + 16 * k8) = lo;
        *reinterpret_cast<u32x4 *>(smem + (2 * cp + 1) * a.pitch + 16 * k8) = hi;
    }
    __syncthreads();

    const char *const arow = smem + (lane & 31) * a.pitch + 16 * (lane >> 5);
    const char *const brow = area + (lane & 31) * a.S * 2 + 16 * (lane >> 5);
    constexpr uint32_t SP = 64 * WM + 16;  // bytes of a staged output row
    for (; blk < a.nblk; blk += step) {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const uint32_t off = (g * 64 + lane) * 16;
            if (off < a.segb)
                *reinterpret_cast<u32x4 *>(area + off) = pre[g];
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the wave's span is in LDS
        wave_lds_handoff();
        if (blk + step < a.nblk)
            load(blk + step);

        floatx16 acc[WM];
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                acc[i][e] = 0.f;
        auto frags = [&](uint32_t ks, v8 (&af)[WM], u32x4 &b) {
#pragma unroll
            for (int i = 0; i < WM; ++i)
                af[i] = *reinterpret_cast<const v8 *>(arow + 32 * i * a.pitch + 32 * ks);
            const char *p = brow + 32 * ks;
            if constexpr (AL == 8) {
                const uint2 b0 = *reinterpret_cast<const uint2 *>(p), b1 = *reinterpret_cast<const uint2 *>(p + 8);
                b = u32x4{b0.x, b0.y, b1.x, b1.y};
            } else if constexpr (AL == 4) {
                const uint32_t *w = reinterpret_cast<const uint32_t *>(p);
                b = u32x4{w[0], w[1], w[2], w[3]};
            } else {
                // five aligned dwords, shifted by half a dword where the
                // pixel starts on one
                const uint32_t o = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char *)p;
                const uint32_t *w = reinterpret_cast<const uint32_t *>(p - (o & 2u));
                const uint32_t d[5] = {w[0], w[1], w[2], w[3], w[4]};
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    b[t] = __builtin_amdgcn_alignbyte(d[t + 1], d[t], o & 2u);
            }
        };
        v8 af[2][WM];
        u32x4 bf[2];
        frags(0, af[0], bf[0]);
        const uint32_t last = a.nks - 1;
        uint32_t ks = 0;
#pragma unroll 1
        for (; ks + 2 <= last; ks += 2) {
            frags(ks + 1, af[1], bf[1]);
#pragma unroll
            for (int i = 0; i < WM; ++i)
                acc[i] = E::mfma(af[0][i], __builtin_bit_cast(v8, bf[0]), acc[i]);
            frags(ks + 2, af[0], bf[0]);
#pragma unroll
            for (int i = 0; i < WM; ++i)
                acc[i] = E::mfma(af[1][i], __builtin_bit_cast(v8, bf[1]), acc[i]);
        }
        if (ks < last) {
#pragma unroll
            for (int i = 0; i < WM; ++i)
                acc[i] = E::mfma(af[0][i], __builtin_bit_cast(v8, bf[0]), acc[i]);
            frags(last, af[0], bf[0]);
        }
        // the last step: taps past K belong to the next pixel and are cleared
        const uint32_t k = 16 * last + 8 * (lane >> 5), nv = k < a.K ? a.K - k : 0u;
#pragma unroll
        for (uint32_t d = 0; d < 4; ++d)
            bf[0][d] &= (2 * d < nv ? 0xffffu : 0u) | (2 * d + 1 < nv ? 0xffff0000u : 0u);
#pragma unroll
        for (int i = 0; i < WM; ++i)
            acc[i] = E::mfma(af[0][i], __builtin_bit_cast(v8, bf[0]), acc[i]);

        // round once, stage the block as [pixel][channel] in the wave's area,
        // and store whole output rows
        wave_lds_handoff();
        const uint32_t q = fdiv(blk, a.div_wps), n0 = (blk - q * a.wps) * 32;
        const uint32_t npx = a.Wo - n0 < 32 ? a.Wo - n0 : 32;
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                uint32_t h[4];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    h[e] = E::bits(acc[i][4 * g + e]);
                *reinterpret_cast<uint2 *>(area + (lane & 31) * SP + (32 * i + 8 * g + 4 * (lane >> 5)) * 2) =
                    make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
            }
        __builtin_amdgcn_s_waitcnt(0xC07F);
        wave_lds_handoff();
        uint16_t *const o = a.out + ((uint64_t)q * a.Wo + n0) * a.Co + ch0;
#pragma unroll
        for (int t = 0; t < 2 * WM; ++t) {
            const uint32_t c = t * 64 + lane, px = c / (4 * WM), cc = 8 * (c - px * (4 * WM));
            const u32x4 v = *reinterpret_cast<const u32x4 *>(area + px * SP + 2 * cc);
            if (px >= npx || ch0 + cc >= a.Co)
                continue;
            uint16_t *d = o + (uint64_t)px * a.Co + cc;
            if (a.Co % 8 == 0) {
                *reinterpret_cast<u32x4 *>(d) = v;
            } else {
#pragma unroll
                for (uint32_t e = 0; e < 8; ++e)
                    if (ch0 + cc + e < a.Co)
                        d[e] = (uint16_t)(v[e / 2] >> (16 * (e % 2)));
            }
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);  // the rows are read before the next span lands on them
        wave_lds_handoff();
    }
}

struct SegWPlan {
    const char *name;
    int wm;
};

// Channels a workgroup keeps; the LDS the layer takes with them (0: more
// than there is), and 16-byte granules of a span per lane.
const SegWPlan kSegW[] = {{"w32", 1}, {"w64", 2}, {"w96", 3}, {"w128", 4}};
constexpr int kSegWN = 4;
constexpr int64_t kLds = 160 * 1024;
constexpr int kSegWSmall = 4, kSegWLarge = 11;

struct SegWDims {
    int64_t nks, pitch, segb, lds, grans;
};

SegWDims segw_dims(const Shape &sh, int wm)
{
    SegWDims d;
    d.nks = (sh.K + 15) / 16;
    d.pitch = d.nks * 32 + 16;  // 32*nks is an even number of chunks
    const int64_t npx = sh.Wo < 32 ? sh.Wo : 32;
    const int64_t span = round_up(((npx - 1) * sh.S + 16 * d.nks) * 2, 16);
    d.grans = (span / 16 + 63) / 64;
    // a pixel past the strip's last one reads from the area's other bytes:
    // 32 pixels' worth of them exist in every area
    const int64_t full = round_up((31 * sh.S + 16 * d.nks) * 2 + 4, 16);
    const int64_t stage = 32 * (64 * wm + 16);
    d.segb = full > stage ? full : stage;
    d.lds = 32 * wm * d.pitch + kSegWWaves * d.segb;
    return d;
}

// Kernel instances by [32-channel rows][large spans][AL 8, 4, 2].
template <class E, int WM, int NG, int WPE>
const void *segw_al(int al)
{
    return al == 0   ? (const void *)&conv_fp16_segw<E, WM, NG, 8, WPE>
           : al == 1 ? (const void *)&conv_fp16_segw<E, WM, NG, 4, WPE>
                     : (const void *)&conv_fp16_segw<E, WM, NG, 2, WPE>;
}

template <class E, int WM>
const void *segw_fn(bool large, int al)
{
    return large ? segw_al<E, WM, kSegWLarge, 2>(al) : segw_al<E, WM, kSegWSmall, WM <= 2 ? 4 : 2>(al);
}

template <class E>
const void *segw_fn(int wm, bool large, int al)
{
    return wm == 1   ? segw_fn<E, 1>(large, al)
           : wm == 2 ? segw_fn<E, 2>(large, al)
           : wm == 3 ? segw_fn<E, 3>(large, al)
                     : segw_fn<E, 4>(large, al);
}

// Workgroups of instance f (number id) that are resident at once with `lds`
// bytes of dynamic LDS.  The LDS limit is an attribute of the function, shared
// by the layers and host threads that run it: it is set to the CU's whole LDS,
// the same value whoever sets it, so that no thread lowers it between
// another's query and launch.  The last answer of every instance and device is
// kept (one 64-bit word: the LDS size and the workgroups for it), so that a
// repeated call asks the driver for the device alone.
hipError_t segw_resident(const void *f, int id, int64_t lds, int64_t *wgs)
{
    constexpr int kDevices = 64, kInstances = 2 * kSegWN * 2 * 3;
    static std::atomic<uint64_t> kept[kDevices][kInstances];
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return e;
    std::atomic<uint64_t> *const slot = dev >= 0 && dev < kDevices ? &kept[dev][id] : nullptr;
    const uint64_t k = slot ? slot->load(std::memory_order_acquire) : 0u;
    if (k >> 32 == (uint64_t)lds) {
        *wgs = (int64_t)(k & 0xffffffffu);
        return hipSuccess;
    }
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess)
        e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds);
    if (e == hipSuccess)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, 64 * kSegWWaves, (size_t)lds);
    if (e != hipSuccess)
        return e;
    *wgs = (int64_t)(cus > 0 ? cus : 1) * (per_cu > 0 ? per_cu : 1);
    if (slot)
        slot->store((uint64_t)lds << 32 | (uint64_t)*wgs, std::memory_order_release);
    return hipSuccess;
}

bool segw_fits(const Shape &sh, int w)
{
    const SegWDims d = segw_dims(sh, kSegW[w].wm);
    return sh.Ci % 8 != 0 && sh.d == 1 && d.grans <= kSegWLarge && d.lds <= kLds;
}

hipError_t launch_segw(const Shape &sh, int w, const void *ws, const uint16_t *filt, uint16_t *out, hipStream_t st,
                       Op16 op)
{
    const int wm = kSegW[w].wm;
    const SegWDims d = segw_dims(sh, wm);
    SegWArgs a;
    a.ws = static_cast<const uint16_t *>(ws);
    a.filt = filt;
    a.out = out;
    a.K = (uint32_t)sh.K; a.Co = (uint32_t)sh.Co; a.Wo = (uint32_t)sh.Wo;
    a.Ci = (uint32_t)sh.Ci; a.Kh = (uint32_t)sh.Kh; a.Kw = (uint32_t)sh.Kw; a.S = (uint32_t)sh.S;
    a.L = (uint64_t)sh.L;
    a.wps = (uint32_t)((sh.Wo + 31) / 32);
    a.nblk = (uint32_t)(sh.strips * a.wps);  // at most P
    a.nks = (uint32_t)d.nks; a.pitch = (uint32_t)d.pitch; a.segb = (uint32_t)d.segb;
    a.div_wps = make_fastdiv(a.wps);
    a.div_khci = make_fastdiv(a.Kh * a.Ci);
    a.div_ci = make_fastdiv(a.Ci);
    const bool large = d.grans > kSegWSmall;
    const int al = sh.S * 2 % 8 == 0 ? 0 : sh.S * 2 % 4 == 0 ? 1 : 2;
    const void *f = op == Op16::BF16 ? segw_fn<BF16Op>(wm, large, al) : segw_fn<F16Op>(wm, large, al);
    const int id = (((op == Op16::BF16) * kSegWN + wm - 1) * 2 + large) * 3 + al;
    int64_t wgs;
    const hipError_t e = segw_resident(f, id, d.lds, &wgs);
    if (e != hipSuccess)
        return e;
    // one resident round of workgroups over the channel groups
    const int64_t gy = (sh.Co + 32 * wm - 1) / (32 * wm), need = ((int64_t)a.nblk + kSegWWaves - 1) / kSegWWaves;
    int64_t gx = wgs / gy;
    gx = gx < 1 ? 1 : gx > need ? need : gx;
    void *args[] = {&a};
    return hipLaunchKernel(f, dim3((uint32_t)gx, (uint32_t)gy), dim3(64 * kSegWWaves), args, (size_t)d.lds, st);
}

}  // namespace

// Variants of the tiled kernel, then the one-wave kernel's by channels.
int seg_find(const char *name)
{
    int n;
    const SegVariant *v = seg_variants(&n);
    for (int t = 0; t < n; ++t)
        if (strcmp(name, v[t].name) == 0)
            return t;
    for (int t = 0; t < kSegWN; ++t)
        if (strcmp(name, kSegW[t].name) == 0)
            return n + t;
    return -1;
}

const char *seg_name(int v)
{
    int n;
    const SegVariant *t = seg_variants(&n);
    return v < n ? t[v].name : kSegW[v - n].name;
}

bool seg_reads_filter(int v)
{
    int n;
    seg_variants(&n);
    return v >= n;
}

bool seg_fits(const Shape &sh, int pick)
{
    int n;
    const SegVariant *v = seg_variants(&n);
    if (pick >= n && pick < n + kSegWN)
        return segw_fits(sh, pick - n);
    if (pick < 0 || pick >= n)
        return false;
    if (sh.d != 1)
        return false;  // strip segments assume windows s*K_h*C_i apart
    // strips a tile of bn pixels can touch, wherever it starts in a strip
    const int64_t runs = (v[pick].bn - 1 + sh.Wo - 1) / sh.Wo + 1;
    if (runs > v[pick].rmax || seg_granules_needed(sh, v[pick].bn, runs) > v[pick].gmax)
        return false;
    // byte offsets inside the tile's strips stay below the buffer limit, and
    // pixel indices of the strips after the tile's last one fit 32 bits
    if ((runs * sh.L + sh.K_pad + 8) * 2 >= (int64_t)kMaxRecords)
        return false;
    if (sh.P + (int64_t)v[pick].rmax * sh.Wo >= (int64_t)1 << 32)
        return false;
    return true;
}

int seg_default(const Shape &sh)
{
    if (sh.Ci % 8 == 0)
        return -1;  // 16-byte-aligned windows have their own kernels
    // The one-wave kernel wherever its filter rows and spans fit LDS (strips
    // of at least 8 pixels, a quarter of a block), conv call in us against
    // the tiled or register-staged kernel, each with its pack: 11x11 stride 4
    // 3 -> 96 at 227x227 76 -> 50, 7x7 stride 2 3 -> 64 at 227x227 115 -> 74
    // (16 images 20.8 -> 16.7), 5x5 stride 2 3 -> 96 37.6 -> 20.6; 3x3 52 ->
    // 51 at 81x81, 92 images, 253 -> 76; 5x5 25 -> 273 at 34x34 80 -> 54; 1x1
    // 100 -> 100 at 28x28 34.9 -> 25.3; 3x3 70 -> 150 at 14x14 29.5 -> 13.2.
    // A block costs about 3 + wm for wm 32-channel rows (reading its span and
    // storing it, against its matrix steps), so: few channel groups, little
    // padding, and enough blocks for the 2048 waves.
    if (sh.Wo >= 8) {
        int n, best = -1;
        int64_t least = 0;
        seg_variants(&n);
        const int64_t nblk = sh.strips * ((sh.Wo + 31) / 32);
        for (int w = 0; w < kSegWN; ++w) {
            if (!segw_fits(sh, w))
                continue;
            const int64_t groups = (sh.Co + 32 * kSegW[w].wm - 1) / (32 * kSegW[w].wm);
            const int64_t blocks = nblk * groups < 2048 ? 2048 : nblk * groups;
            const int64_t cost = blocks * (3 + kSegW[w].wm);
            if (best < 0 || cost < least) {
                best = n + w;
                least = cost;
            }
        }
        // Strips of at most 12 pixels (3/8 of a block) lose to the tiled and
        // register-staged kernels once windows are long and every wave has
        // many such blocks (32-channel pieces of them): 3x3 73 -> 536 with 10
        // pixels a strip, 11550 in all, 54.8 us against 29.1; 7x7 13 -> 344
        // with 9, 9954, 35.2 against 24.9.  With 300 to 500 taps and with
        // fewer blocks it is ahead as often as behind.
        if (best >= 0) {
            const int wm = kSegW[best - n].wm;
            const int64_t pieces = nblk * ((sh.Co + 32 * wm - 1) / (32 * wm)) * wm;
            if (sh.Wo > 12 || sh.K < 500 || pieces < 12288)
                return best;
        }
    }
    // C_o <= 64: 64 x 128 tiles with a 16 KiB segment area when the
    // segments fit it (five workgroups per CU instead of two: 7x7 s2 C_i=3
    // at 227x227 284 vs 245 TFLOP/s, 3x3 C_i=3 at 224x224 83 vs 79)
    if (sh.Co <= 64 && seg_fits(sh, seg_find("s64p128g1024")))
        return seg_find("s64p128g1024");
    const int pick = sh.Co <= 64 ? 0 : sh.Co <= 96 ? 1 : 2;
    return seg_fits(sh, pick) ? pick : -1;
}

hipError_t launch_conv_fp16_seg(const Shape &sh, int plan, const void *ws, const uint16_t *filt, const void *packed,
                                uint16_t *out, hipStream_t st, Op16 op)
{
    int n;
    const SegVariant *t = seg_variants(&n);
    if (plan >= n)
        return launch_segw(sh, plan - n, ws, filt, out, st, op);
    const SegVariant &v = t[plan];
    SegArgs a;
    a.ws = static_cast<const uint16_t *>(ws);
    a.packed = static_cast<const uint16_t *>(packed);
    a.out = out;
    a.pad_end = (uint64_t)sh.pad_end;
    a.pk_bytes = (uint32_t)(sh.Co_pad * sh.K_pad * 2);
    a.P = (uint32_t)sh.P; a.K = (uint32_t)sh.K; a.K_pad = (uint32_t)sh.K_pad;
    a.Co = (uint32_t)sh.Co; a.Co_pad = (uint32_t)sh.Co_pad;
    a.Wo = (uint32_t)sh.Wo; a.L = (uint32_t)sh.L; a.S = (uint32_t)sh.S;
    a.div_Wo = make_fastdiv((uint32_t)sh.Wo);
    void *args[] = {&a};
    dim3 grid((uint32_t)((sh.P + v.bn - 1) / v.bn), (uint32_t)((sh.Co + v.bm - 1) / v.bm));
    return hipLaunchKernel(v.f[op == Op16::BF16], grid, dim3(v.nt), args, 0, st);
}

}  // namespace im2win
