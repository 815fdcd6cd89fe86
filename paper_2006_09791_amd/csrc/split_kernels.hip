// Pointwise (1x1, stride 1, no padding) layers as a dense product on v_mfma_f32_16x16x32_bf16: fp32
// layers through the exact three-way split of split_common.h, bf16 layers as they are.
//
// Y[filter][pixel] = sum_c W[filter][c] X[c][pixel] per group; the pixels of all images are numbered flat,
// so no tile is padded for a plane's size.  Block = WM x WP waves, 16*MI*WM filters x 16*NI*WP pixels; the
// reduction runs over chunks of 32 channels (one instruction deep).
//
// What bounds it, at 128 filters x 128 pixels: a chunk is 3072 clocks of matrix work per SIMD for the two
// blocks of a compute unit (128 registers, 76 KB of LDS each), during which the LDS moves 2 x 18 KB per wave
// to the operands and 2 x 48 KB in; the two blocks cover each other's barriers, and the matrix unit is busy
// 0.60 of a compute unit's busy time, the LDS 0.38 (counters), at a clock of 1.84 GHz.  512 -> 1024 on 14x14,
// N = 256: 278 us = 189 TFLOP/s (572 us on the fp32 instruction); a register loop of the same products reaches 300.
//  - filters: in operand order; split at packing time (PRE): global -> LDS directly (no registers), the next
//    chunk's while this one multiplies (two buffers); or, filter matrices of up to 64 KB, as fp32 words that
//    are split on the way through registers;
//  - inputs: a thread loads 2 pixels x 4 channels of the next chunk into registers while this one
//    multiplies, splits them and writes them channel-innermost, [part][8 channels][pixel] units of 16
//    bytes.  Even and odd pixels lie apart (and 64 bytes off), so that the writes of a wave and the
//    operand reads each fall on all banks.
//
// The sum of a split product is not the fp32 sum where a part overflows or is multiplied by an infinity: a wave
// that finds a scaled sum that is not finite recomputes its outputs as plain fp32 sums.
#include <cstring>

#include "split_common.h"

namespace gspc {

struct TileSplit {
    int nchunks, mtiles;          // chunks of 32 channels; 16-filter tiles per group
    int oc_blocks, px_blocks;
    int pre;                      // fp32: the packed filters are split
    unsigned HW, npix;            // plane size, N * HW
    unsigned m_HW, m_ocb;
    unsigned x_bytes, w_bytes, y_bytes;
};
static_assert(sizeof(TileSplit) <= sizeof(((SplitPlan *)0)->data), "plan storage too small");

template <typename TIN> struct SplitTraits;
template <> struct SplitTraits<float> { static constexpr int parts = 3; };
template <> struct SplitTraits<uint16_t> { static constexpr int parts = 1; };

template <int MI, int NI, int WM, int WP, typename TIN, bool VO, bool PRE>
__global__ __launch_bounds__(64 * WM * WP, WM * WP / 2) void conv_mfma16s(ConvParams p, TileSplit t) {
    constexpr int NT = 64 * WM * WP, MT = MI * WM, PB = 16 * NI * WP;
    constexpr int NP = SplitTraits<TIN>::parts, ES = (int)sizeof(TIN);
    constexpr int HALF = PB / 2 + 4, PLANE = 2 * HALF;           // 16-byte units: even pixels, odd pixels
    constexpr unsigned A_BYTES = MT * NP * 1024, PART = 4 * PLANE * 16;
    constexpr int TS = PB / 2 * 8 / NT;                          // staging slots: pixel pair x 4 channels
    constexpr int AP = PRE ? MT * NP : MT;                       // filter pieces of a chunk: 64 lanes x 16 or 32 bytes
    constexpr int AS = (AP + WM * WP - 1) / (WM * WP);           // of them per wave
    static_assert(TS * NT == PB / 2 * 8, "whole staging slots");
    extern __shared__ f32x4 smem4[];
    char *bbuf = reinterpret_cast<char *>(smem4) + (PRE ? 2 : 1) * A_BYTES;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WP, wp = wave % WP;

    // Tiles: the blocks of one XCD (block % 8) take consecutive (pixel tile, filter block) pairs, filter
    // blocks innermost, so that the filter blocks of a pixel tile read it from that XCD's L2.
    const unsigned per = gridDim.x >> 3;
    const unsigned id = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (id >= (unsigned)(t.px_blocks * t.oc_blocks)) return;
    const unsigned pt = fast_div_any(id, t.oc_blocks, t.m_ocb), ob = id - pt * t.oc_blocks;
    const unsigned j = blockIdx.y;
    const unsigned q0 = pt * PB, n0 = fast_div_any(q0, t.HW, t.m_HW), r0 = q0 - n0 * t.HW;

    const __amdgpu_buffer_rsrc_t rx = make_rsrc(p.x, t.x_bytes);
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(p.ws, t.w_bytes);

    // ---- staging plan -------------------------------------------------------------------------
    const unsigned cstep = t.HW * ES;                            // bytes from channel to channel
    const unsigned xbase = (n0 * p.Cin + j * p.CPG) * cstep;
    // byte offset of pixel q0 + d in plane 0 of its image, relative to the first image's
    auto px_off = [&](unsigned d, unsigned planes, unsigned elem) -> unsigned {
        const unsigned r = r0 + d, img = fast_div(r, t.m_HW);
        return (img * (planes - 1) * t.HW + r) * elem;
    };
    // A wave's task: 32 pixel pairs x 8 channels; its lower lanes load channels 0-3, its upper lanes 4-7.
    unsigned xoff[TS][VO ? 1 : 2];
#pragma unroll
    for (int k = 0; k < TS; ++k) {
        const unsigned task = wave + k * (WM * WP), pg = task % (PB / 64), cg = task / (PB / 64);
#pragma unroll
        for (int i = 0; i < (VO ? 1 : 2); ++i) {
            const unsigned d = pg * 64 + (lane & 31) * 2 + i;
            xoff[k][i] = q0 + d < t.npix ? xbase + px_off(d, p.Cin, ES) + (8 * cg + (lane >> 5) * 4) * cstep : kOob;
        }
    }
    u32x2 xv[TS][4];
    auto fetch_x = [&](int ch) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < TS; ++k) {
            const int c0 = ch * 32 + 8 * (int)((wave + k * (WM * WP)) / (PB / 64)) + (lane >> 5) * 4;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                // channels past the group's carry zero weights; their inputs must be zeros too (0 * inf)
                const bool live = c0 + e < p.CPG;
                const unsigned so = (ch * 32 + e) * cstep;
                if (VO) {
                    const unsigned vo = live ? xoff[k][0] : kOob;
                    if (ES == 4)
                        xv[k][e] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rx, vo, so, 0));
                    else
                        xv[k][e].x = __builtin_amdgcn_raw_buffer_load_b32(rx, vo, so, 0);
                } else {
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const unsigned vo = live ? xoff[k][VO ? 0 : i] : kOob;
                        xv[k][e][i] = ES == 4 ? __builtin_amdgcn_raw_buffer_load_b32(rx, vo, so, 0)
                                              : (unsigned)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(rx, vo, so, 0);
                    }
                }
            }
        }
    };
    // The loaded values as operand units: split (or packed) two channels at a time, then the lower lanes'
    // second pixel is exchanged with the upper lanes' first one, which leaves every lane all eight channels
    // of one pixel: 16 bytes per part, written without bank conflicts.
    unsigned xs[2][2][NP];      // [pixel][channel pair][part]
    auto split_x = [&](int k, int i, int c) __attribute__((always_inline)) {
        if constexpr (NP == 3) {
            split3(__uint_as_float(xv[k][2 * c][i]) * kSplitScale, __uint_as_float(xv[k][2 * c + 1][i]) * kSplitScale, xs[i][c]);
        } else {
            // two pixels per dword when loaded together, one otherwise
            xs[i][c][0] = __builtin_amdgcn_perm(xv[k][2 * c + 1][VO ? 0 : i], xv[k][2 * c][VO ? 0 : i],
                                                VO && i ? 0x07060302u : 0x05040100u);
        }
    };
    auto write_x = [&](int k, int q) __attribute__((always_inline)) {
        const unsigned task = wave + k * (WM * WP), pg = task % (PB / 64), cg = task / (PB / 64);
        u32x4 u;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const auto r = __builtin_amdgcn_permlane32_swap(xs[0][c][q], xs[1][c][q], false, false);
            u[c] = r[0];
            u[2 + c] = r[1];
        }
        *reinterpret_cast<u32x4 *>(bbuf + q * PART + (cg * PLANE + (lane >> 5) * HALF + pg * 32 + (lane & 31)) * 16) = u;
    };
    auto put_x = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < TS; ++k) {
#pragma unroll
            for (int i = 0; i < 4; ++i) split_x(k, i >> 1, i & 1);
#pragma unroll
            for (int q = 0; q < NP; ++q) write_x(k, q);
        }
    };
    constexpr unsigned TILE = PRE ? NP * 1024 : 2048;            // packed bytes of a filter tile and chunk
    const unsigned wgrp = j * t.nchunks * t.mtiles * TILE;
    u32x4 wv[PRE ? 1 : AS][2];
    auto fetch_w = [&](int ch) __attribute__((always_inline)) {
        const unsigned so = wgrp + (ch * t.mtiles + ob * MT) * TILE;
#pragma unroll
        for (int k = 0; k < AS; ++k) {
            const unsigned piece = k * (WM * WP) + wave;
            if (AS * WM * WP != AP && piece >= AP) break;
            const bool live = (int)(ob * MT + piece / (PRE ? NP : 1)) < t.mtiles;
            if constexpr (PRE) {
                load_to_lds16(rw, smem4, (ch & 1) * A_BYTES + piece * 1024, live ? lane * 16u : kOob, so + piece * 1024);
            } else {
                wv[k][0] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rw, live ? lane * 32u : kOob, so + piece * 2048, 0));
                wv[k][1] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rw, live ? lane * 32u + 16u : kOob, so + piece * 2048, 0));
            }
        }
    };
    auto put_w = [&]() __attribute__((always_inline)) {
        if constexpr (!PRE) {
#pragma unroll
            for (int k = 0; k < AS; ++k) {
                const unsigned piece = k * (WM * WP) + wave;
                if (AS * WM * WP != AP && piece >= AP) break;
                unsigned u[4][3];
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    split3(__uint_as_float(wv[k][c / 2][c % 2 * 2]) * kSplitScale,
                           __uint_as_float(wv[k][c / 2][c % 2 * 2 + 1]) * kSplitScale, u[c]);
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    *reinterpret_cast<u32x4 *>(reinterpret_cast<char *>(smem4) + (piece * 3 + q) * 1024 + lane * 16) =
                        u32x4{u[0][q], u[1][q], u[2][q], u[3][q]};
            }
        }
    };

    fetch_w(0);
    fetch_x(0);

    const int li = lane & 15, lg = lane >> 4;
    const char *aop = reinterpret_cast<const char *>(smem4) + (wm * MI * NP * 64 + lane) * 16;
    const char *bop = bbuf + (lg * PLANE + (li & 1) * HALF + (wp * NI * 16 + li) / 2) * 16;

    f32x4 acc[MI][NI], low[NP == 3 ? MI : 1][NI];
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            acc[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (NP == 3) low[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    auto mma = [](bf16x8 a, bf16x8 b, f32x4 c) __attribute__((always_inline)) {
        // VO: pixels are the rows of the product, a lane ends up with four consecutive pixels of a filter
        return VO ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, a, c, 0, 0, 0)
                  : __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    };

    // One input buffer, two barriers per chunk: the blocks of a compute unit cover each other's staging.
    // (Measured and not kept: a second input buffer with one barrier and the staging spread between the
    // products, 273 against 270 us at 512 -> 1024 on 14x14 planes, N = 256, and behind on short reductions;
    // loads two chunks ahead in the small blocks, which cost them a block per compute unit: 20.3 -> 24.3 us
    // at 96 -> 24 on 56x56, N = 64.)
    for (int ch = 0; ch < t.nchunks; ++ch) {
        if (ch) __syncthreads();     // the previous chunk's inputs have been read
        put_w();
        put_x();
        if (PRE) wait_vmem0();       // this wave's share of the chunk's filters has arrived
        __syncthreads();
        if (ch + 1 < t.nchunks) {
            fetch_w(ch + 1);
            fetch_x(ch + 1);
        }
        const char *ab = aop + (PRE ? (ch & 1) * A_BYTES : 0u);
        bf16x8 opb[NI][NP];
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int q = 0; q < NP; ++q) opb[ni][q] = *reinterpret_cast<const bf16x8 *>(bop + q * PART + ni * 128);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            bf16x8 opa[NP];
#pragma unroll
            for (int q = 0; q < NP; ++q) opa[q] = *reinterpret_cast<const bf16x8 *>(ab + (mi * NP + q) * 1024);
            if constexpr (NP == 3) {
#pragma unroll
                for (int e = 0; e < 6; ++e)
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni) {
                        f32x4 &c = e == 5 ? acc[mi][ni] : low[mi][ni];
                        c = mma(opa[kSplitA[e]], opb[ni][kSplitB[e]], c);
                    }
            } else {
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) acc[mi][ni] = mma(opa[0], opb[ni][0], acc[mi][ni]);
            }
        }
    }

    // ---- epilogue: residual, ReLU, NCHW stores ---------------------------------------------------
    const __amdgpu_buffer_rsrc_t ry = make_rsrc(p.y, t.y_bytes);
    const __amdgpu_buffer_rsrc_t rr = make_rsrc(p.res ? p.res : p.y, t.y_bytes);
    const unsigned oc0 = ob * (MT * 16) + wm * (MI * 16);
    const unsigned ystep = t.HW * 4, ybase = (n0 * p.Cout + j * p.KPG) * ystep;
    SplitOverflow over;
    if (NP == 3) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                acc[mi][ni] += low[mi][ni];
#pragma unroll
                for (int r = 0; r < 4; ++r) over.see(acc[mi][ni][r]);
                acc[mi][ni] *= kSplitUnscale;
            }
    }
    // offset of a lane's first output of column block ni (its filter 0): pixel 4*lg (VO) or li of the block
    unsigned poff[NI];
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
        const unsigned d = (wp * NI + ni) * 16 + (VO ? 4 * lg : li);
        poff[ni] = q0 + d < t.npix ? ybase + px_off(d, p.Cout, 4) : kOob;
    }
    const unsigned f0 = oc0 + (VO ? li : 4 * lg);    // a lane's first filter
    auto out_off = [&](int mi, int ni, int r) -> unsigned {
        const unsigned f = f0 + mi * 16 + r;
        return f < (unsigned)p.KPG && poff[ni] != kOob ? poff[ni] + f * ystep : kOob;
    };
    if (p.res) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                if (VO) {
                    acc[mi][ni] += __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rr, out_off(mi, ni, 0), 0, 0));
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        acc[mi][ni][r] += __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rr, out_off(mi, ni, r), 0, 0));
                }
            }
    }
    if (p.relu) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[mi][ni][r] = fmaxf(acc[mi][ni][r], 0.f);
    }
    // (all results first, then the stores: a store's data registers are not written again)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            if (VO) {
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[mi][ni]), ry, out_off(mi, ni, 0), 0, 0);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[mi][ni][r]), ry, out_off(mi, ni, r), 0, 0);
            }
        }
    __builtin_amdgcn_sched_barrier(0);
    if (NP == 3 && __ballot(over.any())) {
        // plain fp32 sums of this wave's outputs
        wait_vmem0();   // the stores above come first
        const float *wd = p.wd + (size_t)j * p.CPG * p.KPGd;
        const float *x = static_cast<const float *>(p.x);
#pragma unroll 1
        for (int o = 0; o < MI * NI * 4; ++o) {
            const int mi = o / (NI * 4), ni = o / 4 % NI, r = o % 4;
            const unsigned d = (wp * NI + ni) * 16 + (VO ? 4 * lg + r : li);
            const unsigned f = f0 + mi * 16 + (VO ? 0 : r);
            if (q0 + d >= t.npix || f >= (unsigned)p.KPG) continue;
            const unsigned q = r0 + d, img = fast_div(q, t.m_HW), px = q - img * t.HW;
            const float *xp = x + (size_t)((n0 + img) * p.Cin + j * p.CPG) * t.HW + px;
            float s = 0.f;
#pragma unroll 1
            for (int c = 0; c < p.CPG; ++c) s = fmaf(xp[(size_t)c * t.HW], wd[(size_t)c * p.KPGd + f], s);
            const size_t yo = (size_t)((n0 + img) * p.Cout + j * p.KPG + f) * t.HW + px;
            if (p.res) s += p.res[yo];
            p.y[yo] = p.relu ? fmaxf(s, 0.f) : s;
        }
    }
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
namespace {

struct CfgS {
    int MI, NI, WM, WP;
    int min_blocks;   // fewest blocks of a launch for which the shape is taken
    int cost;         // time per filter and pixel (padding included), relative to the first shape's 100
};
// Block shapes, measured on the pointwise layers of the MobileNet-shaped and paper-form networks (fp32, N = 1,
// 16, 64, 256; us, the four shapes in one session):
//   512 -> 1024 on 14x14, N = 256: 270 / 311 / 413 / 455 (572 for the fp32 instruction in 128 x 128 blocks);
//   32 -> 64 on 112x112, N = 256: 281 / 237 / 273 / 322 (291); 96 -> 24 on 56x56, N = 64: 31 / 25 / 20.3 / 21.5 (26.9);
//   512 -> 512 on 14x14, N = 64 (392 / 784 / .. blocks): 41 / 55 / 57 / 60 (77), N = 16 (100 / 200 / 400 / 800 blocks):
//   26.4 / 24.2 / 21.8 / 21.1 (33.4), N = 4 (208 blocks of the last shape): 15.6 (14.7).
// So the first shape already pays with four blocks for every five compute units, the others want one and a half
// per unit; smaller launches run faster with the reduction split over a block's waves (conv_mfma16).
const CfgS kCfgS[] = {{4, 2, 2, 4, 200, 100}, {4, 2, 1, 4, 384, 114}, {2, 2, 1, 4, 384, 150}, {2, 2, 1, 2, 384, 165}};
constexpr int kNumCfgS = sizeof(kCfgS) / sizeof(kCfgS[0]);

template <int MI, int NI, int WM, int WP, typename TIN, bool VO, bool PRE>
hipError_t launchS(const ConvParams &p, const TileSplit &t, hipStream_t s) {
    constexpr int NP = SplitTraits<TIN>::parts, PB = 16 * NI * WP;
    constexpr size_t lds = (PRE ? 2 : 1) * (size_t)MI * WM * NP * 1024 + (size_t)NP * 4 * (PB + 8) * 16;
    auto kern = conv_mfma16s<MI, NI, WM, WP, TIN, VO, PRE>;
    if (lds > 64 * 1024) {
        static thread_local bool raised = false;   // per instantiation and thread
        if (!raised) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            raised = true;
        }
    }
    const unsigned blocks = (unsigned)round_up(t.px_blocks * t.oc_blocks, 8);
    hipLaunchKernelGGL(kern, dim3(blocks, p.groups), dim3(64 * WM * WP), lds, s, p, t);
    return hipGetLastError();
}

template <int MI, int NI, int WM, int WP>
hipError_t launchS_type(const ConvParams &p, const TileSplit &t, bool vo, hipStream_t s) {
    if (p.in_bf16)
        return vo ? launchS<MI, NI, WM, WP, uint16_t, true, true>(p, t, s) : launchS<MI, NI, WM, WP, uint16_t, false, true>(p, t, s);
    if (t.pre)
        return vo ? launchS<MI, NI, WM, WP, float, true, true>(p, t, s) : launchS<MI, NI, WM, WP, float, false, true>(p, t, s);
    return vo ? launchS<MI, NI, WM, WP, float, true, false>(p, t, s) : launchS<MI, NI, WM, WP, float, false, false>(p, t, s);
}

}  // namespace

bool plan_split(const ConvParams &p, const PackGeom &g, bool any_size, SplitPlan *out) {
    if (!p.ws || p.KH != 1 || p.KW != 1 || p.stride != 1 || p.pad != 0) return false;
    const double npix = (double)p.N * p.H * p.W;
    const double xb = npix * p.Cin * (p.in_bf16 ? 2 : 4), yb = npix * p.Cout * 4;
    if (xb >= (double)kOob || yb >= (double)kOob || (double)g.split_bytes >= (double)kOob || p.groups > 65535) return false;
    // One filter tile and at most 12 channels per group leave half of this kernel's smallest block and two thirds of its
    // k-step empty; where the staged kernel's planes need no ragged loads it is then ahead from 250k pixels times groups
    // on (split / staged, us: 8 -> 16 on 56x56, N = 247 22.3 / 17.9; 64 -> 128 on 32x32, g = 8, N = 169 46.5 / 32.1;
    // 48 -> 64 on 64x64, g = 4, N = 78 39.2 / 31.6; at 220k 32 -> 64 on 20x20, g = 4, N = 138 9.4 / 9.6).
    if (!any_size && !p.in_bf16 && g.split_mtiles == 1 && g.CPG <= 12 && (p.H * p.W) % 4 == 0 && npix * p.groups > 250e3)
        return false;
    // One filter tile on odd planes that the staged kernel's 64-pixel tiles fit: 640 -> 32 on 5x11, g = 2, N = 252 17.2 /
    // 10.6, 2048 -> 128 on 7x7, g = 8, N = 82 14.6 / 11.4, 1280 -> 128, N = 81 10.5 / 8.9 (36 layers 0.79).
    if (!any_size && !p.in_bf16 && g.split_mtiles == 1 && fills_image_tiles(p, 1)) return false;
    if ((long)p.H * p.W > 60000) return false;   // offsets inside a block are divided by the plane size exactly
    TileSplit t{};
    t.nchunks = g.split_chunks;
    t.mtiles = g.split_mtiles;
    t.pre = g.split_parts == 3;
    t.HW = p.H * p.W;
    t.npix = (unsigned)npix;
    t.m_HW = div_magic(t.HW);
    t.x_bytes = (unsigned)xb;
    t.y_bytes = (unsigned)yb;
    t.w_bytes = (unsigned)g.split_bytes;
    long best = 0;
    for (int i = 0; i < kNumCfgS; ++i) {
        const CfgS &c = kCfgS[i];
        const int ocb = (t.mtiles + c.MI * c.WM - 1) / (c.MI * c.WM);
        const long pxb = (long)((npix + 16 * c.NI * c.WP - 1) / (16 * c.NI * c.WP));
        if (pxb * ocb > 0x7ffffff0L) continue;
        if (pxb * ocb * p.groups < c.min_blocks && !(any_size && i == kNumCfgS - 1)) continue;
        const long cost = (long)ocb * c.MI * c.WM * c.cost;
        if (best && cost >= best) continue;
        best = cost;
        t.oc_blocks = ocb;
        t.m_ocb = div_magic(ocb);
        t.px_blocks = (int)pxb;
        out->inst = i;
        std::memcpy(out->data, &t, sizeof(t));
    }
    return best != 0;
}

hipError_t launch_split(const ConvParams &p, const SplitPlan &plan, hipStream_t s, const char **name) {
    TileSplit t;
    std::memcpy(&t, plan.data, sizeof(t));
    const CfgS &c = kCfgS[plan.inst];
    const bool vo = t.HW % 4 == 0;
    if (!*name)
        *name = intern_name("conv_mfma16s<" + std::to_string(c.MI) + "," + std::to_string(c.NI) + "," + std::to_string(c.WM) + "," +
                            std::to_string(c.WP) + (p.in_bf16 ? ",bf16," : ",f32,") + (vo ? "true," : "false,") +
                            (p.in_bf16 || t.pre ? "true>" : "false>"));
    switch (plan.inst) {
    case 0: return launchS_type<4, 2, 2, 4>(p, t, vo, s);
    case 1: return launchS_type<4, 2, 1, 4>(p, t, vo, s);
    case 2: return launchS_type<2, 2, 1, 4>(p, t, vo, s);
    case 3: return launchS_type<2, 2, 1, 2>(p, t, vo, s);
    }
    return hipErrorNotSupported;
}

}  // namespace gspc
