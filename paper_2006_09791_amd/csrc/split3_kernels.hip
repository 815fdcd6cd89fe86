// 3x3 layers with padding 1 on v_mfma_f32_16x16x32_bf16, fp32 layers through the exact three-way split
// (split_common.h), bf16 layers as they are: implicit GEMM per group over a staged input tile.
//
// Output pixels of all images are numbered flat; a block owns 16*NI*WP consecutive ones and 16*MI*WM
// filters of a group.  Rows are numbered over the padded images too, P = n * (H + 2) + ih + 1: the rows a
// tile needs are then one contiguous range of P (rows -1 and H of an image are zeros), whatever the plane
// and wherever images meet, and no pixel of a tile is padding.  Per chunk of 8*CGS channels the block
// stages that range once, split and channel-innermost - [part][8 channels][row][column] units of 16 bytes -
// and multiplies it nine taps long; the filters go from memory (L2) straight into the registers of the wave that
// multiplies them, split at packing time or (PLAIN: up to 256 weights per tap and group) by that wave.
//
// A unit of the reduction is 8 channels at one tap; a k-step is four units: with CGS = 4 one tap, the lane
// group lane/16 picks the channels; with CGS = 2 (tiles too large for four, or fewer channels) two taps.
//
// Small launches: WK groups of waves split the chunks, each with a tile of its own, and the partial sums
// meet in LDS.
//
// What bounds it: a wave tile of 32 filters x 64 pixels takes 768 matrix clocks per k-step, 12 KB of operands
// from LDS (64 of 128 bytes per clock with all four SIMDs busy) and six 1 KB filter loads (half of what the
// vector memory path issues).  128 -> 128 on 28x28, g = 2, N = 64 (784 blocks on 512 slots): a compute unit is busy
// 0.63 of the launch and its matrix unit 0.57 of that; 0.55 of the cycles of the LDS's operand accesses are bank
// conflicts (counters).
#include <algorithm>
#include <cstring>

#include "split_common.h"

namespace gspc {

struct TileH {
    int nchunks, ncg, mtiles;     // chunks of 8*CGS channels, blocks of 8 channels, 16-filter tiles per group
    int oc_blocks, px_blocks;
    int LW, PW, ROWS, PLANE;      // row pitch in units, column pairs per row, rows allocated, units per 8 channels
    unsigned npix, HWo;
    unsigned m_HWo, m_Wout, m_PW, m_H2, m_ocb;
    unsigned x_bytes, w_bytes, y_bytes;
};
static_assert(sizeof(TileH) <= sizeof(((Split3Plan *)0)->data), "plan storage too small");

// Waves per SIMD.  The bf16 instances of 16 channels per chunk, even rows and 4-byte stores come out one register past the step of
// five (four) waves if they are left to it: 384 -> 240 on 33x34 at stride 2, g = 8, N = 110 35.5 us for 25.8.
template <int MI, int CGS, typename TIN, bool EVEN, bool VO>
constexpr int kWavesH = sizeof(TIN) == 2 && CGS == 2 && EVEN && !VO ? (MI == 1 ? 5 : 4) : 2;

template <int MI, int NI, int WM, int WP, int WK, int CGS, int S, typename TIN, bool EVEN, bool VO, bool PLAIN>
__global__ __launch_bounds__(64 * WM * WP * WK, (kWavesH<MI, CGS, TIN, EVEN, VO>)) void conv_split3(ConvParams p, TileH t) {
    constexpr int NP = sizeof(TIN) == 4 ? 3 : 1, ES = (int)sizeof(TIN);
    constexpr int NT = 64 * WM * WP, PB = 16 * NI * WP, KS = CGS == 4 ? 9 : 5;
    constexpr int NA = 3;           // filter sets: k-step ks in set ks % NA, requested NA - 1 k-steps ahead
    constexpr int TS = 4;                         // staging tasks (32 column pairs x 8 channels) per wave in flight
    extern __shared__ f32x4 smem4[];

    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lg = lane >> 4;
    const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave_all / (WM * WP), wave = wave_all % (WM * WP);
    const int wm = wave / WP, wp = wave % WP;
    const unsigned part_bytes = CGS * t.PLANE * 16, tile_bytes = NP * part_bytes;
    char *tile = reinterpret_cast<char *>(smem4) + wk * tile_bytes;

    // the blocks of one XCD (block % 8) take consecutive (pixel tile, filter block) pairs
    const unsigned per = gridDim.x >> 3;
    const unsigned id = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (id >= (unsigned)(t.px_blocks * t.oc_blocks)) return;
    const unsigned pt = fast_div_any(id, t.oc_blocks, t.m_ocb), ob = id - pt * t.oc_blocks;
    const unsigned j = blockIdx.y;
    const unsigned q0 = pt * PB;
    const unsigned n0 = fast_div_any(q0, t.HWo, t.m_HWo), r0 = q0 - n0 * t.HWo;
    const unsigned H2 = p.H + 2, HW = p.H * p.W;
    const unsigned P0 = fast_div(r0, t.m_Wout) * S;              // first padded row, relative to image n0
    // pixel q0 + d: its image relative to n0, row and column
    auto pixel = [&](unsigned d, unsigned &img, unsigned &oh, unsigned &ow) {
        const unsigned r = r0 + d;
        img = fast_div(r, t.m_HWo);
        const unsigned rem = r - img * t.HWo;
        oh = fast_div(rem, t.m_Wout);
        ow = rem - oh * p.Wout;
    };
    const unsigned dlast = min((unsigned)PB, t.npix - q0) - 1;
    unsigned li_img, li_oh, li_ow;
    pixel(dlast, li_img, li_oh, li_ow);
    const unsigned rows = li_img * H2 + li_oh * S + 3 - P0;      // <= ROWS

    const __amdgpu_buffer_rsrc_t rx = make_rsrc(p.x, t.x_bytes);
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(p.wh, t.w_bytes);

    // ---- filters: [g][8 channels][tap][filter tile][part][16 filters][8], PLAIN: fp32 [16 filters][8], split below ------
    constexpr unsigned WT = PLAIN ? 512 : NP * 256;      // bytes of a filter tile at one tap
    const unsigned wtap = t.mtiles * WT;
    const unsigned wlane = (CGS == 4 ? lg * 9 * wtap : (lg & 1) * 9 * wtap + (lg >> 1) * wtap) + li * (PLAIN ? 32 : 16);
    const unsigned mt0 = ob * (MI * WM) + wm * MI;
    u32x4 wv[NA][MI][NP];
    auto fetch_w = [&](int ch, int ks, u32x4 (&v)[MI][NP]) __attribute__((always_inline)) {
        const unsigned so = ((j * t.ncg + ch * CGS) * 9 + (CGS == 4 ? ks : 2 * ks)) * wtap + mt0 * WT;
        const bool live = ch * CGS + (CGS == 4 ? lg : lg & 1) < t.ncg && (CGS == 4 || ks < 4 || lg < 2);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int q = 0; q < (PLAIN ? 2 : NP); ++q)
                v[mi][q] = __builtin_amdgcn_raw_buffer_load_b128(
                    rw, live && (int)mt0 + mi < t.mtiles ? wlane : kOob, so + mi * WT + q * (PLAIN ? 16u : 256u), 0);
    };
    auto split_w = [&](u32x4 (&v)[MI][NP]) __attribute__((always_inline)) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            u32x4 o[3];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                unsigned s[3];
                split3(__uint_as_float(v[mi][c / 2][c % 2 * 2]) * kSplitScale, __uint_as_float(v[mi][c / 2][c % 2 * 2 + 1]) * kSplitScale, s);
#pragma unroll
                for (int q = 0; q < 3; ++q) o[q][c] = s[q];
            }
#pragma unroll
            for (int q = 0; q < NP; ++q) v[mi][q] = o[q];
        }
    };

    // ---- staging: a wave's task is 32 column pairs of one 8-channel block; lower lanes load channels 0-3,
    // upper lanes 4-7 of both pixels, then exchange, so that a lane writes all eight channels of one pixel.
    // Addresses are the same for every chunk and computed once for the tasks that have a slot.
    const unsigned pairs = rows * t.PW, pgroups = (pairs + 31) >> 5, tasks = pgroups * CGS;
    struct Task {
        unsigned at;     // byte offset of (first channel of the lane, first pixel) in chunk 0, kOob: nothing to load;
                         // bit 0: the second pixel is outside the row
        unsigned lds;    // byte offset in the tile of the pixel the lane writes, kOob: nothing to write
    };
    // first channel of a task's lanes within a chunk
    auto task_c0 = [&](unsigned task) -> int { return (int)(task & (CGS - 1)) * 8 + (lane >> 5) * 4; };
    auto make_task = [&](unsigned task) __attribute__((always_inline)) -> Task {
        const unsigned cg = task & (CGS - 1), pair = (task / CGS) * 32 + (lane & 31);   // (CGS is a power of two)
        const unsigned row = fast_div(pair, t.m_PW), col = 2 * (pair - row * t.PW);
        const unsigned P = P0 + row, img = fast_div(P, t.m_H2);
        const int ih = (int)(P - img * H2) - 1;
        const bool in = task < tasks && pair < pairs;
        Task k;
        k.at = in && (unsigned)ih < (unsigned)p.H && n0 + img < (unsigned)p.N
                   ? ((((n0 + img) * p.Cin + j * p.CPG + task_c0(task)) * HW + ih * p.W + col) * (unsigned)ES |
                      (col + 1 >= (unsigned)p.W ? 1u : 0u))
                   : kOob;
        const unsigned wcol = col + (lane >> 5);
        k.lds = in && wcol < (unsigned)p.W ? (cg * t.PLANE + row * t.LW + 1 + wcol) * 16 : kOob;
        return k;
    };
    Task slot[TS];
#pragma unroll
    for (int k = 0; k < TS; ++k) slot[k] = make_task(wave + k * (WM * WP));
    u32x2 xv[TS][4];
    auto fetch_x = [&](int ch, unsigned task, const Task &k, u32x2 (&v)[4]) __attribute__((always_inline)) {
        const int left = p.CPG - ch * CGS * 8;      // channels from the chunk's first one on
        const unsigned so = (unsigned)(ch * CGS * 8) * HW * ES;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const unsigned vo = task_c0(task) + e < left ? k.at & ~1u : kOob, se = so + e * HW * ES;
            if constexpr (EVEN) {
                if (ES == 4) v[e] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rx, vo, se, 0));
                else v[e].x = __builtin_amdgcn_raw_buffer_load_b32(rx, vo, se, 0);       // both pixels
            } else {
                const unsigned v1 = vo != kOob && !(k.at & 1u) ? vo + ES : kOob;
                if (ES == 4) {
                    v[e].x = __builtin_amdgcn_raw_buffer_load_b32(rx, vo, se, 0);
                    v[e].y = __builtin_amdgcn_raw_buffer_load_b32(rx, v1, se, 0);
                } else {
                    v[e].x = (unsigned)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(rx, vo, se, 0);
                    v[e].y = (unsigned)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(rx, v1, se, 0);
                }
            }
        }
    };
    auto put_x = [&](const Task &k, const u32x2 (&v)[4]) __attribute__((always_inline)) {
        unsigned s[2][2][NP];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                if constexpr (NP == 3) {
                    split3(__uint_as_float(v[2 * c][i]) * kSplitScale, __uint_as_float(v[2 * c + 1][i]) * kSplitScale, s[i][c]);
                } else {
                    const bool both = EVEN;
                    const unsigned a0 = i && !both ? v[2 * c].y : v[2 * c].x, a1 = i && !both ? v[2 * c + 1].y : v[2 * c + 1].x;
                    s[i][c][0] = __builtin_amdgcn_perm(a1, a0, i && both ? 0x07060302u : 0x05040100u);
                }
            }
        char *d = tile + k.lds;
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            u32x4 u;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const auto r = __builtin_amdgcn_permlane32_swap(s[0][c][q], s[1][c][q], false, false);
                u[c] = r[0];
                u[2 + c] = r[1];
            }
            if (k.lds != kOob) *reinterpret_cast<u32x4 *>(d + q * part_bytes) = u;
        }
    };

    fetch_w(wk, 0, wv[0]);
    if (NA == 3) fetch_w(wk, 1, wv[1]);
#pragma unroll
    for (int k = 0; k < TS; ++k) fetch_x(wk, wave + k * (WM * WP), slot[k], xv[k]);

    // columns -1 and W of every row, never written by the staging: zeros
    for (unsigned i = tid % NT; i < (unsigned)NP * CGS * t.ROWS * 2; i += NT) {
        const unsigned side = i & 1, r = i >> 1, row = r % t.ROWS, pl = r / t.ROWS;   // pl: (part, 8 channels)
        *reinterpret_cast<u32x4 *>(tile + ((pl / CGS) * part_bytes) + ((pl % CGS) * t.PLANE + row * t.LW + side * (p.W + 1)) * 16) =
            u32x4{0u, 0u, 0u, 0u};
    }

    // ---- operand addresses ---------------------------------------------------------------------------
    // unit offset of a lane's pixel, and what its taps add to it (CGS = 2: the lane's tap of each k-step)
    unsigned bpix[NI];
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
        unsigned img, oh, ow;
        pixel(min((unsigned)((wp * NI + ni) * 16 + li), dlast), img, oh, ow);
        bpix[ni] = ((CGS == 4 ? lg : lg & 1) * t.PLANE + (img * H2 + oh * S - P0) * t.LW + ow * S) * 16;
    }
    auto tap_off = [&](int ks) -> unsigned {
        if (CGS == 4) return ((ks / 3) * t.LW + ks % 3) * 16u;
        const int t0 = 2 * ks, t1 = 2 * ks + 1 < 9 ? 2 * ks + 1 : 8;
        return (lg >> 1) ? ((t1 / 3) * t.LW + t1 % 3) * 16u : ((t0 / 3) * t.LW + t0 % 3) * 16u;
    };

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

    const int rounds = (t.nchunks + WK - 1) / WK;
    for (int rd = 0; rd < rounds; ++rd) {
        const int ch = rd * WK + wk;
        if (rd) __syncthreads();                  // the previous chunk has been read
#pragma unroll
        for (int k = 0; k < TS; ++k) put_x(slot[k], xv[k]);
        for (unsigned k = TS * (WM * WP); k < tasks; k += WM * WP) {   // (wide planes: more tasks than slots)
            const Task more = make_task(wave + k);
            fetch_x(ch, wave + k, more, xv[0]);
            put_x(more, xv[0]);
        }
        __syncthreads();
        // A k-step goes pixel tile by pixel tile: the inputs of the next one are read from LDS while the matrix
        // unit works on this one; the next chunk's inputs are requested one task per k-step.
        bf16x8 opb[2][NP];
        // (an offset the compiler cannot see through: it would otherwise keep the operand addresses of all k-steps,
        // a hundred registers, across the chunks)
        unsigned opaque = 0;
        asm volatile("" : "+s"(opaque));
        auto load_b = [&](int ks, int ni) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                const char *b = tile + q * part_bytes + bpix[ni] + (tap_off(ks) + opaque);
                // (CGS = 2: the last k-step's second tap does not exist.  Its weights are zeros, and so must the inputs
                // be, lest an infinity times zero come into the sum: a unit of column -1)
                if (CGS == 2 && ks == KS - 1 && lg >= 2) b = tile + q * part_bytes;
                opb[(ks * NI + ni) & 1][q] = *reinterpret_cast<const bf16x8 *>(b);
            }
        };
        load_b(0, 0);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            constexpr int AH = NA - 1;
            if (ks + AH < KS) fetch_w(ch, ks + AH, wv[(ks + AH) % NA]);
            else fetch_w(ch + WK, ks + AH - KS, wv[(ks + AH) % NA]);
            if (ks < TS) fetch_x(ch + WK, wave + ks * (WM * WP), slot[ks], xv[ks]);
            if constexpr (PLAIN) split_w(wv[ks % NA]);
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                if (ni + 1 < NI) load_b(ks, ni + 1);
                else if (ks + 1 < KS) load_b(ks + 1, 0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int e = 0; e < (NP == 3 ? 6 : 1); ++e)
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi) {
                        f32x4 &c = NP == 1 || e == 5 ? acc[mi][ni] : low[NP == 3 ? mi : 0][ni];
                        c = mma(__builtin_bit_cast(bf16x8, wv[ks % NA][mi][NP == 3 ? kSplitA[e] : 0]),
                                opb[(ks * NI + ni) & 1][NP == 3 ? kSplitB[e] : 0], c);
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (KS % NA) {                            // the next chunk's first filters move to set 0 (and 1)
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int q = 0; q < NP; ++q) {
                    if (NA == 3) wv[1][mi][q] = wv[0][mi][q];
                    wv[0][mi][q] = wv[NA - 1][mi][q];
                }
        }
    }

#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
            if (NP == 3) acc[mi][ni] += low[mi][ni];
    if (WK > 1) {
        // partial sums of the other groups, [group - 1][wave][tile][lane]
        __syncthreads();
        f32x4 *ps = smem4;
        if (wk > 0) {
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
                    ps[((((wk - 1) * (WM * WP) + wave) * MI + mi) * NI + ni) * 64 + lane] = acc[mi][ni];
        }
        __syncthreads();
        if (wk > 0) return;
#pragma unroll
        for (int k = 1; k < WK; ++k)
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
                    acc[mi][ni] += ps[((((k - 1) * (WM * WP) + wave) * MI + mi) * NI + ni) * 64 + lane];
    }
    SplitOverflow over;
    if (NP == 3) {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
#pragma unroll
                for (int r = 0; r < 4; ++r) over.see(acc[mi][ni][r]);
                acc[mi][ni] *= kSplitUnscale;
            }
    }

    // ---- epilogue: residual, ReLU, NCHW stores ---------------------------------------------------------
    const __amdgpu_buffer_rsrc_t ry = make_rsrc(p.y, t.y_bytes);
    const __amdgpu_buffer_rsrc_t rr = make_rsrc(p.res ? p.res : p.y, t.y_bytes);
    const unsigned ystep = t.HWo * 4, ybase = (n0 * p.Cout + j * p.KPG) * ystep;
    unsigned poff[NI];
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) {
        const unsigned d = (wp * NI + ni) * 16 + (VO ? 4 * lg : li);
        const unsigned r = r0 + d, img = fast_div(r, t.m_HWo);
        poff[ni] = q0 + d < t.npix ? ybase + (img * (p.Cout - 1) * t.HWo + r) * 4 : kOob;
    }
    const unsigned f0 = mt0 * 16 + (VO ? li : 4 * lg);           // a lane's first filter
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
        const float *wd = p.wd + (size_t)j * p.CPG * 9 * p.KPGd;
        const float *x = static_cast<const float *>(p.x);
#pragma unroll 1
        for (int o = 0; o < MI * NI * 4; ++o) {
            const int mi = o / (NI * 4), ni = o / 4 % NI, r = o % 4;
            const unsigned d = (wp * NI + ni) * 16 + (VO ? 4 * lg + r : li);
            const unsigned f = f0 + mi * 16 + (VO ? 0 : r);
            if (q0 + d >= t.npix || f >= (unsigned)p.KPG) continue;
            unsigned img, oh, ow;
            pixel(d, img, oh, ow);
            const float *xp = x + (size_t)((n0 + img) * p.Cin + j * p.CPG) * HW;
            float s = 0.f;
#pragma unroll 1
            for (int k = 0; k < p.CPG * 9; ++k) {
                const int ih = (int)oh * S - 1 + k % 9 / 3, iw = (int)ow * S - 1 + k % 3;
                if ((unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W)
                    s = fmaf(xp[(size_t)(k / 9) * HW + ih * p.W + iw], wd[(size_t)k * p.KPGd + f], s);
            }
            const size_t yo = (size_t)((n0 + img) * p.Cout + j * p.KPG + f) * t.HWo + oh * p.Wout + ow;
            if (p.res) s += p.res[yo];
            p.y[yo] = p.relu ? fmaxf(s, 0.f) : s;
        }
    }
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
namespace {

struct CfgH {
    int MI, NI, WM, WP, WK;
    float kstep;      // fp32 layers: microseconds per k-step of a block alone on its compute unit
    // bf16 layers: microseconds per launch and per block, chunk, k-step and 1000 staged units (16 bytes) of a compute unit
    float launch, block, chunk, step, stage;
};
const CfgH kCfgH[] = {
    {2, 4, 2, 2, 1, 0.75f, 5.3f, 0.59f, 0.36f, 0.027f, 0.49f},
    {2, 2, 2, 2, 1, 0.5f, 4.5f, 0.53f, 0.30f, 0.040f, 0.22f},
    {2, 4, 2, 1, 2, 0.75f},
    {2, 2, 1, 1, 4, 0.5f},
    {2, 4, 1, 4, 1, 0.82f, 5.3f, 0.74f, 0.19f, 0.f, 0.75f},     // up to 32 filters per group
    {1, 4, 1, 4, 1, 0.52f, 5.3f, 0.58f, 0.034f, 0.f, 0.63f},     // up to 16
    {1, 2, 1, 4, 1, 0.31f},
};
constexpr int kNumCfgH = sizeof(kCfgH) / sizeof(kCfgH[0]);
constexpr int kFirstFew = 4;     // blocks of at most 32 filters
constexpr int kFirstPlain = 5;   // shapes of one filter tile, which have an instance that splits the filters itself
constexpr int kLdsBlockH = 78 * 1024;   // two blocks per compute unit

size_t lds_bytes_h(const CfgH &c, int cgs, int parts, const TileH &t) {
    const size_t tiles = (size_t)c.WK * parts * cgs * t.PLANE * 16;
    const size_t sums = (size_t)(c.WK - 1) * c.WM * c.WP * c.MI * c.NI * 1024;
    return tiles > sums ? tiles : sums;
}

template <int MI, int NI, int WM, int WP, int WK, int CGS, int S, typename TIN, bool EVEN, bool VO, bool PLAIN>
hipError_t launchH(const ConvParams &p, const TileH &t, hipStream_t s) {
    const size_t lds = lds_bytes_h(CfgH{MI, NI, WM, WP, WK, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, CGS, sizeof(TIN) == 4 ? 3 : 1, t);
    auto kern = conv_split3<MI, NI, WM, WP, WK, CGS, S, TIN, EVEN, VO, PLAIN>;
    if (lds > 64 * 1024) {
        static thread_local bool raised = false;   // per instantiation and thread
        if (!raised) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBlockH);
            if (e != hipSuccess) return e;
            raised = true;
        }
    }
    const unsigned blocks = (unsigned)round_up(t.px_blocks * t.oc_blocks, 8);
    hipLaunchKernelGGL(kern, dim3(blocks, p.groups), dim3(64 * WM * WP * WK), lds, s, p, t);
    return hipGetLastError();
}

// 16-byte stores (VO) go with 8-byte loads: an odd row width takes the 4-byte forms of both
template <int MI, int NI, int WM, int WP, int WK, int CGS, int S, typename TIN, bool PLAIN>
hipError_t launchH_form(const ConvParams &p, const TileH &t, hipStream_t s) {
    if (p.W & 1) return launchH<MI, NI, WM, WP, WK, CGS, S, TIN, false, false, PLAIN>(p, t, s);
    if (t.HWo % 4) return launchH<MI, NI, WM, WP, WK, CGS, S, TIN, true, false, PLAIN>(p, t, s);
    return launchH<MI, NI, WM, WP, WK, CGS, S, TIN, true, true, PLAIN>(p, t, s);
}

template <int MI, int NI, int WM, int WP, int WK, typename TIN, bool PLAIN = false>
hipError_t launchH_cgs(const ConvParams &p, const TileH &t, int cgs, hipStream_t s) {
    if (cgs == 4)
        return p.stride == 1 ? launchH_form<MI, NI, WM, WP, WK, 4, 1, TIN, PLAIN>(p, t, s) : launchH_form<MI, NI, WM, WP, WK, 4, 2, TIN, PLAIN>(p, t, s);
    return p.stride == 1 ? launchH_form<MI, NI, WM, WP, WK, 2, 1, TIN, PLAIN>(p, t, s) : launchH_form<MI, NI, WM, WP, WK, 2, 2, TIN, PLAIN>(p, t, s);
}

bool planH_cfg(const ConvParams &p, const PackGeom &g, const CfgH &c, int cgs, TileH *out) {
    const int PB = 16 * c.NI * c.WP, MT = c.MI * c.WM;
    const double npix = (double)p.N * p.Hout * p.Wout;
    const double xb = (double)p.N * p.Cin * p.H * p.W * (p.in_bf16 ? 2 : 4), yb = (double)p.N * p.Cout * p.Hout * p.Wout * 4;
    if (xb >= (double)kOob || yb >= (double)kOob || (double)g.h3_bytes >= (double)kOob || p.groups > 65535) return false;
    TileH t{};
    t.ncg = (g.CPG + 7) / 8;
    t.nchunks = (t.ncg + cgs - 1) / cgs;
    t.mtiles = (g.KPG + 15) / 16;
    t.oc_blocks = (t.mtiles + MT - 1) / MT;
    const long pxb = (long)((npix + PB - 1) / PB);
    if (pxb * t.oc_blocks > 0x7ffffff0L) return false;
    t.px_blocks = (int)pxb;
    t.HWo = p.Hout * p.Wout;
    t.npix = (unsigned)npix;
    // rows of a tile: those its pixels span, three taps, and at every change of image the rows between the last
    // window of one and the first of the next
    const int span = (PB - 2) / p.Wout + 2, cross = p.N > 1 ? (PB - 2) / (int)t.HWo + 1 : 0;
    const int out_rows = span, extra = p.H + 2 - p.Hout * p.stride;
    const int crossings = cross < out_rows - 1 ? cross : out_rows - 1;
    t.ROWS = (out_rows - 1) * p.stride + 3 + crossings * (extra > 0 ? extra : 0);
    t.LW = p.W + 2;
    t.PW = (p.W + 1) / 2;
    t.PLANE = t.ROWS * t.LW;
    t.m_ocb = div_magic(t.oc_blocks);
    t.m_HWo = div_magic(t.HWo);
    t.m_Wout = div_magic(p.Wout);
    t.m_PW = div_magic(t.PW);
    t.m_H2 = div_magic(p.H + 2);
    t.x_bytes = (unsigned)xb;
    t.y_bytes = (unsigned)yb;
    t.w_bytes = (unsigned)g.h3_bytes;
    // exact reciprocals: offsets inside a tile stay below 2^32 / divisor
    if ((double)(t.HWo + PB) * t.HWo >= 4.0e9 || (double)(t.ROWS + p.H + 2) * (p.H + 2) >= 4.0e9 ||
        (double)(t.ROWS * t.PW + 64) * t.PW >= 4.0e9)
        return false;
    if (lds_bytes_h(c, cgs, p.in_bf16 ? 1 : 3, t) > (size_t)kLdsBlockH) return false;
    *out = t;
    return true;
}

// Microseconds of a bf16 launch, for comparison with the 16x16x32 kernel: start and stores, then per chunk a fixed part, the
// products, the staging of odd rows (element by element), and the tasks that have no slot; blocks that share a compute unit
// take 1.43 times one's time (fitted to 1100 layers of 4 .. 240 us: nine in ten within a sixth).
double bf16_estimate(const ConvParams &p, const CfgH &c, int cgs, const TileH &t, long blocks) {
    const double mm = c.MI * c.NI, units = (double)blocks / kNumCU, n = (double)((blocks + kNumCU - 1) / kNumCU);
    const double shared = n <= 1.0 ? 1.0 : n <= 2.0 ? 1.43 : 0.715 * (0.5 * n + 0.5 * units);
    const int waves = c.WM * c.WP, tasks = ((t.ROWS * t.PW + 31) / 32 * cgs + waves - 1) / waves;
    return 3.32 + 0.2 * mm + shared * t.nchunks * (0.577 + 0.0101 * (cgs == 4 ? 9 : 5) * mm + (p.W % 2 ? 0.182 * tasks : 0.0) +
                                                   (tasks > 4 ? 0.219 * (tasks - 4) : 0.0));
}

// Microseconds of an fp32 launch, for comparison with the kernels that have the layer otherwise: start and stores, then per
// chunk a fixed part, the products and filter loads, and the staging of odd rows and of tasks that have no slot (fitted to
// 2600 layers in each shape that takes them: nine in ten within a sixth).
double f32_estimate(const ConvParams &p, const CfgH &c, int cgs, const TileH &t, bool plain, long blocks) {
    const double mm = c.MI * c.NI, units = (double)blocks / kNumCU, n = (double)((blocks + kNumCU - 1) / kNumCU);
    const double shared = n <= 1.0 ? 1.0 : n <= 2.0 ? 1.78 : 0.89 * (0.5 * n + 0.5 * units);
    const int waves = c.WM * c.WP, tasks = ((t.ROWS * t.PW + 31) / 32 * cgs + waves - 1) / waves;
    const double chunk = 1.26 + (cgs == 4 ? 9 : 5) * (0.0514 * mm + 0.0216 * c.MI + (plain ? 0.124 : 0.0)) +
                         (p.W % 2 ? 0.1325 * tasks : 0.0) + (tasks > 4 ? 0.328 * (tasks - 4) : 0.0);
    return 3.61 + 0.176 * mm * (p.W % 2 || t.HWo % 4 ? 1.83 : 1.0) + (c.WK > 1 ? 0.37 : 0.0) + shared * ((t.nchunks + c.WK - 1) / c.WK) * chunk;
}

}  // namespace

// Block shape: the one with the shortest estimated launch.  A block alone on its compute unit needs `kstep` per k-step
// (1.3 times that for the half-size chunks), 1 us per chunk and 1.5 us besides; two share the unit at 1.45 times that,
// more follow in pairs; the sum of split chunks adds a tenth (N = 64, us, estimate / measured: 256 -> 256 on 14x14 g = 2
// 47 / 40, 512 -> 512 on 7x7 g = 2 47 / 43, 128 -> 128 on 8x8 11.2 / 10.8, 50 -> 75 on 31x23 at N = 100 66 / 58 and 69 / 65
// for the next best shape).
//
// Which layers (N = 64 unless stated, us, before / with this kernel; channels and filters are the layer's):
//  - rows that are not a multiple of 4 or channels per group that are not: the fp32 kernels stage those 4 bytes at a
//    time, or in one chunk: 256 -> 256 on 14x14 g = 2 68 / 40, g = 4 38 / 24, 512 -> 512 on 7x7 g = 2 89 / 43,
//    192 -> 192 on 13x17 g = 2 104 / 33, 50 -> 75 on 31x23 at N = 100 423 / 58, 110 -> 100 on 40x40 stride 2 at N = 20
//    281 / 22, 80 -> 72 on 18x18 at N = 128 76 / 48, with almost half of the filters padding 144 -> 144 on 14x14 g = 2
//    33.7 / 31.3;
//  - planes of more than 256 pixels whose 2x2 tiles leave a tenth of Winograd's 32-tile blocks empty, in whole chunks and
//    filter tiles (40 -> 48 on 28x28: 17.5 / 22.4) and with more than a block per compute unit (128 -> 128 on 28x28 g = 2
//    at N = 16, 196 blocks: 15.9 / 16.8; at N = 24 24.7 / 23.5): 128 -> 128 on 28x28 g = 2 47.4 / 43.5, g = 1 85 / 77,
//    256 -> 256 g = 4 92 / 76, 128 -> 128 on 20x20 g = 2 at N = 100 49 / 34, 64 -> 64 25.8 / 22.7.  Planes that fill the
//    blocks are level or Winograd's (64 -> 64 on 32x32 25.8 / 25.4, on 56x56 91 / 95);
//  - stride 2 from two blocks per compute unit on: 128 -> 256 on 28x28 g = 2 50 / 31, 256 -> 512 on 14x14 g = 2 59 / 30,
//    64 -> 128 on 56x56 83 / 62; with one block the fp32 kernels are level (64 -> 128 on 16x16: 11.7 / 13.7);
//  - other stride-1 layers: with at least 128 channels per group where neither Winograd (64 -> 64 on 16x16 at N = 256
//    25.6 / 25.3) nor a launch of more blocks than the chip holds covers the fp32
//    kernel's waits: 128 -> 128 on 8x8 13.4 / 10.3 (64 channels per group: 8.6 / 10.2).
// (from here on channels and filters are per group)
//  - other planes whose 2x2 tiles do not fill Winograd's blocks whole, where the estimate here is shorter than Winograd's:
//    32 -> 32 on 18x18, g = 32 138 / 75, 92 on 24x24, g = 2, N = 198 325 / 176, 112 on 36x36, g = 3, N = 40 330 / 203,
//    16 on 72x72, g = 32, N = 5 67.5 / 47.  Planes that fill them stay: 16 -> 16 on 32x32, g = 2 8.9 / 10.4, 32 -> 32 at N = 256
//    34.9 / 34.4;
//  - odd rows or channels with few weights, against the estimates of the kernels that these layers have otherwise: 16 -> 16 on 98x98, g = 16, N = 13 418 / 112, 32 -> 10 on 33x33, g = 4 41.6 / 23.9 with
//    72, 126 -> 12 on 38x38, g = 3, N = 4 258 / 15, 80 -> 12 on 85x85, g = 2, N = 27 641 / 89; not: 8 -> 8 per group, which the
//    4x4x1 kernel takes (29x29, g = 32, N = 143 106 / 219), and up to 256 weights per tap on small planes (16 -> 16 on 17x19,
//    g = 2, N = 207 18.1 / 16.8, which is level where launches are smaller).
// With Winograd switched off (gspc_set_winograd(0)) every fp32 3x3 layer stays on the fp32 instruction.
//
// (Blocks of 128 filters x 128 pixels and 64 x 256 for bf16 layers, with half the operand reads per product: 0.99 and 1.10 times
// the time on the 14x14 layer below, up to 1.6 times elsewhere.)
//
// bf16 layers that the 16x16x32 kernel takes too, where the estimate here is shorter than that kernel's as well (738 random
// layers of these kinds: level with the faster of the two within 0.4 % in the geometric mean; without the estimates 102 of them
// were up to 2.6 times slower than that kernel: 6 -> 6 on 107x107, g = 16, N = 23 43 / 113, 12 -> 12 on 33x33 at stride 2, g = 4,
// N = 4 4.3 / 5.6, 272 -> 68 on 90x13, g = 2, N = 2 13.8 / 27.5) (us, that kernel / this one):
//  - groups that it merges (channels not a multiple of 8), eight channels apart: 63 -> 63 on 8x8, g = 8 54 / 5.7, 80 -> 57 on 36x18
//    at stride 2 166 / 25, 128 -> 25 on 88x88 597 / 98, 6 -> 64 on 72x72 60 / 39; 8 -> 8 merged in pairs stays (13.7 / 25.6);
//  - 40 channels and more that it takes in chunks of 8 (104 on 20x79 127 / 63, 72 on 75x75 241 / 137) or 16 (48 on 44x44
//    151 / 83, 112 on 25x25 281 / 169; 16 channels 0.5-0.9 of its speed), below 80 channels on rows of an even length only (48 on
//    21x21 18.5 / 21.3);
//  - from 64 channels in chunks of 32 at stride 1, on rows it loads in less than 16 bytes (96 on 71x75 137 / 93): 128 -> 128 on 14x14, g = 2, N = 256
//    45.3 / 36.0, on 18x18 59 / 40, 64 on 52x52 18.7 / 13.9; rows of whole octets (32 on 56x56 72 / 91, 128 on 48x48 at stride 2
//    83 / 104), long rows (96 on 110x110 61 / 75) and 7x7 planes (44 / 55) stay.
bool prefers_split3_bf16(const ConvParams &p, const PackGeom &g) {
    if (!p.in_bf16 || !p.wh || !g.bf16_bytes) return false;
    if (g.mb > 1) return g.CPG != 8;
    const double macs = (double)p.N * p.Cout * p.Hout * p.Wout * g.CPG * 9;
    if (g.CPG < 40 || macs < 3e8) return false;
    if (g.CPG % 16) return true;
    if (g.KPG < 32 || (p.W % 2 && g.CPG < 80)) return false;
    return g.CPG % 32 || (g.CPG >= 64 && p.stride == 1 && p.W % 8 && p.W <= 80 && p.H * p.W >= 100 && macs >= 1e9);
}

bool plan_split3(const ConvParams &p, const PackGeom &g, int when, Split3Plan *out) {
    if (!p.wh || p.KH != 3 || p.KW != 3 || p.pad != 1 || (p.stride != 1 && p.stride != 2)) return false;
    const bool odd = p.W % 4 != 0 || g.CPG % 4 != 0;
    // layers of more than 16384 weights per group, or whose channels only this kernel takes in whole chunks
    const bool large = g.KPG >= 16 && g.CPG >= 8 && ((long)g.CPG * g.KPG * 9 > 16384 || g.CPG % 4 != 0);
    const int ft = (g.KPG + 63) / 64 * 64;
    const int wt = (p.Hout + 1) / 2 * ((p.Wout + 1) / 2), wr = (wt + 31) / 32 * 32;
    const bool ragged = p.H * p.W > 256 && 10 * (wr - wt) > wr && g.CPG % 32 == 0 && ft == g.KPG &&
                        (double)p.N * p.Hout * p.Wout * p.Cout > kNumCU * 64 * 128.0;
    const bool sure = large && (odd ? ft < 2 * g.KPG : ragged);   // Winograd's estimate is not asked
    if (when == kSplit3BeforeWinograd && (p.stride != 1 || (!sure && (!g.wino_bytes || wt == wr || 32 % wt == 0)))) return false;
    if (when != kSplit3Rest && (g.CPG < 5 || g.KPG < 5)) return false;
    if (when == kSplit3Else && !odd && (p.stride == 1 ? g.CPG < 128 : !large)) return false;
    if (when == kSplit3Else && !large && g.CPG * g.KPG <= 256 && p.H * p.W < 400) return false;
    bool wide = false;        // a block of 64 filters passes the bounds below
    double best = 0.0, est64[kFirstFew] = {};
    Split3Plan plan64[kFirstFew]{};   // the blocks of 64 filters (and of 32 in four chunks at a time)
    for (int i = 0; i < kNumCfgH; ++i) {
        const CfgH &c = kCfgH[i];
        if (p.in_bf16 && c.launch == 0.f) continue;
        if (g.h3_plain && i < kFirstPlain) continue;
        for (int cgs : {4, 2}) {
            TileH t;
            if (cgs == 4 && (g.CPG + 15) / 16 * 16 < (g.CPG + 31) / 32 * 32 - 8) continue;
            if (!planH_cfg(p, g, c, cgs, &t)) continue;
            const long blocks = (long)t.px_blocks * t.oc_blocks * p.groups, n = (blocks + kNumCU - 1) / kNumCU;
            if ((when < kSplit3Rest && blocks < kNumCU / 4) || (when == kSplit3Else && !odd && p.stride == 2 && n < 2) ||
                (when == kSplit3Else && !odd && p.stride == 1 && n > 2))
                continue;
            wide |= i < kFirstFew;
            const double rounds = (t.nchunks + c.WK - 1) / c.WK, ks = rounds * (cgs == 4 ? 9 : 5 * 1.3);
            const double stretch = p.stride == 1 ? 1.0 : c.WM == 1 ? (c.NI == 4 ? 1.4 : 1.35) : c.WK > 1 ? 1.4 : c.NI == 4 ? 1.15 : 0.75;
            const double one = ks * c.kstep * stretch + rounds + 1.5;
            double est = (c.WK > 1 ? 1.1 : 1.0) * one * (1.45 * (double)(n / 2) + (double)(n % 2));
            if (p.in_bf16) {
                const double per_unit = n > 1 ? 0.5 * (double)n + 0.5 * (double)blocks / kNumCU : 1.0;
                est = c.launch + per_unit * (c.block + t.nchunks * (c.chunk + (cgs == 4 ? 9 : 5) * c.step + 1e-3 * cgs * t.PLANE * c.stage));
            }
            const auto keep = [&](Split3Plan *o) {
                o->inst = i;
                o->cgs = cgs;
                o->plain = g.h3_plain;
                o->us = p.in_bf16 ? bf16_estimate(p, c, cgs, t, blocks) : f32_estimate(p, c, cgs, t, g.h3_plain, blocks);
                std::memcpy(o->data, &t, sizeof(t));
            };
            if (i < kFirstFew && (est64[i] == 0.0 || est < est64[i])) {
                est64[i] = est;
                keep(&plan64[i]);
            }
            if (best != 0.0 && est >= best) continue;
            best = est;
            keep(out);
        }
    }
    if (best == 0.0) return false;
    out->sure = large && wide;
    // The choice between near ties is asked again of the second estimate, which is fitted over all shapes at once.  Blocks of
    // few filters stage the tile once per 16 or 32 filters, a cost for long reductions in few blocks (bf16, 323 -> 32 on 17x17,
    // g = 3, N = 3 33.5 / 29.2 us, 116 -> 72 on 19x19, g = 3, N = 9 15.7 / 12.7), and at stride 2 large blocks can leave one per
    // compute unit (bf16, 68 -> 68 on 56x56, N = 18 14.7 / 11.9) and smaller ones only share it (fp32, 76 -> 152 on 32x16, g = 3, N = 93
    // 73.9 / 66.9, 96 -> 96 on 22x37, g = 8, N = 45 136 / 123).  Nearer than 5.5 % it is no better than the first (bf16: of 29
    // random layers that it moves 25 gain, 1.09 in the mean, the worst loses 6 %; fp32: 10 of 1042, 7 gain, the worst loses 5 %), nor is
    // it for bf16 layers in large blocks at stride 1.
    if (!p.in_bf16 || out->inst >= kFirstFew || p.stride == 2)
        for (int i = 0; i < kFirstFew; ++i)
            if (est64[i] != 0.0 && est64[i] < 1.06 * best && plan64[i].us < 0.945 * out->us) {
                plan64[i].sure = out->sure;
                *out = plan64[i];
            }
    if (when == kSplit3BeforeWinograd && !sure) {
        WinoPlan px;
        return plan_wino(p, g, true, &px) && (g.h3_plain ? best + 4.0 : 0.82 * best + 3.0) < wino_estimate(p, px);
    }
    // (a first bound, before the estimates of those kernels: what is left runs at up to 9.5 Tera-products per second; with no
    // other matrix-core kernel at 0.13 us or more per term of a sum: 40 -> 2 on 44x44, g = 3, N = 7 51 / 13 before / with this kernel, 100 -> 3 on 9x9, N = 8
    // 119 / 11, 300 -> 6 on 17x17, g = 3, N = 40 in bf16 168 / 14)
    const double macs = (double)p.N * p.Cout * p.Hout * p.Wout * g.CPG * 9;
    if (when == kSplit3Else && !large) return 0.87 * best < 3.0 + macs / 9.5e6;
    if (when == kSplit3Rest) return 0.87 * best < 3.0 + std::max(macs / 9.5e6, 0.13 * 9 * g.CPG);
    return true;
}

hipError_t launch_split3(const ConvParams &p, const Split3Plan &plan, hipStream_t s, const char **name) {
    TileH t;
    std::memcpy(&t, plan.data, sizeof(t));
    const CfgH &c = kCfgH[plan.inst];
    const bool even = p.W % 2 == 0;
    // (a plan for another form of the shape must not run with this one's filter layout)
    if ((plan.plain && plan.inst < kFirstPlain) || (p.in_bf16 && (plan.plain || c.launch == 0.f))) return hipErrorNotSupported;
    if (!*name)
        *name = intern_name("conv_split3<" + std::to_string(c.MI) + "," + std::to_string(c.NI) + "," + std::to_string(c.WM) +
                            "," + std::to_string(c.WP) + "," + std::to_string(c.WK) + "," + std::to_string(plan.cgs) + "," +
                            std::to_string(p.stride) + (p.in_bf16 ? ",bf16" : ",f32") + (even ? ",true" : ",false") +
                            (even && t.HWo % 4 == 0 ? ",true>" : ",false>") + (plan.plain ? "/plain" : ""));
    if (plan.plain) return plan.inst == 5 ? launchH_cgs<1, 4, 1, 4, 1, float, true>(p, t, plan.cgs, s) : launchH_cgs<1, 2, 1, 4, 1, float, true>(p, t, plan.cgs, s);
    switch (plan.inst) {
    case 0: return p.in_bf16 ? launchH_cgs<2, 4, 2, 2, 1, uint16_t>(p, t, plan.cgs, s) : launchH_cgs<2, 4, 2, 2, 1, float>(p, t, plan.cgs, s);
    case 1: return p.in_bf16 ? launchH_cgs<2, 2, 2, 2, 1, uint16_t>(p, t, plan.cgs, s) : launchH_cgs<2, 2, 2, 2, 1, float>(p, t, plan.cgs, s);
    case 2: return launchH_cgs<2, 4, 2, 1, 2, float>(p, t, plan.cgs, s);
    case 3: return launchH_cgs<2, 2, 1, 1, 4, float>(p, t, plan.cgs, s);
    case 4: return p.in_bf16 ? launchH_cgs<2, 4, 1, 4, 1, uint16_t>(p, t, plan.cgs, s) : launchH_cgs<2, 4, 1, 4, 1, float>(p, t, plan.cgs, s);
    case 5: return p.in_bf16 ? launchH_cgs<1, 4, 1, 4, 1, uint16_t>(p, t, plan.cgs, s) : launchH_cgs<1, 4, 1, 4, 1, float>(p, t, plan.cgs, s);
    case 6: return launchH_cgs<1, 2, 1, 4, 1, float>(p, t, plan.cgs, s);
    }
    return hipErrorNotSupported;
}

}  // namespace gspc
