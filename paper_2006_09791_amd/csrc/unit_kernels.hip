// Small launches (batch 1 and the like): per-group implicit GEMM on v_mfma_f32_16x16x4_f32 without staging.
//
// A block owns one tile of 16 filters x 16 output pixels and its waves split the reduction; every operand
// goes from global memory (L2) straight into the registers of the lane that multiplies it, so that all loads
// of a wave are on their way before the first product, and the only barrier is the one before the partial
// sums are added.  Such a launch is a chain of latencies - kernel start, addresses, one trip to memory,
// products, the sum, the store - and conv_mfma16's chunks put three or four more trips into it.
//
// A channel block is four channels (lane / 16); for 3x3 layers a lane loads the three taps of its pixel (lane % 16) and
// the three weights of its filter in one kernel row with one 12-byte load each and multiplies three times; for 1x1
// layers a block is sixteen channels, one 16-byte load of weights and four of inputs.  A row of a block costs the vector
// memory path two (1x1: five) instructions of up to 16 clocks for one tile, and nothing is shared between tiles: that is
// why the dispatch rule counts loads.
//
// What a launch takes beyond the 1.8 us of an empty one that depends on another is this chain, and instructions are a
// large part of it: a block has up to 16 waves, which share four instruction streams, so that a hundred more per wave are
// 0.2-0.7 us.  Hence: one struct of arguments, read in one round; divisions without branches, the tile's share of them in
// scalar registers; an address per kernel row, which the channel blocks move by a scalar offset; validity as a choice
// of address; the residual requested with the inputs; and no code for shared blocks where none are.  The trivial
// kernel with the same blocks, loads, products and sum takes 4.1 us on cold weights in a graph (14x14, 64 channels per
// group: 1.0 us of them the weights, 0.6 the inputs, 0.5 the products).  Per layer of the batch-1 ResNet-34-shaped chain,
// g = 4: 4.4 -> 3.7 us (169 -> 145 us in all), MobileNetV2-shaped 236 -> 205, the pointwise form of the WRN stack 306 -> 238;
// 60 -> 84 on 29x37, g = 3, N = 5 6.9 -> 5.5.  (One chain of products instead of two is level and
// 5-20 % less exact.)
#include <algorithm>
#include <cstring>

#include "conv_common.h"
#include "unit_index.h"

namespace gspc {

typedef float f32x3 __attribute__((ext_vector_type(3)));
typedef unsigned int u32x3 __attribute__((ext_vector_type(3)));

static_assert(sizeof(TileUnit) <= sizeof(((UnitPlan *)0)->data), "plan storage too small");

// SHARE: two or three waves share a channel block (t.parts).
template <int NW, int KH, int S, bool SHARE>
__global__ __launch_bounds__(64 * NW, 8) void conv_mfma16u(TileUnit t) {
    constexpr bool ROW = KH == 3;
    constexpr int UB = ROW ? 2 : 4;                     // channel blocks in flight per wave
    constexpr int KR = ROW ? 3 : 1, PR = ROW ? 3 : 4;   // kernel rows; products of a block's row
    constexpr int OT = NW * 64 < 256 ? NW * 64 : 256, OPT = 256 / OT;   // threads that store, outputs of each
    __shared__ f32x4 part[NW][64];

    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const UnitTileAt tile = unit_tile(t, blockIdx.x);
    const unsigned mt = tile.mt, j = tile.j;
    const unsigned HW = t.H * t.W;

    const __amdgpu_buffer_rsrc_t rx = make_rsrc(t.x, t.x_bytes);
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(t.w, t.w_bytes);

    int first = wave, rows = 7;
    if constexpr (SHARE) {
        const UnitWave shared = unit_share(t, wave);
        first = shared.first;
        rows = shared.rows;
    }
    const auto row_on = [&](int k) { return !SHARE || (rows >> k & 1); };

    // ---- weights (they do not wait for the pixel arithmetic) ---------------------------------------
    constexpr unsigned WLANE = ROW ? 12 : 16;
    u32x4 wv[UB][KR];
    const unsigned wstep = unit_w_step<KR, WLANE>(t), wbase = unit_w_base<KR, WLANE>(t, tile);
    auto fetch_w = [&](int u, int s) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < KR; ++k) {
            const unsigned vo = unit_w_lane<WLANE>(t, u, row_on(k), lane), so = wbase + u * wstep + k * (64 * WLANE);
            if constexpr (ROW) {
                const u32x3 v = __builtin_amdgcn_raw_buffer_load_b96(rw, vo, so, 0);
                wv[s][k] = u32x4{v.x, v.y, v.z, 0u};
            } else {
                wv[s][k] = __builtin_amdgcn_raw_buffer_load_b128(rw, vo, so, 0);
            }
        }
    };
#pragma unroll
    for (int s = 0; s < UB; ++s) fetch_w(first + s * NW, s);

    // ---- this lane's pixel ------------------------------------------------------------------------
    const UnitPixel pix = unit_pixel<KH, S>(t, tile, li);
    const unsigned n = pix.n, rem = pix.rem;
    const bool live = pix.live;
    unsigned xo[KR];
#pragma unroll
    for (int k = 0; k < KR; ++k) xo[k] = unit_x_row<KH>(t, tile, pix, lg, k, row_on(k));
    u32x3 xr[UB][KR];
    unsigned xs[UB][4];
    auto fetch_x = [&](int u, int s) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < (ROW ? 3 : 4); ++e) {
            const int c = ROW ? u * 4 : u * 16 + 4 * e;      // (waves past the last block are past the channels)
            const unsigned vo = unit_x_lane(t, xo[ROW ? e : 0], lg, c), so = c * HW * 4;
            if constexpr (ROW) xr[s][e] = __builtin_amdgcn_raw_buffer_load_b96(rx, vo, so, 0);
            else xs[s][e] = __builtin_amdgcn_raw_buffer_load_b32(rx, vo, so, 0);
        }
    };
#pragma unroll
    for (int s = 0; s < UB; ++s) fetch_x(first + s * NW, s);

    // ---- this thread's outputs: filters tid / 16 (+ 8) of the tile at the lane's pixel --------------
    const unsigned f0 = mt * 16 + tid / 16;
    const size_t at = (size_t)(n * t.Cout + j * t.KPG + f0) * t.HWo + rem;
    float res[OPT];
    if (t.res && tid < OT) {
#pragma unroll
        for (int o = 0; o < OPT; ++o) res[o] = live && f0 + o * (OT / 16) < (unsigned)t.KPG ? t.res[at + (size_t)o * (OT / 16) * t.HWo] : 0.f;
    }
    __builtin_amdgcn_sched_barrier(0);

    f32x4 acc = {0.f, 0.f, 0.f, 0.f}, odd = {0.f, 0.f, 0.f, 0.f};   // even and odd blocks: two chains of products
    const bool left_end = pix.start > pix.iw0, right_end = pix.start < pix.iw0;
    for (int u0 = first; u0 < t.blocks; u0 += UB * NW) {
#pragma unroll
        for (int s = 0; s < UB; ++s) {
            const int u = u0 + s * NW;
            if (u >= t.blocks) break;
#pragma unroll
            for (int k = 0; k < KR; ++k) {
                if (SHARE && !(rows >> k & 1)) continue;
                float b[4];
                if constexpr (ROW) {
                    const float x0 = __uint_as_float(xr[s][k].x), x1 = __uint_as_float(xr[s][k].y), x2 = __uint_as_float(xr[s][k].z);
                    b[0] = left_end ? 0.f : right_end ? x1 : x0;
                    b[1] = left_end ? x0 : right_end ? x2 : x1;
                    b[2] = left_end ? x1 : right_end ? 0.f : x2;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) b[e] = __uint_as_float(xs[s][e]);
                }
#pragma unroll
                for (int e = 0; e < PR; ++e) {
                    f32x4 &c = s & 1 ? odd : acc;
                    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(wv[s][k][e]), b[e], c, 0, 0, 0);
                }
            }
            if (u + UB * NW < t.blocks) {
                fetch_w(u + UB * NW, s);
                fetch_x(u + UB * NW, s);
            }
        }
    }

    // ---- the waves' partial sums; residual, ReLU, NCHW store ---------------------------------------
    part[wave][lane] = acc + odd;
    __syncthreads();
    const float *sum = reinterpret_cast<const float *>(part) + (tid / 64 * 16 + li) * 4 + lg;   // filter tid / 16, pixel li
    if (wave >= OT / 64) return;
#pragma unroll
    for (int o = 0; o < OPT; ++o) {
        float v = sum[o * OT];
#pragma unroll
        for (int k = 1; k < NW; ++k) v += sum[o * OT + k * 256];
        if (live && f0 + o * (OT / 16) < (unsigned)t.KPG) {
            if (t.res) v += res[o];
            t.y[at + (size_t)o * (OT / 16) * t.HWo] = t.relu ? fmaxf(v, 0.f) : v;
        }
    }
}

namespace {

template <int NW, int KH, int S, bool SHARE = false>
hipError_t launchU(const TileUnit &t, hipStream_t s) {
    if constexpr (KH == 3 && !SHARE) {
        if (t.parts > 1) return launchU<NW, KH, S, true>(t, s);
    }
    hipLaunchKernelGGL((conv_mfma16u<NW, KH, S, SHARE>), dim3(unit_blocks(t)), dim3(64 * NW), 0, s, t);
    return hipGetLastError();
}

template <int NW>
hipError_t launchU_shape(const ConvParams &p, const TileUnit &t, hipStream_t s) {
    if (p.KH == 3) return p.stride == 1 ? launchU<NW, 3, 1>(t, s) : launchU<NW, 3, 2>(t, s);
    return p.stride == 1 ? launchU<NW, 1, 1>(t, s) : launchU<NW, 1, 2>(t, s);
}

}  // namespace

bool plan_unit(const ConvParams &p, const PackGeom &g, UnitPlan *out, double more) {
    if (!p.wu || p.in_bf16 || (p.stride != 1 && p.stride != 2)) return false;
    const bool row = p.KH == 3;
    if (row ? p.pad != 1 || p.W < 3 : p.pad != 0) return false;
    const double npix = (double)p.N * p.Hout * p.Wout;
    const double xb = (double)p.N * p.Cin * p.H * p.W * 4;
    if (xb >= (double)kOob || npix >= 1e6 || (double)g.unit_bytes >= (double)kOob) return false;
    if ((double)p.Hout * p.Wout * (p.Hout * p.Wout + 16.0) > 4294967296.0) return false;
    const long px_tiles = ((long)npix + 15) / 16, tiles = px_tiles * g.mtiles * p.groups;
    if ((double)(tiles + 8) * px_tiles >= 4294967296.0 || (double)(g.mtiles * (double)p.groups + 1) * g.mtiles >= 4294967296.0)
        return false;
    TileUnit t{};
    unit_layer(t, p.N, p.Cin, p.H, p.W, p.Cout, p.groups, p.KH, p.Hout, p.Wout, g.mtiles);
    const int units = row ? 3 * t.blocks : t.blocks;     // of the reduction in the rules below: 3x3, a kernel row of a block
    t.w_bytes = (unsigned)g.unit_bytes;
    // Where it pays (us per layer of a recorded chain, the kernel that has the layer otherwise / this one): 256 -> 256 on 14x14, g = 4,
    // N = 2 6.5 / 4.3; 1024 -> 1024 pointwise on 7x7, N = 1 19.5 / 4.9; 60 -> 84 on 29x37, g = 3, N = 5 8.8 / 5.6.  The lines below were
    // drawn for a form of this kernel that took 1.05 to 2 times as long, 1x1 most of all: where the far side of one has this kernel
    // ahead, marked *, it could lie further out.  Operands are loaded once per tile that uses them, so the loads decide:
    //  - 3x3, stride 1, rows of a multiple of 4 (16-byte staging on the other side): 75k loads 6.2 / 5.7 (256 -> 256 on 28x28, g = 8,
    //    N = 2) and 6.6 / 6.0 (on 14x14, g = 4, N = 4), twice the batch 8.9 / 8.8 and 8.5 / 9.6, four times 10.3 / 15.1 and 11.3 / 15.6;
    //  - stride 2, other widths, 1x1: 32 -> 64 on 32x32 at stride 2, g = 2 98k 7.8 / 6.8, 147k 9.4 / 9.1, 197k 11.3 / 11.6, 295k
    //    16.5 / 15.9; 256 -> 256 on 15x15, g = 2, N = 6 (261k) 13.5 / 14.0; 1x1 on planes of a multiple of 4, 512 -> 128 on 14x14 173k
    //    16.0 / 8.8, *188k 15.0 / 9.4 and 251k 14.6 / 11.8, which choose() gives to this kernel after all.
    // With few units a block is mostly its start and its sum, and once the blocks no longer run together that counts:
    //  - fewer than six: 3 -> 32 on 32x32, N = 8 3.5 / 3.0, N = 32 5.1 / 5.5; pointwise on planes that are staged 16 bytes
    //    at a time 64 -> 64 on 16x16, N = 16 (1024 tiles) 4.2 / 3.1, *64 -> 128 (2048) 4.8 / 4.2, *64 -> 64 on 56x56, N = 3
    //    (2352) 5.3 / 4.9, on other planes 64 -> 80 on 55x55, N = 2 (1895) 6.9 / 4.2;
    //  - six, 3x3 with stride 1: 64 -> 64, g = 8 on 16-pixel rows (2048) 5.0 / 3.7, on 20x20, N = 16 (3200) 4.8 / 4.8, *on
    //    13x13, N = 50 (4232) 6.7 / 5.5; with nine 96 -> 96, g = 8 on 17x17 (2312) 7.2 / 4.8;
    //  - six at stride 2, from 17 filters per group on, which the other side then multiplies out of one staged tile: *32 -> 192
    //    on 40x40, g = 4, N = 14 (4200) 7.3 / 5.9, 32 -> 128 on 16x16, g = 4, N = 187 (5984) 6.8 / 7.5;
    //  - ten, pointwise: 160 -> 144 on 20x20, N = 5 (1125) 8.7 / 4.4, *N = 10 (2250) 8.1 / 6.1, and with nine *144 -> 24 on 64x64,
    //    N = 4 (2048) 6.0 / 5.5, 576 -> 96 on 32x32, g = 4 (512) 4.7 / 3.0.
    const double loads = (double)tiles * units * (row ? 2 : 5);
    const bool wide = p.stride == 1 && (row ? p.W % 4 == 0 : (p.Hout * p.Wout) % 4 == 0);   // staged 16 bytes at a time
    if (loads > more * (row ? wide ? 80e3 : p.W % 4 == 0 ? 160e3 : 200e3 : wide ? 180e3 : 200e3)) return false;
    if (units < (row || wide ? 6 : 4) && tiles > 4 * kNumCU) return false;
    if (row && p.stride == 1 && units < 9 && tiles > 8 * kNumCU) return false;
    if (row && p.stride == 2 && units < 9 && g.KPG > 16 && tiles > 12 * kNumCU) return false;
    if (!row && wide && units < 12 && tiles >= 8 * kNumCU) return false;
    // Odd pointwise planes handed over as one row are staged 16 bytes at a time as well:
    //  - 40 .. 63 pixels, which fill most of a 64-pixel tile, while the staged kernel has a block per image (see
    //    fills_image_tiles), from 4 tiles per compute unit on: *384 -> 32 on 7x7, g = 2, N = 178 (1092 tiles) 6.9 / 4.8,
    //    *768 -> 192, g = 8, N = 27 (1328) 5.0 / 4.1, *192 -> 48, g = 2, N = 150 (1840) 5.7 / 4.6;
    //  - more, from 12 on: *256 -> 40 on 9x9, g = 4, N = 170 (3444) 6.5 / 5.7, *512 -> 48 on 11x11, g = 4, N = 133 (4024)
    //    10.0 / 7.8; past the bound on the loads 320 -> 48 on 11x11, N = 212 19.4 / 21.2.
    if (!row && p.stride == 1 && p.H == 1 && p.W % 4 != 0 && p.W >= 64 && p.W <= 256 && g.CPG % 4 == 0 && tiles > 12 * kNumCU)
        return false;
    if (tiles > 4 * kNumCU && fills_image_tiles(p, g.mtiles)) return false;
    // waves per block: what lets every wave request all of its units at once, more as long as all of the launch's waves
    // still start together, eight per compute unit: one block too many costs its start anew (the kernel's earlier form, 8 -> 16
    // on 12x12, g = 2, N = 21: 378 blocks of eight waves 4.4 us, of four 3.6; 230 layers with 230 .. 1000 tiles 0.81 of their time;
    // now 2.8 with four)
    int nw = 2;
    while (nw < 16 && (units > nw * (row ? 6 : 4) || (tiles * nw * 2 <= 8 * kNumCU && units > nw))) nw *= 2;
    // Large 3x3 layers whose waves have places for a third more units than there are (9, 15, 18, 27, 30 of them) go to the
    // kernel that keeps its filters where that takes the layer and the rows fill its 16-pixel tiles (there / here): 144 -> 192 on
    // 16x16, g = 4, N = 7 (1344 tiles) 6.3 / 6.6, *80 -> 256 on 16x16, g = 2, N = 5 (1280) 6.3 / 6.1.  On rows of 12, 20, 24, 28
    // and 40 pixels 28 layers were level with this kernel's earlier form (0.83 .. 1.09), and so were 12 and 24 units, which leave no
    // place empty.
    // Six units leave half of the places empty, and five tiles per compute unit are enough: 16 -> 64 on 16x16, g = 2, N = 29
    // (1856) 3.9 / 3.9, *8 -> 128 on 14x16, N = 15 (1680) 3.9 / 3.7; not on planes that the 32 pixels of its two waves do not
    // divide (16 -> 32 on 14x8, g = 2, N = 144 (2016) 5.1 / 4.0).
    Mfma16wPlan pw;
    if (row && wide && (16 % p.W == 0 || p.W % 16 == 0) && 4 * units <= 3 * 6 * nw &&
        tiles * nw >= (units < 9 && p.H * p.W % 32 == 0 ? 10 : 24) * kNumCU && plan_mfma16w(p, g, &pw))
        return false;
    t.parts = row && nw >= 2 * t.blocks ? std::min(nw / t.blocks, 3) : 1;
    out->nw = nw;
    std::memcpy(out->data, &t, sizeof(t));
    return true;
}

hipError_t launch_unit(const ConvParams &p, const UnitPlan &plan, hipStream_t s, const char **name) {
    TileUnit t;
    std::memcpy(&t, plan.data, sizeof(t));
    t.x = static_cast<const float *>(p.x);
    t.w = p.wu;
    t.y = p.y;
    t.res = p.res;
    t.relu = p.relu;
    if (!*name)
        *name = intern_name("conv_mfma16u<" + std::to_string(plan.nw) + "," + std::to_string(p.KH) + "," + std::to_string(p.stride) + ">");
    switch (plan.nw) {
    case 2: return launchU_shape<2>(p, t, s);
    case 4: return launchU_shape<4>(p, t, s);
    case 8: return launchU_shape<8>(p, t, s);
    case 16: return launchU_shape<16>(p, t, s);
    }
    return hipErrorNotSupported;
}

}  // namespace gspc
