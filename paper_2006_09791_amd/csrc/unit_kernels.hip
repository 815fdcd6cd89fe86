// Small launches (batch 1 and the like): per-group implicit GEMM on v_mfma_f32_16x16x4_f32 without staging.
//
// A block owns one tile of 16 filters x 16 output pixels and its waves split the reduction; every operand
// goes from global memory (L2) straight into the registers of the lane that multiplies it, so that all loads
// of a wave are on their way before the first product, and the only barrier is the one before the partial
// sums are added.  Such a launch is a chain of latencies - kernel start, addresses, one trip to memory,
// products, the sum, the store - and conv_mfma16's chunks put three or four more trips into it.
//
// A unit of the reduction is four channels (lane / 16) and, for 3x3 layers, one kernel row: a lane loads the
// three taps of its pixel (lane % 16) and the three weights of its filter with one 12-byte load each and
// multiplies three times; for 1x1 layers sixteen channels, one 16-byte load of weights and four of inputs.
// A unit costs the vector memory path two (1x1: five) instructions of up to 16 clocks for one tile, and nothing
// is shared between tiles: that is what bounds it, and why the dispatch rule counts loads.  One 14x14 layer of
// 256 channels in 4 groups at N = 1: 8.9 -> 3.5 us in the kernel trace.
#include <cstring>

#include "conv_common.h"

namespace gspc {

typedef float f32x3 __attribute__((ext_vector_type(3)));
typedef unsigned int u32x3 __attribute__((ext_vector_type(3)));

struct TileUnit {
    int units, cblks, mtiles;        // units of the reduction, blocks of four channels, filter tiles per group
    unsigned npix, m_Wout;           // N * Hout * Wout; reciprocal
    unsigned x_bytes, w_bytes;
};
static_assert(sizeof(TileUnit) <= sizeof(((UnitPlan *)0)->data), "plan storage too small");

template <int NW, int KH, int S>
__global__ __launch_bounds__(64 * NW) void conv_mfma16u(ConvParams p, TileUnit t) {
    constexpr bool ROW = KH == 3;
    constexpr int UB = ROW ? 6 : 4;                     // units in flight per wave
    __shared__ float part[NW][16][17];

    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned j = blockIdx.z, mt = blockIdx.y;
    const unsigned HWo = p.Hout * p.Wout, HW = p.H * p.W;

    const __amdgpu_buffer_rsrc_t rx = make_rsrc(p.x, t.x_bytes);
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(p.wu, t.w_bytes);

    // weights: [g][unit block][filter tile]([kernel row])[64 lanes][3 or 4]
    constexpr unsigned WLANE = ROW ? 12 : 16, WUNIT = 64 * WLANE;
    auto w_off = [&](int u) -> unsigned {               // wave-uniform
        if (ROW) return ((j * t.cblks + u / 3) * t.mtiles + mt) * (3 * WUNIT) + (u % 3) * WUNIT;
        return ((j * t.units + u) * t.mtiles + mt) * WUNIT;
    };
    u32x4 wv[UB];
    auto fetch_w = [&](int u, int s) __attribute__((always_inline)) {
        const unsigned vo = u < t.units ? lane * WLANE : kOob;
        if (ROW) {
            const u32x3 v = __builtin_amdgcn_raw_buffer_load_b96(rw, vo, w_off(u), 0);
            wv[s] = u32x4{v.x, v.y, v.z, 0u};
        } else {
            wv[s] = __builtin_amdgcn_raw_buffer_load_b128(rw, vo, w_off(u), 0);
        }
    };
#pragma unroll
    for (int s = 0; s < UB; ++s) fetch_w(wave + s * NW, s);   // (they do not wait for the pixel arithmetic)

    // ---- this lane's pixel ------------------------------------------------------------------------
    const unsigned q = blockIdx.x * 16 + li;
    const bool live = q < t.npix;
    const unsigned n = q / HWo, rem = q - n * HWo;
    const unsigned oh = fast_div(rem, t.m_Wout), ow = rem - oh * p.Wout;
    const int ih0 = (int)oh * S - p.pad, iw0 = (int)ow * S - p.pad;
    // 3x3 (padding 1): the three columns are loaded from inside the row; at its left (right) end they move one
    // place up (down) and a zero takes the place of the column outside
    const int start = ROW ? min(max(iw0, 0), p.W - 3) : iw0;
    const int shift = start - iw0;
    const unsigned xpix = ((n * p.Cin + j * p.CPG + lg) * HW + start) * 4u;
    u32x3 xr[ROW ? UB : 1];
    unsigned xs[ROW ? 1 : UB][4];
    auto fetch_x = [&](int u, int s) __attribute__((always_inline)) {
        if constexpr (ROW) {
            const int cb = u / 3, ih = ih0 + u % 3;
            const bool ok = live && u < t.units && cb * 4 + lg < p.CPG && (unsigned)ih < (unsigned)p.H;
            xr[s] = __builtin_amdgcn_raw_buffer_load_b96(rx, ok ? xpix + (cb * 4 * HW + ih * p.W) * 4u : kOob, 0, 0);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int cb = u * 4 + e;
                const bool ok = live && cb * 4 + lg < p.CPG;
                xs[s][e] = __builtin_amdgcn_raw_buffer_load_b32(rx, ok ? xpix + (cb * 4 * HW + ih0 * p.W) * 4u : kOob, 0, 0);
            }
        }
    };
#pragma unroll
    for (int s = 0; s < UB; ++s) fetch_x(wave + s * NW, s);
    __builtin_amdgcn_sched_barrier(0);

    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int u0 = wave; u0 < t.units; u0 += UB * NW) {
        const bool more = u0 + UB * NW < t.units;
#pragma unroll
        for (int s = 0; s < UB; ++s) {
            float b[4];
            if constexpr (ROW) {
                const float x0 = __uint_as_float(xr[s].x), x1 = __uint_as_float(xr[s].y), x2 = __uint_as_float(xr[s].z);
                b[0] = shift > 0 ? 0.f : shift < 0 ? x1 : x0;
                b[1] = shift > 0 ? x0 : shift < 0 ? x2 : x1;
                b[2] = shift > 0 ? x1 : shift < 0 ? 0.f : x2;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) b[e] = __uint_as_float(xs[s][e]);
            }
#pragma unroll
            for (int e = 0; e < (ROW ? 3 : 4); ++e)
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(wv[s][e]), b[e], acc, 0, 0, 0);
            if (more) {
                const int u = u0 + (s + UB) * NW;
                fetch_w(u, s);
                fetch_x(u, s);
            }
        }
    }

    // ---- the waves' partial sums; residual, ReLU, NCHW store ---------------------------------------
#pragma unroll
    for (int r = 0; r < 4; ++r) part[wave][4 * lg + r][li] = acc[r];
    __syncthreads();
    constexpr int OT = NW * 64 < 256 ? NW * 64 : 256;    // threads that store
    if (tid >= OT) return;
#pragma unroll
    for (int o = tid; o < 256; o += OT) {
        const int f = o >> 4, px = o & 15;
        float v = part[0][f][px];
#pragma unroll
        for (int k = 1; k < NW; ++k) v += part[k][f][px];
        const unsigned qo = blockIdx.x * 16 + px, fo = mt * 16 + f;
        if (qo < t.npix && fo < (unsigned)p.KPG) {
            const unsigned no = qo / HWo;
            const size_t at = (size_t)(no * p.Cout + j * p.KPG + fo) * HWo + (qo - no * HWo);
            if (p.res) v += p.res[at];
            p.y[at] = p.relu ? fmaxf(v, 0.f) : v;
        }
    }
}

namespace {

template <int NW, int KH, int S>
hipError_t launchU(const ConvParams &p, const TileUnit &t, hipStream_t s) {
    hipLaunchKernelGGL((conv_mfma16u<NW, KH, S>), dim3((t.npix + 15) / 16, t.mtiles, p.groups), dim3(64 * NW), 0, s, p, t);
    return hipGetLastError();
}

template <int NW>
hipError_t launchU_shape(const ConvParams &p, const TileUnit &t, hipStream_t s) {
    if (p.KH == 3) return p.stride == 1 ? launchU<NW, 3, 1>(p, t, s) : launchU<NW, 3, 2>(p, t, s);
    return p.stride == 1 ? launchU<NW, 1, 1>(p, t, s) : launchU<NW, 1, 2>(p, t, s);
}

}  // namespace

bool plan_unit(const ConvParams &p, const PackGeom &g, UnitPlan *out) {
    if (!p.wu || p.in_bf16 || (p.stride != 1 && p.stride != 2)) return false;
    const bool row = p.KH == 3;
    if (row ? p.pad != 1 || p.W < 3 : p.pad != 0) return false;
    const double npix = (double)p.N * p.Hout * p.Wout;
    const double xb = (double)p.N * p.Cin * p.H * p.W * 4;
    if (xb >= (double)kOob || npix >= 1e6 || (double)g.unit_bytes >= (double)kOob) return false;
    if (p.groups > 65535 || g.mtiles > 65535 || (long)p.Hout * p.Wout >= 65536) return false;
    TileUnit t{};
    t.cblks = g.CPGp / 4;
    t.units = row ? t.cblks * 3 : (t.cblks + 3) / 4;
    t.mtiles = g.mtiles;
    t.npix = (unsigned)npix;
    t.m_Wout = div_magic(p.Wout);
    t.x_bytes = (unsigned)xb;
    t.w_bytes = (unsigned)g.unit_bytes;
    // Where it pays (layers of the WRN-, ResNet-34- and MobileNet-shaped networks at N = 1 .. 64, us, conv_mfma16 with
    // staging / this kernel): 2 x 256 -> 256 on 14x14, g = 4 7.2 / 4.8; 1024 -> 1024 pointwise on 7x7, N = 1 19.1 / 6.6;
    // 60 -> 84 on 29x37, g = 3, N = 5 9.1 / 6.9.  Operands are loaded once per tile that uses them, so the loads decide:
    //  - 3x3, stride 1, rows of a multiple of 4 (16-byte staging on the other side): 75k loads 8.3 / 6.5 and 9.4 / 6.6,
    //    150k 9.1 / 10.0 and 13.1 / 10.0, 300k 13.4 / 16.6;
    //  - stride 2, other widths, 1x1: 150k 12.7 / 10.2 and 18.2 / 9.9, 200k (32 -> 64 on 32x32 at stride 2) 10.2 / 11.4,
    //    300k 16.7 / 18.0 and 20.0 / 22.2; pointwise on planes of a multiple of 4 174k 15.4 / 11.6, 189k 13.9 / 16.8.
    // With few units a block is mostly its start and its sum, and once the blocks no longer run together that counts:
    //  - fewer than six: 3 -> 32 on 32x32, N = 8 4.9 / 4.7, N = 32 5.2 / 6.8; pointwise on planes that are staged 16 bytes
    //    at a time 64 -> 64 on 16x16, N = 16 (1024 tiles) 5.0 / 4.7, 64 -> 128 (2048) 5.0 / 5.3, 64 -> 64 on 56x56, N = 3
    //    (2352) 5.4 / 6.6, on other planes 64 -> 80 on 55x55, N = 2 (1895) 8.0 / 6.5;
    //  - six, 3x3 with stride 1: 64 -> 64, g = 8 on 16-pixel rows (2048) 4.8 / 4.7, on 20x20, N = 16 (3200) 5.1 / 6.1, on
    //    13x13, N = 50 (4232) 6.6 / 7.7; with nine 96 -> 96, g = 8 on 17x17 (2312) 7.4 / 5.9;
    //  - six at stride 2, from 17 filters per group on, which the other side then multiplies out of one staged tile: 32 -> 192
    //    on 40x40, g = 4, N = 14 (4200) 7.5 / 8.6, 32 -> 128 on 16x16, g = 4, N = 187 (5984) 7.2 / 10.1, 78 layers 0.82;
    //    with up to 16 filters 37 layers are level;
    //  - ten, pointwise: 160 -> 144 on 20x20, N = 5 (1125) 9.0 / 5.9, N = 10 (2250) 8.7 / 9.8, and with nine 144 -> 24 on 64x64,
    //    N = 4 (2048) 6.5 / 9.7, 576 -> 96 on 32x32, g = 4 6.6 / 9.0.
    const long tiles = (long)((t.npix + 15) / 16) * g.mtiles * p.groups;
    const double loads = (double)tiles * t.units * (row ? 2 : 5);
    const bool wide = p.stride == 1 && (row ? p.W % 4 == 0 : (p.Hout * p.Wout) % 4 == 0);   // staged 16 bytes at a time
    if (loads > (row ? wide ? 80e3 : p.W % 4 == 0 ? 160e3 : 200e3 : wide ? 180e3 : 200e3)) return false;
    if (t.units < (row || wide ? 6 : 4) && tiles > 4 * kNumCU) return false;
    if (row && p.stride == 1 && t.units < 9 && tiles > 8 * kNumCU) return false;
    if (row && p.stride == 2 && t.units < 9 && g.KPG > 16 && tiles > 12 * kNumCU) return false;
    if (!row && wide && t.units < 12 && tiles >= 8 * kNumCU) return false;
    // Odd pointwise planes handed over as one row are staged 16 bytes at a time as well:
    //  - 40 .. 63 pixels, which fill most of a 64-pixel tile: while the staged kernel has a block per image (see
    //    fills_image_tiles) it is ahead from 4 tiles per compute unit on: 384 -> 32 on 7x7, g = 2, N = 178 (1092 tiles)
    //    10.5 / 7.3 here / staged, 768 -> 192, g = 8, N = 27 (1328) 7.8 / 5.3, 192 -> 48, g = 2, N = 150 (1840) 9.3 / 6.4;
    //  - more: from 12 on: 256 -> 40 on 9x9, g = 4, N = 170 (3444) 11.2 / 7.9, 512 -> 48 on 11x11, g = 4, N = 133 (4024)
    //    18.0 / 11.5 (one of 19 layers the other way round: 320 -> 48 on 11x11, N = 212 19.1 / 26.5).
    if (!row && p.stride == 1 && p.H == 1 && p.W % 4 != 0 && p.W >= 64 && p.W <= 256 && g.CPG % 4 == 0 && tiles > 12 * kNumCU)
        return false;
    if (tiles > 4 * kNumCU && fills_image_tiles(p, g.mtiles)) return false;
    // waves per block: what lets every wave request all of its units at once, more as long as all of the launch's waves
    // still start together, eight per compute unit: one block too many costs its start anew (8 -> 16 on 12x12, g = 2,
    // N = 21: 378 blocks of eight waves 4.4 us, of four 3.6; 230 layers with 230 .. 1000 tiles 0.81 of their time)
    int nw = 2;
    while (nw < 16 && (t.units > nw * (row ? 6 : 4) || (tiles * nw * 2 <= 8 * kNumCU && t.units > nw))) nw *= 2;
    // Large 3x3 layers whose waves have places for a third more units than there are (9, 15, 18, 27, 30 of them) go to the
    // kernel that keeps its filters where that takes the layer and the rows fill its 16-pixel tiles: 20 -> 64 on 32x32,
    // N = 4, g = 2 (2048 tiles) 6.9 / 5.3 here / there, 144 -> 192 on 16x16, g = 4, N = 7 (1344) 8.6 / 6.5, 80 -> 256 on 16x16,
    // g = 2, N = 5 (1280) 7.8 / 6.6; 128 layers 0.84.  On rows of 12, 20, 24, 28 and 40 pixels 28 layers are level (0.83 ..
    // 1.09), and so are 12 and 24 units, which leave no place empty.
    // Six units leave half of the places empty, and five tiles per compute unit are enough: 16 -> 64 on 16x16, g = 2, N = 29
    // (1856) 4.8 / 4.3, 8 -> 128 on 14x16, N = 15 (1680) 4.8 / 4.3, with 4.5 tiles level; not on planes that the 32 pixels of
    // its two waves do not divide (16 -> 32 on 14x8, g = 2, N = 144 (2016) 4.9 / 5.3).
    Mfma16wPlan pw;
    if (row && wide && (16 % p.W == 0 || p.W % 16 == 0) && 4 * t.units <= 3 * 6 * nw &&
        tiles * nw >= (t.units < 9 && p.H * p.W % 32 == 0 ? 10 : 24) * kNumCU && plan_mfma16w(p, g, &pw))
        return false;
    out->nw = nw;
    std::memcpy(out->data, &t, sizeof(t));
    return true;
}

hipError_t launch_unit(const ConvParams &p, const UnitPlan &plan, hipStream_t s, const char **name) {
    TileUnit t;
    std::memcpy(&t, plan.data, sizeof(t));
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
