// Depthwise 3x3 convolution, padding 1 (g = Cin = Cout, the G(N) end of the paper's sweep,
// Section IV of arXiv 2006.09791).
//
// With one channel per group the input planes of consecutive (image, channel)
// pairs are consecutive in NCHW memory, and so are the output planes: a wavefront
// takes a contiguous piece of the input (whole planes, or a band of rows of one),
// copies it flat into an LDS region of its own with 16-byte accesses and reads its
// windows there.  LDS operations of one wavefront execute in order, so nothing here
// needs a barrier.  HBM-bound.
//
//   conv_dw_wave      whole 56x56, 28x28, 14x14 and 7x7 planes, launches that fill the chip;
//   conv_dw_band      112x112 planes, a band of 16 rows per wavefront;
//   conv_direct_rows  fp32 planes that the strip kernel (conv_direct_small) does not take and four output rows of which need at
//                     most 2048 floats of input (rows of up to 340 elements at stride 1 and 227 at stride 2, wider on planes of
//                     few rows), but for launches of few large planes; small and large launches of small planes that it would take;
//   conv_direct_narrow  the same with one output row at a time, larger launches of short rows.
// Other planes and bf16 inputs stay on conv_direct_flat.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>

#include "split_common.h"

namespace gspc {

// n / d with mul = floor(2^32 / d) + 1, 0 for d = 1, while n * d < 2^32.  In the wave kernels the branch (or select) keeps the loads of the
// weights behind those of the input: with fast_div the compiler moves them in front, 448 channels on 56x56, N = 6 14.6 / 15.8 us
// (14.9 with a scheduling barrier between them).
__device__ __forceinline__ unsigned div_in_order(unsigned n, unsigned mul) { return mul ? __umulhi(n, mul) : n; }
inline unsigned magic_in_order(unsigned d) { return d > 1 ? 0xffffffffu / d + 1u : 0u; }

// ---- whole planes per wavefront -------------------------------------------------------------
// For the square planes of the network tails (28x28, 14x14, 7x7) a wavefront takes G consecutive
// planes by itself: their floats are one contiguous, 16-byte aligned piece of the input and their
// outputs one contiguous piece of the output.  The piece is copied flat into a wave-private LDS
// region (16-byte loads and LDS writes, no re-pitch and no halo: the left and right padding
// columns are dropped from the unrolled sums at compile time, the top and bottom padding rows are
// selected to zero per lane), a lane reads the (R-1)*S + 3 input rows of its R output rows as one
// contiguous window into registers, multiplies them out, writes the R*Wout results back into the
// region at their flat output position (the region is reused: every lane has its window in
// registers by then), and the wave reads the results back 16 bytes per lane in flat order for
// coalesced stores (residual and ReLU applied there).  LDS operations of one wavefront execute in
// order, so no barrier is needed anywhere; memory clobbers keep the compiler from reordering the
// phases.  Per lane and R*Wout outputs this takes a few dozen wide LDS operations where the
// sum read per output takes nine 4-byte reads.
template <int S, int H, int W, int R, int CP = -1>
struct DwWaveGeom {
    static constexpr int Hout = (H - 1) / S + 1, Wout = (W - 1) / S + 1;
    static constexpr int HW = H * W, HoWo = Hout * Wout;
    static constexpr int LP = (Hout + R - 1) / R;           // lanes per plane (the last one may own fewer rows)
    static constexpr bool RAG = Hout % R != 0;
    static constexpr int pick_g() {
        for (int g = 64 / LP; g >= 1; --g)
            if ((g * HW) % 4 == 0 && (g * HoWo) % 4 == 0) return g;
        return 0;
    }
    static constexpr int G = pick_g();                      // planes per wavefront
    static constexpr int IN = G * HW, OUT = G * HoWo;       // floats per wavefront
    static constexpr int NSI = (IN / 4 + 63) / 64, NSO = (OUT / 4 + 63) / 64;
    static constexpr int NR = (R - 1) * S + 3;              // input rows of a lane's window
    static constexpr int FRONT = (W + 3) / 4 * 4;           // the first plane's row -1
    static constexpr int over = (LP * R - 1) * S + 2 - H;   // rows the last window reaches past its plane
    static constexpr int BACK = (over > 0 ? over : 0) * W;
    static constexpr int REGION = (FRONT + IN + BACK + 3) / 4 * 4;   // floats per wavefront
    static constexpr int VR = W % 4 == 0 ? 4 : W % 2 == 0 ? 2 : 1;   // window reads
    static constexpr int ao = RAG ? Wout : R * Wout;        // floats written at one aligned position
    static constexpr int VO = (ao % 4 == 0 && HoWo % 4 == 0) ? 4 : (ao % 2 == 0 && HoWo % 2 == 0) ? 2 : 1;
    // the nine weights of the wave's planes: fetched lane by lane (9 loads), or, when the wave has few planes,
    // as one flat list of G*9 values through LDS (NWS loads)
    static constexpr int NWS = (G * 9 + 63) / 64;
    static constexpr bool COOP = CP < 0 ? NWS <= 4 : CP != 0;
    static constexpr int WTS = COOP ? (G * 9 + 3) / 4 * 4 : 0;
    static constexpr int WAVE_FLOATS = REGION + WTS;
    static_assert(G > 0 && OUT <= IN, "unsupported shape");
};

struct TileW {
    unsigned chunks, planes, m_C;
    unsigned x_bytes, y_bytes, w_bytes;
};

template <int S, int H, int W, int R, int CP>
__global__ __launch_bounds__(256) void conv_dw_wave(ConvParams p, TileW t) {
    using Q = DwWaveGeom<S, H, W, R, CP>;
    extern __shared__ f32x4 smem4[];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const unsigned chunk = blockIdx.x * 4 + wv;
    if (chunk >= t.chunks) return;   // wave-uniform; the kernel has no barriers
    float *reg = reinterpret_cast<float *>(smem4) + wv * Q::WAVE_FLOATS;
    float *data = reg + Q::FRONT;
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(p.x, t.x_bytes);
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(p.wd, t.w_bytes);

    // ---- the wave's planes, requested first ----
    const unsigned gbase = chunk * (unsigned)(Q::IN * 4);
    f32x4 pin[Q::NSI];
#pragma unroll
    for (int j = 0; j < Q::NSI; ++j) {
        const int q = lane + 64 * j;
        pin[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rx, q * 4 < Q::IN ? gbase + q * 16 : kOob, 0, 0));
    }
    // ---- the lane's plane, rows and weights ----
    const bool active = lane < Q::G * Q::LP;
    const int la = active ? lane : 0;
    const int pl = Q::LP == 1 ? la : la / Q::LP;
    const int oh0 = Q::LP == 1 ? 0 : (la - pl * Q::LP) * R;
    float w[9];
    if constexpr (Q::COOP) {
        float *wts = reg + Q::REGION;
#pragma unroll
        for (int j = 0; j < Q::NWS; ++j) {
            const int i = lane + 64 * j;
            if (i < Q::G * 9) {
                const int wp = i / 9, k = i - wp * 9;
                unsigned pg = chunk * Q::G + wp;
                pg = pg < t.planes ? pg : t.planes - 1;
                const unsigned c = pg - div_in_order(pg, t.m_C) * p.Cin;
                wts[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rw, ((c * 9 + k) * p.KPGd) * 4, 0, 0));
            }
        }
    } else {
        unsigned pg = chunk * Q::G + pl;
        pg = pg < t.planes ? pg : t.planes - 1;
        const unsigned c = pg - div_in_order(pg, t.m_C) * p.Cin;
#pragma unroll
        for (int k = 0; k < 9; ++k)
            w[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rw, ((c * 9 + k) * p.KPGd) * 4, 0, 0));
    }
#pragma unroll
    for (int j = 0; j < Q::NSI; ++j) {
        const int q = lane + 64 * j;
        if (q * 4 < Q::IN) *reinterpret_cast<f32x4 *>(data + q * 4) = pin[j];
    }
    asm volatile("" ::: "memory");
    if constexpr (Q::COOP) {
        const float *wts = reg + Q::REGION;
#pragma unroll
        for (int k = 0; k < 9; ++k) w[k] = wts[pl * 9 + k];
    }
    // ---- window: rows oh0*S - 1 .. oh0*S - 1 + NR - 1 of the plane ----
    float xr[Q::NR][W];
    {
        const int ih0 = oh0 * S - 1;
        const float *wp = data + pl * Q::HW + ih0 * W;
#pragma unroll
        for (int i = 0; i < Q::NR; ++i) {
            const bool valid = (unsigned)(ih0 + i) < (unsigned)H;
#pragma unroll
            for (int x = 0; x < W; x += Q::VR) {
                if constexpr (Q::VR == 4) {
                    const f32x4 v = *reinterpret_cast<const f32x4 *>(wp + i * W + x);
                    xr[i][x] = valid ? v.x : 0.f;
                    xr[i][x + 1] = valid ? v.y : 0.f;
                    xr[i][x + 2] = valid ? v.z : 0.f;
                    xr[i][x + 3] = valid ? v.w : 0.f;
                } else if constexpr (Q::VR == 2) {
                    const float2 v = *reinterpret_cast<const float2 *>(wp + i * W + x);
                    xr[i][x] = valid ? v.x : 0.f;
                    xr[i][x + 1] = valid ? v.y : 0.f;
                } else {
                    const float v = wp[i * W + x];
                    xr[i][x] = valid ? v : 0.f;
                }
            }
        }
    }
    asm volatile("" ::: "memory");
    // ---- R rows of Wout outputs, written to their flat position in the region ----
    {
        float *op = data + pl * Q::HoWo + oh0 * Q::Wout;
        float acc[R * Q::Wout];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int ow = 0; ow < Q::Wout; ++ow) {
                float a = 0.f;
#pragma unroll
                for (int kh = 0; kh < 3; ++kh)
#pragma unroll
                    for (int kw = 0; kw < 3; ++kw) {
                        const int col = ow * S - 1 + kw;
                        if (col >= 0 && col < W) a = fmaf(xr[r * S + kh][col], w[kh * 3 + kw], a);
                    }
                acc[r * Q::Wout + ow] = a;
            }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            // without ragged rows the lane's R rows are written as one run
            if (active && (!Q::RAG || oh0 + r < Q::Hout)) {
#pragma unroll
                for (int x = 0; x < Q::Wout; x += (Q::RAG ? Q::VO : 1)) {
                    const int e = r * Q::Wout + x;
                    if (!Q::RAG && e % Q::VO != 0) continue;
                    if constexpr (Q::VO == 4) *reinterpret_cast<f32x4 *>(op + e) = f32x4{acc[e], acc[e + 1], acc[e + 2], acc[e + 3]};
                    else if constexpr (Q::VO == 2) *reinterpret_cast<float2 *>(op + e) = float2{acc[e], acc[e + 1]};
                    else op[e] = acc[e];
                }
            }
        }
    }
    asm volatile("" ::: "memory");
    // ---- flat read-back, residual, ReLU, 16-byte stores ----
    const __amdgpu_buffer_rsrc_t ry = make_rsrc(p.y, t.y_bytes);
    const __amdgpu_buffer_rsrc_t rr = make_rsrc(p.res ? p.res : p.y, t.y_bytes);
    const unsigned obase = chunk * (unsigned)(Q::OUT * 4);
#pragma unroll
    for (int j = 0; j < Q::NSO; ++j) {
        const int q = lane + 64 * j;
        if (q * 4 < Q::OUT) {
            f32x4 v = *reinterpret_cast<const f32x4 *>(data + q * 4);
            if (p.res) v += __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rr, obase + q * 16, 0, 0));
            if (p.relu) v = f32x4{fmaxf(v.x, 0.f), fmaxf(v.y, 0.f), fmaxf(v.z, 0.f), fmaxf(v.w, 0.f)};
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), ry, obase + q * 16, 0, 0);
        }
    }
}

constexpr int kDwKind = 23, kDwInst = 22;   // plan slots: 1 = whole planes per wavefront, and its instance

// Instances of conv_dw_wave: (stride, plane edge, output rows per lane, weights through LDS), each the fastest of
// the forms measured at N = 256 (one row per lane except on 7x7 planes at stride 2; the 56x56 stride-2 layer
// is faster on the strip kernel and has no instance).
template <int I> struct DwWaveInst;
#define GSPC_DW_WAVE_INST(I, S_, E_, R_, CP_) \
    template <> struct DwWaveInst<I> { using Q = DwWaveGeom<S_, E_, E_, R_, CP_>; static constexpr int S = S_, E = E_, R = R_, CP = CP_; }
GSPC_DW_WAVE_INST(0, 1, 28, 1, 0);
GSPC_DW_WAVE_INST(1, 2, 28, 1, 0);
GSPC_DW_WAVE_INST(2, 1, 14, 1, 0);
GSPC_DW_WAVE_INST(3, 2, 14, 1, 0);
GSPC_DW_WAVE_INST(4, 1, 7, 1, 1);
GSPC_DW_WAVE_INST(5, 2, 7, 2, 0);
GSPC_DW_WAVE_INST(6, 1, 56, 1, 0);
constexpr int kDwWaveInsts = 7;

template <int I>
bool plan_dw_wave_inst(const ConvParams &p, DwPlan *out) {
    using T = DwWaveInst<I>;
    using Q = typename T::Q;
    if (p.stride != T::S || p.H != T::E || p.W != T::E) return false;
    const double planes = (double)p.N * p.Cin;
    const double chunks = (planes + Q::G - 1) / Q::G;
    // small launches: the forms that spread over the chip
    static const bool force = std::getenv("GSPC_DW_WAVE") != nullptr;   // tuning aid
    if (!force && chunks < 4.0 * 2 * kNumCU) return false;
    const double xb = planes * Q::HW * 4, yb = planes * Q::HoWo * 4, wb = (double)p.groups * 9 * p.KPGd * 4;
    const double slack = 4.0 * Q::IN * 4 + 65536;   // offsets past the tensor's end must not wrap
    if (planes >= 2147483648.0 || xb + slack >= (double)kOob || yb + slack >= (double)kOob || wb >= (double)kOob ||
        planes * p.Cin >= 4.29e9)
        return false;
    TileW t{};
    t.planes = (unsigned)planes;
    t.chunks = (unsigned)((t.planes + Q::G - 1) / Q::G);
    t.m_C = magic_in_order(p.Cin);
    t.x_bytes = (unsigned)xb;
    t.y_bytes = (unsigned)yb;
    t.w_bytes = (unsigned)wb;
    static_assert(sizeof(TileW) <= sizeof(int) * kDwInst, "plan storage too small");
    std::memcpy(out->data, &t, sizeof(t));
    out->data[kDwKind] = 1;
    out->data[kDwInst] = I;
    return true;
}

template <int I = 0>
bool plan_dw_wave(const ConvParams &p, DwPlan *out) {
    static const bool off = std::getenv("GSPC_NO_DWWAVE") != nullptr;   // tuning aid
    if (off) return false;
    if constexpr (I < kDwWaveInsts) return plan_dw_wave_inst<I>(p, out) || plan_dw_wave<I + 1>(p, out);
    else return false;
}

template <int I = 0>
hipError_t launch_dw_wave(int inst, const ConvParams &p, const TileW &t, hipStream_t s, const char **name) {
    if constexpr (I < kDwWaveInsts) {
        if (inst != I) return launch_dw_wave<I + 1>(inst, p, t, s, name);
        using T = DwWaveInst<I>;
        using Q = typename T::Q;
        *name = intern_name("conv_dw_wave<" + std::to_string(T::S) + "," + std::to_string(T::E) + "," + std::to_string(T::E) +
                            "," + std::to_string(T::R) + "," + std::to_string(T::CP) + ">");
        const size_t lds = (size_t)4 * Q::WAVE_FLOATS * sizeof(float);
        hipLaunchKernelGGL((conv_dw_wave<T::S, T::E, T::E, T::R, T::CP>), dim3((t.chunks + 3) / 4), dim3(256), lds, s, p, t);
        return hipGetLastError();
    } else {
        return hipErrorNotSupported;
    }
}

// ---- bands of rows per wavefront (planes too large for the form above) ---------------------------
// The same scheme for one band of BR output rows of one plane per wavefront: the (BR-1)*S + 3 input rows the
// band needs are contiguous in memory and are copied flat (the rows above the first and below the last band are
// other planes' rows, or lie outside the tensor and arrive as zeros: either way they are selected to zero).  A lane
// owns CW = Wout / NQ consecutive outputs of one row; its 3-row window is read with aligned 8- or 16-byte LDS reads
// that start VR floats to the left of its first column, the columns left of the plane and right of it are selected
// to zero.  The plane's nine weights are uniform over the wavefront and sit in scalar registers.
template <int S, int H, int W, int BR, int NQ>
struct DwBandGeom {
    static constexpr int Hout = (H - 1) / S + 1, Wout = (W - 1) / S + 1;
    static constexpr int NBD = Hout / BR;                    // bands per plane
    static constexpr int CW = Wout / NQ;                     // outputs per lane
    static constexpr int NRB = (BR - 1) * S + 3;             // input rows per band
    static constexpr int IN = NRB * W, OUT = BR * Wout;      // floats per band
    static constexpr int NSI = (IN / 4 + 63) / 64, NSO = (OUT / 4 + 63) / 64;
    static constexpr int VR = (CW * S) % 4 == 0 ? 4 : 2;     // alignment (floats) of a lane's first column
    static constexpr int WIN = (CW - 1) * S + 3;             // window columns
    static constexpr int XW = (VR - 1 + WIN + VR - 1) / VR * VR;   // floats read per window row
    static constexpr int REGION = (VR + IN + XW + 3) / 4 * 4;
    static constexpr int VO = CW % 4 == 0 ? 4 : CW % 2 == 0 ? 2 : 1;
    static_assert(Hout % BR == 0 && Wout % NQ == 0 && BR * NQ <= 64 && W % 4 == 0 && OUT % 4 == 0 &&
                      (Hout * Wout) % 4 == 0 && (CW * S) % 2 == 0 && VR >= 2,
                  "unsupported band shape");
};

template <int S, int H, int W, int BR, int NQ>
__global__ __launch_bounds__(256) void conv_dw_band(ConvParams p, TileW t) {
    using Q = DwBandGeom<S, H, W, BR, NQ>;
    extern __shared__ f32x4 smem4[];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const unsigned chunk = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + wv);
    if (chunk >= t.chunks) return;   // wave-uniform; the kernel has no barriers
    float *data = reinterpret_cast<float *>(smem4) + wv * Q::REGION + Q::VR;
    const unsigned plane = chunk / Q::NBD, band = chunk - plane * Q::NBD;
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(p.x, t.x_bytes);

    // ---- the band's input rows, requested first (the row above the first band of the first plane has a
    // "negative" offset, which wraps to out of range and reads as zero) ----
    const int ihb = (int)band * (BR * S) - 1;   // first input row of the band
    const unsigned gbase = (plane * (unsigned)(H * W) + (unsigned)(ihb * W)) * 4u;
    f32x4 pin[Q::NSI];
#pragma unroll
    for (int j = 0; j < Q::NSI; ++j) {
        const int q = lane + 64 * j;
        pin[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rx, q * 4 < Q::IN ? gbase + q * 16 : kOob, 0, 0));
    }
    // ---- weights: uniform over the wave ----
    float w[9];
    {
        const unsigned c = plane - div_in_order(plane, t.m_C) * p.Cin;
#pragma unroll
        for (int k = 0; k < 9; ++k) w[k] = p.wd[(c * 9 + k) * p.KPGd];
    }
    const bool active = lane < BR * NQ;
    const int la = active ? lane : 0;
    const int r = la / NQ, qs = la - r * NQ;
#pragma unroll
    for (int j = 0; j < Q::NSI; ++j) {
        const int q = lane + 64 * j;
        if (q * 4 < Q::IN) *reinterpret_cast<f32x4 *>(data + q * 4) = pin[j];
    }
    asm volatile("" ::: "memory");
    // ---- window: 3 rows x XW floats from column qs*CW*S - VR ----
    float acc[Q::CW];
#pragma unroll
    for (int x = 0; x < Q::CW; ++x) acc[x] = 0.f;
    {
        const float *wp = data + (r * S) * W + qs * (Q::CW * S) - Q::VR;
#pragma unroll
        for (int kh = 0; kh < 3; ++kh) {
            const bool rvalid = (unsigned)(ihb + r * S + kh) < (unsigned)H;
            float xr[Q::XW];
#pragma unroll
            for (int x = 0; x < Q::XW; x += Q::VR) {
                if constexpr (Q::VR == 4) {
                    const f32x4 v = *reinterpret_cast<const f32x4 *>(wp + kh * W + x);
                    xr[x] = v.x;
                    xr[x + 1] = v.y;
                    xr[x + 2] = v.z;
                    xr[x + 3] = v.w;
                } else {
                    const float2 v = *reinterpret_cast<const float2 *>(wp + kh * W + x);
                    xr[x] = v.x;
                    xr[x + 1] = v.y;
                }
            }
            // window column j is xr[j + VR - 1]; column 0 lies left of the plane for the first segment, the last one
            // right of it for the last segment of a stride-1 row
#pragma unroll
            for (int j = 0; j < Q::WIN; ++j) {
                bool ok = rvalid;
                if (j == 0) ok = ok && qs != 0;
                if (S == 1 && j == Q::WIN - 1) ok = ok && qs != NQ - 1;
                xr[j + Q::VR - 1] = ok ? xr[j + Q::VR - 1] : 0.f;
            }
#pragma unroll
            for (int kw = 0; kw < 3; ++kw)
#pragma unroll
                for (int x = 0; x < Q::CW; ++x) acc[x] = fmaf(xr[x * S + kw + Q::VR - 1], w[kh * 3 + kw], acc[x]);
        }
    }
    asm volatile("" ::: "memory");
    // ---- results to their flat position in the region (every lane has read its window) ----
    if (active) {
        float *op = data + r * Q::Wout + qs * Q::CW;
#pragma unroll
        for (int e = 0; e < Q::CW; e += Q::VO) {
            if constexpr (Q::VO == 4) *reinterpret_cast<f32x4 *>(op + e) = f32x4{acc[e], acc[e + 1], acc[e + 2], acc[e + 3]};
            else if constexpr (Q::VO == 2) *reinterpret_cast<float2 *>(op + e) = float2{acc[e], acc[e + 1]};
            else op[e] = acc[e];
        }
    }
    asm volatile("" ::: "memory");
    const __amdgpu_buffer_rsrc_t ry = make_rsrc(p.y, t.y_bytes);
    const __amdgpu_buffer_rsrc_t rr = make_rsrc(p.res ? p.res : p.y, t.y_bytes);
    const unsigned obase = (plane * (unsigned)(Q::Hout * Q::Wout) + band * (unsigned)Q::OUT) * 4u;
#pragma unroll
    for (int j = 0; j < Q::NSO; ++j) {
        const int q = lane + 64 * j;
        if (q * 4 < Q::OUT) {
            f32x4 v = *reinterpret_cast<const f32x4 *>(data + q * 4);
            if (p.res) v += __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rr, obase + q * 16, 0, 0));
            if (p.relu) v = f32x4{fmaxf(v.x, 0.f), fmaxf(v.y, 0.f), fmaxf(v.z, 0.f), fmaxf(v.w, 0.f)};
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), ry, obase + q * 16, 0, 0);
        }
    }
}

template <int I> struct DwBandInst;
#define GSPC_DW_BAND_INST(I, S_, E_, BR_, NQ_) \
    template <> struct DwBandInst<I> { using Q = DwBandGeom<S_, E_, E_, BR_, NQ_>; static constexpr int S = S_, E = E_, BR = BR_, NQ = NQ_; }
// One instance, the only shape where the form measured faster than the strip kernel at N = 256: 112x112 stride 1
// (168 -> 144 and 316 -> 291 us for 32 and 64 channels).  Within 2 % either way: 112x112 stride 2 in bands of 14 rows;
// slower: 56x56 in bands of 14 rows (stride 1: 173 against 150 us for whole planes; stride 2: 107 against 100 us for
// the strip kernel), lanes of 14 instead of 28 outputs on 112x112 (169 us).
GSPC_DW_BAND_INST(0, 1, 112, 16, 4);
constexpr int kDwBandInsts = 1;

template <int I = 0>
bool plan_dw_band(const ConvParams &p, DwPlan *out) {
    if constexpr (I < kDwBandInsts) {
        using T = DwBandInst<I>;
        using Q = typename T::Q;
        const bool shape = p.stride == T::S && p.H == T::E && p.W == T::E;
        const double planes = (double)p.N * p.Cin, chunks = planes * Q::NBD;
        const double xb = planes * (T::E * T::E) * 4, yb = planes * (Q::Hout * Q::Wout) * 4, wb = (double)p.groups * 9 * p.KPGd * 4;
        const double slack = 4.0 * Q::IN * 4 + 65536;
        if (!shape || chunks < 4.0 * 2 * kNumCU || chunks >= 4.0e9 || xb + slack >= (double)kOob || yb + slack >= (double)kOob ||
            wb >= (double)kOob || planes * p.Cin >= 4.29e9)
            return plan_dw_band<I + 1>(p, out);
        TileW t{};
        t.planes = (unsigned)planes;
        t.chunks = (unsigned)chunks;
        t.m_C = magic_in_order(p.Cin);
        t.x_bytes = (unsigned)xb;
        t.y_bytes = (unsigned)yb;
        t.w_bytes = (unsigned)wb;
        std::memcpy(out->data, &t, sizeof(t));
        out->data[kDwKind] = 2;
        out->data[kDwInst] = I;
        return true;
    } else {
        return false;
    }
}

template <int I = 0>
hipError_t launch_dw_band(int inst, const ConvParams &p, const TileW &t, hipStream_t s, const char **name) {
    if constexpr (I < kDwBandInsts) {
        if (inst != I) return launch_dw_band<I + 1>(inst, p, t, s, name);
        using T = DwBandInst<I>;
        using Q = typename T::Q;
        *name = intern_name("conv_dw_band<" + std::to_string(T::S) + "," + std::to_string(T::E) + "," + std::to_string(T::E) +
                            "," + std::to_string(T::BR) + "," + std::to_string(T::NQ) + ">");
        const size_t lds = (size_t)4 * Q::REGION * sizeof(float);
        hipLaunchKernelGGL((conv_dw_band<T::S, T::E, T::E, T::BR, T::NQ>), dim3((t.chunks + 3) / 4), dim3(256), lds, s, p, t);
        return hipGetLastError();
    } else {
        return hipErrorNotSupported;
    }
}

// ---- bands of rows or groups of planes per wavefront, any plane ----------------------------------------
// Planes that the forms above do not take: a wavefront owns one band of BR output rows of one plane or, of small
// planes, G whole ones (MULTI).  Either way its input is one contiguous range of memory, which goes flat, from the 16-byte
// boundary at or below its start, straight into a wave-private LDS region (16 bytes per lane, no registers in between).  Rows
// above and below the plane are overwritten with zeros there, or, between planes, selected to zero.  A lane takes one
// column of R consecutive output rows at a time - the (plane, strip, column) items are numbered flat, so odd widths fill
// the lanes - and reads the three columns of its (R-1)*S + 3 input rows, 4.5 words per output at stride 1.  Neighbouring
// lanes store neighbouring elements.
//
// conv_direct_narrow is the same with R = 1: one output per item and nine words read for it, but every store of a wavefront is
// one contiguous piece, where strips of four rows write segments of a row each time, and four stores fill a line.  Beyond
// the last-level cache such partial lines cost memory bandwidth.  It has the larger launches of short rows.
struct TileRows {
    unsigned chunks, planes;      // wavefronts with work, planes
    int NBD, BR, G;               // bands per plane, output rows per band; planes per wavefront
    int front, region, witem;     // floats before the rows, floats per wavefront, (strip, column) items of a plane
    int R;                        // output rows per item
    unsigned m_NBD, m_Wout, m_C, m_item;
    unsigned x_bytes, y_bytes;
};

constexpr int kRowsStrip = 4;     // R of conv_direct_rows
constexpr int kRowsSlots = 8;     // 16-byte loads per lane, at most: 2048 floats per wavefront
constexpr int kRowsLds = 150 * 1024;   // (rows of several hundred elements; square planes stay below 48 KB per block)

template <int S, bool MULTI, int R>
__device__ __forceinline__ void rows_body(const ConvParams &p, const TileRows &t) {
    constexpr int NR = (R - 1) * S + 3;
    extern __shared__ f32x4 smem4[];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned chunk = blockIdx.x * 4 + wv;
    if (chunk >= t.chunks) return;   // wave-uniform; the kernel has no barriers
    float *reg = reinterpret_cast<float *>(smem4) + wv * t.region;
    const unsigned plane = MULTI ? chunk * t.G : fast_div(chunk, t.m_NBD), band = MULTI ? 0 : chunk - plane * t.NBD;
    const unsigned np = MULTI ? min((unsigned)t.G, t.planes - plane) : 1;
    const int W = p.W, H = p.H;
    const int oh0 = (int)band * t.BR, nr = min(t.BR, p.Hout - oh0);   // the band's output rows
    const int ih0 = oh0 * S - 1, ih1 = ih0 + (nr - 1) * S + 3;        // its input rows [ih0, ih1)
    const unsigned pbase = plane * (unsigned)(H * W);
    const unsigned first = pbase + (unsigned)(max(ih0, 0) * W);       // floats
    const unsigned last = MULTI ? pbase + np * (unsigned)(H * W) : pbase + (unsigned)(min(ih1, H) * W);
    const unsigned a0 = first & ~3u, len = last - a0;
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(p.x, t.x_bytes);
    for (unsigned j = 0; j < len; j += 256) {
        const unsigned e = j + lane * 4;
        load_to_lds16(rx, smem4, (wv * t.region + t.front + j) * 4, e < len ? (a0 + e) * 4 : kOob, 0);
    }
    float w[9];
    float *wl = reg + t.region - t.G * 9;                             // (MULTI) the planes' weights
    if constexpr (MULTI) {
        for (unsigned i = lane; i < np * 9; i += 64) {
            const unsigned pl = fast_div(i, 0x1c71c71cu), pg = plane + pl;   // i / 9, exact for i < 2^16
            wl[i] = p.wd[((pg - fast_div(pg, t.m_C) * p.Cin) * 9 + (i - pl * 9)) * p.KPGd];
        }
    } else {
        const unsigned c = plane - fast_div(plane, t.m_C) * p.Cin;
#pragma unroll
        for (int k = 0; k < 9; ++k) w[k] = p.wd[(c * 9 + k) * p.KPGd];
    }
    if (MULTI)               // a row of zeros before the data, which the rows between planes are read from
        for (int i = lane; i < t.front; i += 64) reg[i] = 0.f;
    wait_vmem0();
    asm volatile("" ::: "memory");
    // input row ih, column w: top[(ih - ih0) * W + w]
    float *top = reg + t.front + (first - a0) - (ih0 < 0 ? W : 0);
    if (!MULTI && ih0 < 0)
        for (int i = lane; i < W; i += 64) top[i] = 0.f;
    if (!MULTI && ih1 > H)   // (one row, at stride 2 too)
        for (int i = lane; i < W; i += 64) top[(H - ih0) * W + i] = 0.f;
    asm volatile("" ::: "memory");

    const __amdgpu_buffer_rsrc_t ry = make_rsrc(p.y, t.y_bytes);
    const __amdgpu_buffer_rsrc_t rr = make_rsrc(p.res ? p.res : p.y, t.y_bytes);
    const unsigned ybase = plane * (unsigned)(p.Hout * p.Wout) + (unsigned)(oh0 * p.Wout);   // floats
    const unsigned Wout = p.Wout, items = MULTI ? np * t.witem : (unsigned)((nr + R - 1) / R) * Wout;
    const unsigned qstrip = (unsigned)(R * S) * W, ostrip = (R - 1) * Wout;
    for (unsigned it = lane; it < items; it += 64) {
        const unsigned pl = MULTI ? fast_div(it, t.m_item) : 0, i0 = MULTI ? it - __umul24(pl, t.witem) : it;
        const unsigned strip = fast_div(i0, t.m_Wout), ow = i0 - __umul24(strip, Wout);
        const float *q = top + __umul24(strip, qstrip) + ow * S;
        if (MULTI) q += __umul24(pl, (unsigned)(H * W));
        float v[NR][3];      // (all reads before any selection: they are in bounds whatever the lane's column)
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const float *row = q + i * W;
            if (MULTI && i != 1 && (unsigned)((int)(strip * (R * S)) - 1 + i) >= (unsigned)H) row = reg + 1;
#pragma unroll
            for (int k = 0; k < 3; ++k) v[i][k] = row[k - 1];
        }
        if constexpr (MULTI) {
#pragma unroll
            for (int k = 0; k < 9; ++k) w[k] = wl[pl * 9 + k];
        }
        const bool lok = ow > 0, rok = (int)(ow * S) + 1 < W;
        float acc[R];
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] = 0.f;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const float v0 = lok ? v[i][0] : 0.f, v2 = rok ? v[i][2] : 0.f;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int kh = i - r * S;
                if (kh < 0 || kh > 2) continue;
                acc[r] = fmaf(v0, w[kh * 3], acc[r]);
                acc[r] = fmaf(v[i][1], w[kh * 3 + 1], acc[r]);
                acc[r] = fmaf(v2, w[kh * 3 + 2], acc[r]);
            }
        }
        const unsigned o = (ybase + (MULTI ? __umul24(pl, (unsigned)(p.Hout * p.Wout)) : 0) + i0 + __umul24(strip, ostrip)) * 4u;
        const int left = nr - (int)strip * R;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const unsigned off = r < left ? o + (unsigned)r * Wout * 4u : kOob;
            if (p.res) acc[r] += __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rr, off, 0, 0));
            if (p.relu) acc[r] = fmaxf(acc[r], 0.f);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[r]), ry, off, 0, 0);
        }
    }
}

template <int S, bool MULTI>
__global__ __launch_bounds__(256) void conv_direct_rows(ConvParams p, TileRows t) {
    rows_body<S, MULTI, kRowsStrip>(p, t);
}

template <int S, bool MULTI>
__global__ __launch_bounds__(256) void conv_direct_narrow(ConvParams p, TileRows t) {
    rows_body<S, MULTI, 1>(p, t);
}

// GSPC_NO_DWPLANES (tuning aid): depthwise layers on the strip, flat and generic kernels only
static bool planes_off() {
    static const bool off = std::getenv("GSPC_NO_DWPLANES") != nullptr;
    return off;
}

static_assert(sizeof(TileRows) <= sizeof(int) * kDwInst, "plan storage too small");

// The band height, or the planes per wavefront, with the shortest estimated launch: a wavefront's instructions (120, 10 per
// load slot, 100 per round of items, 200 where planes are mixed), times the rounds of wavefronts over the chip's 1024
// SIMDs, of which each after the first adds half (fitted to sweeps over plane sizes at 3 .. 1000 images of 96 channels).
// us, a block of planes in LDS tiles or a thread per output (what these layers ran on before) / this: 95x95 with 1040 planes
// 52 / 17, 86x86 with 4480 179 / 45, 27x79 at stride 2 with 18400 82 / 29, 43x43 with 3264 16.3 / 13.0 (stride 2 9.5 / 7.9),
// 23x23 with 11424 15.0 / 11.9 (9.4 / 6.5), 15x15 with 26688 15.2 / 12.8 (10.2 / 6.2), 9x9 with 74112 16.9 / 15.7 (11.0 / 9.2).
bool plan_dw_rows(const ConvParams &p, DwPlan *out) {
    if (planes_off() || p.CPG != 1 || p.KPG != 1 || p.in_bf16 || p.KH != 3 || p.KW != 3 || p.pad != 1 || (p.stride != 1 && p.stride != 2))
        return false;
    const int R = kRowsStrip, S = p.stride, HW = p.H * p.W, limit = kRowsSlots * 256;
    const double planes = (double)p.N * p.Cin, xb = planes * HW * 4, yb = planes * p.Hout * p.Wout * 4;
    if (xb + 65536 >= (double)kOob || yb + 65536 >= (double)kOob || planes * p.Cin >= 4.29e9 || p.W > 1024) return false;
    TileRows t{};
    double best = 0.0, best_wave = 0.0;
    const auto consider = [&](int g, int br) {
        const int rows = br < p.Hout ? br : p.Hout, nrb = (rows - 1) * S + 3;
        const int len = g * (nrb < p.H ? nrb : p.H) * p.W + 3;      // floats loaded, with the alignment's
        const int nbd = (p.Hout + br - 1) / br, strips = (rows + R - 1) / R, items = g * strips * p.Wout;
        const double chunks = g > 1 ? std::ceil(planes / g) : planes * nbd;
        // the last strip's window may reach past the band's rows, for outputs that are not stored
        // (and the loads fill whole pieces of 64 lanes x 4 floats)
        const int window = 3 + (g - 1) * HW + ((strips * R - 1) * S + 3) * p.W + 4, pieces = round_up(len, 256);
        const int front = round_up(p.W, 4) + 4;
        const int region = front + round_up(window > pieces ? window : pieces, 4) + (g > 1 ? round_up(g * 9, 4) : 0);
        if (len > limit || chunks * nbd >= 4.29e9 || region * 16 > kRowsLds) return;
        const double wave = 120.0 + 10.0 * ((len + 255) / 256) + (g > 1 ? 200.0 : 100.0) * ((items + 63) / 64);
        const double est = wave * (0.5 + 0.5 * std::ceil(chunks / (4 * kNumCU)));
        if (best != 0.0 && est >= best) return;
        best = est;
        best_wave = wave;
        t.chunks = (unsigned)chunks;
        t.NBD = nbd;
        t.BR = br;
        t.G = g;
        t.witem = strips * p.Wout;
        t.front = front;
        t.region = region;
    };
    // one plane or less: the largest bands that fit, and up to three more per plane
    const int fit = ((limit - 3) / p.W - 3) / S + 1, brmax = HW + 3 <= limit ? p.Hout : fit / R * R;
    if (brmax < 1) return false;
    const int n0 = (p.Hout + brmax - 1) / brmax;
    for (int n = n0, br = 0; n < n0 + 4; ++n) {
        const int b = round_up((p.Hout + n - 1) / n, R);
        if (b == br) break;
        br = b;
        consider(1, br);
    }
    // several planes, where that leaves no compute unit idle.  Short rows from 60 MB of input and output on (40 MB at stride 2): fewer
    // than 16 outputs, at stride 1 fewer than 24 on planes of up to 256 elements and than 18 on larger ones: the launch waits for memory, a compute unit holds 16 wavefronts of 8 KB regions and 32 of smaller ones, and the
    // estimate's single small planes load too little each.  With buffers that take turns over 2 GB, us, 8 KB or as estimated / the
    // most planes of 3 KB (planes of up to 256 elements) or 4 KB: 8x8 at 95 MB 31.0 / 27.0, 9x9 at stride 2 at 94 MB 29.3 / 24.3; over 520
    // random layers 0.86 .. 1.00 of the time by size, width and stride, below these bounds 1.04.
    const int longest = S == 2 ? 16 : HW <= 256 ? 24 : 18;
    const bool narrow = p.Wout < longest && xb + yb >= (S == 1 ? 60e6 : 40e6);
    const int group = !narrow ? limit : HW <= 256 ? 768 : 1024;
    if (planes > 4 * kNumCU) {
        if (narrow && HW <= 256) best = 0.0;
        for (int g = std::min(32, (group - 3) / HW); g > 1; g = narrow ? 1 : g > 8 ? g / 2 : g - 1) consider(g, round_up(p.Hout, R));
    }
    if (best == 0.0) return false;
    // Few planes of more than about 40x40: a wavefront works through its band for longer than a launch with a thread per output
    // takes (both in microseconds, fitted to 122 launches of up to 3 million outputs: of 24 that were slower here, by up to
    // 1.62 times, one is left, by 5 %; none that was faster returns): 98x98 with 20 planes 3.4 / 5.6, 66x66 with 10 2.7 / 4.1, 89x89 with
    // 15 3.0 / 4.7; 52x52 with 87 2.8 / 2.8, 60x60 at stride 2 with 208 4.0 / 3.0.
    const double outputs = planes * p.Hout * p.Wout;
    if ((p.H + 2) * (p.W + 2) > 2048 && outputs < 3e6) {
        const double sets = std::ceil(t.chunks / (4.0 * kNumCU));
        const double rows = 1.53 + best_wave * (0.00439 + 0.0013 * (sets - 1.0)) + 0.332e-6 * planes * HW;
        if (rows > 0.95 * (2.51 + 7.76e-6 * outputs)) return false;
    }
    // The same layers with one output row per item, bands from 60 MB and groups of planes from 100 MB on, where buffers have left the
    // last-level cache when a program comes back to them.  Buffers that take turns over 2 GB, us, four rows / one (and a block
    // that copied whole planes and stored them contiguously): 86x9 at 176 MB 48.7 / 37.1 (41.7), 65x6 at 228 MB 60.2 / 45.8 (53.9), 8x8 at
    // 130 MB 36.2 / 31.9 (34.0), 13x13 at 331 MB 81.6 / 71.1 (74.7), 15x15 at stride 2 at 129 MB 26.3 / 26.0 (30.4).  On one buffer that
    // stays in the cache bands are level and groups of 100 .. 240 MB 0.97 (12x12 at 133 MB 23.9 / 28.8).  Rows of
    // 16 and 17 outputs at stride 1 on planes of more than 256 elements: 17x17 at 214 MB 53.4 / 48.4 (48.9), 28x17 at 214 MB 46.4 /
    // 40.3 (45.9), 22x16 level; from 18 on four rows are ahead of that block, 0.95 with buffers that take turns and 1.05 on one.
    t.R = kRowsStrip;
    if (narrow && (p.Wout < 16 || HW > 256) && xb + yb >= (t.G == 1 ? 60e6 : 100e6)) {
        t.R = 1;       // (bands, planes and LDS as above: the windows reach less far)
        t.witem = p.Hout * p.Wout;
    }
    t.planes = (unsigned)planes;
    t.m_NBD = div_magic(t.NBD);
    t.m_Wout = div_magic(p.Wout);
    t.m_C = div_magic(p.Cin);
    t.m_item = div_magic(t.witem);
    t.x_bytes = (unsigned)xb;
    t.y_bytes = (unsigned)yb;
    std::memcpy(out->data, &t, sizeof(t));
    out->data[kDwKind] = 3;
    return true;
}

template <int S, bool MULTI>
hipError_t launch_dw_rows(const ConvParams &p, const TileRows &t, hipStream_t s) {
    const size_t lds = (size_t)4 * t.region * sizeof(float);
    if (t.R == 1) {   // (rows of at most 31 elements: a region is far below 64 KB / 4)
        hipLaunchKernelGGL((conv_direct_narrow<S, MULTI>), dim3((t.chunks + 3) / 4), dim3(256), lds, s, p, t);
        return hipGetLastError();
    }
    auto kern = conv_direct_rows<S, MULTI>;
    if (lds > 64 * 1024) {
        static thread_local bool raised = false;   // per instantiation and thread
        if (!raised) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kRowsLds);
            if (e != hipSuccess) return e;
            raised = true;
        }
    }
    hipLaunchKernelGGL(kern, dim3((t.chunks + 3) / 4), dim3(256), lds, s, p, t);
    return hipGetLastError();
}

bool plan_dw_planes(const ConvParams &p, DwPlan *out) {
    if (planes_off() || p.CPG != 1 || p.KPG != 1 || p.in_bf16 || p.KH != 3 || p.KW != 3 || p.pad != 1 ||
        (p.stride != 1 && p.stride != 2))
        return false;
    if (plan_dw_wave(p, out)) return true;
    {
        static const bool off = std::getenv("GSPC_NO_DWBAND") != nullptr;   // tuning aid
        if (!off && plan_dw_band(p, out)) return true;
    }
    return false;
}

hipError_t launch_dw_planes(const ConvParams &p, const DwPlan &plan, hipStream_t s, const char **name) {
    if (plan.data[kDwKind] == 3) {
        TileRows tr;
        std::memcpy(&tr, plan.data, sizeof(tr));
        static const char *const names[2][2][2] = {{{"conv_direct_rows<1,false>", "conv_direct_rows<1,true>"},
                                                    {"conv_direct_rows<2,false>", "conv_direct_rows<2,true>"}},
                                                   {{"conv_direct_narrow<1,false>", "conv_direct_narrow<1,true>"},
                                                    {"conv_direct_narrow<2,false>", "conv_direct_narrow<2,true>"}}};
        *name = names[tr.R == 1][p.stride - 1][tr.G > 1];
        if (tr.G > 1) return p.stride == 1 ? launch_dw_rows<1, true>(p, tr, s) : launch_dw_rows<2, true>(p, tr, s);
        return p.stride == 1 ? launch_dw_rows<1, false>(p, tr, s) : launch_dw_rows<2, false>(p, tr, s);
    }
    if (plan.data[kDwKind] == 2) {
        TileW tw;
        std::memcpy(&tw, plan.data, sizeof(tw));
        return launch_dw_band(plan.data[kDwInst], p, tw, s, name);
    }
    if (plan.data[kDwKind] == 1) {
        TileW tw;
        std::memcpy(&tw, plan.data, sizeof(tw));
        return launch_dw_wave(plan.data[kDwInst], p, tw, s, name);
    }
    return hipErrorNotSupported;
}

}  // namespace gspc
