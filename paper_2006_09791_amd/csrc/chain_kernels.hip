// Non-convolution steps of the residual stacks of Section IV-A of
// arXiv 2006.09791: ReLU, element-wise add, max pooling.  All fp32.
#include "divide.h"
#include "gspc_internal.h"

namespace gspc {

__global__ void relu_kernel(const float *__restrict__ x, float *__restrict__ y, size_t count) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t step = (size_t)gridDim.x * blockDim.x;
    for (; i < count; i += step) y[i] = fmaxf(x[i], 0.f);
}

__global__ void add_kernel(const float *__restrict__ a, const float *__restrict__ b,
                           float *__restrict__ y, size_t count, int relu) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t step = (size_t)gridDim.x * blockDim.x;
    for (; i < count; i += step) {
        float v = a[i] + b[i];
        y[i] = relu ? fmaxf(v, 0.f) : v;
    }
}

// One thread per output; K = 0: any window size.  Taps outside the plane are moved to its nearest row or column, which a
// window whose padding is at most half of it contains, so that every load is requested before the first maximum is taken.
// (With 64-bit divisions, a branch per tap and a wait per load the 3x3 stride-2 window on 112x112, 64 channels, took 3.85 us
// at N = 1, 15.5 at 8 and 96 at 64; now 3.06, 10.0 and 59.  A launch with nothing to do takes 1.8.)
template <int K>
__global__ void maxpool_kernel(const float *__restrict__ x, float *__restrict__ y, int H, int W, int Kany, int stride, int pad,
                               int Hout, int Wout, unsigned total, unsigned m_Wout, unsigned m_Hout) {
    const unsigned i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    const int k = K ? K : Kany;
    const unsigned r = fast_div_any(i, Wout, m_Wout), plane = fast_div_any(r, Hout, m_Hout);   // n * C + c
    const int iw0 = (int)(i - r * Wout) * stride - pad, ih0 = (int)(r - plane * Hout) * stride - pad;
    const float *xp = x + (size_t)plane * H * W;
    float m = -INFINITY;
    if constexpr (K > 0) {
        float v[K][K];
#pragma unroll
        for (int kh = 0; kh < K; ++kh)
#pragma unroll
            for (int kw = 0; kw < K; ++kw)
                v[kh][kw] = xp[(unsigned)(min(max(ih0 + kh, 0), H - 1) * W + min(max(iw0 + kw, 0), W - 1))];
#pragma unroll
        for (int kh = 0; kh < K; ++kh)
#pragma unroll
            for (int kw = 0; kw < K; ++kw) m = fmaxf(m, v[kh][kw]);
    } else {
        for (int kh = 0; kh < k; ++kh)
            for (int kw = 0; kw < k; ++kw)
                m = fmaxf(m, xp[(unsigned)(min(max(ih0 + kh, 0), H - 1) * W + min(max(iw0 + kw, 0), W - 1))]);
    }
    y[i] = m;
}

static unsigned grid_for(size_t count) {
    size_t b = (count + 255) / 256;
    if (b > 262144) b = 262144;
    if (b == 0) b = 1;
    return (unsigned)b;
}

hipError_t launch_relu(const float *x, float *y, size_t count, hipStream_t s) {
    hipLaunchKernelGGL(relu_kernel, dim3(grid_for(count)), dim3(256), 0, s, x, y, count);
    return hipGetLastError();
}

hipError_t launch_add(const float *a, const float *b, float *y, size_t count, int relu,
                      hipStream_t s) {
    hipLaunchKernelGGL(add_kernel, dim3(grid_for(count)), dim3(256), 0, s, a, b, y, count, relu);
    return hipGetLastError();
}

hipError_t launch_maxpool(const float *x, float *y, int N, int C, int H, int W, int K, int stride,
                          int pad, int Hout, int Wout, hipStream_t s) {
    const auto kern = K == 2 ? maxpool_kernel<2> : K == 3 ? maxpool_kernel<3> : maxpool_kernel<0>;
    const size_t plane = (size_t)Hout * Wout, planes = (size_t)N * C;
    const size_t step = plane < 0x80000000u ? 0x80000000u / plane : 1;   // planes per launch: outputs are numbered in 32 bits
    for (size_t at = 0; at < planes; at += step) {
        const unsigned total = (unsigned)((planes - at < step ? planes - at : step) * plane);
        hipLaunchKernelGGL(kern, dim3((total + 255) / 256), dim3(256), 0, s, x + at * H * W, y + at * plane, H, W, K, stride, pad,
                           Hout, Wout, total, div_magic(Wout), div_magic(Hout));
    }
    return hipGetLastError();
}

}  // namespace gspc
