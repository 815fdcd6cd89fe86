// Device and host helpers shared by the convolution kernels of libgspc.
#pragma once

#include <mutex>
#include <set>
#include <string>

#include "divide.h"
#include "gspc_internal.h"

namespace gspc {

typedef float f32x4 __attribute__((ext_vector_type(4)));

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Buffer descriptors: raw (stride 0) buffers (see kOob).
constexpr int kRsrcFlags = 0x00020000;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, kRsrcFlags);
}
// 64 lanes x 16 bytes from global memory straight into LDS: lane l's bytes land at byte offset dst + 16 l of
// the dynamic LDS array (dst wave-uniform).  (A device-only function: the host pass does not know that this
// GPU takes 16 bytes per lane in this instruction, and inside a lambda it would be checked there.)
__device__ __forceinline__ void load_to_lds16(__amdgpu_buffer_rsrc_t r, f32x4 *lds_base, unsigned dst, unsigned voff,
                                              unsigned soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        r, (__attribute__((address_space(3))) void *)(reinterpret_cast<char *>(lds_base) + dst), 16, voff, soff, 0, 0);
}
// Four (vec) or one consecutive input elements as fp32.
template <typename TIN> __device__ __forceinline__ f32x4 buf_load_in(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff, int vec);
template <> __device__ __forceinline__ f32x4 buf_load_in<float>(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff, int vec) {
    if (vec) return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
    return f32x4{__uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0)), 0.f, 0.f, 0.f};
}
template <> __device__ __forceinline__ f32x4 buf_load_in<uint16_t>(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff, int vec) {
    if (vec) {
        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
        return f32x4{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u),
                     __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u)};
    }
    const unsigned h = __builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0);
    return f32x4{__uint_as_float(h << 16), 0.f, 0.f, 0.f};
}


// ---- host-side helpers --------------------------------------------------------
// Kernel names are reported as the template arguments of the instance that ran,
// so they can be matched one to one with a profiler's kernel names.  The
// returned pointer stays valid for the life of the process.
inline const char *intern_name(const std::string &s) {
    static std::mutex mu;
    static std::set<std::string> names;
    std::lock_guard<std::mutex> lock(mu);
    return names.insert(s).first->c_str();
}

constexpr int kNumCU = 256;

// Odd pointwise planes of 40 .. 63 pixels, handed over as one row: conv_mfma16 gives every image and 16 filters a block of
// one 64-pixel tile, up to three blocks per compute unit (with more it takes two images per block, a third of it padding).
inline bool fills_image_tiles(const ConvParams &p, int mtiles) {
    return p.KH == 1 && p.stride == 1 && p.pad == 0 && p.H == 1 && p.W % 4 != 0 && p.W >= 40 && p.W < 64 && p.CPG % 4 == 0 &&
           (long)((p.N + 1) / 2) * mtiles * p.groups < 3 * kNumCU / 2;
}

// Splits the output into NB images x TH rows per block for a pixel capacity PB.
inline bool split_pixels(const ConvParams &p, int PB, int *NB, int *TH) {
    if (p.Wout > PB) return false;
    const int HWo = p.Hout * p.Wout;
    if (HWo <= PB) {
        *TH = p.Hout;
        *NB = PB / HWo;
        if (*NB > p.N) *NB = p.N;
    } else {
        *NB = 1;
        const int thmax = PB / p.Wout;
        const int rbk = (p.Hout + thmax - 1) / thmax;
        *TH = (p.Hout + rbk - 1) / rbk;
    }
    return true;
}

}  // namespace gspc
