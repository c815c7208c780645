// Small device helpers shared by the gfx950 kernels: vector types, wavefront reductions, activations.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>

#include "kernels.h"

namespace mt {

// Host: raise a kernel's dynamic-LDS limit once per device (the attribute belongs to the function ON a device).
// `done` is the call site's bit set of devices already served; concurrent first calls both set the same value.
inline hipError_t ensure_dynamic_lds(const void* fn, int bytes, std::atomic<uint64_t>& done)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = 1ull << (dev & 63);
    if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess) return e;
    done.fetch_or(bit, std::memory_order_release);
    return hipSuccess;
}

typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

// The values of a lane and of the lane whose number differs in the bit M, as two registers of every lane: one or two vector instructions, where a
// shuffle is an LDS round trip of about 0.1 us in a chain that little else covers.  M = 4: only of values that agree in lanes 8 apart.
template <int M>
__device__ __forceinline__ void lane_pair(uint32_t v, uint32_t& a, uint32_t& b)
{
    static_assert(M == 1 || M == 2 || M == 4 || M == 8 || M == 16 || M == 32, "");
    if constexpr (M == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        a = r[0];
        b = r[1];
    } else if constexpr (M == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        a = r[0];
        b = r[1];
    } else {
        constexpr int ctrl = M == 1 ? 0xB1 : M == 2 ? 0x4E : M == 4 ? 0x124 : 0x128;     // quad_perm [1,0,3,2], [2,3,0,1]; row_ror:4, :8
        a = v;
        b = __builtin_amdgcn_update_dpp((int)v, (int)v, ctrl, 0xF, 0xF, false);
    }
}
template <int M>
__device__ __forceinline__ float lane_pair_sum(float v)
{
    uint32_t a, b;
    lane_pair<M>(__builtin_bit_cast(uint32_t, v), a, b);
    return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}
template <int M>
__device__ __forceinline__ float lane_pair_max(float v)
{
    uint32_t a, b;
    lane_pair<M>(__builtin_bit_cast(uint32_t, v), a, b);
    return fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
}
template <int M>
__device__ __forceinline__ int lane_pair_sum(int v)
{
    uint32_t a, b;
    lane_pair<M>((uint32_t)v, a, b);
    return (int)(a + b);
}

// Sum / max over the 64 lanes of a wavefront; every lane receives the result.
template <typename T>
__device__ __forceinline__ T wave_sum_any(T v)
{
    v = lane_pair_sum<32>(v);
    v = lane_pair_sum<16>(v);
    v = lane_pair_sum<8>(v);
    v = lane_pair_sum<4>(v);
    v = lane_pair_sum<2>(v);
    return lane_pair_sum<1>(v);
}
__device__ __forceinline__ float wave_sum(float v) { return wave_sum_any(v); }
__device__ __forceinline__ int wave_sum_int(int v) { return wave_sum_any(v); }
__device__ __forceinline__ float wave_max(float v)
{
    v = lane_pair_max<32>(v);
    v = lane_pair_max<16>(v);
    v = lane_pair_max<8>(v);
    v = lane_pair_max<4>(v);
    v = lane_pair_max<2>(v);
    return lane_pair_max<1>(v);
}

// Block w of what is to be read ahead.
__device__ __forceinline__ void read_ahead(const ReadAhead& r, uint32_t w)
{
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t n = (r.bytes[i] + kAheadBlock - 1) / kAheadBlock;
        if (w < n) {
            const unsigned char* p = static_cast<const unsigned char*>(r.base) + (size_t)r.at[i] * 256 + (size_t)w * kAheadBlock;
            const uint32_t end = min(r.bytes[i] - w * kAheadBlock, kAheadBlock), step = blockDim.x * 16;
            for (uint32_t o = threadIdx.x * 16; o < end; o += 8 * step) {
                u32x4 v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = *reinterpret_cast<const u32x4*>(p + min(o + k * step, end - 16));
#pragma unroll
                for (int k = 0; k < 8; ++k) asm volatile("" ::"v"(v[k]));
            }
            return;
        }
        w -= n;
    }
}

// LayerNorm's arithmetic on a lane's four values, contractions written out: the row-major and the panel kernels give the same bits (E4M3 roundings
// behind them amplify a last bit to 5 % of the logits), whatever the compiler would fuse in either.
__device__ __forceinline__ float ln_squares(const float4& v, float mean)
{
#pragma clang fp contract(off)
    const float a = v.x - mean, b = v.y - mean, c = v.z - mean, d = v.w - mean;
    return fmaf(a, a, b * b) + fmaf(c, c, d * d);
}
__device__ __forceinline__ float4 ln_normalise(const float4& v, float mean, float inv, const float4& g, const float4& b)
{
#pragma clang fp contract(off)
    return make_float4(fmaf(g.x, (v.x - mean) * inv, b.x), fmaf(g.y, (v.y - mean) * inv, b.y), fmaf(g.z, (v.z - mean) * inv, b.z),
                       fmaf(g.w, (v.w - mean) * inv, b.w));
}

// GELU(x) = x * Phi(x).  Exact form through erff; tanh form as the published approximation.
__device__ inline float gelu_erf(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
// The erf form for bf16 epilogues.  GELU(x) = x * Phi(x) and Phi(x) = 1 / (1 + exp(-z(x))) with z = ln(Phi(x) / Phi(-x)),
// an odd function of x; z is replaced by the odd polynomial x * (c0 + c1 x^2 + c2 x^4) whose coefficients minimise the
// largest absolute error of x * Phi(x) on [-9, 9] (fitted against erf in float64: 2.6e-5, reached near x = -0.56; the
// published tanh form, the same shape with two coefficients chosen differently, is off by 4.7e-4).  That is a
// twentieth of the bf16 rounding step of a typical activation (0.3 .. 1) and is what every bf16 kernel stores;
// the float32 validation mode uses erff.  6 multiply-adds, one exp2, one reciprocal per element.
__device__ __forceinline__ float gelu_erf_fast(float x)
{
    constexpr float kLog2e = 1.4426950408889634f;
    const float xc = __builtin_amdgcn_fmed3f(x, -9.0f, 9.0f);  // the fit's range; beyond it Phi is 0 or 1 to float32 anyway
    const float x2 = xc * xc;
    float p = fmaf(x2, -7.03037878e-04f * kLog2e, 7.40113199e-02f * kLog2e);
    p = fmaf(x2, p, 1.59501574e+00f * kLog2e);
    const float e = __builtin_amdgcn_exp2f(-xc * p);          // exp(-z), between 2^-39 and 2^39
    return x * __builtin_amdgcn_rcpf(1.0f + e);
}
__device__ inline float gelu_tanh(float x)
{
    const float u = 0.79788456080286536f * (x + 0.044715f * x * x * x);
    return 0.5f * x * (1.0f + tanhf(u));
}

// four float32 -> four OCP FP8 E4M3 bytes in one dword (round to nearest even, saturating at +-448)
__device__ __forceinline__ uint32_t pack_e4m3(float a, float b, float c, float d)
{
    a = __builtin_amdgcn_fmed3f(a, -448.f, 448.f);
    b = __builtin_amdgcn_fmed3f(b, -448.f, 448.f);
    c = __builtin_amdgcn_fmed3f(c, -448.f, 448.f);
    d = __builtin_amdgcn_fmed3f(d, -448.f, 448.f);
    int v = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false);
    v = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, v, true);
    return (uint32_t)v;
}

__device__ inline float apply_act(float v, int act)
{
    switch (act) {
        case 1: return gelu_erf(v);
        case 2: return gelu_tanh(v);
        case 3: return tanhf(v);
        default: return v;
    }
}

}  // namespace mt
