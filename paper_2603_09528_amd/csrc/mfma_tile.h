// MFMA and buffer access of the GEMM tiles (gemm_impl.h, fold_impl.h).
#pragma once
#include "device_common.h"

namespace tpt {

// ---------------------------------------------------------------------------
// FP64 / FP32 MFMA (v_mfma_f64_16x16x4f64, v_mfma_f32_16x16x4f32).
// Operand fragments: lane l holds A[m0 + l%16][k0 + l/16] and
// B[k0 + l/16][n0 + l%16]; the 16x16 result of lane l is column l%16, rows
// l/16 + 4r (f64, measured on gfx950) or 4(l/16) + r (f32), r = 0..3.
// ---------------------------------------------------------------------------
template <typename TM> struct Mfma;
template <> struct Mfma<double> {
    typedef d4 acc;
    static __device__ __forceinline__ acc zero() { return (acc){0.0, 0.0, 0.0, 0.0}; }
    static __device__ __forceinline__ acc mma(double a, double b, acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lg, int r) { return lg + 4 * r; }
};
template <> struct Mfma<float> {
    typedef f4 acc;
    static __device__ __forceinline__ acc zero() { return (acc){0.f, 0.f, 0.f, 0.f}; }
    static __device__ __forceinline__ acc mma(float a, float b, acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lg, int r) { return 4 * lg + r; }
};

typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
constexpr int BUF_RSRC_WORD3 = 0x00020000;  // raw 32-bit buffer (gfx9 family)

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* base) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, 0x7fffffff, BUF_RSRC_WORD3);
}
// buffer resource over [base, base + bytes), bytes clamped to the 31-bit range
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc_n(const void* base, long long bytes) {
    const int n = bytes <= 0 ? 0 : (bytes > 0x7ffffff0LL ? 0x7ffffff0 : (int)bytes);
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, n, BUF_RSRC_WORD3);
}
template <typename T> struct BufIO;
template <> struct BufIO<double> {
    static __device__ __forceinline__ double ld(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so) {
        return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)vo, (int)so, 0));
    }
    static __device__ __forceinline__ void st(double v, __amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so) {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_t, v), r, (int)vo, (int)so, 0);
    }
};
template <> struct BufIO<float> {
    static __device__ __forceinline__ float ld(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so) {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)vo, (int)so, 0));
    }
    static __device__ __forceinline__ void st(float v, __amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, (int)vo, (int)so, 0);
    }
};

}  // namespace tpt
