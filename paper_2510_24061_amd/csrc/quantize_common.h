// Device helpers of the quantizer, shared by its own launches (quantize.hip) and the products that quantize their
// input themselves (gemm_thin.hip).
#pragma once
#include "falqon_internal.h"
#include "gemm_common.h"

namespace falqon {
namespace {

// the maximum over the workgroup's N waves, in all threads.  The barrier is behind LDS accesses only: loads in flight
// stay in flight.
template <int N>
__device__ __forceinline__ float block_max(float v, float* smem /* [N] */)
{
    v = wave_max(v);
    if ((threadIdx.x & 63) == 0) smem[threadIdx.x >> 6] = v;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    barrier_lds_only();
    float r = smem[0];
    for (int w = 1; w < N; ++w) r = fmaxf(r, smem[w]);
    return r;
}

// 16 bytes of a tensor per lane: E elements, whose codes are E bytes.  A wave reads and writes without gaps (32 or 64
// bytes per lane, in two or four instructions over the same lines, took 9 to 15 % more at 33 MB).
typedef unsigned v4u __attribute__((ext_vector_type(4)));
template <typename T> struct Piece;
template <> struct Piece<uint16_t> { static constexpr int E = 8; typedef unsigned codes_t __attribute__((ext_vector_type(2))); };
template <> struct Piece<float> { static constexpr int E = 4; typedef unsigned codes_t; };

__device__ __forceinline__ void widen(v4u w, float (&f)[8])          // bf16 -> fp32 is exact
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = __uint_as_float(w[i] << 16);
        f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
}
__device__ __forceinline__ void widen(v4u w, float (&f)[4])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = __uint_as_float(w[i]);
}

template <typename T>
__device__ __forceinline__ float abs_max(v4u w, float m)
{
    float f[Piece<T>::E];
    widen(w, f);
#pragma unroll
    for (int i = 0; i < Piece<T>::E; ++i) m = fmaxf(m, fabsf(f[i]));
    return m;
}

// Saturating round-to-nearest-even cast of four fp32 values to one dword of FP8 codes.
// The hardware conversion rounds to nearest even but turns out-of-range inputs into
// NaN (E4M3) or Inf (E5M2), so the value is clamped to the largest finite one first.
template <int FMT>
__device__ __forceinline__ uint32_t cast4(float a, float b, float c, float d)
{
    constexpr float mx = FMT == FALQON_E4M3 ? 448.0f : 57344.0f;
    a = __builtin_amdgcn_fmed3f(a, -mx, mx);
    b = __builtin_amdgcn_fmed3f(b, -mx, mx);
    c = __builtin_amdgcn_fmed3f(c, -mx, mx);
    d = __builtin_amdgcn_fmed3f(d, -mx, mx);
    int w = 0;
    if (FMT == FALQON_E4M3) {
        w = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, w, false);
        w = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, w, true);
    } else {
        w = __builtin_amdgcn_cvt_pk_bf8_f32(a, b, w, false);
        w = __builtin_amdgcn_cvt_pk_bf8_f32(c, d, w, true);
    }
    return static_cast<uint32_t>(w);
}

template <typename T, int FMT>
__device__ __forceinline__ typename Piece<T>::codes_t cast_piece(v4u w, float s)
{
    float f[Piece<T>::E];
    widen(w, f);
#pragma unroll
    for (int i = 0; i < Piece<T>::E; ++i) f[i] = __fmul_rn(f[i], s);
    typename Piece<T>::codes_t o;
    if constexpr (Piece<T>::E == 8) {
        o[0] = cast4<FMT>(f[0], f[1], f[2], f[3]);
        o[1] = cast4<FMT>(f[4], f[5], f[6], f[7]);
    } else {
        o = cast4<FMT>(f[0], f[1], f[2], f[3]);
    }
    return o;
}

}  // namespace
}  // namespace falqon
