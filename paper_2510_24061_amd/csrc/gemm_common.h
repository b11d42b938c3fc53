// Device helpers shared by the two families of FP8 product kernels (gemm.hip: tiles of 128 to 256 tokens on rings two and
// three stages deep; gemm_mid.hip: tiles of 32 to 128 tokens on deep rings).
#pragma once
#include <type_traits>

#include "falqon_internal.h"

namespace falqon {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

#define FQ_GLOBAL_PTR(p) ((const void __attribute__((address_space(1)))*)(p))
#define FQ_LDS_PTR(p) ((void __attribute__((address_space(3)))*)(p))

__device__ __attribute__((aligned(16))) uint8_t g_zero16[16];

constexpr int BK = 128;   // bytes of K per step (two 64-deep MFMAs)

// Swizzle of a K-contiguous tile (128 B = 8 chunks of 16 B per row): the physical chunk of
// logical chunk c in row `row` is c ^ swz_kc(row).  Any 8 or 16 consecutive rows land on
// distinct 16-byte bank groups for a fixed logical chunk.
__device__ __forceinline__ int swz_kc(int row) { return ((row >> 1) ^ ((row & 1) << 2)) & 7; }

// Swizzle of a [K][N] tile with CH chunks of 16 B per K-row.
template <int CH>
__device__ __forceinline__ int swz_kn(int krow) { return CH >= 16 ? ((krow & 7) << 1) : (krow & (CH - 1)); }

// Operand of lane `lane` for a 32x32x64 instruction from half kh of a K-contiguous tile (128-byte rows, swizzle swz_kc):
// lane l holds row (l % 32), which the caller names, and the 32 K-bytes [32 (l / 32), +32) of the 64-deep half.
// Its two 16-byte chunks may come from two tiles.
__device__ __forceinline__ v8i read_kc_tiles(const uint8_t* tile_lo, const uint8_t* tile_hi, int row, int kh, int lane)
{
    const int cb = kh * 4 + (lane >> 5) * 2;
    const int sw = swz_kc(row);
    const v4i lo = *reinterpret_cast<const v4i*>(tile_lo + row * BK + ((cb ^ sw) << 4));
    const v4i hi = *reinterpret_cast<const v4i*>(tile_hi + row * BK + (((cb + 1) ^ sw) << 4));
    v8i r;
    r[0] = lo[0]; r[1] = lo[1]; r[2] = lo[2]; r[3] = lo[3];
    r[4] = hi[0]; r[5] = hi[1]; r[6] = hi[2]; r[7] = hi[3];
    return r;
}

__device__ __forceinline__ v8i read_kc_tile(const uint8_t* tile, int row, int kh, int lane)
{
    return read_kc_tiles(tile, tile, row, kh, lane);
}

__device__ __forceinline__ const uint8_t* opaque_uniform(const uint8_t* p)
{
    const uint64_t u = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(u));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(u >> 32));
    return reinterpret_cast<const uint8_t*>((static_cast<uint64_t>(hi) << 32) | lo);
}

// Workgroup barrier that orders LDS accesses only.  __syncthreads() also waits for every
// outstanding global access, which would drain the global_load_lds fetches that are meant to
// stay in flight across the barrier; their completion is awaited explicitly where needed.
__device__ __forceinline__ void barrier_lds_only()
{
    asm volatile("" ::: "memory");               // compiler-level: no LDS access moves across
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
}

// The same behind LDS writes of this wave: they have been carried out, loads from memory may still be in flight.
__device__ __forceinline__ void barrier_lds_written()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt 0 only
    barrier_lds_only();
}

// The maximum over a wave, in all lanes.  Within rows of 16 lanes by DPP, across rows by lane swaps: about 60 cycles; six
// exchanges through LDS (__shfl_xor) take 600, which a kernel of a few microseconds feels.
__device__ __forceinline__ float wave_max(float v)
{
    auto moved = [](float x, auto ctrl) {
        constexpr int C = decltype(ctrl)::value;
        const int i = static_cast<int>(__float_as_uint(x));
        return __uint_as_float(static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(i, C, 0xf, 0xf, true)));
    };
    v = fmaxf(v, moved(v, std::integral_constant<int, 0xB1>{}));      // quad_perm [1, 0, 3, 2]
    v = fmaxf(v, moved(v, std::integral_constant<int, 0x4E>{}));      // quad_perm [2, 3, 0, 1]
    v = fmaxf(v, moved(v, std::integral_constant<int, 0x141>{}));     // row_half_mirror
    v = fmaxf(v, moved(v, std::integral_constant<int, 0x140>{}));     // row_mirror
    uint32_t u = __float_as_uint(v);
    const auto rows = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    v = fmaxf(__uint_as_float(rows[0]), __uint_as_float(rows[1]));
    u = __float_as_uint(v);
    const auto halves = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(halves[0]), __uint_as_float(halves[1]));
}

// two fp32 -> two bf16 (round to nearest even) in one dword: v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    typedef float v2f __attribute__((ext_vector_type(2)));
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
    const v2f f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, v2bf));
}

// a + b of eight bf16 each, every sum rounded once (what adding two bf16 tensors gives)
__device__ __forceinline__ uint4 add_bf16x8(uint4 a, uint4 b)
{
    auto add2 = [](uint32_t x, uint32_t y) {
        return pack_bf16x2(__uint_as_float(x << 16) + __uint_as_float(y << 16),
                           __uint_as_float(x & 0xffff0000u) + __uint_as_float(y & 0xffff0000u));
    };
    return make_uint4(add2(a.x, b.x), add2(a.y, b.y), add2(a.z, b.z), add2(a.w, b.w));
}

}  // namespace
}  // namespace falqon
