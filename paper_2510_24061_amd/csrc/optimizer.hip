// Optimizer step into the proxy buffer ("DeltaBuffer <- Optimizer(dL/dB, lr)", second line of
// the loop of the backward-and-update algorithm) with the optimizer the paper's experiments name:
// AdamW under gradient-norm clipping.  B is never stored, only its change, so the decoupled
// weight decay has nothing to act on; what remains is Adam with bias correction, writing the
// change of B into the buffer.
//
// Both kernels stream a few MB once: HBM/launch bound, 16-byte accesses per lane.  The sum of
// squares is formed in fp64 with a fixed assignment of elements to threads and fixed reduction
// trees, so it is bitwise reproducible (no floating-point atomics).
#include <type_traits>

#include "falqon_internal.h"

namespace falqon {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxNormBlocks = 256;     // partial sums of squares (doubles) in the workspace

// The sum over a workgroup of four waves, in its first thread, in a fixed tree: within rows of 16 lanes by DPP, across rows by
// lane swaps, across waves through LDS.  (With a tree through LDS, a barrier per level, the two launches of a layer of 4096 x 64 took 3.1 and 1.7 us; 2.7 and 1.45 now.)
__device__ __forceinline__ double block_sum(double v)
{
    static_assert(kThreads == 256 && kMaxNormBlocks == 256, "four waves");
    __shared__ double s_wave[4];
    auto moved = [](double x, auto ctrl) {
        constexpr int C = decltype(ctrl)::value;
        return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(x), C, 0xf, 0xf, true), __builtin_amdgcn_mov_dpp(__double2loint(x), C, 0xf, 0xf, true));
    };
    v += moved(v, std::integral_constant<int, 0xB1>{});               // quad_perm [1, 0, 3, 2]
    v += moved(v, std::integral_constant<int, 0x4E>{});               // quad_perm [2, 3, 0, 1]
    v += moved(v, std::integral_constant<int, 0x141>{});              // row_half_mirror
    v += moved(v, std::integral_constant<int, 0x140>{});              // row_mirror
    auto both = [](auto lo, auto hi) {
        return __hiloint2double(static_cast<int>(hi[0]), static_cast<int>(lo[0])) + __hiloint2double(static_cast<int>(hi[1]), static_cast<int>(lo[1]));
    };
    unsigned lo = static_cast<unsigned>(__double2loint(v)), hi = static_cast<unsigned>(__double2hiint(v));
    v = both(__builtin_amdgcn_permlane16_swap(lo, lo, false, false), __builtin_amdgcn_permlane16_swap(hi, hi, false, false));
    lo = static_cast<unsigned>(__double2loint(v));
    hi = static_cast<unsigned>(__double2hiint(v));
    v = both(__builtin_amdgcn_permlane32_swap(lo, lo, false, false), __builtin_amdgcn_permlane32_swap(hi, hi, false, false));
    if ((threadIdx.x & 63) == 0) s_wave[threadIdx.x >> 6] = v;
    __syncthreads();
    return (s_wave[0] + s_wave[1]) + (s_wave[2] + s_wave[3]);
}

__global__ void __launch_bounds__(kThreads)
sqnorm_partial_kernel(const float* __restrict__ g, int64_t count, double* __restrict__ partial)
{
    double acc = 0.0;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads * 4;
    for (int64_t e = (static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x) * 4; e < count; e += stride) {
        const float4 v = *reinterpret_cast<const float4*>(g + e);
        acc += static_cast<double>(v.x) * v.x;
        acc += static_cast<double>(v.y) * v.y;
        acc += static_cast<double>(v.z) * v.z;
        acc += static_cast<double>(v.w) * v.w;
    }
    acc = block_sum(acc);
    if (threadIdx.x == 0) partial[blockIdx.x] = acc;
}

// one workgroup: partials added in a fixed tree, result added to the accumulator
__global__ void __launch_bounds__(kMaxNormBlocks)
sqnorm_final_kernel(const double* __restrict__ partial, int n_partials, double* sum_sq)
{
    const double before = *sum_sq;                                    // on its way beside the partials
    const double sum = block_sum(static_cast<int>(threadIdx.x) < n_partials ? partial[threadIdx.x] : 0.0);
    if (threadIdx.x == 0) *sum_sq = before + sum;
}

__global__ void __launch_bounds__(kThreads)
adamw_delta_kernel(const float* __restrict__ d_b, float* __restrict__ exp_avg, float* __restrict__ exp_avg_sq,
                   float* __restrict__ delta_buf, int64_t count, const AdamFactors f,
                   const double* __restrict__ sum_sq)
{
    float c = 1.0f;
    if (sum_sq) {
        const double cc = f.max_norm / (sqrt(*sum_sq) + 1e-6);
        c = cc < 1.0 ? static_cast<float>(cc) : 1.0f;
    }
    const float beta1 = f.beta1, omb1 = f.one_minus_beta1, beta2 = f.beta2, omb2 = f.one_minus_beta2;
    const float eps = f.eps, step_size = f.step_size, inv_sqrt_bias2 = f.inv_sqrt_bias2;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads * 4;
    for (int64_t e = (static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x) * 4; e < count; e += stride) {
        const float4 g4 = *reinterpret_cast<const float4*>(d_b + e);
        float4 m4 = *reinterpret_cast<const float4*>(exp_avg + e);
        float4 v4 = *reinterpret_cast<const float4*>(exp_avg_sq + e);
        float4 b4 = *reinterpret_cast<const float4*>(delta_buf + e);
        const float g[4] = {g4.x, g4.y, g4.z, g4.w};
        float m[4] = {m4.x, m4.y, m4.z, m4.w}, v[4] = {v4.x, v4.y, v4.z, v4.w}, b[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float gi = c * g[i];
            m[i] = beta1 * m[i] + omb1 * gi;
            v[i] = beta2 * v[i] + omb2 * gi * gi;
            const float denom = sqrtf(v[i]) * inv_sqrt_bias2 + eps;
            b[i] += -step_size * m[i] / denom;
        }
        *reinterpret_cast<float4*>(exp_avg + e) = make_float4(m[0], m[1], m[2], m[3]);
        *reinterpret_cast<float4*>(exp_avg_sq + e) = make_float4(v[0], v[1], v[2], v[3]);
        *reinterpret_cast<float4*>(delta_buf + e) = make_float4(b[0], b[1], b[2], b[3]);
    }
}

unsigned blocks_for(int64_t count, int64_t cap)
{
    int64_t b = (count / 4 + kThreads - 1) / kThreads;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return static_cast<unsigned>(b);
}

}  // namespace

hipError_t launch_grad_sqnorm(const float* g, int64_t count, double* sum_sq, double* partials, hipStream_t stream)
{
    const unsigned nb = blocks_for(count, kMaxNormBlocks);
    sqnorm_partial_kernel<<<nb, kThreads, 0, stream>>>(g, count, partials);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    sqnorm_final_kernel<<<1, kMaxNormBlocks, 0, stream>>>(partials, static_cast<int>(nb), sum_sq);
    return hipGetLastError();
}

hipError_t launch_adamw_delta(const float* d_b, float* exp_avg, float* exp_avg_sq, float* delta_buf, int64_t count,
                              const AdamFactors& f, const double* sum_sq, hipStream_t stream)
{
    adamw_delta_kernel<<<blocks_for(count, 4096), kThreads, 0, stream>>>(d_b, exp_avg, exp_avg_sq, delta_buf, count, f,
                                                                         sum_sq);
    return hipGetLastError();
}

}  // namespace falqon
