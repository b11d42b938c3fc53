// Initialization (the paper's initialization algorithm): the quantization residual
//   E = DQ(W~) - W            (its residual step, with the sign the reformulation equation fixes)
// and the right factor of its rank-r truncated SVD,  A^ = sqrt(S_r) V_r^T  (its decomposition step),
// which the caller then casts with the backbone's scale (its last step, falqon_quantize with scale_in).
//
// This runs once per layer, before training; it is off the hot path.  The SVD is a randomized
// subspace iteration (the paper only says "SVD"; a truncated factor is all it needs):
//   Z0 = orth(Omega)                         l = r + 8 rows of length n, Omega Gaussian (caller's);
//                                            orth = Cholesky QR applied twice
//   repeat q times:  Y = orth(Z E^T);  Z = orth(Y E)
//   Y = Z E^T;  H = Y Y^T (l x l, fp64);  H = P diag(lambda) P^T  (cyclic Jacobi, fp64)
//   A^[i,:] = lambda_i^(1/4) * sum_c P[c,i] Z[c,:]      for the r largest lambda_i = sigma_i^2
// Products with E accumulate in fp32 (matrix cores, slices of the contraction added in order);
// everything l x l (Gram matrices, Cholesky factors, the eigenproblem) is fp64.
#include "falqon_internal.h"
#include "jacobi_rotation.h"

namespace falqon {
namespace {

constexpr int kThreads = 256;

__global__ void __launch_bounds__(kThreads)
init_residual_kernel(const float* __restrict__ w, const uint8_t* __restrict__ wq, const float* __restrict__ s_w,
                     int64_t count, float* __restrict__ e)
{
    const float s = *s_w;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads * 4;
    for (int64_t i = (static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x) * 4; i < count; i += stride) {
        const float4 wv = *reinterpret_cast<const float4*>(w + i);
        const uint32_t c = *reinterpret_cast<const uint32_t*>(wq + i);
        float4 o;
        // IEEE division and subtraction, unfused, as the definition has them
        o.x = __fsub_rn(__fdiv_rn(__builtin_amdgcn_cvt_f32_fp8(static_cast<int>(c), 0), s), wv.x);
        o.y = __fsub_rn(__fdiv_rn(__builtin_amdgcn_cvt_f32_fp8(static_cast<int>(c), 1), s), wv.y);
        o.z = __fsub_rn(__fdiv_rn(__builtin_amdgcn_cvt_f32_fp8(static_cast<int>(c), 2), s), wv.z);
        o.w = __fsub_rn(__fdiv_rn(__builtin_amdgcn_cvt_f32_fp8(static_cast<int>(c), 3), s), wv.w);
        *reinterpret_cast<float4*>(e + i) = o;
    }
}

__global__ void __launch_bounds__(kThreads)
copy_kernel(const float* __restrict__ src, float* __restrict__ dst, int64_t count)
{
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; i < count; i += stride) dst[i] = src[i];
}

constexpr int kMaxL = 128;                 // vectors in the subspace (r + 8 <= 128)
constexpr int kMaxSlices = 16;             // slices of the contracted dimension in the two products

typedef float v16f __attribute__((ext_vector_type(16)));

// The two products with E run on the fp32 matrix cores (v_mfma_f32_32x32x2_f32), operands loaded
// straight from memory into the instruction's layout: lane t supplies row (t % 32) of its
// operand and depth index (t / 32).  A contraction does not care in which order its terms are
// taken as long as both operands agree, so depth index h of four consecutive instructions stands
// for four consecutive memory elements 4 h .. 4 h + 3 of an eight-element step: one 16-byte load
// per lane and operand where the operand is contiguous along the contracted dimension.
// The accumulator of (first, second) operand holds, in lane t, column (t % 32) = the second
// operand's row, and in register v the first operand's row 8 (v / 4) + 4 (t / 32) + v % 4.
// One wave owns 32 rows (or columns) of E and all l <= 32 NBV vectors over one slice of the
// contracted dimension; the slices' results are added in order by sum_slices_kernel.

// part[s][c][i] = sum over columns j of slice s of Z[c][j] E[i][j]
template <int NBV>
__global__ void __launch_bounds__(kThreads)
apply_e_kernel(const float* __restrict__ e, int64_t m, int64_t n, const float* __restrict__ z, int l,
               float* __restrict__ part, int64_t per_slice)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, h = lane >> 5;
    const int64_t i0 = (static_cast<int64_t>(blockIdx.x) * (kThreads / 64) + wave) * 32;
    if (i0 >= m) return;                                             // (no barrier in this kernel)
    const int64_t j_begin = static_cast<int64_t>(blockIdx.y) * per_slice;
    const int64_t j_end = j_begin + per_slice < n ? j_begin + per_slice : n;
    const int64_t row = i0 + (lane & 31);
    const float* const erow = e + (row < m ? row : m - 1) * n;
    v16f acc[NBV];
#pragma unroll
    for (int b = 0; b < NBV; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[b][v] = 0.0f;
    const float4 zero = make_float4(0.0f, 0.0f, 0.0f, 0.0f);

    for (int64_t j0 = j_begin; j0 < j_end; j0 += 8) {
        const int64_t jj = j0 + 4 * h;                               // n and per_slice are multiples of 4 and 8
        const bool in = jj < j_end;
        const float4 ev = (in && row < m) ? *reinterpret_cast<const float4*>(erow + jj) : zero;
#pragma unroll
        for (int b = 0; b < NBV; ++b) {
            const int c = b * 32 + (lane & 31);
            const float4 zv = (in && c < l) ? *reinterpret_cast<const float4*>(z + static_cast<int64_t>(c) * n + jj) : zero;
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(zv.x, ev.x, acc[b], 0, 0, 0);
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(zv.y, ev.y, acc[b], 0, 0, 0);
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(zv.z, ev.z, acc[b], 0, 0, 0);
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(zv.w, ev.w, acc[b], 0, 0, 0);
        }
    }
    if (row >= m) return;
    float* const out = part + static_cast<int64_t>(blockIdx.y) * l * m;
#pragma unroll
    for (int b = 0; b < NBV; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int c = b * 32 + 8 * (v / 4) + 4 * h + v % 4;
            if (c < l) out[static_cast<int64_t>(c) * m + row] = acc[b][v];
        }
}

// part[s][c][j] = sum over rows i of slice s of Y[c][i] E[i][j]
template <int NBV>
__global__ void __launch_bounds__(kThreads)
apply_et_kernel(const float* __restrict__ e, int64_t m, int64_t n, const float* __restrict__ y, int l,
                float* __restrict__ part, int64_t per_slice)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, h = lane >> 5;
    const int64_t j0 = (static_cast<int64_t>(blockIdx.x) * (kThreads / 64) + wave) * 32;
    if (j0 >= n) return;                                             // (no barrier in this kernel)
    const int64_t i_begin = static_cast<int64_t>(blockIdx.y) * per_slice;
    const int64_t i_end = i_begin + per_slice < m ? i_begin + per_slice : m;
    const int64_t col = j0 + (lane & 31);
    const float* const ecol = e + (col < n ? col : n - 1);
    v16f acc[NBV];
#pragma unroll
    for (int b = 0; b < NBV; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[b][v] = 0.0f;
    const float4 zero = make_float4(0.0f, 0.0f, 0.0f, 0.0f);

    // Operands of the next step are requested before this step's products (92 -> 76 us at 4096 x 4096, l = 72; the
    // other product, whose loads are 16 bytes of a row each, is faster without, 50 against 100 us).
    float ev[4], ev2[4];
    float4 yv[NBV], yv2[NBV];
    auto fetch = [&](int64_t i0, float (&ef)[4], float4 (&yf)[NBV]) {
        const int64_t ii = i0 + 4 * h;                               // m and per_slice are multiples of 4 and 8
        const bool in = ii < i_end;
#pragma unroll
        for (int t = 0; t < 4; ++t) ef[t] = (in && col < n) ? ecol[(ii + t) * n] : 0.0f;
#pragma unroll
        for (int b = 0; b < NBV; ++b) {
            const int c = b * 32 + (lane & 31);
            yf[b] = (in && c < l) ? *reinterpret_cast<const float4*>(y + static_cast<int64_t>(c) * m + ii) : zero;
        }
    };
    auto multiply = [&](const float (&ef)[4], const float4 (&yf)[NBV]) {
#pragma unroll
        for (int b = 0; b < NBV; ++b) {
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(yf[b].x, ef[0], acc[b], 0, 0, 0);
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(yf[b].y, ef[1], acc[b], 0, 0, 0);
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(yf[b].z, ef[2], acc[b], 0, 0, 0);
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(yf[b].w, ef[3], acc[b], 0, 0, 0);
        }
    };
    fetch(i_begin, ev, yv);
    for (int64_t i0 = i_begin; i0 < i_end; i0 += 16) {
        fetch(i0 + 8, ev2, yv2);                                     // (zeros beyond the slice)
        __builtin_amdgcn_sched_barrier(0);
        multiply(ev, yv);
        fetch(i0 + 16, ev, yv);
        __builtin_amdgcn_sched_barrier(0);
        multiply(ev2, yv2);
    }
    if (col >= n) return;
    float* const out = part + static_cast<int64_t>(blockIdx.y) * l * n;
#pragma unroll
    for (int b = 0; b < NBV; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int c = b * 32 + 8 * (v / 4) + 4 * h + v % 4;
            if (c < l) out[static_cast<int64_t>(c) * n + col] = acc[b][v];
        }
}

// out[i] = part[0][i] + part[1][i] + ... in that order
__global__ void __launch_bounds__(kThreads)
sum_slices_kernel(const float* __restrict__ part, int slices, int64_t count, float* __restrict__ out)
{
    const int64_t i = (static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x) * 4;
    if (i >= count) return;                                          // count is a multiple of 4
    float4 s = *reinterpret_cast<const float4*>(part + i);
    for (int k = 1; k < slices; ++k) {
        const float4 v = *reinterpret_cast<const float4*>(part + static_cast<int64_t>(k) * count + i);
        s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    *reinterpret_cast<float4*>(out + i) = s;
}

// Orthonormalisation of the l rows of V[l][len] by Cholesky QR, applied twice: G = V V^T (fp64,
// gram_kernel), G = L L^T and its inverse factor (inverse_factor_kernel), V <- L^-1 V
// (apply_lower_kernel).  Everything of size len runs over the whole chip; only the l x l factorisation is
// one workgroup.  The second application brings the rows to orthonormal at the precision they are stored in
// whenever cond(V) < 1e8, which a product with E of a set of orthonormal vectors is far from reaching.  A
// row whose pivot is not positive (a vector in the span of the earlier ones) is set to zero.
//
// L^-1 by elimination on [G | I]: step c subtracts G[k][c] / d_c times row c from every row k > c, d_c the
// pivot; the right half becomes the inverse of the unit factor L', and L = L' D^(1/2).  Column j of the left
// half is finished in step j, where column j of the right one begins, so one lower triangle of registers
// holds both, in blocks of 4 x 4, one per thread: a step reads eight LDS values per sixteen updates (one
// element per thread and update reads two for each, and the LDS then takes longer than the arithmetic:
// 55 us at l = 72).  A step publishes row c of the right half and column c of the left one in one LDS vector
// and costs a barrier, a reciprocal and the update: a chain of l of them is all there is: 29 us at l = 72, where a factorisation with its trailing block in LDS took
// 130 us and a forward substitution per column of V another 113 us.
constexpr int kFactorThreads = 576;                                   // 32 * 33 / 2 blocks at l = 128, in whole waves

__global__ void __launch_bounds__(kFactorThreads)
inverse_factor_kernel(const double* __restrict__ g, int l, double* __restrict__ linv)
{
    __shared__ __attribute__((aligned(32))) double s_vec[2][kMaxL];
    __shared__ double s_root[kMaxL];
    const int t = threadIdx.x, nb = l / 4;                            // l is a multiple of 8
    int R = static_cast<int>((sqrtf(8.0f * static_cast<float>(t) + 1.0f) - 1.0f) * 0.5f);
    if (R * (R + 1) / 2 > t) --R;
    if ((R + 1) * (R + 2) / 2 <= t) ++R;
    const int C = t - R * (R + 1) / 2;
    const bool live = R < nb;                                         // block row R, block column C <= R
    double x[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) x[i][j] = live ? g[(4 * R + i) * l + 4 * C + j] : 0.0;
    const double tiny = 1e-28 * fmax(g[0], 1e-300);
    for (int cb = 0; cb < nb; ++cb) {
#pragma unroll
        for (int ci = 0; ci < 4; ++ci) {
            const int c = 4 * cb + ci;
            double* const vec = s_vec[ci & 1];                        // (the buffers alternate: one barrier per step)
            if (live && C == cb) {                                    // the pivot and the column below it
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (R > cb || i >= ci) vec[4 * R + i] = x[i][ci];
            }
            if (live && R == cb) {                                    // L'^-1[c][.] before the pivot
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (C < cb || j < ci) vec[4 * C + j] = x[ci][j];
            }
            __syncthreads();
            const double d = vec[c];
            double dinv = __builtin_amdgcn_rcp(d);                    // and two Newton steps: full precision
            dinv = fma(fma(-d, dinv, 1.0), dinv, dinv);
            dinv = fma(fma(-d, dinv, 1.0), dinv, dinv);
            if (!(d > tiny)) dinv = 0.0;                              // a dead row takes no part
            if (t == 0) s_root[c] = dinv;
            if (live && R >= cb) {
                double f[4], v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) { f[i] = vec[4 * R + i] * dinv; v[i] = vec[4 * C + i]; }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (R == cb && i <= ci) continue;                 // rows up to c are finished
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[i][j] = C == cb && j == ci ? -f[i] : x[i][j] - f[i] * v[j];
                }
                if (R == cb && C == cb) x[ci][ci] = 1.0;
            }
        }
    }
    __syncthreads();
    if (t < l) s_root[t] = sqrt(s_root[t]);
    __syncthreads();
    if (!live) return;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (R > C || j <= i) linv[(4 * R + i) * l + 4 * C + j] = x[i][j] * s_root[4 * R + i];
}

// V <- L^-1 V in place: a workgroup owns 64 columns of V, a wave four rows of the result at a time, whose
// factors are uniform over the wave (scalar loads) and share each element of V read from LDS: 9.6 us at
// 72 x 4096.
constexpr int kLowerCols = 64, kLowerThreads = 1024;

__global__ void __launch_bounds__(kLowerThreads)
apply_lower_kernel(float* __restrict__ v, int l, int64_t len, const double* __restrict__ linv)
{
    extern __shared__ double s_v[];                                   // [l][64]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t j = static_cast<int64_t>(blockIdx.x) * kLowerCols + lane;
    for (int c = wave; c < l; c += kLowerThreads / 64)
        s_v[c * kLowerCols + lane] = j < len ? static_cast<double>(v[static_cast<int64_t>(c) * len + j]) : 0.0;
    __syncthreads();
    for (int c0 = 4 * wave; c0 < l; c0 += 4 * (kLowerThreads / 64)) { // l is a multiple of 8
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        const double* const f = linv + static_cast<int64_t>(c0) * l;
        for (int p = 0; p < c0; p += 4) {
            double x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = s_v[(p + u) * kLowerCols + lane];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int u = 0; u < 4; ++u) acc[q] = fma(f[q * l + p + u], x[u], acc[q]);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)                                   // the diagonal block
#pragma unroll
            for (int u = 0; u <= q; ++u) acc[q] = fma(f[q * l + c0 + u], s_v[(c0 + u) * kLowerCols + lane], acc[q]);
        if (j < len) {
#pragma unroll
            for (int q = 0; q < 4; ++q) v[static_cast<int64_t>(c0 + q) * len + j] = static_cast<float>(acc[q]);
        }
    }
}

// H[a][b] = sum_i Y[a][i] Y[b][i] in fp64; grid (l, l), the upper half leaves, the lower one writes both
__global__ void __launch_bounds__(kThreads)
gram_kernel(const float* __restrict__ y, int l, int64_t m, double* __restrict__ h)
{
    __shared__ double s_red[kThreads / 64];
    if (blockIdx.y > blockIdx.x) return;
    const float* ya = y + static_cast<int64_t>(blockIdx.x) * m;
    const float* yb = y + static_cast<int64_t>(blockIdx.y) * m;
    double d = 0.0;
    for (int64_t i = 4 * threadIdx.x; i < m; i += 4 * kThreads) {     // m is a multiple of 4
        const float4 p = *reinterpret_cast<const float4*>(ya + i), q = *reinterpret_cast<const float4*>(yb + i);
        d += static_cast<double>(p.x) * static_cast<double>(q.x);
        d += static_cast<double>(p.y) * static_cast<double>(q.y);
        d += static_cast<double>(p.z) * static_cast<double>(q.z);
        d += static_cast<double>(p.w) * static_cast<double>(q.w);
    }
    for (int off = 32; off > 0; off >>= 1) d += __shfl_xor(d, off, 64);
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = d;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < kThreads / 64; ++w) t += s_red[w];
        h[static_cast<int64_t>(blockIdx.x) * l + blockIdx.y] = t;
        h[static_cast<int64_t>(blockIdx.y) * l + blockIdx.x] = t;
    }
}

// Symmetric eigen-decomposition of H (l x l, l even, fp64) by two-sided Jacobi with the round-robin
// ordering: each round rotates l/2 disjoint index pairs at once.  One workgroup; H lives in LDS, the
// eigenvectors (rows of pt) beside it where both fit (P_IN_LDS, l <= 96: a round then touches no memory), in
// global memory otherwise.  A round is two phases between barriers: one pass that applies the rotations to H
// from both sides at once (a thread owns the 2 x 2 block of two pairs, in the lower half, and writes its
// mirror image too); then the eigenvectors' rotation by fifteen waves, while the first one forms the next
// round's rotations, a chain of fp64 roots and a division.  Rows of H at an odd pitch: at a pitch of 72
// doubles a column sits in four LDS banks.  Stops after the first sweep without a rotation, or after
// `sweeps`.  On exit lambda[i] = H[i][i] and order[k] is the index of the k-th largest eigenvalue.
// 1024 threads; a chain of l - 1 rounds per sweep, 1.4 us each (l = 72: 0.78 ms for the
// whole; 2.85 ms with columns, rows and rotations as three phases at an even pitch).
constexpr int kJacobiThreads = 1024;

template <bool P_IN_LDS>
__global__ void __launch_bounds__(kJacobiThreads)
jacobi_eig_kernel(const double* __restrict__ h_in, int l, double* __restrict__ pt, double* __restrict__ lambda,
                  int* __restrict__ order, int sweeps)
{
    extern __shared__ double s_h[];                                   // [l][l + 1], (pt [l][l],) then rotations and pairs
    const int pitch = l + 1, t = threadIdx.x;
    double* const s_p = P_IN_LDS ? s_h + l * pitch : pt;              // the eigenvectors while they are rotated
    double* const s_cs = s_h + l * pitch + (P_IN_LDS ? l * l : 0);    // two sets of l/2 cosines, l/2 sines
    int* const s_pairs = reinterpret_cast<int*>(s_cs + 2 * l);        // and of l/2 pairs
    int* const s_rot = s_pairs + 2 * l;                               // rotations taken in this sweep and the next
    for (int q = t; q < l * l; q += kJacobiThreads) {
        s_h[q / l * pitch + q % l] = h_in[q];
        s_p[q] = (q / l == q % l) ? 1.0 : 0.0;
    }
    const int half = l / 2;
    // this thread's blocks (k >= j) of H, and its columns of pairs of eigenvectors, as two 16-bit indices
    constexpr int EB = 3, EP = 9;                                     // l <= 128: 2080 blocks, 8192 columns
    int blk[EB], vec[EP];
#pragma unroll
    for (int e = 0; e < EB; ++e) {
        const int q = t + e * kJacobiThreads;
        int k = static_cast<int>((sqrtf(8.0f * static_cast<float>(q) + 1.0f) - 1.0f) * 0.5f);
        if (k * (k + 1) / 2 > q) --k;
        if ((k + 1) * (k + 2) / 2 <= q) ++k;
        blk[e] = k < half ? k << 16 | (q - k * (k + 1) / 2) : -1;
    }
#pragma unroll
    for (int e = 0; e < EP; ++e) {                                    // the first wave forms rotations instead
        const int q = t - 64 + e * (kJacobiThreads - 64);
        vec[e] = t >= 64 && q < half * l ? (q / l) << 16 | q % l : -1;
    }
    if (t == 0) s_rot[0] = s_rot[1] = 0;
    __syncthreads();
    // round-robin ordering: position 0 keeps index 0, positions 1 .. l-1 rotate by one per round
    auto at = [&](int pos, int round) { return pos == 0 ? 0 : (pos - 1 >= round ? pos - round : pos - round + l - 1); };
    // pairs (positions k and l-1-k) of a round and their rotations from the current 2x2 blocks
    auto form = [&](int round, int set, int* rot) {
        if (t >= half) return;
        int a = at(t, round), b = at(l - 1 - t, round);
        if (a > b) { const int x = a; a = b; b = x; }
        s_pairs[set * l + 2 * t] = a; s_pairs[set * l + 2 * t + 1] = b;
        const double haa = s_h[a * pitch + a], hbb = s_h[b * pitch + b], hab = s_h[a * pitch + b];
        double c, s;
        if (jacobi_rotation(haa, hbb, hab, c, s)) atomicAdd(rot, 1);
        s_cs[set * l + t] = c; s_cs[set * l + half + t] = s;
    };
    form(0, 0, s_rot);
    __syncthreads();
    int set = 0;
    for (int sweep = 0; sweep < sweeps; ++sweep) {
        for (int round = 0; round < l - 1; ++round, set ^= 1) {
            const double* const s_c = s_cs + set * l;
            const double* const s_s = s_c + half;
            const int* const s_pp = s_pairs + set * l;
            const bool last = round == l - 2;
            if (last && t == 0) s_rot[(sweep + 1) & 1] = 0;
            // H <- J^T H J   (pairs are disjoint, so all of them at once)
#pragma unroll
            for (int e = 0; e < EB; ++e) {
                if (blk[e] < 0) continue;
                const int k = blk[e] >> 16, j = blk[e] & 0xffff;
                const int ak = s_pp[2 * k], bk = s_pp[2 * k + 1], aj = s_pp[2 * j], bj = s_pp[2 * j + 1];
                const double ck = s_c[k], sk = s_s[k], cj = s_c[j], sj = s_s[j];
                const double x00 = s_h[ak * pitch + aj], x01 = s_h[ak * pitch + bj];
                const double x10 = s_h[bk * pitch + aj], x11 = s_h[bk * pitch + bj];
                const double y00 = cj * x00 - sj * x01, y01 = sj * x00 + cj * x01;
                const double y10 = cj * x10 - sj * x11, y11 = sj * x10 + cj * x11;
                const double z00 = ck * y00 - sk * y10, z01 = ck * y01 - sk * y11;
                const double z10 = sk * y00 + ck * y10, z11 = sk * y01 + ck * y11;
                s_h[ak * pitch + aj] = z00; s_h[ak * pitch + bj] = z01;
                s_h[bk * pitch + aj] = z10; s_h[bk * pitch + bj] = z11;
                if (k != j) {
                    s_h[aj * pitch + ak] = z00; s_h[bj * pitch + ak] = z01;
                    s_h[aj * pitch + bk] = z10; s_h[bj * pitch + bk] = z11;
                }
            }
            __syncthreads();
            // the next round's rotations (first wave) beside pt <- J^T pt (the others)
            form(last ? 0 : round + 1, set ^ 1, s_rot + ((sweep + (last ? 1 : 0)) & 1));
#pragma unroll
            for (int e = 0; e < EP; ++e) {
                if (vec[e] < 0) continue;
                const int k = vec[e] >> 16, i = vec[e] & 0xffff;
                double* const pa = s_p + s_pp[2 * k] * l + i;
                double* const pb = s_p + s_pp[2 * k + 1] * l + i;
                const double c = s_c[k], s = s_s[k], va = *pa, vb = *pb;
                *pa = c * va - s * vb;
                *pb = s * va + c * vb;
            }
            __syncthreads();
        }
        if (s_rot[sweep & 1] == 0) break;                             // converged (same value in every lane)
    }
    if (P_IN_LDS)
        for (int q = t; q < l * l; q += kJacobiThreads) pt[q] = s_p[q];
    for (int i = t; i < l; i += kJacobiThreads) lambda[i] = s_h[i * pitch + i];
    __syncthreads();
    // rank by eigenvalue, larger first, equal values by smaller index.  A NaN (a matrix that is not finite) ranks
    // last: the ranks have to be a permutation, since the entries of `order` are used as indices.
    auto value = [&](int i) { const double x = s_h[i * pitch + i]; return x == x ? x : -HUGE_VAL; };
    for (int i = t; i < l; i += kJacobiThreads) {
        const double li = value(i);
        int rank = 0;
        for (int j = 0; j < l; ++j) {
            const double lj = value(j);
            rank += (lj > li || (lj == li && j < i)) ? 1 : 0;
        }
        order[rank] = i;
    }
}

// A^[k][j] = lambda_k^(1/4) * sum_c pt[order[k]][c] Z[c][j];  sigma[k] = sqrt(lambda_k)
__global__ void __launch_bounds__(kThreads)
rotate_kernel(const float* __restrict__ z, int l, int64_t n, const double* __restrict__ pt,
              const double* __restrict__ lambda, const int* __restrict__ order, int r,
              float* __restrict__ a_out, float* __restrict__ sigma_out, int inverse_scale)
{
    const int k = blockIdx.y;
    const int col = order[k];
    const double lam = lambda[col] > 0.0 ? lambda[col] : 0.0;
    // right factor: z holds unit vectors, row k becomes sqrt(sigma_k) v_k.  Left factor (inverse_scale):
    // z holds E v (length sigma_k u_k after the rotation), row k becomes sqrt(sigma_k) u_k.
    const double root = sqrt(sqrt(lam));
    const double scale = inverse_scale ? (root > 0.0 ? 1.0 / root : 0.0) : root;
    const int64_t j = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (j < n) {
        double acc = 0.0;
        for (int c = 0; c < l; ++c) acc += pt[col * l + c] * static_cast<double>(z[static_cast<int64_t>(c) * n + j]);
        a_out[static_cast<int64_t>(k) * n + j] = static_cast<float>(scale * acc);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0 && sigma_out) sigma_out[k] = static_cast<float>(sqrt(lam));
}

}  // namespace

hipError_t launch_init_residual(const float* w, const uint8_t* wq, const float* s_w, int64_t count, float* e,
                                hipStream_t stream)
{
    int64_t blocks = (count / 4 + kThreads - 1) / kThreads;
    if (blocks < 1) blocks = 1;
    if (blocks > 8192) blocks = 8192;
    init_residual_kernel<<<static_cast<unsigned>(blocks), kThreads, 0, stream>>>(w, wq, s_w, count, e);
    return hipGetLastError();
}

SvdLayout svd_layout(int64_t m, int64_t n, int64_t r)
{
    const size_t l = static_cast<size_t>(r) + 8;
    auto up = [](size_t v) { return (v + 255) / 256 * 256; };
    SvdLayout L;
    size_t off = 0;
    L.z = off;      off = up(off + sizeof(float) * l * static_cast<size_t>(n));
    L.y = off;      off = up(off + sizeof(float) * l * static_cast<size_t>(m));
    L.h = off;      off = up(off + sizeof(double) * l * l);
    L.p = off;      off = up(off + sizeof(double) * l * l);
    L.lambda = off; off = up(off + sizeof(double) * l);
    L.order = off;  off = up(off + sizeof(int) * l);
    L.part = off;   off = up(off + sizeof(float) * kMaxSlices * l * static_cast<size_t>(m > n ? m : n));
    L.total = off;
    return L;
}

// rows of v[l][len] <- orthonormal (Cholesky QR twice); h and lfac are l x l fp64 scratch
static hipError_t orthonormalize_rows(float* v, int l, int64_t len, double* h, double* lfac, hipStream_t stream)
{
    const size_t lds = sizeof(double) * static_cast<size_t>(l) * kLowerCols;                  // 64 KB at most
    hipError_t err;
    for (int pass = 0; pass < 2; ++pass) {
        gram_kernel<<<dim3(l, l), kThreads, 0, stream>>>(v, l, len, h);
        inverse_factor_kernel<<<1, kFactorThreads, 0, stream>>>(h, l, lfac);
        apply_lower_kernel<<<static_cast<unsigned>((len + kLowerCols - 1) / kLowerCols), kLowerThreads, lds, stream>>>(v, l, len, lfac);
        err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

hipError_t launch_svd_right_factor(const float* e, int64_t m, int64_t n, int64_t r, const float* omega, int iters,
                                   float* a_out, float* sigma_out, float* bt_out, uint8_t* ws, hipStream_t stream)
{
    const int l = static_cast<int>(r) + 8;
    const SvdLayout L = svd_layout(m, n, r);
    float* z = reinterpret_cast<float*>(ws + L.z);
    float* y = reinterpret_cast<float*>(ws + L.y);
    double* h = reinterpret_cast<double*>(ws + L.h);
    double* p = reinterpret_cast<double*>(ws + L.p);
    double* lambda = reinterpret_cast<double*>(ws + L.lambda);
    int* order = reinterpret_cast<int*>(ws + L.order);
    float* part = reinterpret_cast<float*>(ws + L.part);
    // Y[l][m] = Z E^T (transposed == false) or Z[l][n] = Y E: slices of the contracted dimension so that about
    // 2048 waves stream E, then the ordered sum of the slices
    auto product = [&](bool transposed, const float* vec, float* out) -> hipError_t {
        const int64_t rows = transposed ? n : m, depth = transposed ? m : n;
        const int64_t blocks = (rows + 31) / 32;
        int64_t slices = 2048 / blocks;
        if (slices < 1) slices = 1;
        if (slices > kMaxSlices) slices = kMaxSlices;
        int64_t per = ((depth + slices - 1) / slices + 7) / 8 * 8;
        slices = (depth + per - 1) / per;
        const dim3 grid(static_cast<unsigned>((blocks + kThreads / 64 - 1) / (kThreads / 64)), static_cast<unsigned>(slices));
        float* dst = slices > 1 ? part : out;
        const int nbv = (l + 31) / 32;
#define FQ_PRODUCT(NBV)                                                                                   \
        if (transposed) apply_et_kernel<NBV><<<grid, kThreads, 0, stream>>>(e, m, n, vec, l, dst, per);   \
        else apply_e_kernel<NBV><<<grid, kThreads, 0, stream>>>(e, m, n, vec, l, dst, per)
        if (nbv == 1) { FQ_PRODUCT(1); } else if (nbv == 2) { FQ_PRODUCT(2); } else if (nbv == 3) { FQ_PRODUCT(3); } else { FQ_PRODUCT(4); }
#undef FQ_PRODUCT
        hipError_t pe = hipGetLastError();
        if (pe != hipSuccess || slices == 1) return pe;
        const int64_t count = static_cast<int64_t>(l) * rows;          // a multiple of 4 (m and n are)
        sum_slices_kernel<<<static_cast<unsigned>((count / 4 + kThreads - 1) / kThreads), kThreads, 0, stream>>>(
            part, static_cast<int>(slices), count, out);
        return hipGetLastError();
    };
    hipError_t err;
#define FQ_CHECK_LAUNCH() do { err = hipGetLastError(); if (err != hipSuccess) return err; } while (0)
    copy_kernel<<<1024, kThreads, 0, stream>>>(omega, z, static_cast<int64_t>(l) * n);
    FQ_CHECK_LAUNCH();
    err = orthonormalize_rows(z, l, n, h, p, stream);
    if (err != hipSuccess) return err;
    for (int it = 0; it < iters; ++it) {
        err = product(false, z, y);
        if (err != hipSuccess) return err;
        err = orthonormalize_rows(y, l, m, h, p, stream);
        if (err != hipSuccess) return err;
        err = product(true, y, z);
        if (err != hipSuccess) return err;
        err = orthonormalize_rows(z, l, n, h, p, stream);
        if (err != hipSuccess) return err;
    }
    err = product(false, z, y);
    if (err != hipSuccess) return err;
    gram_kernel<<<dim3(l, l), kThreads, 0, stream>>>(y, l, m, h);
    FQ_CHECK_LAUNCH();
    // H, and the eigenvectors too while both fit the LDS (l <= 96; rotated in memory otherwise)
    const size_t mat = sizeof(double) * static_cast<size_t>(l) * l;
    const size_t rest = sizeof(double) * 3 * static_cast<size_t>(l) + sizeof(int) * (2 * static_cast<size_t>(l) + 2);
    const bool p_in_lds = 2 * mat + rest <= 160 * 1024;
    const size_t lds = (p_in_lds ? 2 : 1) * mat + rest;
    const void* jacobi = p_in_lds ? reinterpret_cast<const void*>(&jacobi_eig_kernel<true>)
                                  : reinterpret_cast<const void*>(&jacobi_eig_kernel<false>);
    err = hipFuncSetAttribute(jacobi, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    if (err != hipSuccess) return err;
    if (p_in_lds) jacobi_eig_kernel<true><<<1, kJacobiThreads, lds, stream>>>(h, l, p, lambda, order, 14);
    else jacobi_eig_kernel<false><<<1, kJacobiThreads, lds, stream>>>(h, l, p, lambda, order, 14);
    FQ_CHECK_LAUNCH();
    rotate_kernel<<<dim3(static_cast<unsigned>((n + kThreads - 1) / kThreads), static_cast<unsigned>(r)), kThreads, 0,
                    stream>>>(z, l, n, p, lambda, order, static_cast<int>(r), a_out, sigma_out, 0);
    FQ_CHECK_LAUNCH();
    if (bt_out) {
        // y still holds E z^T: its rotation by the same eigenvectors is sigma_k u_k, the left singular vectors
        rotate_kernel<<<dim3(static_cast<unsigned>((m + kThreads - 1) / kThreads), static_cast<unsigned>(r)), kThreads, 0,
                        stream>>>(y, l, m, p, lambda, order, static_cast<int>(r), bt_out, nullptr, 1);
        FQ_CHECK_LAUNCH();
    }
#undef FQ_CHECK_LAUNCH
    return hipSuccess;
}

}  // namespace falqon
