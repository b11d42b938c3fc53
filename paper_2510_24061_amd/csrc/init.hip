// Initialization (the paper's initialization algorithm): the quantization residual
//   E = DQ(W~) - W            (its residual step, with the sign the reformulation equation fixes)
// and the right factor of its rank-r truncated SVD,  A^ = sqrt(S_r) V_r^T  (its decomposition step),
// which the caller then casts with the backbone's scale (its last step, falqon_quantize with scale_in).
//
// This runs once per layer, before training; it is off the hot path.  The SVD is a randomized
// subspace iteration (the paper only says "SVD"; a truncated factor is all it needs):
//   Z0 = orth(Omega)                         l = r + 8 rows of length n, Omega Gaussian (caller's);
//                                            orth = Cholesky QR (the last one twice)
//   repeat q times:  Y = orth(Z E^T);  Z = orth(Y E)
//   Y = Z E^T;  H = Y Y^T (l x l, fp64);  H = P diag(lambda) P^T  (Cholesky factor, one-sided Jacobi, fp64)
//   A^[i,:] = lambda_i^(1/4) * sum_c P[c,i] Z[c,:]      for the r largest lambda_i = sigma_i^2
// Products with E accumulate in fp32 (matrix cores, slices of the contraction added in order);
// everything l x l (Gram matrices, Cholesky factors, the eigenproblem) is fp64.
#include <type_traits>

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

constexpr int kMaxL = 128;                 // vectors in the subspace (r + 8 <= 128)
constexpr int kMaxSlices = 12;             // slices of the contracted dimension in the two products

typedef float v4f __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));

// The two products with E run on the bf16 matrix cores, with both operands in three parts: an fp32 number is the sum of its
// rounding to bf16, the rounding of what that leaves, and what is left then (8 bits and a sign each, exact).  Six of the
// nine products of parts are formed (v_mfma_f32_16x16x32_bf16, exact products added in fp32, small ones first).  The
// others are at most 2^-24 of the whole (parts of 2^-8 and 2^-17 of their elements, twice), 2^-27.4 of it in the mean square (the largest of 4
// million drawn pairs 2^-24.2): what rounding a term to fp32 could cost, which the fp32 cores do not do.  An instruction adds 32
// terms where the fp32 one adds four, and sums come out nearer to 64 bits all the same (3.7e-7 against 5.4e-7 of a sum of 4096 terms of random sign).  At 4096 x 4096,
// l = 72, the fp32 cores need 17 us for a product, the six on the bf16 ones 6.5, and E, split on the way from memory to the
// operands, becomes what bounds it: a launch takes 21.6 us (30.5 on the fp32 cores; 25 with the operands of two steps in registers instead of three).
// Elements whose parts bf16 does not hold (look_at_range) take the fp32 cores, without packing or a ring: initialization of 4096 x 4096, r = 64,
// 1460 us (1275 in parts, 1563 with packed vectors on the fp32 cores for all).
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v8f __attribute__((ext_vector_type(8)));
constexpr int kParts = 3;

__device__ __forceinline__ void split(v8f x, v8bf (&part)[kParts])
{
#pragma unroll
    for (int k = 0; k < kParts; ++k) {
        part[k] = __builtin_convertvector(x, v8bf);
        if (k + 1 < kParts) x -= __builtin_convertvector(part[k], v8f);
    }
}

// Vectors as the products read them: blocks of 32 elements x 16 vectors, per block its three parts in the operand layout of
// the instruction, so that a wave reads 1 KB in a row.  Lane t holds row t % 16 of an operand and depths 8 (t / 16) .. + 7:
// element j of vector c lies in block (j / 32, c / 16) at lane c % 16 + 16 (j % 32 / 8), component j % 8.  Vectors are
// padded to whole blocks of 16, elements to blocks of 32, both with zeros.
//
// The vectors are packed, and every operand of E comes with 128 or 256 bytes of its row.  The next step's operands are
// requested before this step's products.  The four waves of a workgroup share out the steps of a slice and add up in LDS,
// which leaves a quarter of the partial sums in memory.  The accumulator of (first, second) operand holds, in lane t,
// column t % 16 = the second operand's row, and in register v the first operand's row 4 (t / 16) + v.
template <int CB>
struct Products {
    static_assert(CB <= 7, "eight blocks are two halves");
    v4f acc[4][CB];
    static constexpr int DEPTH = CB <= 5 ? 3 : 2;                     // steps whose operands are in registers or on their way
    v8bf zf[DEPTH][CB][kParts];

    __device__ __forceinline__ Products()
    {
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) acc[x][cb] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    }
    // blocks [first, first + CB) of `blocks`
    __device__ __forceinline__ void fetch(const v8bf* __restrict__ packed, int64_t step, int blocks, int first, int lane, int which)
    {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int k = 0; k < kParts; ++k) zf[which][cb][k] = packed[((step * blocks + first + cb) * kParts + k) * 64 + lane];
    }
    // steps first, first + 4, ... below end; none where the word says so, which is looked at behind the first requests
    template <class F, class M>
    __device__ __forceinline__ static void run(int64_t first, int64_t end, int outside, F fetch, M multiply)
    {
#pragma unroll
        for (int d = 0; d + 1 < DEPTH; ++d)
            if (first + 4 * d < end) fetch(first + 4 * d, d);
        if (outside) return;
        for (int64_t b = first; b < end; b += 4 * DEPTH) {
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                if (b + 4 * d >= end) break;
                if (b + 4 * (d + DEPTH - 1) < end) fetch(b + 4 * (d + DEPTH - 1), (d + DEPTH - 1) % DEPTH);
                __builtin_amdgcn_sched_barrier(0);
                multiply(d);
            }
        }
    }
    // The same on the fp32 matrix cores, with the vectors as they are.  vector: the one of this lane in the first block, of `length`
    // elements, with `vectors` from it on; operand(i, k): elements i .. i + 3 of this lane's row of E in block k (ROWS) or those of its
    // column in all four blocks from row i + k.  Depth index `quad` of four consecutive instructions stands for four elements in a row.
    template <bool ROWS, class O>
    __device__ __forceinline__ void run_fp32(const float* vector, int vectors, int64_t length, int64_t first, int64_t end, int quad, O operand)
    {
        for (int64_t b = first; b < end; b += 4) {
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const int64_t i = b * 32 + 16 * half + 4 * quad;      // (lengths are multiples of 4)
                const bool in = i < length;
                v4f o[4], z[CB];
#pragma unroll
                for (int k = 0; k < 4; ++k) o[k] = in ? operand(i, k) : v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
                    z[cb] = in && 16 * cb < vectors ? *reinterpret_cast<const v4f*>(vector + 16 * cb * length + i) : v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int x = 0; x < 4; ++x)
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb)
                            acc[x][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(z[cb][u], ROWS ? o[x][u] : o[u][x], acc[x][cb], 0, 0, 0);
            }
        }
    }
    // 16 vectors x CB by 16 rows of E, 32 deep
    __device__ __forceinline__ void multiply(int x, v8f e, int which)
    {
        v8bf ef[kParts];
        split(e, ef);
        constexpr int Z[6] = {2, 0, 1, 1, 0, 0}, E[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int q = 0; q < 6; ++q)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
                acc[x][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zf[which][cb][Z[q]], ef[E[q]], acc[x][cb], 0, 0, 0);
    }
};

// part[s][c][i] = sum over columns j of slice s of Z[c][j] E[i][j]; a workgroup owns 64 rows of E and CB blocks of vectors (all
// up to seven, at 424 of 512 registers; eight, which spilled 66 where seven took 508, are two halves, which give the same bits)
template <int CB>
__global__ void __launch_bounds__(kThreads)
apply_e_kernel(const float* __restrict__ e, int64_t m, int64_t n, const v8bf* __restrict__ zp, const float* __restrict__ z, int l,
               const int* __restrict__ wide, float* __restrict__ part, int64_t per_slice)
{
    constexpr int PITCH = 68;
    __shared__ __attribute__((aligned(16))) float s_sum[4][CB * 16 * PITCH];
    const int outside = *wide;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, row16 = lane & 15, quad = lane >> 4;
    const int64_t i0 = static_cast<int64_t>(blockIdx.x) * 64, steps = (n + 31) / 32;
    const int64_t begin = static_cast<int64_t>(blockIdx.y) * per_slice;
    const int64_t end = begin + per_slice < steps ? begin + per_slice : steps;
    const float* erow[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        const int64_t row = i0 + 16 * x + row16;
        erow[x] = e + (row < m ? row : m - 1) * n;                   // rows beyond E are computed and not stored
    }
    Products<CB> p;
    v4f ef[Products<CB>::DEPTH][4][2];
    auto fetch = [&](int64_t b, int which) {
        int64_t j[2] = {b * 32 + 8 * quad, b * 32 + 8 * quad + 4};
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (j[h] >= n) j[h] = n - 4;                             // (the vectors are zero there)
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int h = 0; h < 2; ++h) ef[which][x][h] = *reinterpret_cast<const v4f*>(erow[x] + j[h]);
        p.fetch(zp, b, CB * static_cast<int>(gridDim.z), CB * static_cast<int>(blockIdx.z), lane, which);
    };
    auto multiply = [&](int which) {
#pragma unroll
        for (int x = 0; x < 4; ++x) p.multiply(x, __builtin_shufflevector(ef[which][x][0], ef[which][x][1], 0, 1, 2, 3, 4, 5, 6, 7), which);
    };
    const int c0 = 16 * CB * static_cast<int>(blockIdx.z);
    p.run(begin + wave, end, outside, fetch, multiply);
    if (outside)
        p.template run_fp32<true>(z + (c0 + row16) * n, l - c0 - row16, n, begin + wave, end, quad,
                                  [&](int64_t j, int x) { return *reinterpret_cast<const v4f*>(erow[x] + j); });
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int v = 0; v < 4; ++v) s_sum[wave][(cb * 16 + 4 * quad + v) * PITCH + x * 16 + row16] = p.acc[x][cb][v];
    __syncthreads();
    const int vectors = l - c0 < 16 * CB ? l - c0 : 16 * CB;
    float* const out = part + (static_cast<int64_t>(blockIdx.y) * l + c0) * m;
    for (int q = threadIdx.x; q < vectors * 16; q += kThreads) {
        const int c = q >> 4, i4 = (q & 15) * 4;
        if (i0 + i4 >= m) continue;                                  // m is a multiple of 4
        v4f s = *reinterpret_cast<const v4f*>(&s_sum[0][c * PITCH + i4]);
#pragma unroll
        for (int w = 1; w < 4; ++w) s += *reinterpret_cast<const v4f*>(&s_sum[w][c * PITCH + i4]);
        *reinterpret_cast<v4f*>(out + static_cast<int64_t>(c) * m + i0 + i4) = s;
    }
}

// part[s][c][j] = sum over rows i of slice s of Y[c][i] E[i][j]; a workgroup owns 64 columns of E: lane t reads four
// columns 4 (t % 16) + x of eight rows, one for each of four column blocks
template <int CB>
__global__ void __launch_bounds__(kThreads)
apply_et_kernel(const float* __restrict__ e, int64_t m, int64_t n, const v8bf* __restrict__ yp, const float* __restrict__ y, int l,
                const int* __restrict__ wide, float* __restrict__ part, int64_t per_slice)
{
    constexpr int PITCH = 68;
    __shared__ __attribute__((aligned(16))) float s_sum[4][CB * 16 * PITCH];
    const int outside = *wide;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, row16 = lane & 15, quad = lane >> 4;
    const int64_t j0 = static_cast<int64_t>(blockIdx.x) * 64, steps = (m + 31) / 32;
    const int64_t begin = static_cast<int64_t>(blockIdx.y) * per_slice;
    const int64_t end = begin + per_slice < steps ? begin + per_slice : steps;
    const int64_t col = j0 + 4 * row16 < n ? j0 + 4 * row16 : n - 4; // columns beyond E are computed and not stored
    Products<CB> p;
    v4f ef[Products<CB>::DEPTH][8];
    auto fetch = [&](int64_t b, int which) {
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const int64_t i = b * 32 + 8 * quad + v;
            ef[which][v] = *reinterpret_cast<const v4f*>(e + (i < m ? i : m - 1) * n + col);   // (the vectors are zero beyond)
        }
        p.fetch(yp, b, CB * static_cast<int>(gridDim.z), CB * static_cast<int>(blockIdx.z), lane, which);
    };
    auto multiply = [&](int which) {
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            v8f column;
#pragma unroll
            for (int v = 0; v < 8; ++v) column[v] = ef[which][v][x];
            p.multiply(x, column, which);
        }
    };
    const int c0 = 16 * CB * static_cast<int>(blockIdx.z);
    p.run(begin + wave, end, outside, fetch, multiply);
    if (outside)
        p.template run_fp32<false>(y + (c0 + row16) * m, l - c0 - row16, m, begin + wave, end, quad,
                                   [&](int64_t i, int v) { return *reinterpret_cast<const v4f*>(e + (i + v) * n + col); });
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            *reinterpret_cast<v4f*>(&s_sum[wave][(cb * 16 + 4 * quad + v) * PITCH + 4 * row16]) =
                v4f{p.acc[0][cb][v], p.acc[1][cb][v], p.acc[2][cb][v], p.acc[3][cb][v]};
    __syncthreads();
    const int vectors = l - c0 < 16 * CB ? l - c0 : 16 * CB;
    float* const out = part + (static_cast<int64_t>(blockIdx.y) * l + c0) * n;
    for (int q = threadIdx.x; q < vectors * 16; q += kThreads) {
        const int c = q >> 4, j4 = (q & 15) * 4;
        if (j0 + j4 >= n) continue;                                  // n is a multiple of 4
        v4f s = *reinterpret_cast<const v4f*>(&s_sum[0][c * PITCH + j4]);
#pragma unroll
        for (int w = 1; w < 4; ++w) s += *reinterpret_cast<const v4f*>(&s_sum[w][c * PITCH + j4]);
        *reinterpret_cast<v4f*>(out + static_cast<int64_t>(c) * n + j0 + j4) = s;
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

// Orthonormalisation of the l rows of V[l][len] by Cholesky QR: G = V V^T (fp64, gram_kernel), G = L L^T and its
// inverse factor (factor_kernel), V <- L^-1 V (apply_lower_kernel).  Everything of size len runs over the whole chip;
// only the l x l factorisation is one workgroup.  A row whose pivot is not positive (a vector in the span of the
// earlier ones) is set to zero.  Between two products one application is enough: the iteration needs the span of the
// rows and a basis of it that is well conditioned, and with everything in fp64 one application leaves the rows
// orthonormal to 1e-16 cond(V)^2 before they are rounded to fp32 (a product with E of orthonormal vectors has its
// condition limited by the rounding of the product to about 1e7).  The last basis, which the Rayleigh-Ritz step and
// A^ take as orthonormal, gets a second one: orthonormal at the precision it is stored in while cond(V) < 1e8.
//
// L^-1 by elimination on [G | I] in blocks of 16 x 16, all as accumulators of v_mfma_f64_16x16x4_f64, a wave for each (or up to
// three).  Step b: its pivot block D is factored by one wave (W D W^T diagonal, W unit lower triangular), a row per lane, in 16
// pivots that pass through no memory (row_newbcast, an instruction per element; moved first and added then: 15.1 us the launch); F(R) = P(R) W^T for the blocks P(R) below it and, transposed, W V(C) for those
// of its row in the right half; then block (R, C) loses F(R) diag(1/d) F(C)^T, R > b.  Column b of the left half is
// finished in step b, where column b of the right one begins, so one lower triangle of blocks holds both halves; the rows of
// step b are finished too, and are written scaled with d^(-1/2).  A step costs the chain of 16 pivots (about 2000 cycles), two barriers
// and two chains of four matrix instructions: 12.6 us at l = 72.  (Blocks of 4 x 4, one per thread, the pivot block factored by
// every thread for itself and everything through LDS between steps: 23.3 us; with a scalar pivot per step 29.)
// FACTOR: L^T itself instead (its upper triangle; nothing else is written); pivots below the rounding of their own
// diagonal entry, which the subtractions cannot fall below, are null.  (Entries of G may differ by the square of the range
// of singular values: measured against the largest one, all values below 3e-8 of it would be lost, also those of rows
// that have nothing to do with it.)
constexpr int factor_blocks(int nb) { return nb * (nb + 1) / 2; }
constexpr int factor_waves(int nb) { return factor_blocks(nb) < 16 ? factor_blocks(nb) : 16; }

// lane N of the row of 16 lanes
template <int N>
__device__ __forceinline__ double of_lane(double v)
{
    return __builtin_amdgcn_update_dpp(0.0, v, 0x150 + N, 0xf, 0xf, true);
}

// v[i] += u times the v[i] of lane N of the row of 16, COUNT of them, an instruction each (the compiler takes two and a wait in
// between).  A DPP read has to be two instructions behind a vector write of its source.  The compiler does not look into inline
// assembly for that, and what it puts before a block (a copy, a reload, the select of a start value) may be such a write: so
// every block waits by itself, and within one no source is written before it is read.  Nor does it see that a block writes:
// what it reads by DPP next is a block's first element, so a block of one or two waits at its end, too.
template <int N, int COUNT>
__device__ __forceinline__ void add_of_lane(double* v, double u)
{
    static_assert(COUNT >= 0 && COUNT <= 8, "operands of a block");
#define FQ_ADD(i) "\n\tv_fmac_f64_dpp %" #i ", %" #i ", %[u] row_newbcast:%[lane] row_mask:0xf bank_mask:0xf"
#define FQ_BLOCK(adds, ...) asm volatile("s_nop 1" adds : __VA_ARGS__ : [u] "v"(u), [lane] "n"(N))
    if constexpr (COUNT == 1) FQ_BLOCK(FQ_ADD(0) "\n\ts_nop 1", "+v"(v[0]));
    if constexpr (COUNT == 2) FQ_BLOCK(FQ_ADD(0) FQ_ADD(1) "\n\ts_nop 1", "+v"(v[0]), "+v"(v[1]));
    if constexpr (COUNT == 3) FQ_BLOCK(FQ_ADD(0) FQ_ADD(1) FQ_ADD(2), "+v"(v[0]), "+v"(v[1]), "+v"(v[2]));
    if constexpr (COUNT == 4) FQ_BLOCK(FQ_ADD(0) FQ_ADD(1) FQ_ADD(2) FQ_ADD(3), "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
    if constexpr (COUNT > 4 && COUNT < 8) { add_of_lane<N, 4>(v, u); add_of_lane<N, COUNT - 4>(v + 4, u); }
    if constexpr (COUNT == 8)
        FQ_BLOCK(FQ_ADD(0) FQ_ADD(1) FQ_ADD(2) FQ_ADD(3) FQ_ADD(4) FQ_ADD(5) FQ_ADD(6) FQ_ADD(7),
                 "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7]));
#undef FQ_BLOCK
#undef FQ_ADD
}

template <int N, int END, typename F>
__device__ __forceinline__ void for_each(F f)
{
    if constexpr (N < END) {
        f(std::integral_constant<int, N>{});
        for_each<N + 1, END>(f);
    }
}

// *wide <- 1 where E has entries that the parts of the products do not hold: beyond 2^120 (rounding up must not overflow, nor a sum of
// what was rounded up), not finite, or below 2^-109 but not zero (bits down to 2^-133 are bf16's; conversion and matrix instruction keep
// subnormals).  Elements of the vectors, of length 1, lose no more than 2^-134 and are not looked at.
struct RangeOf {
    const float* e;
    int64_t count;                                                    // a multiple of 16
    int* wide;
};
__device__ __forceinline__ void look_at_range(const RangeOf& r, int64_t first, int64_t stride)
{
    constexpr uint32_t LEAST = uint32_t{127 - 109} << 23, MOST = uint32_t{127 + 120} << 23;
    bool outside = false;
    for (int64_t i = 4 * first; i < r.count; i += 4 * stride) {
        const uint4 v = *reinterpret_cast<const uint4*>(r.e + i);
        const uint32_t bits[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t size = bits[u] & 0x7fffffffu;
            outside |= size != 0 && size - LEAST > MOST - LEAST;
        }
    }
    if (outside) *r.wide = 1;
}

// Workgroups beyond the first (one takes all of the chain) look at E's range meanwhile.
template <int NB, bool FACTOR>
__global__ void __launch_bounds__(64 * factor_waves(NB))
factor_kernel(const double* __restrict__ g, int l, double* __restrict__ out, const RangeOf range)
{
    if (!FACTOR && blockIdx.x > 0) {
        look_at_range(range, static_cast<int64_t>(blockIdx.x - 1) * blockDim.x + threadIdx.x, static_cast<int64_t>(gridDim.x - 1) * blockDim.x);
        return;
    }
    constexpr int WAVES = factor_waves(NB), PER = (factor_blocks(NB) + WAVES - 1) / WAVES;
    constexpr int P = 18;                                             // doubles per row of a block: rows spread over the banks
    __shared__ __attribute__((aligned(16))) double s_in[NB][16 * P], s_f[NB][16 * P], s_w[16 * P], s_inv[2][16];
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), x = t & 15, quad = (t >> 4) & 3;
    // Blocks wave, wave + WAVES, ... of the lower triangle, row by row; register v of a block holds row quad + 4 v, column x.
    int R[PER], C[PER];
    v4d acc[PER];
    double least[PER];                                                // pivots up to this are null (of row x)
    const double largest = FACTOR ? 0.0 : fmax(g[0], 1e-300);
#pragma unroll
    for (int s = 0; s < PER; ++s) {
        const int q = wave + s * WAVES;
        int r = 0;
        while ((r + 1) * (r + 2) / 2 <= q) ++r;
        R[s] = r;                                                     // (beyond the triangle: never equal to, or below, a step)
        C[s] = q - r * (r + 1) / 2;
        if (q >= factor_blocks(NB)) R[s] = -1;
        const int row = 16 * r + x;
        least[s] = row >= l ? 0.0 : FACTOR ? 1e-15 * g[row * l + row] : 1e-28 * largest;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = 16 * r + quad + 4 * v, j = 16 * C[s] + x;
            acc[s][v] = R[s] >= 0 && i < l && j < l ? g[i * l + j] : i == j ? 1.0 : 0.0;     // (padded with the identity)
        }
    }
    // of row x of a block in LDS, the elements 4 quad .. + 3: depth index `quad` of four consecutive instructions
    auto row_part = [&](const double* block, double (&part)[4]) {
#pragma unroll
        for (int u = 0; u < 4; ++u) part[u] = block[x * P + 4 * quad + u];
    };
    auto product = [&](const double (&a)[4], const double (&b)[4], v4d c) {
#pragma unroll
        for (int u = 0; u < 4; ++u) c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[u], c, 0, 0, 0);
        return c;
    };
    for (int b = 0; b < NB; ++b) {
        // what the next products read: the column below the pivot block, its row in the right half transposed
#pragma unroll
        for (int s = 0; s < PER; ++s) {
            if (C[s] == b && R[s] >= b) {
#pragma unroll
                for (int v = 0; v < 4; ++v) s_in[R[s]][(quad + 4 * v) * P + x] = acc[s][v];
            } else if (!FACTOR && R[s] == b) {
#pragma unroll
                for (int v = 0; v < 4; ++v) s_in[C[s]][x * P + quad + 4 * v] = acc[s][v];
            }
            if (R[s] != b || C[s] != b) continue;
            // the pivot block: lane x holds its row x, four times over, and columns 4 quad .. + 3 of row x of W
            asm volatile("" ::: "memory");                            // (a wave's LDS accesses are carried out in order)
            const int row = 16 * b + x;
            double d[16], w[4], own = 0.0;
#pragma unroll
            for (int j = 0; j < 16; ++j) d[j] = s_in[b][x * P + j];
#pragma unroll
            for (int c = 0; c < 4; ++c) w[c] = 4 * quad + c == x ? 1.0 : 0.0;
            for_each<0, 16>([&](auto tag) {
                constexpr int k = decltype(tag)::value;
                const double p = of_lane<k>(d[k]);
                double r = __builtin_amdgcn_rcp(p);                   // and two Newton steps: full precision
                r = fma(fma(-p, r, 1.0), r, r);
                r = fma(fma(-p, r, 1.0), r, r);
                const double inv = p > of_lane<k>(least[s]) ? r : 0.0;   // a dead row takes no part
                if (x == k) own = inv;
                const double u = x > k ? -d[k] * inv : 0.0;
                constexpr int LEFT = 15 - k, FIRST = LEFT > 8 ? 8 : LEFT;
                add_of_lane<k, FIRST>(d + k + 1, u);
                add_of_lane<k, LEFT - FIRST>(d + k + 1 + FIRST, u);
                add_of_lane<k, 4>(w, u);
            });
            if (quad == 0) s_inv[b & 1][x] = own;
            const double root = sqrt(own);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int j = 4 * quad + c;
                s_w[x * P + j] = w[c];
                if (!FACTOR && row < l && j <= x) out[row * l + 16 * b + j] = w[c] * root;
            }
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < PER; ++s) {
            if (!FACTOR && R[s] == b && C[s] == b) {                  // W itself is what its column loses first
                double w[4];
                row_part(s_w, w);
#pragma unroll
                for (int u = 0; u < 4; ++u) s_f[b][(4 * quad + u) * P + x] = w[u];
            }
            const bool below = C[s] == b && (FACTOR ? R[s] >= b : R[s] > b), right = !FACTOR && R[s] == b && C[s] < b;
            if (!below && !right) continue;
            const int which = below ? R[s] : C[s];
            double p[4], w[4];
            row_part(s_in[which], p);
            row_part(s_w, w);
            const v4d f = product(p, w, v4d{0.0, 0.0, 0.0, 0.0});
            const double root = sqrt(s_inv[b & 1][x]);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = quad + 4 * v, j = 16 * b + x;           // element i of the block, column or row j of the result
                s_f[which][i * P + x] = f[v];
                if (FACTOR ? j < l && 16 * R[s] + i < l : right && j < l)
                    out[j * l + 16 * which + i] = FACTOR && R[s] == b && x > i ? 0.0 : f[v] * root;
            }
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < PER; ++s) {
            if (R[s] <= b || (FACTOR && C[s] <= b)) continue;
            double f[4], h[4];
            row_part(s_f[R[s]], f);
            row_part(s_f[C[s]], h);
#pragma unroll
            for (int u = 0; u < 4; ++u) f[u] *= -s_inv[b & 1][4 * quad + u];
            if (C[s] == b) acc[s] = v4d{0.0, 0.0, 0.0, 0.0};
            acc[s] = product(f, h, acc[s]);
        }
    }
}

// dst = L^-1 src on the fp64 matrix cores (v_mfma_f64_16x16x4_f64: lane t holds row t % 16 and depth t / 16 of its
// operand; register v of the accumulator holds row t / 16 + 4 v, column t % 16).  A workgroup owns 16 elements of all
// vectors, a wave 16 vectors of the result; every load is requested at once, so the launch is one memory round trip
// and a chain of up to l / 4 instructions.  dst may be src, and is written only if *asked where
// that is given; `packed` gets the layout above with its padding.
template <int CB>
__global__ void __launch_bounds__(CB * 64)
apply_lower_kernel(const float* src, float* dst, uint32_t* __restrict__ packed, int l, int64_t len,
                   const double* __restrict__ linv, const int* __restrict__ asked)
{
    const bool whole = !asked || *asked;
    const int R = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, row16 = lane & 15, quad = lane >> 4;
    const int64_t j = static_cast<int64_t>(blockIdx.x) * 16 + row16;
    const int64_t jr = j < len ? j : len - 1;
    const int c = 16 * R + row16, cr = c < l ? c : l - 1;
    double a[4 * CB];
    float b[4 * CB];
#pragma unroll
    for (int q = 0; q < 4 * CB; ++q) {
        const int p = 4 * q + quad, pr = p < l ? p : l - 1;
        if (q / 4 <= R) {
            b[q] = src[static_cast<int64_t>(pr) * len + jr];
            a[q] = linv[cr * l + pr];
        }
    }
    v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 4 * CB; ++q) {
        if (q / 4 > R) continue;
        const int p = 4 * q + quad;
        const bool in = p <= c && c < l;                              // (nothing is stored above the diagonal)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? a[q] : 0.0, p < l ? static_cast<double>(b[q]) : 0.0, acc, 0, 0, 0);
    }
    __syncthreads();                                                  // dst may be src
    float o[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int cc = quad + 4 * v;
        const bool in = 16 * R + cc < l && j < len;
        o[v] = in ? static_cast<float>(acc[v]) : 0.0f;
        if (in && whole) dst[static_cast<int64_t>(16 * R + cc) * len + j] = o[v];
    }
    // Elements j and j + 1 share a word: of each two vectors, the lane of the even one writes the first, the odd one the second.
    const bool odd = row16 & 1;
    const int element = static_cast<int>(blockIdx.x & 1) * 16 + row16;                   // of the block of 32
    uint32_t* const block = packed + (static_cast<int64_t>(blockIdx.x >> 1) * CB + R) * (kParts * 256);
#pragma unroll
    for (int pair = 0; pair < 2; ++pair) {
        const float other = __shfl_xor(odd ? o[2 * pair] : o[2 * pair + 1], 1, 64);
        float lo = odd ? other : o[2 * pair], hi = odd ? o[2 * pair + 1] : other;
        const int cc = quad + 4 * (2 * pair + (odd ? 1 : 0));
#pragma unroll
        for (int k = 0; k < kParts; ++k) {
            typedef float v2f __attribute__((ext_vector_type(2)));
            typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
            const uint32_t word = __builtin_bit_cast(uint32_t, __builtin_convertvector(v2f{lo, hi}, v2bf));
            block[k * 256 + (cc + 16 * (element >> 3)) * 4 + ((element & 7) >> 1)] = word;
            lo -= __uint_as_float(word << 16);
            hi -= __uint_as_float(word & 0xffff0000u);
        }
    }
}

// H[a][b] = sum_i Y[a][i] Y[b][i] in fp64.  A workgroup forms a block of 4 x 4 sums, so that a row is read l / 4
// times and not l times, with the next operands in flight (6.2 us at 72 x 4096, 9.7 without; 5.9 with the first two exchanges of the reduction within four lanes, not through LDS); grid (l / 4, l / 4), the upper half leaves, the lower one
// writes both.  CLEARS: *wide <- 0, for the launch that follows.
template <bool CLEARS>
__global__ void __launch_bounds__(kThreads)
gram_kernel(const float* __restrict__ y, int l, int64_t m, double* __restrict__ h, int* wide)
{
    __shared__ double s_red[kThreads / 64][16];
    if (blockIdx.y > blockIdx.x) return;
    if (CLEARS && blockIdx.x == 0 && threadIdx.x == 0) *wide = 0;
    const float* const ya = y + static_cast<int64_t>(4 * blockIdx.x) * m;
    const float* const yb = y + static_cast<int64_t>(4 * blockIdx.y) * m;
    double d[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) d[q] = 0.0;
    v4f p[4], q[4], p2[4], q2[4];
    auto fetch = [&](int64_t i, v4f (&pf)[4], v4f (&qf)[4]) {
        const int64_t ii = i < m ? i : 0;                             // m is a multiple of 4
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            pf[k] = *reinterpret_cast<const v4f*>(ya + k * m + ii);
            qf[k] = *reinterpret_cast<const v4f*>(yb + k * m + ii);
        }
    };
    auto add = [&](const v4f (&pf)[4], const v4f (&qf)[4]) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int ka = 0; ka < 4; ++ka)
#pragma unroll
                for (int kb = 0; kb < 4; ++kb)
                    d[4 * ka + kb] = fma(static_cast<double>(pf[ka][u]), static_cast<double>(qf[kb][u]), d[4 * ka + kb]);
    };
    int64_t i = 4 * threadIdx.x;
    fetch(i, p, q);
    for (; i < m; i += 8 * kThreads) {
        fetch(i + 4 * kThreads, p2, q2);
        __builtin_amdgcn_sched_barrier(0);
        add(p, q);
        if (i + 4 * kThreads >= m) break;
        fetch(i + 8 * kThreads, p, q);
        __builtin_amdgcn_sched_barrier(0);
        add(p2, q2);
    }
    // sixteen sums over a wave: each of four exchanges adds two halves and leaves half as many sums per lane
    const int lane = threadIdx.x & 63;
    auto exchange = [&](auto step_tag) {
        constexpr int step = decltype(step_tag)::value, half = 8 >> step;
        const bool upper = (lane >> step) & 1;
#pragma unroll
        for (int q = 0; q < half; ++q) {
            const double keep = upper ? d[q + half] : d[q], give = upper ? d[q] : d[q + half];
            if constexpr (step < 2) {                                 // within four lanes without LDS
                constexpr int CTRL = step == 0 ? 0xB1 : 0x4E;         // quad_perm [1, 0, 3, 2], [2, 3, 0, 1]
                d[q] = keep + __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(give), CTRL, 0xf, 0xf, true),
                                               __builtin_amdgcn_mov_dpp(__double2loint(give), CTRL, 0xf, 0xf, true));
            } else {
                d[q] = keep + __shfl_xor(give, 1 << step, 64);
            }
        }
    };
    for_each<0, 4>(exchange);
    double s = d[0] + __shfl_xor(d[0], 16, 64);
    s += __shfl_xor(s, 32, 64);
    // lane bits 0 .. 3 are bits 3 .. 0 of the sum's index
    if (lane < 16) s_red[threadIdx.x >> 6][(lane & 1) * 8 + (lane & 2) * 2 + (lane & 4) / 2 + (lane & 8) / 8] = s;
    __syncthreads();
    if (threadIdx.x < 16) {
        const int a = 4 * blockIdx.x + (threadIdx.x >> 2), b = 4 * blockIdx.y + (threadIdx.x & 3);
        double t = 0.0;
        for (int w = 0; w < kThreads / 64; ++w) t += s_red[w][threadIdx.x];
        if (a >= b) h[static_cast<int64_t>(a) * l + b] = h[static_cast<int64_t>(b) * l + a] = t;
    }
}

// the sum over each four lanes, the same in all of them
__device__ __forceinline__ double quad_sum(double v)
{
    auto swapped = [](double x, auto ctrl) {
        constexpr int C = decltype(ctrl)::value;
        return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(x), C, 0xf, 0xf, true),
                                __builtin_amdgcn_mov_dpp(__double2loint(x), C, 0xf, 0xf, true));
    };
    v += swapped(v, std::integral_constant<int, 0xB1>{});             // quad_perm [1, 0, 3, 2]
    return v + swapped(v, std::integral_constant<int, 0x4E>{});       // quad_perm [2, 3, 0, 1]
}

// Eigen-decomposition H = P diag(lambda) P^T of a symmetric positive semidefinite H = L L^T (l x l, fp64) by one-sided
// Jacobi: rotations of the columns of L^T that make them orthogonal.  Their dot products are the entries of H, so the
// rotations are those of the two-sided method on H in the same order, and P is their product; but all that is kept is
// W = L^T P, whose columns have lengths lambda^(1/2) and give P back as L W diag(1/lambda) (eigenvector_kernel, settle_kernel).
// Round-robin ordering, a round rotates l/2 disjoint pairs of columns, each pair in four lanes: the dot product of the two is
// reduced within the lanes, every lane forms the rotation, and both columns go back to LDS; one barrier per round.  Their squared
// lengths follow from the rotation, to 1e-12 of each, and are formed anew once per sweep and where little of one is left: with three dot products
// and a tangent to full precision per pair the launch took 577 us at l = 72, 562 now (flat spectrum, nine sweeps).
// A round is bound by the columns' way through LDS (writes at 76 B/clk) and the instructions that a SIMD issues, and those of
// the rotation count once per wave: four lanes per pair make l / 32 waves, one per SIMD.  (Columns that stay in registers and
// move on by a lane per round, their edges through LDS, took 1.06 us a round at l = 72 against 0.95: a b128 access of four lanes costs
// what one of 64 does.)  (With 16 lanes per pair and up to three waves per SIMD a round took
// 1.17 us at l = 72; rotating H from both sides, which takes a pass over all of H, the eigenvectors' update and two
// barriers per round, 1.4 us.)
// Stops after `sweeps`, or after the first sweep that found all columns orthogonal to 1e-8 and turned none by more than
// 1e-8 radians: what such a sweep leaves is of second order, for a short column beside a long one too (these turn by little
// however far from orthogonal they are, and what a short one keeps of a long one enters P with the ratio of the lengths).
// Not counted are rotations of columns that are orthogonal to 1e-14, the rounding level of the products.  Nine sweeps for
// a flat spectrum; 17 to 24 for one that spans the whole range of fp64 before the basis has seen E (no iterations), where
// 14 left cosines of up to 0.8 and a factor that was wrong altogether.
// On exit w[i][.] the columns of W, lambda[i] their squared lengths.
template <int L8>                                                      // l / 8: 16-byte parts of a column per lane
__global__ void __launch_bounds__(256)
jacobi_eig_kernel(const double* __restrict__ lt, double* __restrict__ w, double* __restrict__ lambda, int sweeps)
{
    typedef double v2d __attribute__((ext_vector_type(2)));
    // columns at an odd multiple of 64 bytes: the sixteen pairs of a wave spread over all banks
    constexpr int l = 8 * L8, PITCH = 8 * (L8 | 1);
    extern __shared__ __attribute__((aligned(16))) double s_v[];      // [l][PITCH], squared lengths, two flags
    JacobiLength* const s_length = reinterpret_cast<JacobiLength*>(s_v + l * PITCH);
    int* const s_turned = reinterpret_cast<int*>(s_length + l);
    const int t = threadIdx.x, pair = t >> 2, e0 = 2 * (t & 3);
    const bool live = pair < l / 2;
    for (int q = t; q < l * l; q += blockDim.x) {
        const int i = q / l, c = q % l;
        s_v[c * PITCH + i] = i <= c ? lt[i * l + c] : 0.0;
    }
    if (t < 2) s_turned[t] = 0;
    __syncthreads();
    // position 0 keeps column 0, positions 1 .. l-1 rotate by one per round
    auto at = [&](int pos, int round) { return pos == 0 ? 0 : (pos - 1 >= round ? pos - round : pos - round + l - 1); };
    auto square = [&](const v2d (&v)[L8]) {
        v2d s = {0.0, 0.0};
#pragma unroll
        for (int e = 0; e < L8; ++e)
#pragma unroll
            for (int u = 0; u < 2; ++u) s[u] = fma(v[e][u], v[e][u], s[u]);
        return quad_sum(s[0] + s[1]);
    };
    for (int sweep = 0; sweep < sweeps; ++sweep) {
        for (int c = pair; c < l; c += static_cast<int>(blockDim.x >> 2)) {
            v2d v[L8];
#pragma unroll
            for (int e = 0; e < L8; ++e) v[e] = *reinterpret_cast<const v2d*>(s_v + c * PITCH + e0 + 8 * e);
            const double length = square(v);
            s_length[c] = JacobiLength{length, length};
        }
        __syncthreads();
        for (int round = 0; round < l - 1; ++round) {
            if (round == l - 2 && t == 0) s_turned[(sweep + 1) & 1] = 0;
            if (live) {
                const int ca = at(pair, round), cb = at(l - 1 - pair, round);
                v2d* const pa = reinterpret_cast<v2d*>(s_v + ca * PITCH + e0);
                v2d* const pb = reinterpret_cast<v2d*>(s_v + cb * PITCH + e0);
                v2d va[L8], vb[L8], ab = {0.0, 0.0};
#pragma unroll
                for (int e = 0; e < L8; ++e) { va[e] = pa[4 * e]; vb[e] = pb[4 * e]; }
                JacobiLength la = s_length[ca], lb = s_length[cb];
#pragma unroll
                for (int e = 0; e < L8; ++e)
#pragma unroll
                    for (int u = 0; u < 2; ++u) ab[u] = fma(va[e][u], vb[e][u], ab[u]);
                const double haa = la.now, hbb = lb.now, hab = quad_sum(ab[0] + ab[1]);
                double c, s, tn;
                if (jacobi_rotation(haa, hbb, hab, c, s, tn)) {
#pragma unroll
                    for (int e = 0; e < L8; ++e) {
                        v2d na, nb;
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            na[u] = fma(c, va[e][u], -s * vb[e][u]);
                            nb[u] = fma(s, va[e][u], c * vb[e][u]);
                        }
                        pa[4 * e] = va[e] = na;
                        pb[4 * e] = vb[e] = nb;
                    }
                    if (!jacobi_follow(c, tn, hab, la, lb)) {
                        la.now = la.carried = square(va);
                        lb.now = lb.carried = square(vb);
                    }
                    s_length[ca] = la;
                    s_length[cb] = lb;
                    // (one comparison: orthogonal to 1e-14 where they turn by more than 1e-8, to 1e-8 where not)
                    if (hab * hab > (fabs(s) > 1e-8 ? 1e-28 : 1e-16) * haa * hbb) s_turned[sweep & 1] = 1;
                }
            }
            __syncthreads();
        }
        if (s_turned[sweep & 1] == 0) break;                          // (same value in every lane)
    }
    for (int i = pair; i < l; i += blockDim.x >> 2) {
        double s = 0.0;
#pragma unroll
        for (int e = 0; e < L8; ++e) {
            const v2d v = *reinterpret_cast<const v2d*>(s_v + i * PITCH + e0 + 8 * e);
            *reinterpret_cast<v2d*>(w + i * l + e0 + 8 * e) = v;
            s = fma(v[0], v[0], fma(v[1], v[1], s));
        }
        s = quad_sum(s);
        if ((t & 3) == 0) lambda[i] = s;
    }
}

// the sums of a and b over the workgroup's kMaxL threads, in all of them
__device__ __forceinline__ void sums_over_all(double& a, double& b, double (&smem)[2][kMaxL / 64])
{
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_xor(a, off, 64);
        b += __shfl_xor(b, off, 64);
    }
    if ((threadIdx.x & 63) == 0) { smem[0][threadIdx.x >> 6] = a; smem[1][threadIdx.x >> 6] = b; }
    __syncthreads();
    a = b = 0.0;
    for (int v = 0; v < kMaxL / 64; ++v) { a += smem[0][v]; b += smem[1][v]; }
}

// p[k][.] <- P's column k, L w_k at length 1, for each k a workgroup.  (Its length is lambda_k, which for a null column
// can be anything down to zero.)
__global__ void __launch_bounds__(kMaxL)
eigenvector_kernel(const double* __restrict__ lt, int l, const double* __restrict__ w, double* __restrict__ p)
{
    __shared__ double s_sum[2][kMaxL / 64];
    const int k = blockIdx.x, i = threadIdx.x, column = i < l ? i : l - 1;
    double a = 0.0;
    for (int e0 = 0; e0 < l; e0 += 8) {                               // l is a multiple of 8: eight loads in flight
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = lt[(e0 + u) * l + column];
#pragma unroll
        for (int u = 0; u < 8; ++u) a = fma(e0 + u <= i ? x[u] : 0.0, w[k * l + e0 + u], a);   // (nothing below the diagonal)
    }
    if (i >= l) a = 0.0;
    double square = a * a, unused = 0.0;
    sums_over_all(square, unused, s_sum);
    if (i < l) p[k * l + i] = square > 0.0 && square < HUGE_VAL ? a / sqrt(square) : 0.0;
}

// L w_k carries the rounding of w_k times the ratio of the largest length to its own: of eigenvalues near the
// rounding of H, p_k keeps parts of the vectors of larger ones, which the products with E bring up again.  Here these
// parts are taken out, the vector is brought to length 1, and its eigenvalue becomes |L^T q|^2, so that values, vectors
// and both factors agree whatever their size.  A vector of which nothing is left is null.
// (This launch and the one before it take 9.8 and 6.1 us at l = 72; with P at hand the rotation of the basis takes 10.7 us,
// 28.6 when each of its workgroups formed its vector.)
__global__ void __launch_bounds__(kMaxL)
settle_kernel(const double* __restrict__ lt, int l, const double* __restrict__ p, const double* __restrict__ lambda,
              double* __restrict__ q, double* __restrict__ settled)
{
    __shared__ double s_p[kMaxL], s_dot[kMaxL], s_sum[2][2][kMaxL / 64];
    const int k = blockIdx.x, i = threadIdx.x, column = i < l ? i : l - 1;
    const double own = i < l ? p[k * l + i] : 0.0;
    s_p[i] = own;
    __syncthreads();
    double dot = 0.0;
    const bool larger = i < l && lambda[i] > lambda[k];
    if (larger)
        for (int c0 = 0; c0 < l; c0 += 8) {
            double x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = p[i * l + c0 + u];
#pragma unroll
            for (int u = 0; u < 8; ++u) dot = fma(x[u], s_p[c0 + u], dot);
        }
    s_dot[i] = dot;
    __syncthreads();
    double rest = own;
    for (int c0 = 0; c0 < l; c0 += 8) {
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = p[(c0 + u) * l + column];
#pragma unroll
        for (int u = 0; u < 8; ++u) rest = fma(-s_dot[c0 + u], x[u], rest);
    }
    if (i >= l) rest = 0.0;
    double before = own * own, after = rest * rest;
    sums_over_all(before, after, s_sum[0]);
    const bool live = after > 1e-4 * before;                          // (not for a NaN)
    rest = live ? rest / sqrt(after) : 0.0;
    s_p[i] = rest;                                                    // (all have read it: two barriers ago)
    __syncthreads();
    double t = 0.0, unused = 0.0;
    for (int c0 = 0; c0 < l; c0 += 8) {
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = lt[column * l + c0 + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) t = fma(c0 + u >= i ? x[u] : 0.0, s_p[c0 + u], t);
    }
    t = i < l ? t * t : 0.0;
    sums_over_all(t, unused, s_sum[1]);
    if (i < l) q[k * l + i] = rest;
    if (i == 0) settled[k] = live && t < HUGE_VAL ? t : 0.0;
}

// A^[k][j] = lambda_k^(1/4) * sum_c P[c][k] Z[c][j], sigma[k] = sqrt(lambda_k), for the k-th largest eigenvalue (equal
// ones by smaller index); p[i][.]: P's column i
__global__ void __launch_bounds__(kThreads)
rotate_kernel(const float* __restrict__ z, int l, int64_t n, const double* __restrict__ p,
              const double* __restrict__ lambda, float* __restrict__ a_out, float* __restrict__ sigma_out, int inverse_scale)
{
    __shared__ double s_p[kMaxL], s_lam[kMaxL];
    __shared__ int s_col;
    const int k = blockIdx.y, t = threadIdx.x;
    if (t < l) s_lam[t] = lambda[t];                                  // (none is a NaN)
    __syncthreads();
    if (t < l) {
        int rank = 0;
        for (int j = 0; j < l; ++j) rank += (s_lam[j] > s_lam[t] || (s_lam[j] == s_lam[t] && j < t)) ? 1 : 0;
        if (rank == k) s_col = t;
    }
    __syncthreads();
    const int col = s_col;
    if (t < l) s_p[t] = p[col * l + t];
    __syncthreads();
    const double lam = s_lam[col];
    // right factor: z holds unit vectors, row k becomes sqrt(sigma_k) v_k.  Left factor (inverse_scale):
    // z holds E v (length sigma_k u_k after the rotation), row k becomes sqrt(sigma_k) u_k.
    const double root = sqrt(sqrt(lam));
    const double scale = inverse_scale ? (root > 0.0 ? 1.0 / root : 0.0) : root;
    const int64_t j = static_cast<int64_t>(blockIdx.x) * kThreads + t;
    if (j < n) {
        double acc = 0.0;
        for (int c = 0; c < l; ++c) acc += s_p[c] * static_cast<double>(z[static_cast<int64_t>(c) * n + j]);
        a_out[static_cast<int64_t>(k) * n + j] = static_cast<float>(scale * acc);
    }
    if (blockIdx.x == 0 && t == 0 && sigma_out) sigma_out[k] = static_cast<float>(sqrt(lam));
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
    // partial sums of the products and the packed vectors: together no more than the 16 slices of partial sums that
    // a workspace has had room for (the packed vectors take less than four slices for l >= 24 and max(m, n) >= 32)
    const size_t longest = static_cast<size_t>(m > n ? m : n), room = sizeof(float) * 16 * l * longest;
    L.part = off;
    L.packed = off + sizeof(float) * kMaxSlices * l * longest;
    off = up(off + room);
    L.wide = off - 256;                                                   // (behind the packed vectors: they leave at least 1.5 KB)
    L.total = off;
    return L;
}

// FQ_BY_BLOCKS(count, F): F<count>() with the number of 16-vector blocks as a constant
#define FQ_BY_BLOCKS(count, F)                                                                              \
    switch (count) {                                                                                        \
        case 2: F(2); break; case 3: F(3); break; case 4: F(4); break; case 5: F(5); break;                 \
        case 6: F(6); break; case 7: F(7); break; default: F(8); break;                                     \
    }

// rows of dst[l][len] <- orthonormal basis of the rows of src (Cholesky QR, `passes` times), and the same packed for
// the products; dst may be src, and is written only if *asked where that is given (one pass then); h and lfac are l x l fp64
// scratch; range: what is looked at beside the first factor
static hipError_t orthonormalize_rows(const float* src, float* dst, uint32_t* packed, int l, int64_t len, double* h,
                                      double* lfac, int passes, hipStream_t stream, const int* asked = nullptr,
                                      RangeOf range = {nullptr, 0, nullptr})
{
    const int nb = l / 4;
    const unsigned blocks = static_cast<unsigned>((len + 31) / 32 * 2);
    for (int pass = 0; pass < passes; ++pass) {
        const float* const v = pass ? dst : src;
        const bool looks = range.wide && !pass;
        const unsigned lookers = looks ? 1020 : 0;
        if (looks) gram_kernel<true><<<dim3(nb, nb), kThreads, 0, stream>>>(v, l, len, h, range.wide);
        else gram_kernel<false><<<dim3(nb, nb), kThreads, 0, stream>>>(v, l, len, h, nullptr);
#define FQ_APPLY(CB)                                                                                         \
        factor_kernel<CB, false><<<1 + lookers, 64 * factor_waves(CB), 0, stream>>>(h, l, lfac, range);      \
        apply_lower_kernel<CB><<<blocks, CB * 64, 0, stream>>>(v, dst, packed, l, len, lfac, asked)
        FQ_BY_BLOCKS((l + 15) / 16, FQ_APPLY)
#undef FQ_APPLY
        const hipError_t err = hipGetLastError();
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
    float* part = reinterpret_cast<float*>(ws + L.part);
    uint32_t* packed = reinterpret_cast<uint32_t*>(ws + L.packed);
    int* wide = reinterpret_cast<int*>(ws + L.wide);
    // Y[l][m] = Z E^T (transposed == false) or Z[l][n] = Y E: slices of the contracted dimension so that about 256
    // workgroups stream E, each with at least one step per wave, then the ordered sum
    auto product = [&](bool transposed, float* out) -> hipError_t {
        const int64_t rows = transposed ? n : m, depth = transposed ? m : n;
        const int64_t blocks = (rows + 63) / 64, steps = (depth + 31) / 32;
        int64_t slices = 256 / blocks;
        if (slices > kMaxSlices) slices = kMaxSlices;
        if (slices > (steps + 3) / 4) slices = (steps + 3) / 4;
        if (slices < 1) slices = 1;
        const int64_t per = (steps + slices - 1) / slices;
        slices = (steps + per - 1) / per;
        const int vector_blocks = (l + 15) / 16, halves = vector_blocks == 8 ? 2 : 1;
        const dim3 grid(static_cast<unsigned>(blocks), static_cast<unsigned>(slices), static_cast<unsigned>(halves));
        float* dst = slices > 1 ? part : out;
        const v8bf* const vectors = reinterpret_cast<const v8bf*>(packed);
#define FQ_PRODUCT(CB)                                                                                       \
        if (transposed) apply_et_kernel<CB><<<grid, kThreads, 0, stream>>>(e, m, n, vectors, y, l, wide, dst, per); \
        else apply_e_kernel<CB><<<grid, kThreads, 0, stream>>>(e, m, n, vectors, z, l, wide, dst, per)
        switch (vector_blocks / halves) {
            case 2: FQ_PRODUCT(2); break; case 3: FQ_PRODUCT(3); break; case 4: FQ_PRODUCT(4); break;
            case 5: FQ_PRODUCT(5); break; case 6: FQ_PRODUCT(6); break; default: FQ_PRODUCT(7); break;
        }
#undef FQ_PRODUCT
        hipError_t pe = hipGetLastError();
        if (pe != hipSuccess || slices == 1) return pe;
        const int64_t count = static_cast<int64_t>(l) * rows;          // a multiple of 4 (m and n are)
        sum_slices_kernel<<<static_cast<unsigned>((count / 4 + kThreads - 1) / kThreads), kThreads, 0, stream>>>(
            part, static_cast<int>(slices), count, out);
        return hipGetLastError();
    };
    hipError_t err;
#define FQ_CHECK(expr) do { err = (expr); if (err != hipSuccess) return err; } while (0)
    FQ_CHECK(orthonormalize_rows(omega, z, packed, l, n, h, p, iters ? 1 : 2, stream, nullptr, RangeOf{e, m * n, wide}));
    for (int it = 0; it < iters; ++it) {
        FQ_CHECK(product(false, y));
        FQ_CHECK(orthonormalize_rows(y, y, packed, l, m, h, p, 1, stream, wide));
        FQ_CHECK(product(true, z));
        FQ_CHECK(orthonormalize_rows(z, z, packed, l, n, h, p, it == iters - 1 ? 2 : 1, stream));
    }
    FQ_CHECK(product(false, y));
    const int nb = l / 4;
    gram_kernel<false><<<dim3(nb, nb), kThreads, 0, stream>>>(y, l, m, h, nullptr);
#define FQ_FACTOR(CB) factor_kernel<CB, true><<<1, 64 * factor_waves(CB), 0, stream>>>(h, l, p, RangeOf{nullptr, 0, nullptr})
    FQ_BY_BLOCKS((l + 15) / 16, FQ_FACTOR)
#undef FQ_FACTOR
    FQ_CHECK(hipGetLastError());
#define FQ_JACOBI(L8)                                                                                        \
    case L8: {                                                                                               \
        const size_t lds = sizeof(double) * 8 * L8 * (8 * (L8 | 1) + 2) + 2 * sizeof(int);                   \
        FQ_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(&jacobi_eig_kernel<L8>),                  \
                                     hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));    \
        jacobi_eig_kernel<L8><<<1, (16 * L8 + 63) / 64 * 64, lds, stream>>>(p, h, lambda, 48);        \
        break;                                                                                               \
    }
    switch (l / 8) {
        FQ_JACOBI(3) FQ_JACOBI(4) FQ_JACOBI(5) FQ_JACOBI(6) FQ_JACOBI(7) FQ_JACOBI(8) FQ_JACOBI(9) FQ_JACOBI(10)
        FQ_JACOBI(11) FQ_JACOBI(12) FQ_JACOBI(13) FQ_JACOBI(14) FQ_JACOBI(15) FQ_JACOBI(16)
        default: return hipErrorInvalidValue;
    }
#undef FQ_JACOBI
    FQ_CHECK(hipGetLastError());
    // the products' partial sums are no longer needed: their room holds the vectors before they are settled
    double* const vectors = reinterpret_cast<double*>(part);
    double* const settled = vectors + l * l;
    eigenvector_kernel<<<l, kMaxL, 0, stream>>>(p, l, h, vectors);
    FQ_CHECK(hipGetLastError());
    settle_kernel<<<l, kMaxL, 0, stream>>>(p, l, vectors, lambda, h, settled);
    FQ_CHECK(hipGetLastError());
    rotate_kernel<<<dim3(static_cast<unsigned>((n + kThreads - 1) / kThreads), static_cast<unsigned>(r)), kThreads, 0,
                    stream>>>(z, l, n, h, settled, a_out, sigma_out, 0);
    FQ_CHECK(hipGetLastError());
    if (bt_out) {
        // y still holds E z^T: its rotation by the same eigenvectors is sigma_k u_k, the left singular vectors
        rotate_kernel<<<dim3(static_cast<unsigned>((m + kThreads - 1) / kThreads), static_cast<unsigned>(r)), kThreads, 0,
                        stream>>>(y, l, m, h, settled, bt_out, nullptr, 1);
        FQ_CHECK(hipGetLastError());
    }
#undef FQ_CHECK
    return hipSuccess;
}

}  // namespace falqon
