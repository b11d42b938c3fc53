// Per-tensor FP8 quantizer Q_fp8 for gfx950: absolute-maximum reduction, then scale and cast.
//
// Follows the quantization equation of the paper's "Low-precision floating-point
// quantization" section, read as s = max(FP8) / max|X| (the scale multiplies up to the
// format's range; the rescale of the FP8 product divides by it).
//
// Both passes stream the tensor with 16-byte accesses per lane.  The reduction leaves one
// partial maximum per workgroup; the cast pass folds them itself, so there is no atomic,
// no counter to clear and no host round trip between the passes.  The tensor (tens of MB)
// stays in the 256 MB last-level cache between the passes, so HBM sees about one read.
#include <type_traits>

#include "falqon_internal.h"
#include "gemm_common.h"
#include "quantize_common.h"

namespace falqon {
namespace {

constexpr int kThreads = 256;
constexpr int kVec = 16;          // elements per lane per step

// Piece v of a [rows, cols] tensor: its row and its place there.  kDense: no gaps between rows, all is one row (an
// instance of its own: a division's code between the loads costs a launch 0.3 us before it ever runs).  kRows: fewer
// than 2^32 pieces; with floor(2^32 / per_row) the product's upper half is the quotient or one less.  kFarRows: more
// (with a 64-bit division per piece 250 KB of fp32 took 7.6 us, 5.5 now).
enum { kDense, kRows, kFarRows };
struct RowSplit { int64_t per_row; uint32_t inverse; };
struct Place { int64_t row, piece; };

template <int ROWS>
__device__ __forceinline__ Place place_of(int64_t v, RowSplit s)
{
    if (ROWS == kDense) return {0, v};
    if (ROWS == kFarRows) {
        const int64_t row = v / s.per_row;
        return {row, v - row * s.per_row};
    }
    const uint32_t u = static_cast<uint32_t>(v), d = static_cast<uint32_t>(s.per_row);
    uint32_t row = __umulhi(u, s.inverse), piece = u - row * d;
    if (piece >= d) { ++row; piece -= d; }
    return {row, piece};
}

// Both passes go over the tensor in blocks of kBlock pieces per workgroup, block b by a workgroup of index b modulo
// 8, so by the same XCD: what its L2 still holds from the first pass need not be fetched again.
constexpr int kAtOnce = 4, kBlock = kThreads * kAtOnce;    // pieces in flight per thread

template <typename T, int ROWS>
__global__ void __launch_bounds__(kThreads)
amax_partial_kernel(const T* __restrict__ x, int64_t n_pieces, const RowSplit split, int64_t ld_x, float* __restrict__ partials)
{
    __shared__ float smem[kThreads / 64];
    float m = 0.0f;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    for (int64_t v0 = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; v0 < n_pieces; v0 += stride) {
        v4u w[kAtOnce];
#pragma unroll
        for (int b = 0; b < kAtOnce; ++b) {
            const int64_t v = v0 + b * kThreads < n_pieces ? v0 + b * kThreads : v0;   // beyond the end: one it has already
            const Place p = place_of<ROWS>(v, split);
            w[b] = *reinterpret_cast<const v4u*>(x + p.row * ld_x + p.piece * Piece<T>::E);
        }
#pragma unroll
        for (int b = 0; b < kAtOnce; ++b) m = abs_max<T>(w[b], m);
    }
    m = block_max<kThreads / 64>(m, smem);
    if (threadIdx.x == 0) partials[blockIdx.x] = m;
}

// The small bf16 tensor that the last workgroups of a cast pass cast to E4M3 (the saved O_A of the layer, for the
// adapter gradient), its maximum known: s = 448 / max(amax, 1e-12f), one fp32 multiply, then the cast.  It rides so that
// no launch, and no reduction pass, exists for it alone.
__device__ __forceinline__ void cast_side(const SideCast& side, int64_t first, int64_t stride)
{
    const float s = 448.0f / fmaxf(*side.amax, 1e-12f);
    for (int64_t v = first; v < side.count / 8; v += stride)
        *reinterpret_cast<Piece<uint16_t>::codes_t*>(side.q + v * 8) =
            cast_piece<uint16_t, FALQON_E4M3>(*reinterpret_cast<const v4u*>(side.x + v * 8), s);
}

// The tensor is read for the last time: non-temporal loads.  PAST: the codes go past the caches too.
// The first pieces are requested before the partial maxima are reduced.
// Both passes, us, against 32 contiguous bytes per lane, no prefetch and ordinary accesses (bf16, back to back, other
// tensors in turn): 4 MB 5.2 (5.8), 16 MB 9.0 (10.1), 33 MB 12.6 (15.6), 90 MB 34.6 (37.1), 226 MB 83 (102).
template <typename T, int FMT, int ROWS, bool PAST>
__global__ void __launch_bounds__(kThreads)
scale_cast_kernel(const T* __restrict__ x, int64_t n_pieces, const RowSplit split, int64_t ld_x,
                  const float* __restrict__ partials, int n_partials, const float* __restrict__ scale_in,
                  uint8_t* __restrict__ q, int64_t ld_q, float* __restrict__ scale_out,
                  float* __restrict__ amax_out, const ZeroWords zero, const SideCast side, int side_blocks)
{
    __shared__ float smem[kThreads / 64];
    constexpr int E = Piece<T>::E;
    typedef typename Piece<T>::codes_t codes_t;
    const int main_blocks = static_cast<int>(gridDim.x) - side_blocks;
    if (static_cast<int>(blockIdx.x) >= main_blocks) {
        cast_side(side, (static_cast<int64_t>(blockIdx.x) - main_blocks) * kThreads + threadIdx.x,
                  static_cast<int64_t>(side_blocks) * kThreads);
        return;
    }
    const int64_t stride = static_cast<int64_t>(main_blocks) * kBlock;
    int64_t v0 = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    v4u w[kAtOnce];
    int64_t to[kAtOnce];                                             // where the codes go
    auto fetch = [&]() {
#pragma unroll
        for (int b = 0; b < kAtOnce; ++b) {
            const Place p = place_of<ROWS>(v0 + b * kThreads < n_pieces ? v0 + b * kThreads : 0, split);
            to[b] = p.row * ld_q + p.piece * E;
            w[b] = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(x + p.row * ld_x + p.piece * E));
        }
    };
    if (n_pieces > 0) fetch();
    __builtin_amdgcn_sched_barrier(0);
    float m = 0.0f;
    for (int i = threadIdx.x; i < n_partials; i += kThreads) m = fmaxf(m, partials[i]);
    const float amax = block_max<kThreads / 64>(m, smem);
    constexpr float mx = FMT == FALQON_E4M3 ? 448.0f : 57344.0f;
    // IEEE fp32 division (hipcc's default for '/' is the correctly rounded one)
    const float s = scale_in ? *scale_in : mx / fmaxf(amax, 1e-12f);
    while (v0 < n_pieces) {
#pragma unroll
        for (int b = 0; b < kAtOnce; ++b)
            if (v0 + b * kThreads < n_pieces) {
                codes_t* const dst = reinterpret_cast<codes_t*>(q + to[b]);
                if constexpr (PAST) __builtin_nontemporal_store(cast_piece<T, FMT>(w[b], s), dst);
                else *dst = cast_piece<T, FMT>(w[b], s);
            }
        v0 += stride;
        if (v0 < n_pieces) fetch();
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *scale_out = s;
        if (amax_out) *amax_out = amax;
    }
    if (blockIdx.x == 0 && static_cast<int>(threadIdx.x) < zero.count) zero.words[threadIdx.x] = 0u;
}

// Both passes in one launch for small tensors: every workgroup takes the maximum of the whole tensor itself
// (it is order free, so all of them and the two-launch form agree to the bit) and casts its share, one vector
// per thread.  The last side_blocks workgroups cast the side tensor.  Bound by reading the tensor through one CU, so the
// limit is where the device takes as long as for two launches; the host saves one at any size.  us on the device, one
// launch (two): 256 KB bf16 4.9 (5.0), fp32 4.5 (4.9).  Without a maximum the other form is one launch too, of more
// workgroups: 160 KB fp32 3.0 us here, 2.7 there, the same up to 16 KB.
constexpr int kOneThreads = 1024;
constexpr int64_t kOneLaunchBytes = 256 * 1024, kOneLaunchGivenBytes = 16 * 1024;

template <typename T, int FMT, int ROWS>
__global__ void __launch_bounds__(kOneThreads)
quantize_one_kernel(const T* __restrict__ x, int n_pieces, const RowSplit split, int64_t ld_x,
                    const float* __restrict__ scale_in, uint8_t* __restrict__ q, int64_t ld_q, float* __restrict__ scale_out,
                    float* __restrict__ amax_out, const ZeroWords zero, const SideCast side, int side_blocks)
{
    __shared__ float smem[kOneThreads / 64];
    constexpr int E = Piece<T>::E, SHARE = kVec / E;                 // pieces of its share per thread
    typedef typename Piece<T>::codes_t codes_t;
    const int main_blocks = static_cast<int>(gridDim.x) - side_blocks;
    if (static_cast<int>(blockIdx.x) >= main_blocks) {
        cast_side(side, (static_cast<int64_t>(blockIdx.x) - main_blocks) * kOneThreads + threadIdx.x,
                  static_cast<int64_t>(side_blocks) * kOneThreads);
        return;
    }
    float m = 0.0f;
    // B pieces in flight per thread, up to 128 KB per workgroup; no more than there are left (pieces that are not there cost
    // as much as others: 141 KB 5.1 us with eight for the last 852, 4.3 with one)
    int begin = 0;
    auto batch = [&](auto at_once) {
        constexpr int B = decltype(at_once)::value;
        v4u w[B];
        const int v0 = begin + static_cast<int>(threadIdx.x);
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int v = v0 + b * kOneThreads;
            const Place p = place_of<ROWS>(v < n_pieces ? v : n_pieces - 1, split);      // beyond the end: the last one
            w[b] = *reinterpret_cast<const v4u*>(x + p.row * ld_x + p.piece * E);
        }
#pragma unroll
        for (int b = 0; b < B; ++b) m = abs_max<T>(w[b], m);
        begin += B * kOneThreads;
    };
    if (!scale_in || amax_out) {                                     // (a given scale needs no maximum unless it is asked for)
        while (n_pieces - begin > 4 * kOneThreads) batch(std::integral_constant<int, 8>{});
        if (n_pieces - begin > kOneThreads) batch(std::integral_constant<int, 4>{});
        else if (n_pieces > begin) batch(std::integral_constant<int, 1>{});
    }
    const float amax = block_max<kOneThreads / 64>(m, smem);
    constexpr float mx = FMT == FALQON_E4M3 ? 448.0f : 57344.0f;
    const float s = scale_in ? *scale_in : mx / fmaxf(amax, 1e-12f);
#pragma unroll
    for (int b = 0; b < SHARE; ++b) {
        const int v = (static_cast<int>(blockIdx.x) * SHARE + b) * kOneThreads + static_cast<int>(threadIdx.x);
        if (v < n_pieces) {
            const Place p = place_of<ROWS>(v, split);
            *reinterpret_cast<codes_t*>(q + p.row * ld_q + p.piece * E) =
                cast_piece<T, FMT>(*reinterpret_cast<const v4u*>(x + p.row * ld_x + p.piece * E), s);
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *scale_out = s;
        if (amax_out) *amax_out = amax;
    }
    if (blockIdx.x == 0 && static_cast<int>(threadIdx.x) < zero.count) zero.words[threadIdx.x] = 0u;
}

__global__ void zero_word_kernel(uint32_t* w) { *w = 0u; }

template <typename T>
hipError_t run(const T* x, int64_t rows, int64_t cols, int64_t ld_x, falqon_fmt fmt, const float* scale_in,
               uint8_t* q, int64_t ld_q, float* scale_out, float* amax_out, float* partials,
               ZeroWords zero, const SideCast* side_job, int64_t next_width, hipStream_t stream)
{
    SideCast side{nullptr, nullptr, nullptr, 0};
    if (side_job) side = *side_job;                                  // (count: a multiple of 16)
    constexpr int E = Piece<T>::E;
    const int64_t per_row = cols / E, n_pieces = rows * per_row;     // (per_row is 2 at least)
    const bool near = n_pieces < (int64_t(1) << 32);
    const RowSplit split{per_row, near ? static_cast<uint32_t>((int64_t(1) << 32) / per_row) : 0u};
    const bool dense = rows <= 1 || (ld_x == cols && ld_q == cols);
    const bool wants_max = !scale_in || amax_out;                    // (a given scale needs no maximum unless it is asked for)
    if (n_pieces * 16 <= (wants_max ? kOneLaunchBytes : kOneLaunchGivenBytes) && side.count / kVec <= 64 * kOneThreads) {
        const int64_t n_vecs = n_pieces * E / kVec;
        const int64_t main_blocks = n_vecs > 0 ? (n_vecs + kOneThreads - 1) / kOneThreads : 1;
        const int side_blocks = static_cast<int>((side.count / kVec + kOneThreads - 1) / kOneThreads);
        const dim3 grid(static_cast<unsigned>(main_blocks + side_blocks));
        auto go = [&](auto kernel) {
            kernel<<<grid, kOneThreads, 0, stream>>>(x, static_cast<int>(n_pieces), split, ld_x, scale_in, q, ld_q, scale_out,
                                                     amax_out, zero, side, side_blocks);
        };
        if (fmt == FALQON_E4M3) { if (dense) go(quantize_one_kernel<T, FALQON_E4M3, kDense>); else go(quantize_one_kernel<T, FALQON_E4M3, kRows>); }
        else { if (dense) go(quantize_one_kernel<T, FALQON_E5M2, kDense>); else go(quantize_one_kernel<T, FALQON_E5M2, kRows>); }
        return hipGetLastError();
    }
    // The amax pass wants few, long-running workgroups (one partial each); the cast pass is a plain stream.  Both grids
    // are multiples of 8 where a workgroup has more than one block (see kBlock).
    const int64_t want = (n_pieces + kBlock - 1) / kBlock;
    int n_partials = 0;
    if (wants_max) {
        n_partials = static_cast<int>(want < kMaxAmaxBlocks ? want : kMaxAmaxBlocks);
        auto go = [&](auto kernel) { kernel<<<n_partials, kThreads, 0, stream>>>(x, n_pieces, split, ld_x, partials); };
        if (dense || ld_x == cols) go(amax_partial_kernel<T, kDense>);
        else if (near) go(amax_partial_kernel<T, kRows>);
        else go(amax_partial_kernel<T, kFarRows>);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const int64_t side_want = (side.count / 8 + kThreads - 1) / kThreads;
    const int side_blocks = static_cast<int>(side_want < 64 ? side_want : 64);
    const int64_t blocks = want < 1 ? 1 : want > 256 * 16 ? 256 * 16 : want;
    const dim3 grid(static_cast<unsigned>(blocks + side_blocks));
    auto go = [&](auto kernel) {
        kernel<<<grid, kThreads, 0, stream>>>(x, n_pieces, split, ld_x, partials, n_partials, scale_in, q, ld_q, scale_out,
                                              amax_out, zero, side, side_blocks);
    };
    // Where the codes go.  A product finds those of ordinary stores in the caches; with stores past them (PAST) it keeps more
    // of its own operands there.  That gains 1 % on average, from 12 MB on, where the product's tiles are many and read whole
    // cache lines: at least 2048 rows, of whole lines of 128 bytes (80 calls of 2048 to 12000 tokens 0.992 to 1.034 times as
    // fast; 4096 x 4096 -> 4096 69.1 us against 70.3).  With fewer rows or rows across lines a product waits for its operands:
    // 600 x 12000 -> 4064 89.1 us against 71.8 backward, 1907 x 6896 -> 5152 85 against 80, step with tensors of 4 MB 65.0
    // against 60.8.  So does a narrow one (next_width columns): 5314 x 2928 -> 496 57.9 us against 55.8.  Its time per code is
    // that of reading it at about 250 columns; the line is at eight times that.
    const bool past = n_pieces * 16 >= (12 << 20) && rows >= 2048 && ((reinterpret_cast<uintptr_t>(q) | static_cast<uintptr_t>(ld_q)) & 127) == 0 &&
                      (next_width == 0 || next_width >= 2048);
    auto by_rows = [&](auto rows_tag) {
        constexpr int R = decltype(rows_tag)::value;
        if (fmt == FALQON_E4M3) { if (past) go(scale_cast_kernel<T, FALQON_E4M3, R, true>); else go(scale_cast_kernel<T, FALQON_E4M3, R, false>); }
        else { if (past) go(scale_cast_kernel<T, FALQON_E5M2, R, true>); else go(scale_cast_kernel<T, FALQON_E5M2, R, false>); }
    };
    if (dense) by_rows(std::integral_constant<int, kDense>{});
    else if (near) by_rows(std::integral_constant<int, kRows>{});
    else by_rows(std::integral_constant<int, kFarRows>{});
    return hipGetLastError();
}

}  // namespace

hipError_t launch_zero_word(uint32_t* w, hipStream_t stream)
{
    zero_word_kernel<<<1, 1, 0, stream>>>(w);
    return hipGetLastError();
}

hipError_t launch_quantize(const void* x, falqon_dtype xt, int64_t rows, int64_t cols, int64_t ld_x,
                           falqon_fmt fmt, const float* scale_in, uint8_t* q, int64_t ld_q,
                           float* scale_out, float* amax_out, float* partials, ZeroWords zero,
                           hipStream_t stream, const SideCast* side, int64_t next_width)
{
    if (xt == FALQON_BF16)
        return run(static_cast<const uint16_t*>(x), rows, cols, ld_x, fmt, scale_in, q, ld_q, scale_out,
                   amax_out, partials, zero, side, next_width, stream);
    return run(static_cast<const float*>(x), rows, cols, ld_x, fmt, scale_in, q, ld_q, scale_out, amax_out,
               partials, zero, side, next_width, stream);
}

}  // namespace falqon
