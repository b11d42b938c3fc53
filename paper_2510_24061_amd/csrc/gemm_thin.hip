// Forward of a few tokens (a step of generation): quantizer, backbone product and O_A in one launch.
//
// With T <= 16 the weight is all there is to move, and in two launches it waits for the quantizer.  Here every
// workgroup quantizes the whole input for itself (at most 64 KB of bf16 from the L2: maximum, scale, codes into LDS),
// while its weights, which do not depend on it, are already on the way.  They go straight from memory into operand
// registers, each byte to one wave: no LDS ring, and no barrier between the steps.
//
// v_mfma_f32_16x16x128: lane t holds row t % 16 of an operand and 32 of its 128 K-bytes; as long as both operands
// agree it does not matter which, so it takes bytes [16 q, +16) and [64 + 16 q, +16), q = t / 16, and a load covers 64
// bytes of a row.  First operand: output columns, second: tokens, so a lane ends with four adjacent columns of one
// token.  Eight waves: NCB column blocks of 16 x KS shares of the K-steps (3 x 2: six waves multiply), which meet in LDS.
// NCB is the smallest that gives every CU one workgroup.  The first ones form O_A.  Its maximum needs no clear before:
// each of them exchanges a word in the workspace for its own maximum under a mark, waits for the exchange and reads the
// words of all; the one whose exchange is the last finds all marked (so may others, which then write the same),
// writes the maximum and takes the words back.  The mark is a NaN's bits, which no maximum in the workspace has.
//
// Against quantizer and product in two launches (gemm_mid.hip), us per forward call, four layers in turn:
//   1 x 4096 -> 4096, r = 64    9.6 (11.0)     2 x 4096 -> 1024, r = 64    6.7 (11.0)     3 x 1040 -> 2000, r = 48   5.0 (8.4)
//   4 x 4096 -> 4096, r = 32    9.1 (12.2)     16 x 2048 -> 2048, r = 64   7.4 (10.4)     1 x 4096 -> 11008, r = 64 11.5 (13.3)
//   8 x 4096 -> 4096, r = 64   11.5 (12.3)     16 x 256 -> 256, r = 16     3.8 (6.6)      8 x 4096 -> 11008, r = 64 13.7 (15.1)
#include "falqon_internal.h"
#include "gemm_common.h"
#include "quantize_common.h"

namespace falqon {
namespace {

constexpr int64_t kThinNarrow = 254 * 32;                  // m + r up to which a workgroup has 16 or 32 columns
typedef unsigned short v2s __attribute__((ext_vector_type(2)));

constexpr int kThinThreads = 512, kThinMaxTokens = 16, kThinMaxRank = 64;
constexpr int64_t kThinMaxCodes = 32 * 1024, kThinMaxK = 4096, kThinTwoRoundsK = 1024;     // T n, n, n
constexpr unsigned long long kThinArrived = 0x7fa57c3eull;
constexpr int kThinPieces = 8;                             // 16-byte pieces of x per thread: 512 x 8 x 8 elements

struct ThinArgs {
    const uint16_t* x; const uint8_t* wq; const float* s_w;
    int T; int64_t n, m; int r;
    uint8_t* xq; float* s_x; void* y; int y_is_f32; uint16_t* o_a; float* amax_oa;
    unsigned long long* words;                             // one per workgroup of O_A, any contents without kThinArrived
    uint32_t per_row_inverse;                              // ceil(2^32 / (n / 8)): quotients below 2^16 are exact
    int pad;                                               // K-bytes per token in LDS, zeros behind n
};

// K-steps (128 bytes) of a wave, all of them in flight before the input is quantized (with half of them, 8 x 4096 -> 11008
// took 15.1 us)
constexpr int thin_steps(int ks) { return static_cast<int>(kThinMaxK) / (ks * BK); }

// accumulates 16 NCB columns (weight rows from `first` on, `last` the last valid one) of all tokens; the result is in the
// waves of share 0, one block of 16 x 16 each
template <int NCB, int KS, typename Codes>
__device__ __forceinline__ v4f thin_columns(const ThinArgs& a, int64_t first, int64_t last, const uint8_t* lds_x, v4f* exchange,
                                            Codes&& codes)
{
    constexpr int D = thin_steps(KS);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int cb = wave % NCB, kh = wave / NCB;
    int64_t row = first + 16 * cb + (lane & 15);
    row = row < last ? row : last;
    const int n = static_cast<int>(a.n), q16 = (lane >> 4) * 16;
    const uint8_t* const w = a.wq + row * a.n;
    // step d of this wave: K-bytes from 128 (kh + KS d) on; beyond n the tokens are zero, and the row's first bytes stand in
    const int steps = kh < KS ? ((n + BK - 1) / BK - kh + KS - 1) / KS : 0;
    v4i lo[D], hi[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const int k = (kh + KS * d) * BK + q16;
        if (d < steps) {                                   // uniform
            lo[d] = *reinterpret_cast<const v4i*>(w + (k < n ? k : 0));
            hi[d] = *reinterpret_cast<const v4i*>(w + (k + 64 < n ? k + 64 : 0));
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    codes();                                               // the tokens' codes are in LDS behind this
    v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
    const int token = (lane & 15) < a.T ? lane & 15 : a.T - 1;
    const uint8_t* const xrow = lds_x + token * (a.pad + 16) + q16;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        if (d >= steps) continue;
        const int k = (kh + KS * d) * BK;
        const v4i xl = *reinterpret_cast<const v4i*>(xrow + k), xh = *reinterpret_cast<const v4i*>(xrow + k + 64);
        v8i wv, xv;
#pragma unroll
        for (int u = 0; u < 4; ++u) { wv[u] = lo[d][u]; wv[4 + u] = hi[d][u]; xv[u] = xl[u]; xv[4 + u] = xh[u]; }
        acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(wv, xv, acc, 0, 0, 0, 0, 0, 0);
    }
    if (kh > 0 && kh < KS) exchange[(wave - NCB) * 64 + lane] = acc;
    __syncthreads();
    if (kh == 0)
        for (int s = 1; s < KS; ++s) acc += exchange[((s - 1) * NCB + cb) * 64 + lane];
    __syncthreads();                                       // the exchange may be written again
    return acc;
}

template <int NCB, int KS>
__global__ void __launch_bounds__(kThinThreads)
fwd_thin_kernel(const ThinArgs a)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_x[];       // [T][pad + 16]
    __shared__ float s_max[kThinThreads / 64];
    __shared__ __attribute__((aligned(16))) v4f s_exchange[6 * 64 + 64];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int pieces = static_cast<int>(a.T * a.n / 8), per_row = static_cast<int>(a.n / 8);
    v4u xr[kThinPieces];
#pragma unroll
    for (int i = 0; i < kThinPieces; ++i) {
        if (i * kThinThreads >= pieces) break;                            // uniform
        const int p = i * kThinThreads + t;
        xr[i] = *reinterpret_cast<const v4u*>(a.x + static_cast<int64_t>(p < pieces ? p : pieces - 1) * 8);
    }
    __builtin_amdgcn_sched_barrier(0);
    float s = 1.0f;
    auto codes = [&]() {
        // bf16 without signs order as integers, NaN above all.  Counted from the first NaN and modulo 2^16 it is the NaN
        // that come below everything else: they leave the maximum of the other values, as in the quantizer.
        constexpr unsigned short kFirstNan = 0x7f81;
        constexpr unsigned short kZero = 65536 - kFirstNan;
        v2s top = {kZero, kZero};
        auto largest = [](v4u w, v2s m) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                m = __builtin_elementwise_max(m, __builtin_bit_cast(v2s, w[u] & 0x7fff7fffu) - v2s{kFirstNan, kFirstNan});
            return m;
        };
#pragma unroll
        for (int i = 0; i < kThinPieces; ++i) {
            if (i * kThinThreads >= pieces) break;
            top = largest(xr[i], top);
        }
        const uint32_t bits = ((top[0] > top[1] ? top[0] : top[1]) + kFirstNan) & 0xffffu;
        const float m = __uint_as_float(bits << 16);
        const float amax = block_max<kThinThreads / 64>(m, s_max);
        s = 448.0f / fmaxf(amax, 1e-12f);                                 // the quantizer's scale
#pragma unroll
        for (int i = 0; i < kThinPieces; ++i) {
            if (i * kThinThreads >= pieces) break;
            const int p = i * kThinThreads + t;
            if (p >= pieces) continue;
            const Piece<uint16_t>::codes_t c = cast_piece<uint16_t, FALQON_E4M3>(xr[i], s);
            const int token = static_cast<int>(__umulhi(static_cast<uint32_t>(p), a.per_row_inverse)), col = (p - token * per_row) * 8;
            *reinterpret_cast<Piece<uint16_t>::codes_t*>(lds_x + token * (a.pad + 16) + col) = c;
            // the workgroups share out the codes in memory
            const unsigned share = i * (kThinThreads / 64) + wave;
            if ((gridDim.x >= kThinPieces * kThinThreads / 64 ? share : share % gridDim.x) == blockIdx.x)
                *reinterpret_cast<Piece<uint16_t>::codes_t*>(a.xq + static_cast<int64_t>(p) * 8) = c;
        }
        const int fill = (a.pad - static_cast<int>(a.n)) / 16;
        for (int q = t; q < a.T * fill; q += kThinThreads)
            *reinterpret_cast<v4u*>(lds_x + (q / fill) * (a.pad + 16) + a.n + (q % fill) * 16) = v4u{0, 0, 0, 0};
        if (blockIdx.x == 0 && t == 0) *a.s_x = s;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        barrier_lds_only();
    };
    const int token = lane & 15, quad = lane >> 4, adapters = (a.r + 16 * NCB - 1) / (16 * NCB);
    const bool adapter = static_cast<int>(blockIdx.x) < adapters;
    const int64_t first = adapter ? a.m + static_cast<int64_t>(blockIdx.x) * 16 * NCB
                                  : (static_cast<int64_t>(blockIdx.x) - adapters) * 16 * NCB;
    const v4f acc = thin_columns<NCB, KS>(a, first, adapter ? a.m + a.r - 1 : a.m - 1, lds_x, s_exchange, codes);
    if (adapter) {
        const float inv = 1.0f / (s * (*a.s_w));
        float top = 0.0f;
        const int64_t col = first - a.m + 16 * (wave % NCB) + 4 * quad;
        if (wave < NCB && token < a.T && col < a.r) {
            uint2 pk;
            pk.x = pack_bf16x2(acc[0] * inv, acc[1] * inv);
            pk.y = pack_bf16x2(acc[2] * inv, acc[3] * inv);
            *reinterpret_cast<uint2*>(a.o_a + static_cast<int64_t>(token) * a.r + col) = pk;
            top = fmaxf(fmaxf(fabsf(__uint_as_float(pk.x << 16)), fabsf(__uint_as_float(pk.x & 0xffff0000u))),
                        fmaxf(fabsf(__uint_as_float(pk.y << 16)), fabsf(__uint_as_float(pk.y & 0xffff0000u))));
        }
        top = block_max<kThinThreads / 64>(top, s_max);
        if (adapters == 1) {
            if (t == 0) *a.amax_oa = top;
            return;
        }
        if (t >= 64) return;
        if (t == 0) {
            const unsigned long long before = atomicExch(&a.words[blockIdx.x], kThinArrived << 32 | __float_as_uint(top));
            asm volatile("s_waitcnt vmcnt(0)" : : "v"(before) : "memory");
        }
        const unsigned long long word = t < adapters ? atomicOr(&a.words[t], 0ull) : kThinArrived << 32;
        if (__ballot(word >> 32 != kThinArrived)) return;
        const float all = wave_max(__uint_as_float(static_cast<uint32_t>(word)));
        if (t == 0) *a.amax_oa = all;
        if (t < adapters) atomicExch(&a.words[t], 0ull);
        return;
    }
    const float inv = 1.0f / (s * (*a.s_w));
    const int64_t col = first + 16 * (wave % NCB) + 4 * quad;
    if (wave >= NCB || token >= a.T || col >= a.m) return;
    if (a.y_is_f32) {
        *reinterpret_cast<v4f*>(static_cast<float*>(a.y) + token * a.m + col) = v4f{acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv};
    } else {
        uint2 pk;
        pk.x = pack_bf16x2(acc[0] * inv, acc[1] * inv);
        pk.y = pack_bf16x2(acc[2] * inv, acc[3] * inv);
        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(a.y) + token * a.m + col) = pk;
    }
}

}  // namespace

// Every workgroup pays for quantizing the whole input: built for T n = 64 K that took longer than a launch (16 x 4096 ->
// 4096 15.2 us against 12.4; 8 tokens 11.5 against 12.3).  Beyond n = 4096 a wave's share of the rows does not fit its registers
// (in two batches 4 x 11008 -> 4096 20.4 us against 18.8).
// And workgroups that find no CU free begin when others have ended, with a quantizer of their own again: in two rounds
// 1 x 4096 -> 16400 took 22.8 us against 19.7 in two launches, 16 x 2048 -> 24000 19.1 against 16.5, 8 x 2048 -> 32512
// 18.8 against 18.7; up to n = 1024 they are still ahead (16 x 1024 -> 16400 11.6 against 12.2, -> 32512 13.2 against 13.6,
// 1 x 256 -> 32512 7.0 against 8.8).  In three or more they are not (16 x 1024 -> 36000 17.5 against 15.8, 16 x 256 -> 49152
// 12.3 against 11.2).
bool fwd_thin_supported(int64_t T, int64_t n, int64_t m, int64_t r)
{
    const int64_t workgroups = (m + 63) / 64 + (r + 63) / 64;          // (fewer columns each as long as that makes one round)
    return T <= kThinMaxTokens && T * n <= kThinMaxCodes && n <= kThinMaxK && r <= kThinMaxRank &&
           workgroups <= (n <= kThinTwoRoundsK ? 512 : 256);
}

hipError_t launch_fwd_thin(const void* x, const uint8_t* wq, const float* s_w, int64_t T, int64_t n, int64_t m, int64_t r,
                           uint8_t* xq, float* s_x, void* y, bool y_is_f32, void* o_a, float* amax_oa, void* words, hipStream_t stream)
{
    ThinArgs a;
    a.x = static_cast<const uint16_t*>(x); a.wq = wq; a.s_w = s_w; a.T = static_cast<int>(T); a.n = n; a.m = m; a.r = static_cast<int>(r);
    a.xq = xq; a.s_x = s_x; a.y = y; a.y_is_f32 = y_is_f32; a.o_a = static_cast<uint16_t*>(o_a); a.amax_oa = amax_oa;
    a.words = static_cast<unsigned long long*>(words);
    a.per_row_inverse = static_cast<uint32_t>(((uint64_t(1) << 32) + n / 8 - 1) / (n / 8));       // n >= 16
    auto go = [&](auto kernel, int ncb) -> hipError_t {
        const int64_t pad = (n + BK - 1) / BK * BK;
        a.pad = static_cast<int>(pad);
        const size_t lds = static_cast<size_t>(T) * (pad + 16);           // 35 KB at most
        kernel<<<static_cast<unsigned>((m + 16 * ncb - 1) / (16 * ncb) + (r + 16 * ncb - 1) / (16 * ncb)), kThinThreads, lds, stream>>>(a);
        return hipGetLastError();
    };
    if (m + r <= 256 * 16) return go(fwd_thin_kernel<1, 8>, 1);
    if (m + r <= kThinNarrow) return go(fwd_thin_kernel<2, 4>, 2);
    if (m + r <= 254 * 48) return go(fwd_thin_kernel<3, 2>, 3);
    return go(fwd_thin_kernel<4, 2>, 4);
}

}  // namespace falqon
