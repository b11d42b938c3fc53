// Row-wise proxy update (update equation; last two lines of the backward-and-update loop):
//   k = topk( sum_j |dB_ij| ; k ),   W~[k] = W~[k] + DeltaBuffer[k] A
//
// Small launches, all latency bound (the update touches k of m rows), so each is shaped to have its loads
// in flight together rather than one after the other:
//   1. row scores: L1 norm of every buffer row, fp64, columns ascending (row_scores.h).  Skipped when the
//      kernel that wrote the buffer has already left them (falqon_melded_bwd with its buffer step).
//   2. selection: the rank of a row is the number of rows that beat it (larger score, or equal score and
//      smaller index): exact and order free, so the result is deterministic and already sorted, with no
//      sort, no atomics on results, no host round trip.  Only rows that can be selected are ranked: the k-th
//      largest of the maxima of disjoint groups of rows is a lower bound on the k-th largest score.  The
//      selected buffer row moves to a compact staging array (and is cleared in the buffer), which lets the
//      third launch spread one row over several workgroups without a hazard on the buffer.
//   3. requantize: value(W~[i,j]) + sum_p delta[p] * value(A~[p,j]) in fp64 (p ascending), rounded to
//      fp32, cast to E4M3, written back.  A~ is rows [m, m+r) of the concatenated weight, in the same
//      scaled domain as W~, so the backbone's scale never enters.
#include <mutex>
#include <type_traits>

#include "falqon_internal.h"
#include "row_scores.h"

namespace falqon {
namespace {

constexpr int kThreads = 256;

// Scratch of the entry point that may not allocate and takes no workspace: row scores for up to
// kStaticMaxRows rows with their block maxima, then the staged buffer rows of the selection (k * r
// floats).  One copy per GPU, held until the process ends; every
// call on a GPU uses it, so calls that overlap on one GPU race.
constexpr size_t kStaticScoreBytes = sizeof(double) * (kStaticMaxRows + kStaticMaxRows / kScoreRows);
constexpr size_t kStaticBytes = kStaticScoreBytes + sizeof(float) * kStaticMaxSelected;
static __device__ __align__(256) unsigned char scratch[kStaticBytes];

// grid: ceil(m / 64); dynamic LDS: 64 * (r + 4) floats.  1024 threads: one round trip up to rank 64.
constexpr int kScoreThreads = 1024;

__global__ void __launch_bounds__(kScoreThreads)
row_score_kernel(const float* __restrict__ buf, int64_t m, int r, double* __restrict__ score)
{
    extern __shared__ float s_rows[];
    const int pitch = r + 4;                                         // +16 B: rows start on different banks
    const int64_t row0 = static_cast<int64_t>(blockIdx.x) * kScoreRows;
    const int r4 = r / 4;
    for (int e = threadIdx.x; e < kScoreRows * r4; e += kScoreThreads) {
        const int row = e / r4, c4 = e - row * r4;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (row0 + row < m) v = *reinterpret_cast<const float4*>(buf + (row0 + row) * r + c4 * 4);
        *reinterpret_cast<float4*>(s_rows + row * pitch + c4 * 4) = v;
    }
    __syncthreads();
    score_rows_from_lds(s_rows, r, row0, m, score);
}

// the first C of four codes
template <int C>
__device__ __forceinline__ void decode_e4m3(uint32_t w, double (&d)[4])
{
    d[0] = static_cast<double>(__builtin_amdgcn_cvt_f32_fp8(static_cast<int>(w), 0));
    d[1] = static_cast<double>(__builtin_amdgcn_cvt_f32_fp8(static_cast<int>(w), 1));
    if constexpr (C == 4) {
        d[2] = static_cast<double>(__builtin_amdgcn_cvt_f32_fp8(static_cast<int>(w), 2));
        d[3] = static_cast<double>(__builtin_amdgcn_cvt_f32_fp8(static_cast<int>(w), 3));
    }
}

__device__ __forceinline__ uint32_t encode4_e4m3(const double (&acc)[4])
{
    float f[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) f[e] = __builtin_amdgcn_fmed3f(static_cast<float>(acc[e]), -448.0f, 448.0f);
    int w = 0;
    w = __builtin_amdgcn_cvt_pk_fp8_f32(f[0], f[1], w, false);
    w = __builtin_amdgcn_cvt_pk_fp8_f32(f[2], f[3], w, true);
    return static_cast<uint32_t>(w);
}

// ---- selection ------------------------------------------------------------------------------------------
// grid (k): workgroup c finds the row of rank c, stages its buffer row and clears it.  Scores are
// non-negative doubles, so their bit patterns order them as 64-bit integers.  Thread t holds the keys of rows
// t, t + 256, ...; threads t and t ^ 1 form one of 128 groups.  The k-th largest group maximum bounds the
// k-th largest key from below, and so does any number below it: tau, its leading bits (every wave finds them
// by bisection on its own, two maxima per lane).  The rows that reach tau, a few dozen, contain the k selected
// ones; they are ranked pairwise.
//
// tau has 12 bits of the range that the maxima span: the exponent and some bits behind it where the
// rows have learned at different rates, bits far behind it where they are alike (the first step of AdamW moves
// every element by about the learning rate).  If far more rows than are looked for reach tau, 12 more bits,
// until tau is the k-th maximum itself; what is left then are equal scores (an untouched buffer), and the row is
// found among those above tau, or by its index among the equal ones.  Only where many rows are above tau (all that
// is large sits in a few threads) is it found by counting over all rows, bit by bit.
//
// All latency: one round trip for the scores, one for the buffer row, and 2 us of comparisons.  Every
// workgroup repeats the comparisons; nothing is exchanged.  Whole update in us (graph of 20, n = 256), against
// ranking 16 rows per workgroup or, beyond 4096 rows, whole blocks:
//                       rows learned at different rates   after the first AdamW step   untouched
//   512 x 16, k = 8              8.5 (9.1)                        8.5 (9.1)              8.4 (9.4)
//   4096 x 64, k = 32           12.1 (15.0)                      12.1 (14.9)            10.9 (15.2)
//   11008 x 64, k = 32          14.8 (25.6)                      14.9 (25.6)            12.9 (132)
// Slower than before only where many of few rows are equal and reach tau: 256 of 512 rows 10.9 (9.4), a third of
// 2000 rows 13.2 (12.4).
// (Requantizing in the same launch was built too: the workgroups that share a row have to agree on when
// its buffer row may be cleared, and their device-scope atomics cost more, 6 us, than the launch saved.)
constexpr int kSelectGroups = 128, kSelectMaxK = 96, kSelectCands = 2 * kSelectMaxK + 32, kSelectMaxRows = 64 * kThreads;
constexpr int kTauBits = 12;                                         // bits of tau found at a time
constexpr int kTauRounds = 6;                                        // that many cover a key

// a combination over the wave that leaves `none` unchanged, the same in every lane
template <typename F>
__device__ __forceinline__ uint32_t wave_combine(uint32_t x, uint32_t none, F f)
{
    const int o = static_cast<int>(none);
    x = f(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(o, static_cast<int>(x), 0x111, 0xf, 0xf, false)));   // row_shr 1, 2,
    x = f(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(o, static_cast<int>(x), 0x112, 0xf, 0xf, false)));   // 4, 8: rows of
    x = f(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(o, static_cast<int>(x), 0x114, 0xf, 0xf, false)));   // 16 lanes
    x = f(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(o, static_cast<int>(x), 0x118, 0xf, 0xf, false)));
    x = f(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(o, static_cast<int>(x), 0x142, 0xa, 0xf, false)));   // row_bcast 15,
    x = f(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(o, static_cast<int>(x), 0x143, 0xc, 0xf, false)));   // 31: across rows
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(x), 63));
}

// kTauBits more bits of the k-th largest of 128 maxima, two per lane (a, b): it lies in [tau, tau + 2^open), and so it
// does afterwards; open = 0: it is tau.
__device__ __forceinline__ void extend_tau(uint64_t a, uint64_t b, int k, uint64_t& tau, int& open)
{
    const uint64_t da = a - tau, db = b - tau;
    const bool in_a = a >= tau && (open > 63 || da >> open == 0), in_b = b >= tau && (open > 63 || db >> open == 0);
    const uint64_t diff = (in_a ? da : 0) | (in_b ? db : 0);
    const auto either = [](uint32_t x, uint32_t y) { return x | y; };
    const uint64_t all = static_cast<uint64_t>(wave_combine(static_cast<uint32_t>(diff >> 32), 0, either)) << 32 |
                         wave_combine(static_cast<uint32_t>(diff), 0, either);
    const int bits = all ? 64 - __builtin_clzll(all) : 0;
    open = bits > kTauBits ? bits - kTauBits : 0;
    // the leading bits of each distance from tau; maxima above the interval always count, those below never
    const uint32_t wa = in_a ? static_cast<uint32_t>(da >> open) : a > tau ? ~0u : 0u;
    const uint32_t wb = in_b ? static_cast<uint32_t>(db >> open) : b > tau ? ~0u : 0u;
    uint32_t w = 0;
#pragma unroll
    for (int bit = kTauBits - 1; bit >= 0; --bit) {
        const uint32_t trial = w | (1u << bit);
        if (__popcll(__ballot(wa >= trial)) + __popcll(__ballot(wb >= trial)) >= k) w = trial;
    }
    tau += static_cast<uint64_t>(w) << open;
}

template <int U>                                                     // U keys per thread: m <= 256 U
__global__ void __launch_bounds__(kThreads)
select_kernel(const double* __restrict__ score, int64_t m, int64_t k, int r, int32_t* __restrict__ idx, float* buf,
              float* __restrict__ delta_sel, int clear_selected)
{
    static_assert(U <= 64, "one lane per key of a thread");
    __shared__ uint64_t s_max[kSelectGroups];
    __shared__ uint64_t s_ckey[kSelectCands];
    __shared__ int s_cidx[kSelectCands];
    __shared__ int s_listed[kTauRounds + 1], s_row, s_count[2][kThreads / 64];
    __shared__ __attribute__((aligned(16))) int s_equal[64][kThreads / 64];
    __shared__ unsigned long long s_all, s_any;
    const uint64_t* key = reinterpret_cast<const uint64_t*>(score);
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    const int rank = static_cast<int>(blockIdx.x);

    uint64_t v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t i = static_cast<int64_t>(u) * kThreads + t;
        v[u] = i < m ? key[i] : 0;                                   // (0 also stands for the rows behind the last one:
    }                                                                // none is looked for but among equals, by index)
    if (t <= kTauRounds) s_listed[t] = 0;
    if (t == 0) s_row = -1;
    double mx = 0.0;                                                 // (a NaN is left out: tau stays a lower bound)
#pragma unroll
    for (int u = 0; u < U; ++u) mx = fmax(mx, __longlong_as_double(static_cast<long long>(v[u])));
    mx = fmax(mx, __shfl_xor(mx, 1, 64));
    if ((t & 1) == 0) s_max[t >> 1] = static_cast<uint64_t>(__double_as_longlong(mx));
    __syncthreads();

    // Ranking is quadratic: with far more rows listed than are looked for, tau gets more bits, or is the k-th
    // maximum itself and many of the listed ones equal it.
    const int limit = 2 * static_cast<int>(k) + 32;
    // rows with key >= bound > 0 (above: > bound) into the list, as far as it goes; which: the counter, used once per
    // launch.  Keys are compared as doubles, in one instruction; a NaN counts as above, as its bits do.
    auto list_rows = [&](uint64_t bound, auto above_tag, int which) __attribute__((always_inline)) {
        constexpr bool ABOVE = decltype(above_tag)::value;
        const double reach = __longlong_as_double(static_cast<long long>(bound));
        uint32_t in[2] = {0, 0};                                     // bit u: key u of this thread
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double x = __longlong_as_double(static_cast<long long>(v[u]));
            in[u / 32] |= (ABOVE ? !(x <= reach) : !(x < reach)) ? 1u << (u % 32) : 0u;
        }
        if (in[0] | in[1]) {
            int pos = atomicAdd(&s_listed[which], __popc(in[0]) + __popc(in[1]));
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int listed = in[u / 32] >> (u % 32) & 1;
                if (listed && pos < limit) { s_ckey[pos] = v[u]; s_cidx[pos] = u * kThreads + t; }
                pos += listed;
            }
        }
        __syncthreads();
        return s_listed[which];
    };
    // the row of rank `rank` among the nc listed ones: four threads per listed row, four others at a time
    auto rank_listed = [&](int nc) __attribute__((always_inline)) {
        for (int c0 = 0; c0 < nc; c0 += kThreads / 4) {
            const int c = c0 + t / 4;
            const bool in = c < nc;
            const uint64_t kc = s_ckey[in ? c : 0];
            const int ic = s_cidx[in ? c : 0];
            int beat = 0;
            for (int j0 = t & 3; j0 < nc; j0 += 16) {
                uint64_t kj[4];
                int ij[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int j = j0 + 4 * q < nc ? j0 + 4 * q : c;  // beyond the list: the row itself, which does not beat itself
                    kj[q] = s_ckey[in ? j : 0];
                    ij[q] = s_cidx[in ? j : 0];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) beat += (kj[q] > kc || (kj[q] == kc && ij[q] < ic)) ? 1 : 0;
            }
            beat += __shfl_xor(beat, 1, 64);
            beat += __shfl_xor(beat, 2, 64);
            if (in && (t & 3) == 0 && beat == rank) s_row = ic;
        }
    };
    // the row with `left` rows of the same key before it
    auto index_among_equal = [&](uint64_t value, int left) __attribute__((always_inline)) {
        uint64_t equal = 0;                                          // bit u: key u of this thread
        int mine = 0;                                                // lane u: rows of the wave's share of key u
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool eq = v[u] == value;
            const int count = __popcll(__ballot(eq));
            equal |= eq ? uint64_t(1) << u : 0;
            mine = lane == u ? count : mine;
        }
        s_equal[lane][wave] = mine;
        __syncthreads();
        const int4 c = *reinterpret_cast<const int4*>(s_equal[lane]);
        int upto = c.x + c.y + c.z + c.w;                            // rows of keys 0 .. lane
        for (int off = 1; off < 64; off <<= 1) {
            const int below = __shfl_up(upto, off, 64);
            if (lane >= off) upto += below;
        }
        const uint64_t reached = __ballot(upto > left);
        if (!reached) return;                                        // (value is a key of more than `left` rows)
        const int u = __builtin_ctzll(reached);
        int before = __shfl(upto - (c.x + c.y + c.z + c.w), u, 64);
        before += wave > 0 ? __shfl(c.x, u, 64) : 0;
        before += wave > 1 ? __shfl(c.y, u, 64) : 0;
        before += wave > 2 ? __shfl(c.z, u, 64) : 0;
        const bool eq = equal >> u & 1;
        before += __popcll(__ballot(eq) & ((uint64_t(1) << lane) - 1));
        if (eq && before == left) s_row = u * kThreads + t;
    };

    uint64_t tau;
    int nc, open = 64;
    {
        const uint64_t a = s_max[lane], b = s_max[lane + 64];
        const uint32_t ha = static_cast<uint32_t>(a >> 32), hb = static_cast<uint32_t>(b >> 32);
        const auto smaller = [](uint32_t x, uint32_t y) { return x < y ? x : y; };
        tau = static_cast<uint64_t>(wave_combine(smaller(ha, hb), ~0u, smaller)) << 32;   // no maximum is below it
        extend_tau(a, b, static_cast<int>(k), tau, open);
        nc = tau ? list_rows(tau, std::false_type{}, 0) : limit + 1;     // (every row reaches 0)
        for (int round = 1; nc > limit && open != 0 && round < kTauRounds; ++round) {
            const uint64_t before = tau;
            extend_tau(a, b, static_cast<int>(k), tau, open);
            if (tau != before) nc = list_rows(tau, std::false_type{}, round);
        }
    }
    const int above = nc > limit ? list_rows(tau, std::true_type{}, kTauRounds) : 0;
    if (nc <= limit) {
        rank_listed(nc);
    } else if (rank >= above) {
        index_among_equal(tau, rank - above);
    } else if (above <= limit) {
        rank_listed(above);
    } else {
        // largest key that more than `rank` rows reach: the key of the row looked for.  One barrier per count:
        // the sums of a count may still be read while the next one writes, so the two use different buffers, and
        // the barrier of the next keeps the one after it apart.  All waves make the same counts.
        int which = 0;
        auto count_reaching = [&](uint64_t bound) __attribute__((always_inline)) {
            which ^= 1;
            int c = 0;
#pragma unroll
            for (int u = 0; u < U; ++u)
                c += v[u] >= bound ? 1 : 0;
            for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
            if (lane == 0) s_count[which][wave] = c;
            __syncthreads();
            return s_count[which][0] + s_count[which][1] + s_count[which][2] + s_count[which][3];
        };
        // bits that all rows from tau on share need no count
        unsigned long long all = ~0ull, any = 0;
        if (t == 0) { s_all = ~0ull; s_any = 0; }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (v[u] >= tau) {
                all &= v[u];
                any |= v[u];
            }
        }
        for (int off = 32; off > 0; off >>= 1) {
            all &= __shfl_xor(all, off, 64);
            any |= __shfl_xor(any, off, 64);
        }
        if (lane == 0) { atomicAnd(&s_all, all); atomicOr(&s_any, any); }
        __syncthreads();
        all = s_all;
        any = s_any;
        uint64_t found = 0;
        for (int bit = 63; bit >= 0; --bit) {                        // (every thread takes the same path)
            const uint64_t trial = found | (uint64_t(1) << bit);
            if ((all & trial & ~found) || ((any & trial & ~found) && count_reaching(trial) > rank)) found = trial;
        }
        index_among_equal(found, rank - count_reaching(found + 1));
    }
    __syncthreads();
    const int64_t row = s_row;
    if (row < 0 || row >= m) return;                                 // cannot happen; keeps every access in range

    if (t == 0) idx[rank] = static_cast<int32_t>(row);
    if (t < r) {
        delta_sel[static_cast<int64_t>(rank) * r + t] = buf[row * r + t];
        if (clear_selected) buf[row * r + t] = 0.0f;
    }
}

constexpr int kChunk = 4096;                                         // scores that fit the small selection's LDS (32 KB)
static_assert(65536 / kScoreRows <= kChunk, "the block maxima of the largest buffer (m <= 65536) fit the LDS chunk");

// Selection for buffers of up to kChunk rows.  A workgroup ranks 16 rows (4 waves x 4 consecutive
// rows).  All scores sit in LDS; lanes stride over them and count the rows that beat each of the
// wave's rows.  Scores are non-negative doubles, so their bit patterns order them as 64-bit
// integers.  Row j beats row i if key_j > key_i, or key_j == key_i and j < i: for all j below the
// wave's rows that is "key_j >= key_i", for all j above them "key_j > key_i", so the inner loop is
// one integer comparison per pair; only the wave's own four rows need the index compared.
constexpr int kRankRows = 4;

__global__ void __launch_bounds__(kThreads)
topk_rank_kernel(const double* __restrict__ score, int64_t m, int64_t k, int r, int32_t* __restrict__ idx,
                 float* buf, float* __restrict__ delta_sel, int clear_selected)
{
    __shared__ uint64_t s_key[kChunk];
    const uint64_t* key = reinterpret_cast<const uint64_t*>(score);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t base = (static_cast<int64_t>(blockIdx.x) * 4 + wave) * kRankRows;
    uint64_t ki[kRankRows];
    int cnt[kRankRows];
#pragma unroll
    for (int q = 0; q < kRankRows; ++q) {
        ki[q] = base + q < m ? key[base + q] : 0;
        cnt[q] = 0;
    }
    const int n_here = static_cast<int>(m);                          // m <= kChunk
    {
        uint64_t v[kChunk / kThreads];                               // all loads in flight together
#pragma unroll
        for (int u = 0; u < kChunk / kThreads; ++u) {
            const int e = u * kThreads + threadIdx.x;
            v[u] = e < n_here ? key[e] : 0;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kChunk / kThreads; ++u) s_key[u * kThreads + threadIdx.x] = v[u];
    }
    __syncthreads();
    // rows below the wave's rows: ties count; rows above: they do not
    const int64_t lo_end = base > n_here ? n_here : base;
    const int64_t hi_begin = base + kRankRows > n_here ? n_here : base + kRankRows;
    // eight keys per lane and step, read together (one LDS latency per step instead of eight);
    // a slot beyond the range reads key 0 and is masked out of the count
    for (int e0 = lane; e0 < lo_end; e0 += 64 * 8) {
        uint64_t kj[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) kj[u] = s_key[e0 + 64 * u < lo_end ? e0 + 64 * u : 0];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const bool in = e0 + 64 * u < lo_end;
#pragma unroll
            for (int q = 0; q < kRankRows; ++q) cnt[q] += (in && kj[u] >= ki[q]) ? 1 : 0;
        }
    }
    for (int e0 = static_cast<int>(hi_begin) + lane; e0 < n_here; e0 += 64 * 8) {
        uint64_t kj[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) kj[u] = s_key[e0 + 64 * u < n_here ? e0 + 64 * u : 0];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const bool in = e0 + 64 * u < n_here;
#pragma unroll
            for (int q = 0; q < kRankRows; ++q) cnt[q] += (in && kj[u] > ki[q]) ? 1 : 0;
        }
    }
    if (lane < kRankRows && base + lane < n_here) {                  // the wave's own rows
        const uint64_t kj = s_key[base + lane];
#pragma unroll
        for (int q = 0; q < kRankRows; ++q) cnt[q] += (kj > ki[q] || (kj == ki[q] && lane < q)) ? 1 : 0;
    }
#pragma unroll
    for (int q = 0; q < kRankRows; ++q) {
        int c = cnt[q];
        for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
        const int64_t i = base + q;
        if (i < m && c < k) {                                        // wave-uniform
            if (lane == 0) idx[c] = static_cast<int32_t>(i);
            for (int64_t p = lane; p < r; p += 64) {
                delta_sel[static_cast<int64_t>(c) * r + p] = buf[i * r + p];
                if (clear_selected) buf[i * r + p] = 0.0f;
            }
        }
    }
}

// Selection for larger buffers: rank only rows that can be selected.  The k-th largest of the block
// maxima is a lower bound tau on the k-th largest score (each maximum is the score of a different
// row), so a row below tau has at least k rows above it.  A workgroup owns one block of 64 rows; it
// needs nothing but the block maxima to know whether it can leave, and most do.  One that stays
// lists its rows that reach tau, takes 128 KB of LDS to fetch up to 16384 scores per round trip, and
// counts, all threads together and one listed row at a time, the rows that beat it.
constexpr int kChunkFiltered = 16384;

__global__ void __launch_bounds__(kThreads)
topk_filtered_kernel(const double* __restrict__ score, int64_t m, int64_t k, int r, int32_t* __restrict__ idx,
                     float* buf, float* __restrict__ delta_sel, int clear_selected)
{
    extern __shared__ uint64_t s_key[];                              // kChunkFiltered keys
    __shared__ uint64_t s_tau;
    __shared__ int s_cand[kScoreRows + 4], s_cnt[kScoreRows + 4], s_ncand;
    __shared__ uint64_t s_ckey[kScoreRows + 4];
    const uint64_t* key = reinterpret_cast<const uint64_t*>(score);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t row0 = static_cast<int64_t>(blockIdx.x) * kScoreRows;

    // ---- tau, and whether this block can hold a selected row ----------------------------------------
    const int nb = static_cast<int>(score_blocks(m));
    if (threadIdx.x == 0) { s_tau = 0; s_ncand = 0; }
    if (threadIdx.x < kScoreRows + 4) s_cnt[threadIdx.x] = 0;
    for (int e = threadIdx.x; e < nb; e += kThreads) s_key[e] = key[m + e];
    __syncthreads();
    if (nb >= k) {
        for (int e = threadIdx.x; e < nb; e += kThreads) {
            const uint64_t mine = s_key[e];
            int above = 0;                                           // maxima that beat this one (ties by position)
            for (int j = 0; j < nb; ++j) {
                const uint64_t o = s_key[j];
                above += (o > mine || (o == mine && j < e)) ? 1 : 0;
            }
            if (above == k - 1) s_tau = mine;                        // exactly one position has this count
        }
    }
    __syncthreads();
    const uint64_t tau = s_tau;
    if (s_key[blockIdx.x] < tau) return;                             // workgroup-uniform
    // ---- the block's rows that reach tau, in row order ------------------------------------------------
    if (wave == 0) {
        const int64_t i = row0 + lane;
        const uint64_t mine = i < m ? key[i] : 0;
        const bool in = i < m && mine >= tau;
        const uint64_t mask = __ballot(in);
        if (in) {
            const int pos = __popcll(mask & ((uint64_t(1) << lane) - 1));
            s_cand[pos] = static_cast<int>(i);
            s_ckey[pos] = mine;
        }
        const int total = __popcll(mask);
        if (lane < 4) {                                              // padding so that listed rows can be taken four at a time
            s_cand[total + lane] = -1;
            s_ckey[total + lane] = ~uint64_t(0);
        }
        if (lane == 0) s_ncand = total;
    }
    __syncthreads();                                                 // also: the block maxima in s_key are no longer read
    const int ncand = s_ncand;
    // ---- count, for every listed row, the rows that beat it ---------------------------------------------
    for (int64_t c0 = 0; c0 < m; c0 += kChunkFiltered) {
        const int n_here = static_cast<int>(m - c0 < kChunkFiltered ? m - c0 : kChunkFiltered);
        if (c0 > 0) __syncthreads();
        for (int e0 = threadIdx.x; e0 < n_here; e0 += 32 * kThreads) {   // 32 loads in flight per thread
            uint64_t v[32];
#pragma unroll
            for (int u = 0; u < 32; ++u) {
                const int e = e0 + u * kThreads;
                v[u] = e < n_here ? key[c0 + e] : 0;
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < 32; ++u) {
                const int e = e0 + u * kThreads;
                if (e < n_here) s_key[e] = v[u];
            }
        }
        __syncthreads();
        for (int c = 0; c < ncand; c += 4) {                         // four listed rows per pass over the scores
            int64_t ri[4];
            uint64_t kc[4];
            int cnt[4] = {0, 0, 0, 0};
#pragma unroll
            for (int q = 0; q < 4; ++q) { ri[q] = s_cand[c + q]; kc[q] = s_ckey[c + q]; }
            for (int e = threadIdx.x; e < n_here; e += kThreads) {
                const uint64_t kj = s_key[e];
#pragma unroll
                for (int q = 0; q < 4; ++q) cnt[q] += (kj > kc[q] || (kj == kc[q] && c0 + e < ri[q])) ? 1 : 0;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                int v = cnt[q];
                for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
                if (lane == 0 && v) atomicAdd(&s_cnt[c + q], v);     // integer sum in LDS: order immaterial
            }
        }
    }
    __syncthreads();
    // ---- selected rows: index out, buffer row staged and cleared (one wave per row) -------------------
    for (int c = wave; c < ncand; c += 4) {
        const int rank = s_cnt[c];
        if (rank >= k) continue;                                     // wave-uniform
        const int64_t i = s_cand[c];
        if (lane == 0) idx[rank] = static_cast<int32_t>(i);
        for (int64_t p = lane; p < r; p += 64) {
            delta_sel[static_cast<int64_t>(rank) * r + p] = buf[i * r + p];
            if (clear_selected) buf[i * r + p] = 0.0f;
        }
    }
}

// grid: (k, ceil(n / (256 C))); a thread owns C adjacent columns of row idx[blockIdx.x]
template <int C> struct Codes;                                       // C adjacent E4M3 codes
template <> struct Codes<4> { typedef uint32_t type; };
template <> struct Codes<2> { typedef uint16_t type; };

template <int C>
__global__ void __launch_bounds__(kThreads)
row_requantize_kernel(uint8_t* wq, int64_t n, int64_t m, int64_t r, const int32_t* __restrict__ idx,
                      const float* __restrict__ delta_sel)
{
    typedef typename Codes<C>::type codes_t;
    __shared__ double s_delta[256];                                  // r <= 256
    const int64_t i = idx[blockIdx.x];
    if (i < 0 || i >= m) return;                                     // cannot happen; keeps every access in range
    for (int p = threadIdx.x; p < r; p += kThreads)
        s_delta[p] = static_cast<double>(delta_sel[static_cast<int64_t>(blockIdx.x) * r + p]);
    __syncthreads();
    const int64_t nc = n / C;
    const int64_t c = static_cast<int64_t>(blockIdx.y) * kThreads + threadIdx.x;
    if (c >= nc) return;
    codes_t* wrow = reinterpret_cast<codes_t*>(wq + i * n);
    const codes_t* arows = reinterpret_cast<const codes_t*>(wq + m * n);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    decode_e4m3<C>(wrow[c], acc);
    constexpr int U = 16;                                            // r is a multiple of 16
    for (int64_t p0 = 0; p0 < r; p0 += U) {
        codes_t aw[U];
#pragma unroll
        for (int u = 0; u < U; ++u) aw[u] = arows[(p0 + u) * nc + c];    // all 16 loads in flight
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            double a[4];
            decode_e4m3<C>(aw[u], a);
            const double d = s_delta[p0 + u];
#pragma unroll
            for (int e = 0; e < C; ++e) acc[e] = fma(d, a[e], acc[e]);  // product is exact in fp64
        }
    }
    wrow[c] = static_cast<codes_t>(encode4_e4m3(acc));
}

}  // namespace

// Device address of `scratch` on the current GPU.  In host code the array's name is only a handle:
// the address is looked up once per device and kept; every launch below receives that pointer.
static hipError_t static_scratch(unsigned char** out)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static unsigned char* ptrs[kMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptrs[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        ptrs[dev] = static_cast<unsigned char*>(p);
    }
    *out = ptrs[dev];
    return hipSuccess;
}

hipError_t launch_proxy_update_static(float* delta_buf, uint8_t* wq, int64_t n, int64_t m, int64_t r, int64_t k,
                                      int32_t* idx_out, int clear_selected, hipStream_t stream)
{
    unsigned char* base = nullptr;
    hipError_t e = static_scratch(&base);
    if (e != hipSuccess) return e;
    return launch_proxy_update(delta_buf, wq, n, m, r, k, idx_out, clear_selected, reinterpret_cast<double*>(base),
                               nullptr, reinterpret_cast<float*>(base + kStaticScoreBytes), stream);
}

hipError_t launch_proxy_update(float* delta_buf, uint8_t* wq, int64_t n, int64_t m, int64_t r, int64_t k,
                               int32_t* idx_out, int clear_selected, double* scores, const double* scores_in,
                               float* delta_sel, hipStream_t stream)
{
    hipError_t e;
    if (!scores_in) {
        const size_t lds = sizeof(float) * kScoreRows * (static_cast<size_t>(r) + 4);
        if (lds > 64 * 1024) {
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&row_score_kernel),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
            if (e != hipSuccess) return e;
        }
        row_score_kernel<<<static_cast<unsigned>(score_blocks(m)), kScoreThreads, lds, stream>>>(delta_buf, m,
                                                                                                 static_cast<int>(r), scores);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        scores_in = scores;
    }
    // The selection that finds one rank per workgroup, while the scores fit a workgroup's registers and the
    // group maxima bound the k-th score well (k of 128 groups).
    // Figures at the kernel; at the edge, 16384 rows and k = 96: 22.9 us against 31.4 for the whole update.
    if (k <= kSelectMaxK && m <= kSelectMaxRows) {
        auto go = [&](auto kernel) {
            kernel<<<static_cast<unsigned>(k), kThreads, 0, stream>>>(scores_in, m, k, static_cast<int>(r), idx_out, delta_buf,
                                                                      delta_sel, clear_selected);
        };
        if (m <= 4 * kThreads) go(select_kernel<4>);
        else if (m <= 16 * kThreads) go(select_kernel<16>);
        else if (m <= 44 * kThreads) go(select_kernel<44>);
        else go(select_kernel<64>);
    } else if (m > kChunk) {
        constexpr size_t lds_sel = sizeof(uint64_t) * kChunkFiltered;
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&topk_filtered_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds_sel));
        if (e != hipSuccess) return e;
        topk_filtered_kernel<<<static_cast<unsigned>(score_blocks(m)), kThreads, lds_sel, stream>>>(
            scores_in, m, k, static_cast<int>(r), idx_out, delta_buf, delta_sel, clear_selected);
    } else {
        topk_rank_kernel<<<static_cast<unsigned>((m + 4 * kRankRows - 1) / (4 * kRankRows)), kThreads, 0, stream>>>(
            scores_in, m, k, static_cast<int>(r), idx_out, delta_buf, delta_sel, clear_selected);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    // The requantize is bound by its fp64 conversions and sums, so two columns per thread while workgroups of
    // four would leave CUs idle (32 rows of 4096: 6.1 -> 5.4 us at r = 64, 14.4 -> 13.8 at r = 256).
    const int64_t groups = (n / 4 + kThreads - 1) / kThreads;
    if (k * groups <= 128) {
        const dim3 grid(static_cast<unsigned>(k), static_cast<unsigned>((n / 2 + kThreads - 1) / kThreads));
        row_requantize_kernel<2><<<grid, kThreads, 0, stream>>>(wq, n, m, r, idx_out, delta_sel);
    } else {
        row_requantize_kernel<4><<<dim3(static_cast<unsigned>(k), static_cast<unsigned>(groups)), kThreads, 0, stream>>>(
            wq, n, m, r, idx_out, delta_sel);
    }
    return hipGetLastError();
}

}  // namespace falqon
