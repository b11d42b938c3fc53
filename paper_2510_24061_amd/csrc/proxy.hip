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
//      largest of the maxima of disjoint groups of rows is a lower bound on the k-th largest score.
//   3. requantize: value(W~[i,j]) + sum_p delta[p] * value(A~[p,j]) in fp64 (p ascending), rounded to
//      fp32, cast to E4M3, written back.  A~ is rows [m, m+r) of the concatenated weight, in the same
//      scaled domain as W~, so the backbone's scale never enters.
// Selection and requantize are one launch where the row of a rank is not spread over too many workgroups.  Otherwise
// the selected buffer row moves to a compact staging array (and is cleared in the buffer), which lets a third launch
// spread one row over several workgroups without a hazard on the buffer.
#include <mutex>
#include <type_traits>

#include "falqon_internal.h"
#include "gemm_common.h"
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

// grid: ceil(m / ROWS); dynamic LDS: ROWS * (r + 4) floats.  Blocks of 64 rows: 1024 threads, one round trip up to rank
// 64; blocks of 16, up to 4096 rows: 4 r threads, one always (update at 4096 x 256 16.7 us, 17.6 in blocks of 64; x 64
// 9.7 and 10.2).
constexpr int kScoreThreads = 1024;

template <int ROWS>
__global__ void __launch_bounds__(kScoreThreads)
row_score_kernel(const float* __restrict__ buf, int64_t m, int r, double* __restrict__ score)
{
    extern __shared__ float s_rows[];
    const int pitch = r + 4;                                         // +16 B: rows start on different banks
    const int64_t row0 = static_cast<int64_t>(blockIdx.x) * ROWS;
    const int r4 = r / 4;
    for (int e = threadIdx.x; e < ROWS * r4; e += blockDim.x) {
        const int row = e / r4, c4 = e - row * r4;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (row0 + row < m) v = *reinterpret_cast<const float4*>(buf + (row0 + row) * r + c4 * 4);
        *reinterpret_cast<float4*>(s_rows + row * pitch + c4 * 4) = v;
    }
    __syncthreads();
    score_rows_from_lds<ROWS>(s_rows, r, row0, m, score);
}

// C adjacent E4M3 codes
template <int C> struct Codes;
template <> struct Codes<4> { typedef uint32_t type; };
template <> struct Codes<2> { typedef uint16_t type; };
template <> struct Codes<1> { typedef uint8_t type; };

// the first C of four codes
template <int C>
__device__ __forceinline__ void decode_e4m3(uint32_t w, double (&d)[4])
{
    d[0] = static_cast<double>(__builtin_amdgcn_cvt_f32_fp8(static_cast<int>(w), 0));
    if constexpr (C >= 2) d[1] = static_cast<double>(__builtin_amdgcn_cvt_f32_fp8(static_cast<int>(w), 1));
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
// A workgroup finds the row of one rank.  Scores are non-negative doubles, so their bit patterns order them as 64-bit
// integers.  Thread t holds the keys of rows t, t + 512, ...; four threads form one of 128 groups.  Up to 512 rows are
// spread evenly over the groups, so that no more of them are empty than must be: with fewer than k maxima there is no
// bound (240 rows in 60 groups, k = 64: 34 us for the update, 9.5 now, 13 with groups of two threads).  The k-th largest group maximum, tau, bounds the
// k-th largest key from below.  The rows that reach tau, a few dozen, contain the k selected ones; they are
// ranked pairwise, as are the maxima.  If far more rows than are looked for reach tau, the row is found among
// those above tau, or by its index among those equal to it (an untouched buffer).  Only where many rows are
// above tau (all that is large sits in a few threads) is it found by counting over all rows, bit by bit.
//
// All latency: a round trip for the scores (0.7 us), then 2.1 us of comparisons (m = 4096: group maxima 0.2, tau 0.5,
// list 0.8, ranking 0.5; tau bit by bit over ballots took 1.5 us more), most of it chains of LDS accesses and
// barriers.  512 threads: with 256 a SIMD has one wave, whose instructions it cannot overlap.  Every workgroup repeats
// the comparisons; nothing is exchanged.
constexpr int kSelectGroups = 128, kSelectMaxK = 96, kSelectCands = 2 * kSelectMaxK + 32, kSelectThreads = 512;
constexpr int kSelectMaxRows = 32 * kSelectThreads;

// f(U) with the fewest keys per thread, of those that the kernels are built for, that hold m <= kSelectMaxRows rows
template <int U, int... More, typename F>
hipError_t first_that_holds(int64_t m, F f)
{
    if constexpr (sizeof...(More) > 0) {
        if (m > static_cast<int64_t>(U) * kSelectThreads) return first_that_holds<More...>(m, f);
    } else {
        static_assert(U * kSelectThreads >= kSelectMaxRows, "every row has a thread that holds its key");
    }
    return f(std::integral_constant<int, U>{});
}
template <typename F>
hipError_t with_keys(int64_t m, F f) { return first_that_holds<2, 8, 22, 32>(m, f); }

// a value of another lane of the same sixteen; 0xB1: lane ^ 1, 0x4E: lane ^ 2 (quad_perm), 0x141 / 0x140: mirrored
// within eight / sixteen, 0x150 + N: lane N
template <int CTRL>
__device__ __forceinline__ int lanes(int v) { return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true); }
template <int CTRL>
__device__ __forceinline__ double lanes(double v)
{
    return __hiloint2double(lanes<CTRL>(__double2hiint(v)), lanes<CTRL>(__double2loint(v)));
}
__device__ __forceinline__ int sum_of_8(int v)                       // over each eight lanes, in all of them
{
    v += lanes<0xB1>(v);
    v += lanes<0x4E>(v);
    return v + lanes<0x141>(v);                                      // row_half_mirror
}

// Workgroup barrier behind the wave's LDS accesses; __syncthreads() would also wait for the loads of A~ in flight.
__device__ __forceinline__ void barrier_lds()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    barrier_lds_only();
}

// the row of this thread's first key, -1 if it has none; ascending over the threads
template <int U>
__device__ __forceinline__ int first_row(int64_t m)
{
    const int t = static_cast<int>(threadIdx.x);
    if (U > 2 || m > kSelectThreads) return t;
    const int rows = static_cast<int>(m), group = t >> 2, row = group * rows / kSelectGroups + (t & 3);
    return row < (group + 1) * rows / kSelectGroups ? row : -1;
}

// keys of rows row0, t + 512, ...
template <int U>
__device__ __forceinline__ void load_keys(const double* __restrict__ score, int64_t m, int row0, uint64_t (&v)[U])
{
    const uint64_t* key = reinterpret_cast<const uint64_t*>(score);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t i = u ? static_cast<int64_t>(u) * kSelectThreads + threadIdx.x : row0;
        v[u] = i >= 0 && i < m ? key[i] : 0;                         // (0 also stands for no row: none is looked for
    }                                                                // but among equals, by index)
}

// the row of rank `rank` (-1 cannot happen), the same in every thread
template <int U>                                                     // U keys per thread: m <= 512 U
__device__ __forceinline__ int select_row(const uint64_t (&v)[U], int row0, int64_t k, int rank)
{
    static_assert(U <= 32, "one lane per key of a thread");
    __shared__ __attribute__((aligned(16))) uint64_t s_max[kSelectGroups];
    __shared__ uint64_t s_tau;
    __shared__ uint64_t s_ckey[kSelectCands];
    __shared__ int s_cidx[kSelectCands];
    __shared__ int s_listed[2], s_row, s_count[2][kSelectThreads / 64];
    __shared__ __attribute__((aligned(16))) int s_equal[64][kSelectThreads / 64];
    __shared__ unsigned long long s_all, s_any;
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    if (t < 2) s_listed[t] = 0;
    if (t == 0) s_row = -1;
    double mx = 0.0;                                                 // (a NaN is left out: tau stays a lower bound)
#pragma unroll
    for (int u = 0; u < U; ++u) mx = fmax(mx, __longlong_as_double(static_cast<long long>(v[u])));
    mx = fmax(mx, lanes<0xB1>(mx));
    mx = fmax(mx, lanes<0x4E>(mx));
    // the group's number in the last bits: no two are equal
    if ((t & 3) == 0) s_max[t >> 2] = (static_cast<uint64_t>(__double_as_longlong(mx)) & ~uint64_t(127)) | (127 - (t >> 2));
    barrier_lds();
    {
        // tau: the maximum with k - 1 others above it, without its last bits; sixteen threads count for four of them
        typedef unsigned long long v2u __attribute__((ext_vector_type(2)));
        const int q = t & 15;
        uint64_t mine[4];
        int above[4] = {0, 0, 0, 0};
#pragma unroll
        for (int x = 0; x < 4; ++x) mine[x] = s_max[4 * (t >> 4) + x];
#pragma unroll
        for (int u = 0; u < kSelectGroups / 32; ++u) {
            const v2u o = *reinterpret_cast<const v2u*>(s_max + 2 * (16 * u + q));
#pragma unroll
            for (int x = 0; x < 4; ++x) above[x] += (o[0] > mine[x] ? 1 : 0) + (o[1] > mine[x] ? 1 : 0);
        }
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            above[x] = sum_of_8(above[x]);
            above[x] += lanes<0x140>(above[x]);                      // row_mirror
            if (q == x && above[x] == static_cast<int>(k) - 1) s_tau = mine[x] & ~uint64_t(127);
        }
    }
    barrier_lds();
    const uint64_t tau = s_tau;

    // Ranking is quadratic: it ends where far more rows are listed than are looked for.
    const int limit = 2 * static_cast<int>(k) + 32;
    // rows with key >= bound into the list, as far as it goes; which: the counter, used once per launch
    auto list_rows = [&](uint64_t bound, int which) __attribute__((always_inline)) {
        uint32_t in = 0;                                             // bit u: key u of this thread
#pragma unroll
        for (int u = 0; u < U; ++u) in |= v[u] >= bound ? 1u << u : 0u;
        if (in) {
            int pos = atomicAdd(&s_listed[which], __popc(in));
            for (; in && pos < limit; in &= in - 1, ++pos) {
                const int first = __builtin_ctz(in);
                uint64_t key = v[0];
#pragma unroll
                for (int u = 1; u < U; ++u) {
                    key = u == first ? v[u] : key;
                    asm volatile("" : "+v"(key));                    // (else an array in memory)
                }
                s_ckey[pos] = key;
                s_cidx[pos] = first ? first * kSelectThreads + t : row0;
            }
        }
        barrier_lds();
        return s_listed[which];
    };
    // the row of rank `rank` among the nc listed ones: eight threads per listed row, eight others at a time
    auto rank_listed = [&](int nc) __attribute__((always_inline)) {
        for (int c0 = 0; c0 < nc; c0 += kSelectThreads / 8) {
            const int c = c0 + t / 8;
            const uint64_t kc = s_ckey[c < nc ? c : 0];
            int larger = 0, equal = 0;
            for (int j0 = t & 7; j0 < nc; j0 += 64) {
                uint64_t kj[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) kj[q] = s_ckey[j0 + 8 * q < nc ? j0 + 8 * q : 0];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const bool in = j0 + 8 * q < nc;
                    larger += in && kj[q] > kc ? 1 : 0;
                    equal += in && kj[q] == kc ? 1 : 0;              // (itself among them)
                }
            }
            larger = sum_of_8(larger);
            equal = sum_of_8(equal);
            if ((t & 7) || c >= nc || rank < larger || rank >= larger + equal) continue;
            int left = rank - larger;                                // equal keys by index
            const int ic = s_cidx[c];
            if (equal > 1)
                for (int j = 0; j < nc; ++j) left -= s_ckey[j] == kc && s_cidx[j] < ic ? 1 : 0;
            if (left == 0) s_row = ic;
        }
    };
    // the row with `left` rows of the same key before it
    auto index_among_equal = [&](uint64_t value, int left) __attribute__((always_inline)) {
        uint32_t equal = 0;                                          // bit u: key u of this thread
        int mine = 0;                                                // lane u: rows of the wave's share of key u
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool eq = v[u] == value && (u > 0 || row0 >= 0);
            const int count = __popcll(__ballot(eq));
            equal |= eq ? 1u << u : 0u;
            mine = lane == u ? count : mine;
        }
        s_equal[lane][wave] = mine;
        barrier_lds();
        int total = 0, earlier = 0;                                  // rows of key `lane`, and those of earlier waves' shares
#pragma unroll
        for (int w = 0; w < kSelectThreads / 64; ++w) {
            const int c = s_equal[lane][w];
            total += c;
            earlier += w < wave ? c : 0;
        }
        int upto = total;                                            // rows of keys 0 .. lane
        for (int off = 1; off < 64; off <<= 1) {
            const int below = __shfl_up(upto, off, 64);
            if (lane >= off) upto += below;
        }
        const uint64_t reached = __ballot(upto > left);
        if (!reached) return;                                        // (value is a key of more than `left` rows)
        const int u = __builtin_ctzll(reached);
        int before = __shfl(upto - total + earlier, u, 64);
        const bool eq = equal >> u & 1;
        before += __popcll(__ballot(eq) & ((uint64_t(1) << lane) - 1));
        if (eq && before == left) s_row = u ? u * kSelectThreads + t : row0;
    };

    // those that reach tau; those above it if they are too many (every row reaches 0)
    int nc = limit + 1, which = tau ? 0 : 1;
    for (; which < 2; ++which) {
        nc = list_rows(tau + which, which);
        if (nc <= limit) break;
    }
    if (which == 1 && rank >= nc) {
        index_among_equal(tau, rank - nc);
    } else if (nc <= limit) {
        rank_listed(nc);
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
            barrier_lds();
            int sum = 0;
#pragma unroll
            for (int w = 0; w < kSelectThreads / 64; ++w) sum += s_count[which][w];
            return sum;
        };
        // bits that all rows from tau on share need no count
        unsigned long long all = ~0ull, any = 0;
        if (t == 0) { s_all = ~0ull; s_any = 0; }
        barrier_lds();
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
        barrier_lds();
        all = s_all;
        any = s_any;
        uint64_t found = 0;
        for (int bit = 63; bit >= 0; --bit) {                        // (every thread takes the same path)
            const uint64_t trial = found | (uint64_t(1) << bit);
            if ((all & trial & ~found) || ((any & trial & ~found) && count_reaching(trial) > rank)) found = trial;
        }
        index_among_equal(found, rank - count_reaching(found + 1));
    }
    barrier_lds();
    return s_row;
}

// grid (k): workgroup c stages the buffer row of rank c and clears it
template <int U>
__global__ void __launch_bounds__(kSelectThreads)
select_kernel(const double* __restrict__ score, int64_t m, int64_t k, int r, int32_t* __restrict__ idx, float* buf,
              float* __restrict__ delta_sel, int clear_selected)
{
    uint64_t v[U];
    const int row0 = first_row<U>(m);
    load_keys(score, m, row0, v);
    const int t = threadIdx.x, rank = static_cast<int>(blockIdx.x);
    const int64_t row = select_row(v, row0, k, rank);
    if (row < 0 || row >= m) return;                                 // cannot happen; keeps every access in range
    if (t == 0) idx[rank] = static_cast<int32_t>(row);
    if (t < r) {
        delta_sel[static_cast<int64_t>(rank) * r + t] = buf[row * r + t];
        if (clear_selected) buf[row * r + t] = 0.0f;
    }
}

constexpr int kChunk = 4096;                                         // scores that fit the small selection's LDS (32 KB)
static_assert(kScoreFew <= kChunk, "the block maxima are there where the selection for larger buffers runs");
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

// Selection and requantize in one launch, grid (k, parts): every workgroup of a rank finds the row by itself, with
// its part of A~ on the way into registers meanwhile (then LDS: a thread's bytes of 16 ranks at a time), and writes
// its C columns per thread of the row.
//
// The buffer row may only be cleared when all parts have read it.  Each part has a word in memory: it exchanges the
// word for `kArrived` once its reads are done, waits for the exchange, and then reads the words of all parts.  The
// exchange that comes last in memory is followed by reads that find all words set, so at least one part clears
// the row; parts that find them set at the same time write the same zeros.  Who clears the row also takes the words
// back, after all have been set, so none is left behind for the next launch or a replay; a word that happens to hold
// kArrived beforehand is the one thing that must not be (any other 64 bits may stand there).  Nothing waits for
// another workgroup.  The words of a rank lie in 64 bytes or more of their own, and the exchange hides under the
// sums; the clear adds 0.7 us to the launch.  (Counters of all ranks in one line took 6 us.)
//
// Bound by latency: scores 0.7 us, selection 2.6, row 0.5, sums 1.2 (r = 64; 4.3 at r = 256), end 0.6 at 4096 x 4096,
// k = 32.  The sums are rolled up to 16 ranks: unrolled over 64 their instructions alone took 0.8 us to arrive.
// Whole update with its score pass, us (graph of 20, with clear), against selection and requantize in two launches:
//   512 x 512, r = 16, k = 8          6.8 (8.6)      4096 x 4096, r = 256, k = 32     16.8 (18.7)
//   2000 x 1040, r = 48, k = 24       8.9 (10.8)     4096 x 11008, r = 64, k = 32     12.0 (13.3)
//   4096 x 4096, r = 64, k = 32       9.7 (11.3)     11008 x 4096, r = 64, k = 32     12.7 (15.6)
// Ranks whose part of A~ takes more than 4 of 16 bytes per thread, and less than 16, read the rest for nothing; they are
// ahead all the same: r = 80 11.1 (12.2), r = 96 11.7 (12.5), r = 128 12.6 (13.6) at 4096 x 4096, k = 32.
constexpr unsigned long long kArrived = 0xa57c3e91d20b68f5ull;

template <int N, typename F, int I = 0>
__device__ __forceinline__ void for_each(F f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        for_each<N, F, I + 1>(f);
    }
}

// element N of the sixteen that each row of 16 lanes holds (row_newbcast: no LDS access, no scalar register)
template <int N>
__device__ __forceinline__ double of_row(double sixteen) { return lanes<0x150 + N>(sixteen); }

// ROW columns per workgroup, C per thread; NA x 16 bytes of A~ per thread: r ROW <= 8192 NA
template <int U, int ROW, int NA>
__global__ void __launch_bounds__(kSelectThreads)
fold_kernel(uint8_t* wq, int64_t n, int64_t m, int r, const double* __restrict__ score, int64_t k,
            int32_t* __restrict__ idx, float* buf, unsigned long long* arrived, int clear_selected)
{
    constexpr int C = ROW <= 1024 ? 2 : 4, CHUNKS = ROW / 16;
    typedef typename Codes<C>::type codes_t;
    extern __shared__ __attribute__((aligned(16))) uint8_t s_a[];    // [r][ROW]
    __shared__ double s_delta[256];                                  // r <= 256
    const int t = threadIdx.x, rank = static_cast<int>(blockIdx.x), part = static_cast<int>(blockIdx.y);
    const int parts = static_cast<int>(gridDim.y);
    uint64_t v[U];
    const int row0 = first_row<U>(m);
    load_keys(score, m, row0, v);
    __builtin_amdgcn_sched_barrier(0);
    typedef unsigned v4u __attribute__((ext_vector_type(4)));
    v4u ahead[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int q = i * kSelectThreads + t, p = q / CHUNKS;
        const int64_t j = static_cast<int64_t>(part) * ROW + q % CHUNKS * 16;         // n is a multiple of 16
        ahead[i] = *reinterpret_cast<const v4u*>(wq + (m + (p < r ? p : r - 1)) * n + (j < n ? j : n - 16));
    }
    __builtin_amdgcn_sched_barrier(0);
    const int64_t row = select_row(v, row0, k, rank);
    if (row < 0 || row >= m) return;                                 // cannot happen; keeps every access in range
    const int64_t col = static_cast<int64_t>(part) * ROW + t * C;     // the first of this thread's columns
    const bool mine = t * C < ROW && col < n;
    codes_t* const w = reinterpret_cast<codes_t*>(wq + row * n + col);
    float delta = 0.0f;
    if (t < r) delta = buf[row * r + t];
    codes_t old = 0;
    if (mine) old = *w;
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int q = i * kSelectThreads + t;
        if (q < r * CHUNKS) *reinterpret_cast<v4u*>(s_a + q * 16) = ahead[i];
    }
    if (t == 0 && part == 0) idx[rank] = static_cast<int32_t>(row);
    if (t < 256) s_delta[t] = static_cast<double>(delta);            // (waits for it)
    barrier_lds();                                              // all waves have read the row
    unsigned long long* const words = arrived + static_cast<int64_t>(rank) * (r / 2);
    unsigned long long before = 0;
    if (clear_selected && parts > 1 && t == 0) before = atomicExch(&words[part], kArrived);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    decode_e4m3<C>(old, acc);
    const uint8_t* column = s_a + (mine ? t * C : 0);
    if (t < ROW / C) {                                               // (whole waves)
        const double* d16 = s_delta + (t & 15);
#pragma unroll 1
        for (int p = 0; p < r; p += 16, column += 16 * ROW, d16 += 16) {   // r is a multiple of 16
            codes_t a[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) a[u] = *reinterpret_cast<const codes_t*>(column + u * ROW);
            const double d = *d16;
            auto add = [&](auto tag) {
                constexpr int N = decltype(tag)::value;
                double x[4];
                decode_e4m3<C>(a[N], x);
                const double dn = of_row<N>(d);
#pragma unroll
                for (int e = 0; e < C; ++e) acc[e] = fma(dn, x[e], acc[e]);      // product is exact in fp64
            };
            for_each<16>(add);
        }
    }
    if (mine) *w = static_cast<codes_t>(encode4_e4m3(acc));
    if (!clear_selected || t >= 64) return;
    if (parts > 1) {
        if (t == 0) asm volatile("s_waitcnt vmcnt(0)" : : "v"(before) : "memory");
        if (__ballot(t < parts && atomicOr(&words[t < parts ? t : 0], 0ull) != kArrived) != 0) return;
    }
    for (int p = t; p < r; p += 64) buf[row * r + p] = 0.0f;
    if (parts > 1 && t < parts) atomicExch(&words[t], 0ull);
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
        const bool few = m <= kScoreFew;
        const int rows = few ? kScoreRowsFew : kScoreRows;
        const size_t lds = sizeof(float) * rows * (static_cast<size_t>(r) + 4);
        if (lds > 64 * 1024) {
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&row_score_kernel<kScoreRows>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
            if (e != hipSuccess) return e;
        }
        const unsigned blocks = static_cast<unsigned>((m + rows - 1) / rows);
        if (few) row_score_kernel<kScoreRowsFew><<<blocks, static_cast<unsigned>(4 * r), lds, stream>>>(delta_buf, m, static_cast<int>(r), scores);
        else row_score_kernel<kScoreRows><<<blocks, kScoreThreads, lds, stream>>>(delta_buf, m, static_cast<int>(r), scores);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        scores_in = scores;
    }
    // One launch where its workgroups, each of which repeats the selection, find room on the 256 CUs at one per CU (two
    // rounds of them, 4096 x 4096 at r = 64, k = 64 with 512 columns each: 12.2 us for the update against 10.8 with 1024),
    // their part of A~ fits into registers and LDS, and a rank's words fit into the room of its staged row.
    if (k <= kSelectMaxK && m <= kSelectMaxRows) {
        int64_t row = 512, parts = 0;
        for (; row <= 2048; row *= 2) {
            parts = (n + row - 1) / row;
            if (k * parts <= 256) break;
        }
        if (row <= 2048 && r * row <= 128 * 1024 && parts <= 64 && 2 * parts <= r) {
            auto go = [&](auto kernel) -> hipError_t {
                const size_t lds = static_cast<size_t>(r * row);
                if (lds > 48 * 1024) {
                    const hipError_t fe = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                              hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
                    if (fe != hipSuccess) return fe;
                }
                kernel<<<dim3(static_cast<unsigned>(k), static_cast<unsigned>(parts)), kSelectThreads, lds, stream>>>(
                    wq, n, m, static_cast<int>(r), scores_in, k, idx_out, delta_buf,
                    reinterpret_cast<unsigned long long*>(delta_sel), clear_selected);
                return hipGetLastError();
            };
            auto pick = [&](auto keys) -> hipError_t {
                constexpr int U = decltype(keys)::value;
                const bool few = r * row <= 4 * 8192;
                if (row == 512) return few ? go(fold_kernel<U, 512, 4>) : go(fold_kernel<U, 512, 16>);
                if (row == 1024) return few ? go(fold_kernel<U, 1024, 4>) : go(fold_kernel<U, 1024, 16>);
                return few ? go(fold_kernel<U, 2048, 4>) : go(fold_kernel<U, 2048, 16>);
            };
            return with_keys(m, pick);
        }
    }
    // The selection that finds one rank per workgroup, while the scores fit a workgroup's registers and the
    // group maxima bound the k-th score well (k of 128 groups).  Whole update around the line on k, 1040 columns, r = 256:
    // 16384 rows 29.9 us at k = 96 and 42.9 at k = 97, 11264 rows 26.0 and 35.5, 4096 rows 23.6 and 24.1.
    if (k <= kSelectMaxK && m <= kSelectMaxRows) {
        e = with_keys(m, [&](auto keys) -> hipError_t {
            select_kernel<decltype(keys)::value><<<static_cast<unsigned>(k), kSelectThreads, 0, stream>>>(
                scores_in, m, k, static_cast<int>(r), idx_out, delta_buf, delta_sel, clear_selected);
            return hipGetLastError();
        });
        if (e != hipSuccess) return e;
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
