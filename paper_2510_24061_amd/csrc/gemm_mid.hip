// FP8 products of small and medium size: tiles of 32, 64 or 128 tokens on deep LDS rings.
//
// Same products as gemm.hip (see there for operand forms), for sizes that give the 256x256 tiles too few
// workgroups to fill the chip.  What bounds them is not the matrix cores but the way of the operands
// through the LDS, and the latency of getting them there:
//   - a workgroup is alone on its CU and spends the whole LDS on one ring of S stages (S = 4 .. 8) that
//     holds both operands, so that 100 to 130 KB are in flight while one stage is multiplied.
//   - fetches write the LDS at 64 B/clk per CU, reads take about 200 B/clk and hide under them (measured:
//     8 fetches per wave 514 clk, with 16 reads beside them 515), so the fetches are what a K-step costs as
//     long as reads and matrix instructions stay beside them.  The four waves split the tile 2 (columns) x 2 (K): each
//     multiplies 32 MB tokens x 32 NB columns over one 64-byte half of every K-step, which reads a third
//     less than a 2 x 2 split of the tile; the two halves meet once, after the loop.
//   - operands of step k + 1 are read into registers under the matrix instructions of step k, so a
//     stage's slot is free for the next fetch one step after it landed; one barrier per step.
// The adapter's products cost no launch of their own:
//   - forward: workgroups of the first ceil(r / 32) tile columns hold 32 adapter rows in their stages and
//     multiply one more 32-column block, or, where a tile row has too few tile columns or the chip has
//     idle CUs, the adapter has tile columns of its own.  O_A and its maximum leave the launch finished.
//   - input gradient: the stages of the left operand also hold what dB needs (see db_stage below).
// Measured against the 128x128 tiles of gemm.hip plus their launches for the adapter (us, kernel trace of
// both in one run): 512 x 4096 x 4096, r = 64: forward 18.4 (20.1 + 7.0 + 3.9), input gradient with dB 20.4
// (20.9 + 7.4); 8 x 4096 x 11008 forward 10.6 (19.4 + 5.8 + 3.1); 256 x 512 x 512 forward 5.2 (6.5 + 5.4 + 3.2),
// input gradient with dB 5.9 (6.7 + 6.2).
#include <type_traits>

#include "db_tile.h"
#include "falqon_internal.h"
#include "gemm_common.h"
#include "gemm_mid.h"

namespace falqon {
namespace {

struct MidArgs {
    GemmArgs g;              // the backbone product; c1, ldc1, amax1: the adapter's output
    const uint8_t* side;     // adapter rows [r][K] (row stride g.ldb); read only if ride or tiles_a > 0
    int64_t r;
    int tiles_m, tiles_n;    // tile rows, tile columns of the backbone
    int tiles_a;             // extra tile columns for the adapter (0: none)
    int ride;                // tile columns that carry 32 adapter rows along (0: none)
    int chunk;               // tiles per XCD
    const uint8_t* oaq;      // input gradient with the adapter gradient: O_A codes [M][r], else null
    float* db_partial;       // [tiles_m][K][r] raw sums
};

template <int N>
struct WaitStages {          // s_waitcnt with `n` stages of LPW loads outstanding, 0 <= n <= N; lgkmcnt(0)
    template <int LPW>
    static __device__ __forceinline__ void run(int n)
    {
        if (n >= N) __builtin_amdgcn_s_waitcnt(((N * LPW) & 15) | (7 << 4) | (((N * LPW) >> 4) << 14));
        else WaitStages<N - 1>::template run<LPW>(n);
    }
};
template <>
struct WaitStages<-1> {
    template <int LPW>
    static __device__ __forceinline__ void run(int) {}
};

constexpr int kMidCus = 256;
constexpr int mid_max(int a, int b) { return a > b ? a : b; }

// LDS: the ring; afterwards the exchange of the two K halves, then the output rows.
template <int MB, int NB, int S, bool RIDE, bool DB>
constexpr int mid_lds_bytes()
{
    constexpr int BM = 32 * MB, BN = 64 * NB;
    constexpr int ring = S * (BM + BN + (RIDE ? 32 : 0)) * BK + (DB ? BM * 256 : 0);
    constexpr int exchange = 2 * (MB * NB + (RIDE ? mid_max(MB / 2, 1) : 0)) * 4096;
    constexpr int rows = BM * (BN * 4 + 16);
    return mid_max(ring, mid_max(exchange, rows));
}

// Rows of an operand that begin anywhere in a cache line (row length no multiple of 128 bytes): fetched from their own
// first byte on, 128 of them lie across two lines, and in long rows the operands take half as long again to arrive.  SKEW
// ([N,K] operands): a stage holds one whole line of every row instead.  A row begins `shift` chunks of 16 bytes into
// its line 0, so chunk c of K-step k lies in stage k + (c + shift) / 8: a step's operands are in two stages, and one more
// of the ring has landed.  In LDS a chunk keeps the place that it has without SKEW.  Rows eight apart have the same
// shift, whatever their length.  (Lanes of a fetch that only changed places, so that every four lay in one half of a line,
// gained nothing.)
struct Skew {
    int first, length;                                           // first row's place in its line, row length: chunks, modulo 8
    __device__ Skew(const uint8_t* p, int64_t ld)
        : first(static_cast<int>(reinterpret_cast<uintptr_t>(p) >> 4) & 7), length(static_cast<int>(ld >> 4) & 7) {}
    __device__ int shift(int row) const { return (first + row * length) & 7; }
};

// One tile.  RIDE: the stages carry 32 adapter rows too and the tile writes its 32 MB x 32 block of O_A.
// ADAPTER (run time): the tile is one of the adapter's own columns (output to c1, bf16, with its maximum).
template <int MB, int NB, int S, bool B_KN, int A_FMT, bool RIDE, bool DB, bool SKEW, bool ADDS>
__device__ __forceinline__ void mid_tile(const MidArgs& t, const int tile_m, const int tile_n, const bool adapter,
                                         uint8_t* const lds)
{
    static_assert(!RIDE || (!B_KN && A_FMT == 0), "the adapter product belongs to the forward product");
    static_assert(!DB || (B_KN && A_FMT == 1), "the adapter gradient belongs to the input-gradient product");
    static_assert(!ADDS || (B_KN && A_FMT == 1), "input gradients are what is added up");
    static_assert(!SKEW || !B_KN, "whole lines of rows are for operands whose rows run along K");
    const GemmArgs& g = t.g;
    constexpr int BM = 32 * MB, BN = 64 * NB;
    constexpr int A_BYTES = BM * BK, B_BYTES = BN * BK, STAGE = A_BYTES + B_BYTES + (RIDE ? 32 * BK : 0);
    constexpr int IT_A = BM / 32, IT_B = BN / 32, LPW = IT_A + IT_B + (RIDE ? 1 : 0);   // 1 KB fetches per wave and stage
    static_assert((S - 1) * LPW < 64, "vmcnt has six bits");
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wn = wave & 1, kh = wave >> 1;
    const int64_t m0 = static_cast<int64_t>(tile_m) * BM;
    const int64_t n0 = static_cast<int64_t>(adapter ? tile_n - t.tiles_n : tile_n) * BN;
    const int64_t M = g.M, N = adapter ? t.r : g.N, K = g.K;
    const uint8_t* const gb = adapter ? t.side : g.b;

    // ---- global -> LDS ----------------------------------------------------------------------
    // As in the large tiles: uniform base + 32-bit lane offset while a stage lies inside K, rows and
    // columns beyond the matrix clamped to the last valid one, the K tail from a block of zeros.
    constexpr int CH = BN / 16, RPI = 64 / CH;                 // [K][N] tile: chunks per K-row, K-rows per fetch
    const int rows_a = static_cast<int>((M - m0) < BM ? (M - m0) : BM);
    const int rows_b = static_cast<int>((N - n0) < BN ? (N - n0) : BN);
    const int r0 = tile_n * 32;                                 // first adapter row that rides on this tile
    const uint8_t* const base_a = g.a + m0 * g.lda;
    const uint8_t* const base_b = B_KN ? gb + n0 : gb + n0 * g.ldb;
    const uint8_t* const base_r = RIDE ? t.side + static_cast<int64_t>(r0) * g.ldb : nullptr;
    const Skew skew_a(base_a, g.lda), skew_b(base_b, g.ldb), skew_r(base_r, g.ldb);
    // K-contiguous operand: what this lane fetches of LDS row `row`, which holds row rr: chunks behind the row's K-byte 128 s
    auto chunk_kc = [&](const Skew& k, int row, int rr) {
        const int c = (lane & 7) ^ swz_kc(row);
        return SKEW && c + k.shift(rr) >= 8 ? c - 8 : c;
    };
    // (SKEW: stages begin one line before a row's line 0, so that the offset is not negative)
    auto offset_kc = [&](const Skew& k, int row, int rr, int64_t ld) {
        return static_cast<uint32_t>(rr) * static_cast<uint32_t>(ld) + static_cast<uint32_t>(chunk_kc(k, row, rr) * 16 + (SKEW ? BK : 0));
    };
    uint32_t off_a[IT_A], off_b[IT_B], off_r = 0;
#pragma unroll
    for (int it = 0; it < IT_A; ++it) {
        const int row = (it * 4 + wave) * 8 + (lane >> 3);
        off_a[it] = offset_kc(skew_a, row, row < rows_a ? row : rows_a - 1, g.lda);
    }
#pragma unroll
    for (int it = 0; it < IT_B; ++it) {
        if (!B_KN) {
            const int row = (it * 4 + wave) * 8 + (lane >> 3);
            off_b[it] = offset_kc(skew_b, row, row < rows_b ? row : rows_b - 1, g.ldb);
        } else {
            const int krow = (it * 4 + wave) * RPI + lane / CH;
            int c = (lane % CH) ^ swz_kn<CH>(krow);
            c = c * 16 < rows_b ? c : rows_b / 16 - 1;
            off_b[it] = static_cast<uint32_t>(krow) * static_cast<uint32_t>(g.ldb) + c * 16;
        }
    }
    const int row_r = wave * 8 + (lane >> 3), rr_r = r0 + row_r < t.r ? row_r : static_cast<int>(t.r) - 1 - r0;
    if constexpr (RIDE) off_r = offset_kc(skew_r, row_r, rr_r, g.ldb);
    auto dma16 = [&](const uint8_t* src, uint8_t* dst_wave_uniform) {
        __builtin_amdgcn_global_load_lds(FQ_GLOBAL_PTR(src), FQ_LDS_PTR(dst_wave_uniform), 16, 0, 0);
    };
    // fetch j of the LPW that a wave makes for a stage that lies fully inside K
    auto fetch_one = [&](const uint8_t* pa, const uint8_t* pb, const uint8_t* pr, uint8_t* dst, int j) {
        if (j < IT_B) dma16(pb + off_b[j], dst + A_BYTES + wave * 1024 + j * 4096);
        else if (j < IT_B + IT_A) dma16(pa + off_a[j - IT_B], dst + wave * 1024 + (j - IT_B) * 4096);
        else if (RIDE) dma16(pr + off_r, dst + A_BYTES + B_BYTES + wave * 1024);
    };
    auto inside_a = [&](int s) { return opaque_uniform(base_a + static_cast<int64_t>(SKEW ? s - 1 : s) * BK); };
    auto inside_b = [&](int s) { return opaque_uniform(base_b + static_cast<int64_t>(SKEW ? s - 1 : s) * BK * (B_KN ? g.ldb : 1)); };
    auto inside_r = [&](int s) { return RIDE ? opaque_uniform(base_r + static_cast<int64_t>(SKEW ? s - 1 : s) * BK) : nullptr; };
    auto fetch = [&](int s, uint8_t* dst) {
        const int64_t k0 = static_cast<int64_t>(s) * BK;
        if (k0 + BK <= K && (!SKEW || s > 0)) {
            const uint8_t *pa = inside_a(s), *pb = inside_b(s), *pr = inside_r(s);
#pragma unroll
            for (int j = 0; j < LPW; ++j) fetch_one(pa, pb, pr, dst, j);
            return;
        }
        uint8_t* const da = dst + wave * 1024;
        uint8_t* const db = dst + A_BYTES + wave * 1024;
        // a lane's 16 bytes of a K-contiguous row, zeros where they lie outside the row
        auto row_chunk = [&](const uint8_t* base, uint32_t off, int chunk) {
            const int64_t gk = k0 + chunk * 16;
            return gk < K && (!SKEW || gk >= 0) ? base + (SKEW ? k0 - BK : k0) + off : g_zero16;
        };
#pragma unroll
        for (int it = 0; it < IT_B; ++it) {
            if (!B_KN) {
                const int row = (it * 4 + wave) * 8 + (lane >> 3);
                dma16(row_chunk(base_b, off_b[it], chunk_kc(skew_b, row, row < rows_b ? row : rows_b - 1)), db + it * 4096);
            } else {
                const int krow = (it * 4 + wave) * RPI + lane / CH;
                dma16(k0 + krow < K ? base_b + k0 * g.ldb + off_b[it] : g_zero16, db + it * 4096);
            }
        }
#pragma unroll
        for (int it = 0; it < IT_A; ++it) {
            const int row = (it * 4 + wave) * 8 + (lane >> 3);
            dma16(row_chunk(base_a, off_a[it], chunk_kc(skew_a, row, row < rows_a ? row : rows_a - 1)), da + it * 4096);
        }
        if constexpr (RIDE) dma16(row_chunk(base_r, off_r, chunk_kc(skew_r, row_r, rr_r)), dst + A_BYTES + B_BYTES + wave * 1024);
    };

    // ---- LDS -> matrix-core operands (layouts as in the large tiles) ----------------------------
    // K-contiguous operand: rows 32 block + lane % 32 of the tile at `offset` of a stage (SKEW: of two)
    auto read_kc = [&](const uint8_t* st, const uint8_t* st_next, int offset, const Skew& k, int block) {
        const int c = kh * 4 + (lane >> 5) * 2 + (SKEW ? k.shift(lane & 31) : 0), row = block * 32 + (lane & 31);
        return read_kc_tiles((SKEW && c >= 8 ? st_next : st) + offset, (SKEW && c >= 7 ? st_next : st) + offset, row, kh, lane);
    };
    // The transposing read goes out as inline assembly (through the builtin the compiler makes it wait
    // for every fetch in flight), so the compiler takes its results as there at once.  It copies registers
    // where control flow meets, so no read stays in flight across a branch: the reads of a stage, the matrix
    // instructions that hide them and the wait that names their results (landed) are one straight run.
    auto read_kn = [&](const uint8_t* tile, int ncol_base, v2i (&d)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int krow = kh * 64 + (lane >> 5) * 32 + q * 8 + ((lane & 15) >> 1);
            const int ncol = ncol_base + ((lane >> 4) & 1) * 16 + (lane & 1) * 8;
            const uint8_t* p = tile + krow * BN + ((((ncol >> 4) ^ swz_kn<CH>(krow)) << 4) | (ncol & 15));
            const uint32_t addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(FQ_LDS_PTR(p)));
            asm volatile("ds_read_b64_tr_b8 %0, %1" : "=v"(d[q]) : "v"(addr));
        }
    };

    constexpr int RBK = RIDE ? mid_max(MB / 2, 1) : 0;           // 32x32 blocks of O_A per wave
    constexpr int NBK = MB * NB + RBK;
    // The wave's token blocks in the order mi ^ perm, so that its blocks of O_A are on its first ones whatever wn is (a
    // branch on wn in the steady loop made the compiler move accumulators about: a step took 1.7 times as long).
    const int perm = RIDE && MB > 1 ? wn * RBK : 0;
    v16f acc[NBK];
#pragma unroll
    for (int b = 0; b < NBK; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[b][v] = 0.0f;
    v8i af[2][MB], bf[2][NB], rf[2];
    v2i bt[2][NB][4];

    const int KT = static_cast<int>((K + BK - 1) / BK), stages = KT + (SKEW ? 1 : 0);
    constexpr int N_FRAG = NB + MB + (RIDE ? 1 : 0);
    // (st_next: the stage behind st, looked at if SKEW)
    auto read_frag = [&](auto parity, const uint8_t* st, const uint8_t* st_next, int f) {
        constexpr int P = decltype(parity)::value;
        if (f < NB) {
            if constexpr (B_KN) read_kn(st + A_BYTES, wn * NB * 32 + f * 32, bt[P][f]);
            else bf[P][f] = read_kc(st, st_next, A_BYTES, skew_b, wn * NB + f);
        } else if (f < NB + MB) {
            af[P][f - NB] = read_kc(st, st_next, 0, skew_a, (f - NB) ^ perm);
        } else if (RIDE) {
            rf[P] = read_kc(st, st_next, A_BYTES + B_BYTES, skew_r, 0);
        }
    };
    auto read_stage = [&](auto parity, const uint8_t* st, const uint8_t* st_next) {
#pragma unroll
        for (int f = 0; f < N_FRAG; ++f) read_frag(parity, st, st_next, f);
    };
    auto landed = [&](auto parity) {
        if constexpr (B_KN) {
            constexpr int P = decltype(parity)::value;
            __builtin_amdgcn_sched_barrier(0);                    // behind the matrix instructions
#pragma unroll
            for (int ni = 0; ni < NB; ++ni) {
                asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(bt[P][ni][0]), "+v"(bt[P][ni][1]), "+v"(bt[P][ni][2]), "+v"(bt[P][ni][3]));
#pragma unroll
                for (int q = 0; q < 4; ++q) { bf[P][ni][2 * q] = bt[P][ni][q][0]; bf[P][ni][2 * q + 1] = bt[P][ni][q][1]; }
            }
        }
    };
    // ---- adapter gradient: dB = dy~^T O_A~ over this tile's tokens ---------------------------------
    // The stages of the left operand are dy~ [tokens][128 features]; the tiles of a tile row share the
    // K-steps out among themselves, and for its own ones a tile also contracts the stage over its
    // tokens with the O_A codes it keeps beside the ring ([token][256 bytes], chunks XOR-swizzled):
    // no second read of dy~, no launch.  Tokens beyond M read zero codes, so the clamped rows of the
    // stage drop out.  Wave w owns features [32 w, +32).
    uint8_t* const lds_oa = lds + S * STAGE;
    const int db_per = DB ? (KT + t.tiles_n - 1) / t.tiles_n : 0;
    const int db_begin = tile_n * db_per, db_end = db_begin + db_per < KT ? db_begin + db_per : KT;
    auto read_tokens = [&](const uint8_t* tile, int pitch, int feat_base, int t0, bool kc) -> v8i {
        // 32 tokens of one feature per lane, as read_kn; waited for in the same asm block
        uint32_t addr[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int tok = t0 + (BM >= 64 ? (lane >> 5) * 32 : 0) + q * 8 + ((lane & 15) >> 1);
            const int feat = feat_base + ((lane >> 4) & 1) * 16 + (lane & 1) * 8;
            const int chunk = (feat >> 4) ^ (kc ? swz_kc(tok) : (tok & 7));
            const uint8_t* p = tile + tok * pitch + (chunk << 4) + (feat & 15);
            addr[q] = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(FQ_LDS_PTR(p)));
        }
        v2i d0, d1, d2, d3;
        asm volatile("ds_read_b64_tr_b8 %0, %4\n\tds_read_b64_tr_b8 %1, %5\n\tds_read_b64_tr_b8 %2, %6\n\t"
                     "ds_read_b64_tr_b8 %3, %7\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(d0), "=&v"(d1), "=&v"(d2), "=&v"(d3) : "v"(addr[0]), "v"(addr[1]), "v"(addr[2]), "v"(addr[3]));
        v8i x;
        x[0] = d0[0]; x[1] = d0[1]; x[2] = d1[0]; x[3] = d1[1]; x[4] = d2[0]; x[5] = d2[1]; x[6] = d3[0]; x[7] = d3[1];
        if (BM < 64 && lane >= 32) {                              // 32 tokens: the upper half of the depth is empty
#pragma unroll
            for (int q = 0; q < 8; ++q) x[q] = 0;
        }
        return x;
    };
    auto db_stage = [&](const uint8_t* st, int kt) {
        constexpr int DEPTH = BM >= 64 ? BM / 64 : 1;
        v8i a[DEPTH];
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) a[d] = read_tokens(st, BK, wave * 32, d * 64, true);
        float* const out = t.db_partial + static_cast<int64_t>(tile_m) * K * t.r;
        const int64_t i0 = static_cast<int64_t>(kt) * BK + wave * 32 + (lane >> 5) * 4;
        for (int pb = 0; pb * 32 < t.r; ++pb) {
            v16f c;
#pragma unroll
            for (int v = 0; v < 16; ++v) c[v] = 0.0f;
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                const v8i b = read_tokens(lds_oa, 256, pb * 32, d * 64, false);
                c = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a[d], b, c, 1 /* E5M2 */, 0 /* E4M3 */, 0, 0, 0, 0);
            }
            const int64_t p = pb * 32 + (lane & 31);
            if (p >= t.r) continue;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t i = i0 + (v >> 2) * 8 + (v & 3);
                if (i < K) out[i * t.r + p] = c[v];
            }
        }
    };
    constexpr int NEED = SKEW ? 2 : 1;                            // operands of step kt + 1 lie in stages up to kt + NEED
    int slot = 0;                                                 // ring slot of stage kt
    // STEADY: stage kt + S exists and lies inside K, so that the body carries no branch.  The others read a
    // stage kt + 1 too where there is none (bytes of the ring that nothing uses): a branch around the reads
    // would end the straight run.
    auto step = [&](auto parity, auto steady_tag, int kt) {
        constexpr int P = decltype(parity)::value;
        constexpr bool STEADY = decltype(steady_tag)::value;
        // the operands of kt are in registers, stage kt + NEED has landed (of the stages behind it, those already
        // fetched stay in flight) ...
        if constexpr (STEADY) {
            __builtin_amdgcn_s_waitcnt((((S - 1 - NEED) * LPW) & 15) | (7 << 4) | ((((S - 1 - NEED) * LPW) >> 4) << 14));
        } else {
            const int out = (stages - 1 < kt + S - 1 ? stages - 1 : kt + S - 1) - (kt + NEED);
            WaitStages<S - 1 - NEED>::template run<LPW>(out > 0 ? out : 0);
        }
        barrier_lds_only();                                       // ... for every wave: the slot of stage kt is free
        uint8_t* const freed = lds + slot * STAGE;
        slot = slot + 1 == S ? 0 : slot + 1;
        const uint8_t* const st = lds + slot * STAGE;
        const uint8_t* const st_next = SKEW ? lds + (slot + 1 == S ? 0 : slot + 1) * STAGE : st;
        const uint8_t *pa = nullptr, *pb = nullptr, *pr = nullptr;
        if constexpr (STEADY) {
            pa = inside_a(kt + S); pb = inside_b(kt + S); pr = inside_r(kt + S);
        } else {
            if (kt + S < stages) fetch(kt + S, freed);
        }
        if constexpr (DB) {
            if (kt + 1 >= db_begin && kt + 1 < db_end) db_stage(st, kt + 1);
        }
        if constexpr (!STEADY) read_stage(std::integral_constant<int, 1 - P>{}, st, st_next);
        // The fetches are spread over the matrix instructions: a wave that issues them back to back, ahead
        // of its LDS reads, stalls on the CU's 64 B/clk vector-memory path.
        constexpr int PER = (LPW + MB * NB - 1) / (MB * NB), FPER = (N_FRAG + MB * NB - 1) / (MB * NB);
#pragma unroll
        for (int b = 0; b < MB * NB; ++b) {
            const int mi = b / NB, ni = b % NB;
            acc[b] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(bf[P][ni], af[P][mi], acc[b], 0 /* E4M3 */, A_FMT, 0, 0, 0, 0);
            if constexpr (STEADY) {
#pragma unroll
                for (int u = 0; u < (PER > FPER ? PER : FPER); ++u) {
                    if (u < FPER && b * FPER + u < N_FRAG)
                        read_frag(std::integral_constant<int, 1 - P>{}, st, st_next, b * FPER + u);
                    if (u < PER && b * PER + u < LPW) fetch_one(pa, pb, pr, freed, b * PER + u);
                    __builtin_amdgcn_sched_barrier(0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (RIDE) {
            // wave column wn takes token blocks [wn * RBK, +RBK) of the tile (MB = 1: both form the one)
#pragma unroll
            for (int j = 0; j < RBK; ++j)
                acc[MB * NB + j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(rf[P], af[P][j], acc[MB * NB + j], 0, 0, 0, 0, 0, 0);
        }
        landed(std::integral_constant<int, 1 - P>{});
    };
    float inv;
    {
        const int first = stages < S ? stages : S;
        if constexpr (DB) {
            if (db_begin < db_end) {                              // 4 token rows of 256 bytes per wave instruction
#pragma unroll
                for (int it = 0; it < BM / 16; ++it) {
                    const int row = (it * 4 + wave) * 4 + (lane >> 4);
                    const int64_t gt = m0 + row, gp = ((lane & 15) ^ (row & 7)) << 4;
                    dma16((gt < M && gp < t.r) ? t.oaq + gt * t.r + gp : g_zero16, lds_oa + (it * 4 + wave) * 1024);
                }
            }
        }
        for (int s = 0; s < first; ++s) fetch(s, lds + s * STAGE);
        // rescale factor: read behind the first fetches, so that its memory round trip hides under theirs
        inv = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(1.0f / ((*g.sa) * (*g.sb)))));
        WaitStages<S - NEED>::template run<LPW>(first - NEED);
        barrier_lds_only();
        read_stage(std::integral_constant<int, 0>{}, lds, lds + STAGE);
        landed(std::integral_constant<int, 0>{});
        if constexpr (DB) {
            if (db_begin == 0 && db_end > 0) db_stage(lds, 0);
        }
        const int steady = static_cast<int>(K / BK) - S;          // steps whose stage kt + S is a full one
        int kt = 0;
        for (; kt + 1 < steady; kt += 2) {
            step(std::integral_constant<int, 0>{}, std::true_type{}, kt);
            step(std::integral_constant<int, 1>{}, std::true_type{}, kt + 1);
        }
        for (; kt < KT; kt += 2) {
            step(std::integral_constant<int, 0>{}, std::false_type{}, kt);
            if (kt + 1 < KT) step(std::integral_constant<int, 1>{}, std::false_type{}, kt + 1);
        }
    }

    // ---- the two K halves meet: each wave finishes the blocks whose index has its parity ------------
    __syncthreads();                                              // the ring is no longer read
#pragma unroll
    for (int b = 0; b < NBK; ++b) {
        if ((b & 1) == kh) continue;
        float4* ex = reinterpret_cast<float4*>(lds) + (wn * NBK + b) * 256 + lane;
#pragma unroll
        for (int q = 0; q < 4; ++q) ex[q * 64] = make_float4(acc[b][4 * q], acc[b][4 * q + 1], acc[b][4 * q + 2], acc[b][4 * q + 3]);
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < NBK; ++b) {
        if ((b & 1) != kh) continue;
        const float4* ex = reinterpret_cast<const float4*>(lds) + (wn * NBK + b) * 256 + lane;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 v = ex[q * 64];
            acc[b][4 * q] = (acc[b][4 * q] + v.x) * inv;
            acc[b][4 * q + 1] = (acc[b][4 * q + 1] + v.y) * inv;
            acc[b][4 * q + 2] = (acc[b][4 * q + 2] + v.z) * inv;
            acc[b][4 * q + 3] = (acc[b][4 * q + 3] + v.w) * inv;
        }
    }
    __syncthreads();

    // ---- O_A blocks straight from registers: lane l holds token row l % 32 and runs of four ranks -----
    float oa_max = 0.0f;
    auto abs_max2 = [](uint32_t w) { return fmaxf(fabsf(__uint_as_float(w << 16)), fabsf(__uint_as_float(w & 0xffff0000u))); };
    if constexpr (RIDE) {
#pragma unroll
        for (int j = 0; j < RBK; ++j) {
            if (((MB * NB + j) & 1) != kh || (MB == 1 && wn)) continue;
            const int64_t row = m0 + (MB > 1 ? wn * RBK + j : 0) * 32 + (lane & 31);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int col = r0 + q * 8 + (lane >> 5) * 4;
                if (row >= M || col >= t.r) continue;
                const v16f& a = acc[MB * NB + j];
                uint2 pk;
                pk.x = pack_bf16x2(a[4 * q], a[4 * q + 1]);
                pk.y = pack_bf16x2(a[4 * q + 2], a[4 * q + 3]);
                *reinterpret_cast<uint2*>(static_cast<uint16_t*>(g.c1) + row * g.ldc1 + col) = pk;
                oa_max = fmaxf(oa_max, fmaxf(abs_max2(pk.x), abs_max2(pk.y)));
            }
        }
    }

    // ---- the tile: convert, stage through LDS, store row-contiguous -----------------------------------
    auto epilogue = [&](auto is_f32, void* out, int64_t ld) {
        constexpr bool F32 = decltype(is_f32)::value;
        constexpr int ES = F32 ? 4 : 2;
        constexpr int PITCH = BN * ES + 16, SEGS = BN * ES / 16, COLS = 16 / ES, PIECES = BM * SEGS / 256;
        uint4 held[ADDS ? PIECES : 1];                            // on its way while the tile is parked
        if constexpr (ADDS) {
#pragma unroll
            for (int it = 0; it < PIECES; ++it) {
                const int sidx = it * 256 + static_cast<int>(threadIdx.x);
                const int64_t row = m0 + sidx / SEGS, col = n0 + sidx % SEGS * COLS;
                if (row < M && col < N) held[it] = *reinterpret_cast<const uint4*>(static_cast<const uint8_t*>(out) + (row * ld + col) * ES);
            }
        }
#pragma unroll
        for (int mi = 0; mi < MB; ++mi)
#pragma unroll
            for (int ni = 0; ni < NB; ++ni) {
                if (((mi * NB + ni) & 1) != kh) continue;
                uint8_t* srow = lds + ((mi ^ perm) * 32 + (lane & 31)) * PITCH;
                const v16f& a = acc[mi * NB + ni];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int c = (wn * NB + ni) * 32 + q * 8 + (lane >> 5) * 4;
                    if (F32) {
                        *reinterpret_cast<float4*>(srow + c * 4) = make_float4(a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]);
                    } else {
                        uint2 pk;
                        pk.x = pack_bf16x2(a[4 * q], a[4 * q + 1]);
                        pk.y = pack_bf16x2(a[4 * q + 2], a[4 * q + 3]);
                        *reinterpret_cast<uint2*>(srow + c * 2) = pk;
                    }
                }
            }
        __syncthreads();
        if constexpr (ADDS) {
#pragma unroll
            for (int it = 0; it < PIECES; ++it) {
                const int sidx = it * 256 + static_cast<int>(threadIdx.x);
                const int srw = sidx / SEGS, seg = sidx % SEGS;
                const int64_t row = m0 + srw, col = n0 + seg * COLS;
                if (row >= M || col >= N) continue;
                *reinterpret_cast<uint4*>(static_cast<uint8_t*>(out) + (row * ld + col) * ES) =
                    add_bf16x8(held[it], *reinterpret_cast<const uint4*>(lds + srw * PITCH + seg * 16));
            }
            return;
        }
        for (int it = 0; it < PIECES; ++it) {
            const int sidx = it * 256 + static_cast<int>(threadIdx.x);
            const int srw = sidx / SEGS, seg = sidx % SEGS;
            const int64_t row = m0 + srw, col = n0 + seg * COLS;
            if (row >= M || col >= N) continue;
            const uint4 d = *reinterpret_cast<const uint4*>(lds + srw * PITCH + seg * 16);
            uint8_t* dst = static_cast<uint8_t*>(out) + (row * ld + col) * ES;
            if (adapter) {
                *reinterpret_cast<uint4*>(dst) = d;
                oa_max = fmaxf(oa_max, fmaxf(fmaxf(abs_max2(d.x), abs_max2(d.y)), fmaxf(abs_max2(d.z), abs_max2(d.w))));
            } else {
                typedef unsigned v4u __attribute__((ext_vector_type(4)));
                const v4u dd = {d.x, d.y, d.z, d.w};
                __builtin_nontemporal_store(dd, reinterpret_cast<v4u*>(dst));
            }
        }
    };
    if (adapter) epilogue(std::false_type{}, g.c1, g.ldc1);
    else if (!ADDS && g.c0_is_f32) epilogue(std::true_type{}, g.c0, g.ldc0);
    else epilogue(std::false_type{}, g.c0, g.ldc0);
    if ((RIDE || adapter) && g.amax1) {
        oa_max = wave_max(oa_max);
        // non-negative floats order like their bit patterns
        if (lane == 0 && oa_max > 0.0f) atomicMax(g.amax1, __float_as_uint(oa_max));
    }
}

// Workgroup -> tile: XCD x (workgroup index modulo 8) takes tiles [x * chunk, (x + 1) * chunk) of a raster
// that walks panels of PH tile rows, tile column by tile column: the token panel of an XCD stays in its
// L2 and every weight column is fetched by one XCD per panel.
template <int MB, int NB, int S, bool B_KN, int A_FMT, bool DB, bool SKEW, bool ADDS>
__device__ __forceinline__ void mid_workgroup(const MidArgs& t, const int bid, uint8_t* const lds)
{
    constexpr bool FWD = !B_KN && A_FMT == 0;
    const int tile_id = (bid & 7) * t.chunk + (bid >> 3);
    const int cols = t.tiles_n + t.tiles_a;
    if (tile_id >= t.tiles_m * cols) return;
    constexpr int PH = 16;
    const int per_panel = PH * cols;
    const int panel = tile_id / per_panel, rem = tile_id - panel * per_panel;
    const int ph = (t.tiles_m - panel * PH) < PH ? (t.tiles_m - panel * PH) : PH;
    const int tile_n = rem / ph, tile_m = panel * PH + (rem - tile_n * ph);
    if constexpr (FWD) {
        if (tile_n < t.ride) {
            mid_tile<MB, NB, S, B_KN, A_FMT, true, DB, SKEW, false>(t, tile_m, tile_n, false, lds);
            return;
        }
    }
    mid_tile<MB, NB, S, B_KN, A_FMT, false, DB, SKEW, ADDS>(t, tile_m, tile_n, tile_n >= t.tiles_n, lds);
}

template <int MB, int NB, int S, bool B_KN, int A_FMT, bool DB, bool SKEW, bool ADDS = false>
__global__ void __launch_bounds__(256)
gemm_mid_kernel(const MidArgs t)
{
    __shared__ __attribute__((aligned(1024))) uint8_t lds[mid_lds_bytes<MB, NB, S, !B_KN && A_FMT == 0, DB>()];
    mid_workgroup<MB, NB, S, B_KN, A_FMT, DB, SKEW, ADDS>(t, blockIdx.x, lds);
}

// The input-gradient product, and behind its `product` workgroups those of the adapter gradient's tiles (db_tile.h): both
// read only dy~, the weight and O_A.  For products that leave CUs idle, which then form dB meanwhile.
template <int MB, int NB, int S, bool ADDS>
__global__ void __launch_bounds__(256)
gemm_mid_db_kernel(const MidArgs t, const DbArgs d, const int product)
{
    constexpr int LDS = mid_max(mid_lds_bytes<MB, NB, S, false, false>(), static_cast<int>(dbt::kDbLdsBytes));
    static_assert(dbt::kThreads == 256, "one workgroup shape for both kinds of tile");
    __shared__ __attribute__((aligned(1024))) uint8_t lds[LDS];
    const int b = static_cast<int>(blockIdx.x) - product;
    if (b >= 0) {
        const int bi = b % d.i_tiles, rest = b / d.i_tiles;
        dbt::db_partial_tile(d, bi, rest % d.splits, rest / d.splits, lds, g_zero16);
        return;
    }
    mid_workgroup<MB, NB, S, true, 1, false, false, ADDS>(t, blockIdx.x, lds);
}

// Adapter columns of their own cost nothing while they make no further round over the CUs; a step of a tile that
// carries them along takes 1.15 times as long.  Returns the extra tile columns, 0: they ride.
int own_columns(int64_t tiles_m, int64_t tiles_n, int64_t r, int bn)
{
    const int64_t own = (r + bn - 1) / bn;
    const bool fits = (tiles_m * (tiles_n + own) - 1) / kMidCus == (tiles_m * tiles_n - 1) / kMidCus;
    return tiles_n < (r + 31) / 32 || fits ? static_cast<int>(own) : 0;
}

// SKEW is for K from long_rows steps on (launch_gemm_mid).
template <int MB, int NB, int S_FWD, int S_KN, int S_DB>
hipError_t launch_cfg(MidArgs t, int long_rows, const DbArgs* db, hipStream_t stream)
{
    constexpr int BM = 32 * MB, BN = 64 * NB;
    t.tiles_m = static_cast<int>((t.g.M + BM - 1) / BM);
    t.tiles_n = static_cast<int>((t.g.N + BN - 1) / BN);
    t.tiles_a = t.ride = 0;
    if (t.side) {
        t.tiles_a = own_columns(t.tiles_m, t.tiles_n, t.r, BN);
        if (!t.tiles_a) t.ride = static_cast<int>((t.r + 31) / 32);
    }
    t.chunk = (t.tiles_m * (t.tiles_n + t.tiles_a) + 7) / 8;
    const dim3 grid(static_cast<unsigned>(8 * t.chunk)), block(256);
    // rows that do not all begin with a cache line (of a single row only its place counts)
    auto across = [](const uint8_t* p, int64_t ld) { return ((reinterpret_cast<uintptr_t>(p) | static_cast<uintptr_t>(ld)) & (BK - 1)) != 0; };
    const bool skew = t.g.K >= long_rows * BK && (across(t.g.a, t.g.lda) || across(t.g.b, t.g.ldb) || (t.side && across(t.side, t.g.ldb)));
    if (db) {
        const dim3 both(grid.x + static_cast<unsigned>(db->i_tiles * db->splits * db->p_tiles));
        if (t.g.c0_adds) gemm_mid_db_kernel<MB, NB, S_KN, true><<<both, block, 0, stream>>>(t, *db, static_cast<int>(grid.x));
        else gemm_mid_db_kernel<MB, NB, S_KN, false><<<both, block, 0, stream>>>(t, *db, static_cast<int>(grid.x));
        return hipGetLastError();
    }
    auto go = [&](auto kernel) { kernel<<<grid, block, 0, stream>>>(t); };
    if (t.g.b_is_kn) {
        if (t.g.a_fmt == 0) go(gemm_mid_kernel<MB, NB, S_KN, true, 0, false, false>);
        else if (t.g.c0_adds && t.oaq) go(gemm_mid_kernel<MB, NB, S_DB, true, 1, true, false, true>);
        else if (t.g.c0_adds) go(gemm_mid_kernel<MB, NB, S_KN, true, 1, false, false, true>);
        else if (t.oaq) go(gemm_mid_kernel<MB, NB, S_DB, true, 1, true, false>);
        else go(gemm_mid_kernel<MB, NB, S_KN, true, 1, false, false>);
    } else if (t.g.a_fmt == 0) {
        if (skew) go(gemm_mid_kernel<MB, NB, S_FWD, false, 0, false, true>);
        else go(gemm_mid_kernel<MB, NB, S_FWD, false, 0, false, false>);
    } else {
        if (skew) go(gemm_mid_kernel<MB, NB, S_KN, false, 1, false, true>);
        else go(gemm_mid_kernel<MB, NB, S_KN, false, 1, false, false>);
    }
    return hipGetLastError();
}

}  // namespace

bool gemm_mid_supported(int64_t M, int64_t N)
{
    return !use_big_tiles(M, N) && ((M + 127) / 128) * ((N + 127) / 128) <= kMidCus;
}

// us = launch + rounds over the CUs x (round + K-steps x (step + step_full x part of the CUs that are busy)): a
// workgroup is alone on its CU, so every round pays the way into its rings and out again, and a step takes longer
// the more CUs draw on the memory.  Fitted to products of 20 sizes with K from 64 to 8192 (graphs of 10; the fit is
// within 5 %, and the choice by it 0.2 % slower than the best of all on average; with the riding steps at 1.15 and 1.0 us
// for their way out, forwards of 44 drawn layers are 0.1 % off the best on average, 3 % at worst).  Tiles that find room in one
// round win; 2 to 8 rounds of smaller ones take up to twice as long (1024 x 4096, K = 128: 12.2 us in four rounds of
// 64x64, 7.7 with 128x128).
MidPlan plan_mid(int64_t M, int64_t N, int64_t K, bool b_is_kn, int64_t r)
{
    struct Cost { double launch, round, step, step_full; };
    struct { int bm, bn; Cost nk, kn; } const cfg[] = {
        {32, 64, {2.2, 2.1, 0.114, 0.041}, {2.2, 2.15, 0.143, 0.105}},
        {64, 64, {2.1, 2.4, 0.138, 0.071}, {2.1, 2.5, 0.178, 0.134}},
        {64, 128, {2.0, 3.3, 0.198, 0.103}, {1.8, 3.6, 0.253, 0.104}},
        {128, 128, {2.9, 4.0, 0.247, 0.241}, {2.4, 4.7, 0.320, 0.226}}};
    const double steps = static_cast<double>((K + BK - 1) / BK);
    MidPlan best{0, 0, 0, 0.0};
    for (int c = 0; c < 4; ++c) {
        const Cost& k = b_is_kn ? cfg[c].kn : cfg[c].nk;
        const int64_t tm = (M + cfg[c].bm - 1) / cfg[c].bm, tn = (N + cfg[c].bn - 1) / cfg[c].bn;
        const int own = r ? own_columns(tm, tn, r, cfg[c].bn) : 0;
        const int64_t tiles = tm * (tn + own);
        const double busy = tiles < kMidCus ? static_cast<double>(tiles) / kMidCus : 1.0;
        const double us = k.launch + (r && !own ? 1.0 : 0.0) +
                          static_cast<double>((tiles + kMidCus - 1) / kMidCus) *
                              (k.round + steps * (r && !own ? 1.15 : 1.0) * (k.step + k.step_full * busy));
        if (c == 0 || us < best.us) best = MidPlan{c, cfg[c].bm, tn, us};
    }
    return best;
}

hipError_t launch_gemm_mid(const GemmArgs& g, const MidSide& side, hipStream_t stream)
{
    MidArgs t;
    t.g = g; t.side = side.rows; t.r = side.r; t.oaq = side.oaq; t.db_partial = side.db_partial;
    // The last argument of a configuration: K-steps from which rows across cache lines are fetched by whole lines.  Where the
    // rows are shorter or the tiles smaller, the line that one step leaves half used is still near when the next one asks for
    // it, and the stage more costs 0.3 to 1 us.  Plain products, us, by whole lines (from the rows' first bytes): 128-token
    // tiles 1500 x 2000, K = 1040 11.5 (11.2), K = 1552 12.8 (13.1), K = 4112 21.0 (25.9), K = 8208 32.9 (41.9); 64 x 128 512 x 4096,
    // K = 1040 8.4 (8.6), K = 1552 9.2 (10.4), K = 4112 15.2 (18.5), K = 8208 24.6 (32.6).
    // The small tiles' lines are for weights that come from memory, as they do in a model, where other layers' calls lie between
    // two of one layer: 64 x 64 256 x 4096, K = 5136 17.5 (24.2), 500 x 1504, K = 5136 12.9 (16.3); 32 x 64 128 x 4096, K = 8208 19.2
    // (23.8), 100 x 3008, K = 8208 16.4 (18.9), 64 x 1024, K = 8208 13.8 (15.8).  For calls back to back on one weight that the caches still
    // hold they can be the slower way: 13.2 (14.6), 12.5 (11.5), 15.4 (16.5), 14.1 (12.5), 13.1 (11.4).  From memory whole lines are ahead
    // from K = 3088 on in all of 120 products of 17 to 500 tokens (1.02 to 1.49 times as fast), from the caches in 39 of 45 from K = 11024 on (the others down to 0.85).
    // [K,N] operands: only the left one has such rows, 0.3 to 0.5 us slower up to K = 2064,
    // 2 to 5 % faster from 4112 on: not built.
    switch (plan_mid(g.M, g.N, g.K, g.b_is_kn != 0, side.rows ? side.r : 0).config) {
        case 0: return launch_cfg<1, 1, 8, 8, 8>(t, 64, side.db, stream);
        case 1: return launch_cfg<2, 1, 7, 8, 8>(t, 40, side.db, stream);
        case 2: return launch_cfg<2, 2, 5, 6, 6>(t, 12, side.db, stream);
        default: return launch_cfg<4, 2, 4, 5, 4>(t, 12, side.db, stream);
    }
}

}  // namespace falqon
