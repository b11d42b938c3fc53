// Launch interface of the small-tile FP8 products (gemm_mid.hip).
#pragma once
#include "falqon_internal.h"

namespace falqon {

bool use_big_tiles(int64_t M, int64_t N);    // gemm.hip: the 256x256 tiles fill the chip
hipError_t launch_gemm_tiles(const GemmArgs& g, hipStream_t stream);   // gemm.hip: the large-tile family whatever the size

// What a launch does for the adapter besides the product g.
struct MidSide {
    const uint8_t* rows = nullptr;   // forward: adapter rows [r][K] (row stride g.ldb): O_A (bf16) goes to g.c1, its
                                     // maximum to g.amax1
    int64_t r = 0;
    const uint8_t* oaq = nullptr;    // input gradient (E5M2 left operand): O_A codes [M][r]; partial sums of
    float* db_partial = nullptr;     // dy~^T O_A~ go to db_partial[tile row][K][r], not rescaled
};
constexpr int kMidConfigs = 4;
bool gemm_mid_supported(int64_t M, int64_t N);                   // products of this size run on the small tiles
int mid_tile_rows(int64_t M, int64_t N, int64_t K);              // tokens per tile row of the configuration chosen by size
int64_t mid_tile_columns(int64_t M, int64_t N, int64_t K);       // tile columns of it
// cfg: tile configuration, -1 to choose by size
hipError_t launch_gemm_mid(const GemmArgs& g, const MidSide& side, int cfg, hipStream_t stream);

}  // namespace falqon
