// Launch interface of the small-tile FP8 products (gemm_mid.hip).
#pragma once
#include "falqon_internal.h"

namespace falqon {

bool use_big_tiles(int64_t M, int64_t N);    // gemm.hip: the 256x256 tiles fill the chip
// gemm.hip: time of launch_gemm for this product, by the cost rules of both families
double product_us(int64_t M, int64_t N, int64_t K, bool b_is_kn);

// What a launch does for the adapter besides the product g.
struct MidSide {
    const uint8_t* rows = nullptr;   // forward: adapter rows [r][K] (row stride g.ldb): O_A (bf16) goes to g.c1, its
                                     // maximum to g.amax1
    int64_t r = 0;
    const uint8_t* oaq = nullptr;    // input gradient (E5M2 left operand): O_A codes [M][r]; partial sums of
    float* db_partial = nullptr;     // dy~^T O_A~ go to db_partial[tile row][K][r], not rescaled
    const DbArgs* db = nullptr;      // instead: these tiles of the adapter gradient are workgroups of their own in the launch
};
bool gemm_mid_supported(int64_t M, int64_t N);                   // the 128x128 tiles of a product of this size all find a CU
// Tile configuration of a product, the one of least time; r: rank of the adapter whose O_A it forms along (0: none).
struct MidPlan { int config; int rows; int64_t columns; double us; };   // tokens per tile row, tile columns
MidPlan plan_mid(int64_t M, int64_t N, int64_t K, bool b_is_kn, int64_t r);
hipError_t launch_gemm_mid(const GemmArgs& g, const MidSide& side, hipStream_t stream);

}  // namespace falqon
