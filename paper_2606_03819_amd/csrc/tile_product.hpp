// The approximator's bf16 products on the block-tiled GEMM: arguments and
// launchers (tile_product.hip), used by the AR approximator (mlp.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "plan.hpp"
#include "rows.hpp"

namespace tf {

// what becomes of a product
constexpr int kTileStore = 0;      // fp32 table [splits][R][N]
constexpr int kTileSwiGLU = 1;     // silu(gate) * up as bf16 hi/lo pairs
constexpr int kTileSiLU = 2;       // silu(gate) as bf16 hi/lo pairs
constexpr int kTileResidual = 3;   // + h, bf16

// One product of a launch: its weight columns, activations and fp32 output.
struct TileSegment {
    const uint16_t *wa, *wb;   // weight rows (gate and up rows where `gateup`)
    const uint16_t* x;
    int R;
    float* table;
};

// The final sums: own-row tables (or the accumulators), the h~ half of each
// row's drafter state and, for the bigram rows, the products of its two
// previous tokens.
struct TileFinish {
    int epi;
    int R, N;             // rows, product columns (gate and up columns interleaved by 8)
    uint16_t* out;        // activation pairs [R, 2 * width] or h' [R, width]
    int width;            // I or d
    const uint16_t* h;    // [states, width] (residual)
    const float* own;     // [nown][R][N]
    int nown;
    const float* hh;      // [nhh][states][N]
    int nhh, states;
    const float *t1, *t2; // [tokens][N], bigram rows only
    RowTable rt;
};

struct TileProductArgs {
    TileSegment seg[3];
    int nseg;
    bool gateup;          // weight rows alternate 8 gate rows, 8 up rows
    int N, Kw, K;         // product columns, weight row stride, reduction range
    long ldx;
    TileFinish fin;       // S == 1 and fin.epi != kTileStore: applied to the accumulators
};

// seg[0 .. nseg) of one shape: tables, or (S == 1, one segment) the finished outputs
hipError_t launch_tile_product(const TilePlan& p, bool paired, const TileProductArgs& a, hipStream_t st);
// the finished outputs from tables
hipError_t launch_tile_finish(const TileFinish& f, hipStream_t st);

}  // namespace tf
