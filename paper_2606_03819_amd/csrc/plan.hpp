// Launch plans and workspace layout shared by the C ABI and the launchers.
// Host-only; every function here is a pure function of the shapes, so the
// workspace size the caller is told and the layout the kernels use agree.
#pragma once

#include <initializer_list>

#include <stddef.h>
#include <stdint.h>

#include "limits.hpp"
#include "rows.hpp"
#include "work.hpp"

namespace tf {

constexpr int kMaxSplits = 2048;       // vocabulary slices (partials per row); kMaxSplits*kKeep <= merge capacity
constexpr int kMaxSplitsLong = 1024;   // slices up to which a launch may keep long lists
constexpr int kMaxTopk = 1024;         // longest top-k list the merge kernel sorts
constexpr int kMaxBudget = 4095;       // tree nodes per sequence
constexpr int kNumCUs = 256;           // compute units of an MI355X

// Tile ranges (workgroups) of the LM head when a single row block streams
// the whole vocabulary.
#ifndef TF_LM_WORKGROUPS
#define TF_LM_WORKGROUPS 256
#endif
// Pipeline depth (k-chunks of loads in flight per wave) when a single row
// block streams the weights once at NT = 4, and otherwise; the launchers pick
// the kernel instance from NT and wnt.
#ifndef TF_PIPE_SINGLE_NT4
#define TF_PIPE_SINGLE_NT4 3
#endif
#ifndef TF_PIPE_DEFAULT
#define TF_PIPE_DEFAULT 2
#endif

inline int cdiv(long long a, long long b) { return (int)((a + b - 1) / b); }
inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

inline int plan_nt(int rows) { return rows <= 32 ? 1 : (rows <= 64 ? 2 : 4); }

// LM head over [rows, d] x [V, d]: vocabulary slices (see SliceMap), one
// workgroup per (tile range, row block), the row blocks of a range on
// consecutive workgroups so that they share its tiles through L2.  One row
// block: the tiles spread over TF_LM_WORKGROUPS workgroups; more row blocks:
// lm_tile_plan below, narrow widths apart.  fp32 (SIMT kernel): 16 rows and 1 to
// 8 tiles (256 tokens) per workgroup.
struct LmPlan {
    int NT, WM, NW, chunk, nrb, ntiles, nk;
    int WB = 1;   // waves along the activation tiles (a grid of NW / WB x WB waves)
    bool grid = false;   // the DMA kernel's 2 x 2 wave grid (33 to 256 rows)
    SliceMap map;
    bool wnt;   // weight loads carry the non-temporal hint
    bool dma;   // the LDS-DMA kernel (32-row tiles, the grid, or 256-row blocks)
    // the block-tiled kernel (tile_gemm.hpp): WM and NT count 16-row tiles of
    // one of its 2 x 2 waves
    bool tile = false;
    int nsplit() const { return map.G * map.rmax; }
    int blocks() const { return map.G * nrb; }
};

// LM-head tile shape per activation-tile count: waves per workgroup and
// weight tiles per wave (one wave per SIMD when NW = 4, so that a wave may
// hold 128 accumulator registers).
#ifndef TF_LM_NW_NT1
#define TF_LM_NW_NT1 4
#endif
#ifndef TF_LM_WM_NT1
#define TF_LM_WM_NT1 4
#endif
#ifndef TF_LM_NW_NT2
#define TF_LM_NW_NT2 8
#endif
#ifndef TF_LM_WM_NT2
#define TF_LM_WM_NT2 1
#endif
#ifndef TF_LM_NW_NT4
#define TF_LM_NW_NT4 8
#endif
#ifndef TF_LM_WM_NT4
#define TF_LM_WM_NT4 1
#endif
// A single row block: four waves, one per SIMD, in a 2 x 2 grid (two along
// the weight tiles, two along the activation tiles), each with 5 weight
// tiles x 2 activation tiles: ten tiles per round, so the 256 ranges of the
// Qwen vocabularies take two rounds, and every SIMD issues the same MFMAs
// and fragment reads (five waves of 2 x 4 tiles left one SIMD with two
// waves' work, which set the pace of every k step).
#ifndef TF_LM_DMA_WM
#define TF_LM_DMA_WM 5
#endif
#ifndef TF_LM_DMA_NW_SINGLE
#define TF_LM_DMA_NW_SINGLE 4
#endif
#ifndef TF_LM_DMA_SINGLE_WB
#define TF_LM_DMA_SINGLE_WB 2
#endif
#ifndef TF_LM_DMA_KC
#define TF_LM_DMA_KC 64
#endif
#ifndef TF_LM_DMA_STAGES
#define TF_LM_DMA_STAGES 3
#endif
// 32-row tiles (stage 1): four waves of three tiles (twelve per round, two
// rounds per range, 152 KiB of rings), about 1% faster per step than the
// register-staged kernel at the 8B shape
#ifndef TF_LM_DMA_NT1_WM
#define TF_LM_DMA_NT1_WM 3
#endif
#ifndef TF_LM_DMA_NT1_NW
#define TF_LM_DMA_NT1_NW 4
#endif
inline int lm_nw(int NT) { return NT == 1 ? TF_LM_NW_NT1 : (NT == 2 ? TF_LM_NW_NT2 : TF_LM_NW_NT4); }
inline int lm_wm(int NT) { return NT == 1 ? TF_LM_WM_NT1 : (NT == 2 ? TF_LM_WM_NT2 : TF_LM_WM_NT4); }

// The block-tiled kernel serves bf16 calls of more rows than one 128-row block
// (widths up to kTileMaxK keep its byte offsets in 30 bits), and of fewer where
// the vocabulary gives a CU at most 7 or 8 tiles (one round of just those tiles;
// the streaming kernels' rounds of 10 or 12 copy and multiply repeats of the
// last tile) or where the width is no multiple of 64.  us, streaming / tiled:
// 16 rows x 32000 x 4096 74 / 56, x 50000 x 2048 50 / 47, 8 x 64000 x 1024
// (8 tiles a CU) 29.3 / 30.1; 48 x 32000 x 4096 77 / 61; 64 x 65000 x 2048
// 86 / 84; 121 x 60000 x 4096 119 / 112; several rounds: 121 x 151936 x 4096
// 233 / 247; width 2000: 121 x 100000 149 / 131, 48 x 151936 199 / 204.
constexpr int kTileMinRows = 129;
constexpr int kTileMaxK = 1 << 20;

// Tile shapes (WM, NT, one row block).
#define TF_LM_TILE_SHAPES(F)                                                                               \
    F(8, 8, false) F(8, 6, false) F(8, 8, true) F(7, 8, true) F(6, 8, true) F(8, 6, true) F(7, 6, true)    \
    F(6, 6, true) F(8, 4, true) F(7, 4, true) F(6, 4, true) F(4, 4, true) F(8, 2, true) F(7, 2, true)      \
    F(6, 2, true) F(4, 2, true)

// Row blocks of at most 256 rows, 192 where the rows then fill them (a wave
// grid of 2 x 2 waves of 16-row tiles: NXT = 8 or 6; 4 and 2 for up to 128 and
// 64 rows).  One row block streams
// the vocabulary once and is as much HBM- as MFMA-bound: the tiles are spread
// evenly over the CUs, in rounds of 6, 7 or 8 tiles (4 too for few rows), whichever leaves the
// least work for padding (a round's epilogue counted as one more tile), while
// that makes no more slices than long lists may have.  Otherwise, and for
// more row blocks: one slice of 8 tiles per workgroup.
inline LmPlan lm_tile_plan(int rows, int V, int d) {
    LmPlan p;
    p.ntiles = cdiv(V, 32);
    p.nk = cdiv(d, 64);
    p.dma = false;
    p.tile = true;
    p.nrb = cdiv(rows, 256);
    p.NT = rows <= 64 ? 2 : rows <= 128 ? 4 : (cdiv(rows, p.nrb * 32) <= 6 ? 6 : 8);
    p.nrb = cdiv(rows, 32 * p.NT);
    p.NW = 4;
    p.WB = 2;
    p.WM = 8;
    p.wnt = p.nrb == 1;
    if (p.nrb == 1) {
        const int G = p.ntiles < kNumCUs ? p.ntiles : kNumCUs;
        const int per = cdiv(p.ntiles, G);
        for (int wm = 7; wm >= (p.NT <= 4 ? 4 : 6); --wm)
            if (wm != 5 && cdiv(per, wm) * (wm + 1) < cdiv(per, p.WM) * (p.WM + 1)) p.WM = wm;
        p.map = make_slice_map(p.ntiles, G, p.WM);
    }
    if (p.nrb > 1 || p.nsplit() > kMaxSplitsLong) {
        p.WM = 8;
        p.map = make_slice_map(p.ntiles, cdiv(p.ntiles, 8), 8);
    }
    p.chunk = p.WM;
    return p;
}

// Calls of several row blocks' worth of narrow products, which the streaming kernels keep: a k loop of few steps
// leaves the epilogue to set the time, and the block-tiled kernel's is longer (16-row tiles: more lanes share a row).
// Whole 256-row blocks at widths of whole k steps; us, streaming / tiled: 400 x 50000 x 128 36 / 42, x 384 49 / 53,
// x 640 64 / 66, x 33000 x 1024 84 / 79; 1000 x 50000 x 128 67 / 76, x 448 102 / 104, x 512 109 / 108; 1936 x 100000 x
// 128 198 / 232; 256 rows x 33000 x 64 18.7 / 21.0, x 192 21.7 / 22.9, x 9000 x 192 22.7 / 21.0 (192-row blocks: 300 x
// 50000 x 64 34.3 / 33.7, x 384 48 / 42).  Other widths, on 128-row blocks, where the tiled kernel's workgroups leave
// half the CUs of their last round idle (400 x 9000 x 272 34 / 40, x 720 58 / 60, 512 x 33000 x 112 40 / 45), and
// of two row blocks at the narrowest (400 x 100000 x 112 74 / 81, x 208 96 / 95).
inline bool lm_narrow(const LmPlan& t, int rows, int d) {
    if (rows < kTileMinRows) return false;
    if (d % TF_LM_DMA_KC == 0) return t.NT == 8 && d <= (t.nrb == 1 ? 128 : t.nrb <= 3 ? 640 : 448);
    if (t.nrb == 1) return false;
    const long long rounds = cdiv(t.blocks(), kNumCUs);
    return d < (100ll * t.blocks() <= 55 * rounds * kNumCUs ? 512 : t.nrb == 2 ? 160 : 0);
}

// `lean`: the plan with the fewest slices (and so partials) for 129-256 rows,
// for callers whose scratch is short; also taken for vocabularies whose
// block-tiled slices would be too many for long lists.
inline LmPlan lm_plan(int rows, int V, int d, bool bf16, bool lean = false) {
    const int per = cdiv(cdiv(V, 32), kNumCUs);   // weight tiles per CU
    const bool few = per > 1 && (per <= (rows <= 32 ? 7 : 8) || (rows > 64 && d % TF_LM_DMA_KC != 0));
    if (bf16 && d <= kTileMaxK && (rows >= kTileMinRows || (few && !lean))) {
        const LmPlan t = lm_tile_plan(rows, V, d);
        if (!lm_narrow(t, rows, d) && (rows > 256 || (!lean && t.nsplit() <= kMaxSplitsLong))) return t;
    }
    LmPlan p;
    p.ntiles = cdiv(V, 32);
    p.nk = cdiv(d, 64);
    p.dma = false;
    if (bf16) {
        p.NT = plan_nt(rows);
        // k in whole 64-wide steps: the DMA kernel -- 32-row tiles, the
        // 2 x 2 wave grid (up to two row blocks), else 256-row blocks
        p.nrb = cdiv(rows, 32 * p.NT);
        p.grid = p.NT >= 2 && p.nrb <= 2 && d % TF_LM_DMA_KC == 0;
        p.dma = d % TF_LM_DMA_KC == 0;
        if (p.dma && p.NT == 1) {
            p.WM = TF_LM_DMA_NT1_WM;
            p.NW = TF_LM_DMA_NT1_NW;
        } else if (p.grid) {
            p.WM = TF_LM_DMA_WM;
            p.NW = TF_LM_DMA_NW_SINGLE;
            p.WB = TF_LM_DMA_SINGLE_WB;
        } else if (p.dma) {
            // eight waves in a 4 x 2 grid of 2 weight x 4 activation tiles, one workgroup per CU
            p.NT = 8;
            p.nrb = cdiv(rows, 256);
            p.WM = 2;
            p.NW = 8;
            p.WB = 2;
        } else {
            p.WM = lm_wm(p.NT);
            p.NW = lm_nw(p.NT);
        }
        p.chunk = p.NW / p.WB * p.WM;
        // one row block, or the grid: TF_LM_WORKGROUPS workgroups in all;
        // else one chunk per range
        const int gw = TF_LM_WORKGROUPS / p.nrb;
        const int G = p.nrb == 1 || p.grid ? (p.ntiles < gw ? p.ntiles : gw) : cdiv(p.ntiles, p.chunk);
        p.map = make_slice_map(p.ntiles, G, p.chunk);
        // the grid's two row blocks share each range's weights, yet stream them no slower with the hint
        // (256 rows, plain / non-temporal: 262208 x 4096 742 / 725 us, 200000 x 4096 524 / 518, 262208 x 1024 221 / 217)
        p.wnt = p.nrb == 1 || p.grid;
    } else {
        p.NT = 1;
        p.WM = 2;
        p.NW = 4;
        p.nrb = cdiv(rows, 16);
        // slices of one tile while that is at most two workgroups a CU, of up
        // to eight where more row blocks or a larger vocabulary fill the chip
        p.chunk = cdiv((long long)p.nrb * p.ntiles, 2 * kNumCUs);
        if (p.chunk > 8) p.chunk = 8;
        p.map = make_slice_map(p.ntiles, cdiv(p.ntiles, p.chunk), p.chunk);
        p.wnt = false;
    }
    return p;
}

// The approximator's products on the block-tiled GEMM (tile_product.hip): tiles
// of 32 WMT weight rows x 32 NXT activation rows, the reduction range cut into
// S splits of `per` 64-wide steps where there are fewer tiles than CUs.
struct TilePlan {
    int WMT, NXT;
    int nrb, ntw;      // row blocks, weight tiles
    int S, per, nk;    // splits, steps of a split, steps in all
    double us;         // the model's time
    bool wide;         // rows past a descriptor's offsets
    int items() const { return nrb * ntw * S; }
};

// Tile shapes (WMT, NXT, activation pairs).
#define TF_TILE_SHAPES(F)                                                                                     \
    F(8, 8, false) F(6, 8, false) F(5, 8, false) F(4, 8, false) F(4, 4, false) F(2, 4, false) F(4, 2, false) \
    F(8, 4, true) F(4, 4, true) F(2, 4, true) F(4, 2, true) F(2, 2, true)

// The one shape of rows past a descriptor's offsets.
constexpr int kTileWideW = 4, kTileWideX = 2;

constexpr int kTileSplits = 8;             // most splits
constexpr int kTileWideSplits = 64;        // ... of such rows: few tiles, and a long reduction
constexpr int kTileSplitFloats = 16384;    // most fp32 partial sums of a row, over its splits
constexpr int kTileSplitRows = 2048;       // rows up to which products are split (more rows make tiles enough)
constexpr int kTileMinSteps = 4;           // fewest steps of a split

// Partial sums a row's split products may take (floats); none once two splits pass the limit.
inline long long tile_split_floats(int rows, long long N, bool wide = false) {
    if (rows > kTileSplitRows || 2 * N > kTileSplitFloats) return 0;
    const long long most = N * (wide ? kTileWideSplits : kTileSplits);
    return most < kTileSplitFloats ? most : kTileSplitFloats;
}

// The shape and split that a simple time model finds fastest.  A step takes
// what its MFMAs take at two thirds of the issue rate at 2.1 GHz (what the
// 256 x 256 tile reaches under the card's power limit), or its copies into LDS
// at 55 GB/s a CU (40 where fewer than four row blocks share a weight tile,
// which then comes from HBM for most of them; 64 for activation pairs, whose
// rows are 256 bytes a step); weights come from HBM at most at 25 GB/s a CU; a split's sums are
// written and read back, and cost a launch.  Measured against the model
// (us, 256 CUs): 1936 x 8192 x 4096 256 x 256 106 / 97, 128 x 256 119 / 120,
// 160 x 256 130 / 130; 455 x 19456 x 2560 160 x 256 55 / 55, 192 x 256 59 / 59, 256 x 256 72 / 67;
// 256 x 8192 x 4096 128 x 128 in two splits 30 / 30, 64 x 128 33 / 41; pairs:
// 905 x 4096 x 4096 128 x 128 56 / 51, 256 x 128 in two splits 60 / 62; at most 64
// rows 64 x 64, which copies half the bytes of 64 x 128 (the SiLU call from cold
// weights, 64 x 128 or 128 x 64 / 64 x 64: 1 row x 4096 x 4096 36.2 / 34.7, x 4096 x 12288
// 78.7 / 73.3, 29 rows x 4096 x 4096 37.6 / 36.0, 61 rows 43.2 / 40.7).
inline TilePlan tile_plan(int rows, int N, int K, int nseg, bool paired, int max_splits, bool tables,
                          bool wide = false) {
    TilePlan best{};
    best.us = 1e30;
    const int np = paired ? 2 : 1;
    const int nk = cdiv(K, 64);
    const double wbytes = 2.0 * N * K * nseg;
    auto consider = [&](int WMT, int NXT) {
        if (wide && (WMT != kTileWideW || NXT != kTileWideX)) return;
        TilePlan p;
        p.wide = wide;
        p.WMT = WMT;
        p.NXT = NXT;
        p.nk = nk;
        p.nrb = cdiv(rows, 32 * NXT);
        p.ntw = cdiv(N, 32 * WMT);
        const double copy = 32.0 * (WMT + NXT * np) * 128 / (paired ? 64e3 : (p.nrb >= 4 ? 55e3 : 40e3));
        const double mfma = 32.0 * WMT * NXT * np * 1.5 / 2100;
        const double step = copy > mfma ? copy : mfma;
        for (int S = 1; S <= max_splits; S += S < 4 ? 1 : S < 16 ? 2 : 8) {
            if (S > 1 && (nk < S * kTileMinSteps || (long long)S * N > tile_split_floats(rows, N))) break;
            p.per = cdiv(nk, S);
            p.S = cdiv(nk, p.per);
            const long long items = (long long)p.items() * nseg;
            const double rounds = (double)cdiv(items, kNumCUs);
            double us = rounds * (p.per * step + 3);
            const double hbm = wbytes / ((items < kNumCUs ? items : kNumCUs) * 25e3) + 4;
            if (hbm > us) us = hbm;
            if (p.S > 1) us += tables ? 4.0 * p.S * rows * N / 8e6 : 4 + 8.0 * p.S * rows * N / 8e6;
            p.us = us;
            if (us < best.us) best = p;
        }
    };
#define TF_TILE_CONSIDER(W, X, P) \
    if (paired == P) consider(W, X);
    TF_TILE_SHAPES(TF_TILE_CONSIDER)
#undef TF_TILE_CONSIDER
    return best;
}

// Widest weight row whose byte offsets within a tile (and its activations')
// stay below kTileSpan; a product of wider ones, of more than 2^20 columns and so
// of few weight rows, takes the wide kernels: one tile shape, up to 64 splits.
// The weight-streaming kernel before them / now, us: 130 rows, d = 16, I = 2^20 +
// 16 1048 / 1916, 17 rows, d = 2^19 + 64, I = 64 1034 / 1262.
inline bool tile_wide(long long width) { return width > kTileMaxK; }

// The h~ half of an input projection ([states, d] into fp32 tables of N
// columns, the readers add its splits), the e~ half, the down projection.
inline TilePlan tile_state_plan(int states, int N, int d, bool wide) {
    return tile_plan(states, N, d, 1, false, wide ? kTileWideSplits : 2, true, wide);
}
inline TilePlan tile_input_plan(int rows, int N, int ew, bool wide) {
    return tile_plan(rows, N, ew, 1, false, wide ? kTileWideSplits : kTileSplits, false, wide);
}
inline TilePlan tile_down_plan(int rows, int d, int I) {
    const bool wide = tile_wide(I);
    return tile_plan(rows, d, I, 1, true, wide ? kTileWideSplits : kTileSplits, false, wide);
}
// the bigram rows' products, once per state and previous token
inline TilePlan tile_token_plan(int tokens, int N, int d) { return tile_plan(tokens, N, d, 3, false, 1, true); }

// The input projections of the AR approximator for few rows (mlp_dma.hpp):
// items of TG weight tiles over their whole reduction range (an h phase of nkh
// and an e phase of nke 64-column chunks), dealt out to G workgroups of at
// least kMlpDmaMinUnits chunks.  Four tiles per item, so that one chunk carries
// 16 MFMAs per wave and 16 KiB of weights: fewer, fatter chunks than with one
// tile, whose per-chunk barrier and latencies otherwise set the pace.
// The down projection (two tiles per item here before) is faster on the
// block-tiled kernel, which copies half the activation bytes per weight byte:
// the approximator at 121 rows, d = I = 4096 66 -> 59 us, 2560 55 -> 46,
// 91 rows 2560 x 9728 95 -> 82.
#ifndef TF_MLP_DMA_TG_IN
#define TF_MLP_DMA_TG_IN 4
#endif
constexpr int kMlpDmaMinUnits = 12;
constexpr int kMlpDmaMaxRows = 128;    // conditional rows (four activation tiles)
constexpr int kMlpDmaMaxGateRows = 256; // the input projections alone (eight activation tiles)
constexpr int kMlpDmaMaxStates = 32;   // drafter states (one activation tile)
struct MlpDmaPlan {
    int TG;       // weight tiles per item
    int NTE;      // 32-row activation tiles of the e phase (1, 2 or 4)
    int ntiles;   // 32-row weight tiles
    int items, nkh, nke, G;
    int wh, we;   // cost of an h chunk and of an e chunk in the split (work.hpp)
    size_t part_floats() const { return (size_t)2 * G * TG * 1024 * (1 + NTE); }
};
inline MlpDmaPlan mlp_dma_plan(int rows, int ntiles, int nkh, int nke, int TG) {
    MlpDmaPlan p;
    p.TG = TG;
    p.NTE = rows <= 32 ? 1 : (rows <= 64 ? 2 : (rows <= 128 ? 4 : 8));
    p.ntiles = ntiles;
    p.items = cdiv(ntiles, TG);
    p.nkh = nkh;
    p.nke = nke;
    const long long U = (long long)p.items * (nkh + nke);
    long long G = U / kMlpDmaMinUnits;
    G = G < kNumCUs ? G : kNumCUs;
    p.G = (int)(G < 1 ? 1 : G);
    // An e chunk against four activation tiles streams its weights at about
    // three fifths of an h chunk's rate (the activation copies from L2 share
    // the CU's load path with the weight stream; 5:3 measured best against
    // 3:2 and 9:5); two tiles take a ratio between that and 1, and one tile,
    // like the h phase, costs the same; eight tiles (the input
    // projections of 129-256 rows) 5:2.
    p.wh = p.NTE == 8 ? 2 : (p.NTE == 4 ? 3 : (p.NTE == 2 ? 4 : 1));
    p.we = p.NTE == 1 ? 1 : 5;
    if (!cost_split_valid(p.items, nkh, nke, p.wh, p.we, p.G)) p.wh = p.we = 1;
    return p;
}
inline bool mlp_dma_plan_ok(const MlpDmaPlan& p) {
    return cost_split_valid(p.items, p.nkh, p.nke, p.wh, p.we, p.G);
}
// gate/up (SwiGLU: tiles of 16 gate + 16 up rows) or the gate alone (the
// plain SiLU MLP: tiles of 32 gate rows) over [h~ ; e~], e~ ew wide
inline MlpDmaPlan mlp_dma_gate_plan(int rows, int d, int ew, int I, bool swiglu) {
    return mlp_dma_plan(rows, swiglu ? cdiv(I, 16) : cdiv(I, 32), d / 64, ew / 64, TF_MLP_DMA_TG_IN);
}
// the linear approximator W_lin [d, 2d] over [h~ ; e~]
inline MlpDmaPlan mlp_dma_linear_plan(int rows, int d) {
    return mlp_dma_plan(rows, cdiv(d, 32), d / 64, d / 64, TF_MLP_DMA_TG_IN);
}
// The input projections of at most 256 rows (bigram rows: 128, beyond that
// their products are taken per token) on the one-row-block kernel; from 129 rows
// on only weight matrices of 30 M elements and more (SwiGLU's two; 40 M the plain
// gate's one), whose stream outweighs what the tiles gain.  The call from cold
// weights, us, here / tiled, at 241 and 136 rows, I x d: SwiGLU 3840 x 2560 71 / 65
// and 64 / 58, 3648 x 4096 83 / 85 and 79 / 77, 4096 x 4096 82 / 87 and 77 / 76,
// 6144 x 4096 103 / 117 and 98 / 101, 12288 x 4096 164 / 169 and 157 / 166; SiLU
// 3648 x 4096 77 / 70 and 72 / 63, 4096 x 4096 73 / 72 and 69 / 65, 6144 x 4096
// 89 / 91 and 83 / 80, 9728 x 2560 89 / 95 and 79 / 76, 12288 x 4096 127 / 138 and
// 118 / 124.  Up to 128 rows: the gate alone, 121 rows, 4096 x 8192 59 / 75, 2560 x
// 5120 46 / 48, 29 rows 2048 x 2048 31 / 30.
inline bool mlp_dma_gate_rows(long long rows, int d, int I, int ew, bool swiglu, int bigram) {
    if (rows > (bigram ? kMlpDmaMaxRows : kMlpDmaMaxGateRows) || d % 64 != 0 || I % 64 != 0 || ew % 64 != 0) return false;
    if (rows > kMlpDmaMaxRows && (long long)I * (d + ew) < (swiglu ? 30000000 : 40000000)) return false;
    return mlp_dma_plan_ok(mlp_dma_gate_plan((int)rows, d, ew, I, swiglu));
}
inline bool mlp_dma_gate_applies(int b, int gamma, int R, int d, int I, int ew, bool swiglu, int bigram) {
    return (long long)b * gamma <= kMlpDmaMaxStates && !tile_wide(d + (long long)ew) &&
           mlp_dma_gate_rows((long long)b * R, d, I, ew, swiglu, bigram);
}
inline bool mlp_dma_linear_rows(long long rows, int d) {
    return rows <= kMlpDmaMaxRows && d % 64 == 0 && mlp_dma_plan_ok(mlp_dma_linear_plan((int)rows, d));
}
inline bool mlp_dma_linear_applies(bool bf16, int b, int gamma, int R, int d) {
    return bf16 && (long long)b * gamma <= kMlpDmaMaxStates && mlp_dma_linear_rows((long long)b * R, d);
}

// Long (row, slice) lists for top-k lists of at least kLongListK entries
// (bf16 kernels, while the merge's candidate buffer holds every entry).
inline bool lm_long_lists(const LmPlan& p, bool bf16, int K) {
    return bf16 && K >= kLongListK && p.nsplit() <= kMaxSplitsLong;
}

// LM-head scratch: the (row, slice) partials, sized for the long lists
// whenever a launch could keep them.
inline size_t lm_scratch_bytes(const LmPlan& p, int rows, bool bf16) {
    const int stride = bf16 && p.nsplit() <= kMaxSplitsLong ? kPartStrideLong : kPartStride;
    return align256((size_t)rows * p.nsplit() * stride * 4);
}
inline size_t lm_scratch_bytes(int rows, int V, int d, bool bf16) {
    return lm_scratch_bytes(lm_plan(rows, V, d, bf16), rows, bf16);
}

// LM-head scratch that serves every call of up to `rows` rows.  bf16: the slices
// of a row change only at these row counts, not always upwards (129 to 256 rows
// may take more than 257).  fp32: slices of one tile shrink in number as more row
// blocks come, and are then at most 512 a row block and one a row more.
inline size_t lm_reserve_bytes(int rows, int V, int d, bool bf16) {
    size_t most = lm_scratch_bytes(rows, V, d, bf16);
    if (bf16) {
        for (int r : {32, 64, 128, 192, 256})
            if (r < rows && lm_scratch_bytes(r, V, d, bf16) > most) most = lm_scratch_bytes(r, V, d, bf16);
        return most;
    }
    const long long tiles = cdiv(V, 32), one = (long long)rows * tiles, few = 2ll * kNumCUs * 16 + cdiv(rows, 16) * 16;
    const long long parts = (long long)rows * cdiv(tiles, 8), fine = one < few ? one : few;
    return align256((size_t)(parts > fine ? parts : fine) * kPartStride * 4);
}

struct Workspace {
    size_t diag, lm, ht, et, act, hp, mlp_part, counters, hh, total;
    int ncounters;
};

// Layout: [diag counters | LM-head scratch (stage 1 or stage 2), or before it the
// approximator's partial sums | normalised h | normalised embeddings | SwiGLU
// activation | h' | SwiGLU arrival counters | h~-half table of the split input
// projections].  Stage 1 uses the first two only.  `bigram` sizes the w/ 2-prev
// rows (two embeddings per row, a 3d-wide input).
//
// No part shrinks as b, gamma or k grow, so that a workspace made for the largest
// call serves the smaller ones: where a plan needs more at fewer rows (pieces of
// the one-row-block kernel, splits of products that have too few tiles), its most
// is reserved from there on.  Nor is the whole ever smaller than at I = 16, which
// the linear layer, whatever I the workspace was sized with, asks for.
inline Workspace workspace_layout(int b, int gamma, int d, int I, int V, int k, bool bf16, bool bigram = false) {
    const int R = (int)cond_rows(gamma, k, bigram ? 1 : 0);
    const int npre = bigram ? 2 : 1;
    const size_t es = bf16 ? 2 : 4;
    const int rows1 = b * gamma, rows2 = b * R;   // R >= gamma
    const size_t tokens = (size_t)b * bigram_tokens(gamma, k);
    const bool tables = bf16 && bigram && !tile_wide(d + (long long)npre * d);
    size_t mp = 0, hhf = 0, erows = (size_t)rows2 * npre;
    Workspace w;
    w.ncounters = 0;
    if (bf16) {
        // split products: at most kTileSplitFloats a row, of at most kTileSplitRows rows
        const int rs = rows2 < kTileSplitRows ? rows2 : kTileSplitRows, ss = rows1 < rs ? rows1 : rs;
        const bool wide = tile_wide(d + (long long)npre * d) || tile_wide(I);
        for (const long long N : {2ll * I, (long long)I, (long long)d}) {
            const long long f = tile_split_floats(1, N, wide);
            mp = mp > (size_t)(rs * f) ? mp : (size_t)(rs * f);
            // the h~ tables: two splits (wide: as above) of up to kTileSplitRows states, one of more
            const long long s2 = ss * (wide || f == 0 ? f : 2 * N), s1 = rows1 * N;
            hhf = hhf > (size_t)(s1 > s2 ? s1 : s2) ? hhf : (size_t)(s1 > s2 ? s1 : s2);
        }
        if (tables) {
            const size_t ld = 2 * (size_t)I > (size_t)d ? 2 * (size_t)I : (size_t)d;
            hhf += 2 * tokens * ld;
            const size_t few = (size_t)(rows2 < kMlpDmaMaxRows ? rows2 : kMlpDmaMaxRows) * npre;
            erows = tokens > few ? tokens : few;
        }
        // the one-row-block kernel at each number of activation tiles up to this call's
        for (int r = 32; r <= kMlpDmaMaxGateRows && (r == 32 || r / 2 < rows2); r *= 2) {
            const int n = r < rows2 ? r : rows2;
            auto need = [&](const MlpDmaPlan& q) {
                mp = mp > q.part_floats() ? mp : q.part_floats();
                w.ncounters = w.ncounters > q.items ? w.ncounters : q.items;
            };
            if (mlp_dma_linear_rows(n, d)) need(mlp_dma_linear_plan(n, d));
            for (const bool swiglu : {true, false})
                if (!tile_wide(d + (long long)npre * d) && mlp_dma_gate_rows(n, d, I, npre * d, swiglu, bigram))
                    need(mlp_dma_gate_plan(n, d, npre * d, I, swiglu));
        }
    }
    const size_t lm = lm_reserve_bytes(rows2, V, d, bf16), part = align256(mp * 4);
    size_t off = 0;
    w.diag = off;
    off += 256;
    w.lm = w.mlp_part = off;   // the LM head reads h' only once the partial sums are finished
    off += lm > part ? lm : part;
    w.ht = off;
    off += align256((size_t)rows1 * d * es);
    w.et = off;
    off += align256(erows * d * es);
    w.act = off;
    off += align256((size_t)rows2 * I * es * (bf16 ? 2 : 1));   // bf16: hi/lo pairs
    w.hp = off;
    off += align256((size_t)rows2 * d * es);
    w.counters = off;
    off += align256((size_t)w.ncounters * 4);
    w.hh = off;
    off += align256(hhf * 4);
    w.total = off;
    return w;
}

}  // namespace tf
