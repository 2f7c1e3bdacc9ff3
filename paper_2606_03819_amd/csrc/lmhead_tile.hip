// LM head on the block-tiled GEMM (bf16; which calls: see lm_plan), with
// the list epilogue, one (row, vocabulary slice) partial per round.
#include "common.hpp"
#include "launch.hpp"
#include "lm_tile.hpp"
#include "plan.hpp"

namespace tf {

struct LmTileArgs {
    const uint16_t* x;
    long ldx;
    const uint16_t* w;
    int R, K, V, nrb, nslices;
    SliceMap map;
    float sl2;
    float* part;
    int* diag;
};

// Workgroup (tile range g, row block rb), the row blocks of a range on
// consecutive workgroups of one XCD so that they share its weights in L2.
// A range is streamed in rounds; the first copies of a round go out before
// the previous round's epilogue, whose lists sit in the weight stage those
// copies leave alone.
template <int WMT, int NXT, bool WNT, bool LONG>
__global__ __launch_bounds__(256, 1) void lmhead_tile_kernel(LmTileArgs a) {
    using G = TileGemm<WMT, NXT, false, (NXT <= 4)>;
    using E = EpiLmTile<WMT, NXT, LONG>;
    static_assert(E::SMEM <= G::WST, "the epilogue's lists fit one weight stage");
    constexpr int CPOL = WNT ? kCpolNt : 0;
    extern __shared__ __align__(16) unsigned char dyn[];
    if (a.diag != nullptr && blockIdx.x == 0 && threadIdx.x == 0) a.diag[0] = 0;
    const int nb = gridDim.x;
    const int id = (nb & 7) != 0 ? (int)blockIdx.x : ((int)blockIdx.x & 7) * (nb >> 3) + ((int)blockIdx.x >> 3);
    const int rb = id % a.nrb, range = id / a.nrb;
    const int row0 = rb * G::XROWS, rows = min(a.R - row0, G::XROWS);
    G g;
    g.init(dyn);
    g.activations(a.x + (size_t)row0 * a.ldx, a.ldx, rows, a.K, 0, (a.K + 63) / 64);
    int t0, t1;
    auto weights = [&](int r) {   // round r's slice, if it has one
        slice_tiles(a.map, range * a.map.rmax + r, t0, t1);
        if (t0 == t1) return false;
        const int n = min(a.V, t1 * 32) - t0 * 32;   // rows past the slice read as zeros
        const auto rs = byte_buffer(a.w + (size_t)t0 * 32 * a.K, (size_t)n * a.K * 2);
        g.weights(rs, rs, [&](int row) { return row < n ? (unsigned)row * (unsigned)a.K * 2u : (unsigned)kTileSpan; });
        return true;
    };
    int r = 0;
    bool more = weights(0);
    if (more) g.template prologue<CPOL>();
    while (more) {
        const int vbase = t0 * 32, vend = min(a.V, t1 * 32);
        g.template loop<CPOL>();
        block_barrier();   // every wave is done with the rings
        const int slice = range * a.map.rmax + r;
        more = ++r < a.map.rmax && weights(r);
        if (more) g.template prologue<CPOL>();
        E::apply(g, dyn + (G::SW - 1) * G::WST, vbase, vend, row0, a.R, slice, a.nslices, a.sl2, a.part);
    }
    // empty slices: partials the merge skips
    for (; r < a.map.rmax; ++r) {
        const int t = threadIdx.x;
        if (t < rows)
            *reinterpret_cast<f32x4*>(a.part + ((size_t)(row0 + t) * a.nslices + range * a.map.rmax + r) *
                                                   part_stride(E::KEEP)) =
                f32x4{neg_inf(), 0.f, neg_inf(), __int_as_float(0)};
    }
}

template <int WMT, int NXT, bool WNT>
static hipError_t launch_shape(const LmTileArgs& a, int blocks, bool longl, hipStream_t st) {
    using G = TileGemm<WMT, NXT, false, (NXT <= 4)>;
    auto kern = longl ? lmhead_tile_kernel<WMT, NXT, WNT, true> : lmhead_tile_kernel<WMT, NXT, WNT, false>;
    const hipError_t e =
        hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, G::SMEM);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(G::NTH), G::SMEM, st, a);
    return hipGetLastError();
}

hipError_t launch_lm_tile(const LmPlan& p, const uint16_t* x, long ldx, const uint16_t* w, int rows, int d, int V,
                          bool longl, float sl2, float* part, int* diag, hipStream_t st) {
    const LmTileArgs a{x, ldx, w, rows, d, V, p.nrb, p.nsplit(), p.map, sl2, part, diag};
    const int nb = p.blocks();
#define TF_LM_TILE_CASE(WMT, NXT, WNT) \
    if (p.WM == WMT && p.NT == NXT && p.wnt == WNT) return launch_shape<WMT, NXT, WNT>(a, nb, longl, st);
    TF_LM_TILE_SHAPES(TF_LM_TILE_CASE)
#undef TF_LM_TILE_CASE
    return hipErrorInvalidValue;
}

}  // namespace tf
