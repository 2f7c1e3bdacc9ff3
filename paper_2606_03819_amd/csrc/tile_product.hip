// The approximator's products where the rows fill more than the one-row-block
// kernels' tiles (bf16): gate/up, the plain gate, the linear layer, the down
// projection over the activation's hi/lo pairs, and the h~ half of an input
// projection as an fp32 table.
//
// Whole sums end in the outputs at once.  A product with too few tiles for the
// chip cuts its reduction range instead: the pieces store fp32 tables, and one
// pass over them (tile_finish_kernel) adds them in order and finishes.  That
// pass costs a launch and 8 bytes per sum and piece; having the last piece to
// arrive read the others' sums back serialises it behind them.
#include "common.hpp"
#include "launch.hpp"
#include "tile_gemm.hpp"
#include "tile_product.hpp"

namespace tf {

__device__ __forceinline__ int state_of(const RowTable& rt, int r) {
    const int s = r / rt.Rs;
    return s * rt.gamma + rt.depth(r - s * rt.Rs) - 1;
}

// silu(g) = g / (1 + e^-g), the quotient by the hardware reciprocal
__device__ __forceinline__ float silu(float g) { return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)); }

// four activations as bf16 hi/lo pairs, interleaved by 8; i % 4 == 0
__device__ __forceinline__ void store_pairs(uint16_t* out, int I, int row, int i, const float (&v)[4]) {
    uint32_t hi[2], lo[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        hi[q] = f32x2_to_bf16x2_bits(v[2 * q], v[2 * q + 1]);
        lo[q] = f32x2_to_bf16x2_bits(v[2 * q] - bf16_bits_to_f32(hi[q] & 0xffffu),
                                     v[2 * q + 1] - bf16_bits_to_f32(hi[q] >> 16));
    }
    uint16_t* o = out + (size_t)row * 2 * I + (size_t)(i >> 3) * 16 + (i & 7);
    *reinterpret_cast<uint2*>(o) = uint2{hi[0], hi[1]};
    *reinterpret_cast<uint2*>(o + 8) = uint2{lo[0], lo[1]};
}
__device__ __forceinline__ void store_residual(const TileFinish& f, int row, int state, int n, const f32x4& y) {
    const uint2 hv = *reinterpret_cast<const uint2*>(f.h + (size_t)state * f.width + n);
    const uint32_t o01 =
        f32x2_to_bf16x2_bits(bf16_bits_to_f32(hv.x & 0xffffu) + y[0], bf16_bits_to_f32(hv.x >> 16) + y[1]);
    const uint32_t o23 =
        f32x2_to_bf16x2_bits(bf16_bits_to_f32(hv.y & 0xffffu) + y[2], bf16_bits_to_f32(hv.y >> 16) + y[3]);
    *reinterpret_cast<uint2*>(f.out + (size_t)row * f.width + n) = uint2{o01, o23};
}

__device__ const __align__(16) uint16_t zero_piece[8] = {};   // what wide operands read past their ends

struct TileGrid {
    int nrb, ntw, S, per, nk;   // row blocks, weight tiles, splits of `per` steps, steps in all
};

// Workgroup (row block, weight tile, split, segment), the row blocks of a
// weight tile on consecutive workgroups of one XCD: they share its weights in
// that XCD's L2, and the tiles of one split share the activations.
template <int WMT, int NXT, bool PAIRED, bool WIDE>
__global__ __launch_bounds__(256, (TileGemm<WMT, NXT, PAIRED, true>::SMEM <= 80 * 1024 ? 2 : 1)) void tile_product_kernel(
    TileProductArgs a, TileGrid t) {
    using G = TileGemm<WMT, NXT, PAIRED, true, WIDE>;
    extern __shared__ __align__(16) unsigned char dyn[];
    const int nb = gridDim.x, xcd = blockIdx.x & 7;
    int id = xcd * (nb >> 3) + min(xcd, nb & 7) + ((int)blockIdx.x >> 3);
    const int rb = id % t.nrb;
    id /= t.nrb;
    const int wt = id % t.ntw;
    id /= t.ntw;
    const int split = id % t.S, sg = id / t.S;
    const TileSegment seg = a.seg[sg];
    const int row0 = rb * G::XROWS, v0 = wt * G::WROWS;
    if (row0 >= seg.R) return;   // segments of fewer row blocks
    const int rows = min(seg.R - row0, G::XROWS);
    G g;
    g.init(dyn);
    g.activations(seg.x + (size_t)row0 * a.ldx, a.ldx, rows, a.K, split * t.per, min(t.nk, (split + 1) * t.per));
    const int n = min(a.N - v0, G::WROWS);   // product columns of this tile
    if constexpr (WIDE) {
        g.weights(zero_piece, [&](int r) -> const uint16_t* {
            if (!a.gateup) return r < n ? seg.wa + (size_t)(v0 + r) * a.Kw : nullptr;
            const int o = (r >> 4) * 8 + (r & 7);
            return o < n >> 1 ? ((r & 8) != 0 ? seg.wb : seg.wa) + (size_t)((v0 >> 1) + o) * a.Kw : nullptr;
        });
    } else if (a.gateup) {
        const int no = n >> 1, o0 = v0 >> 1;
        const size_t bytes = ((size_t)(no - 1) * a.Kw + a.K) * 2;
        g.weights(byte_buffer(seg.wa + (size_t)o0 * a.Kw, bytes), byte_buffer(seg.wb + (size_t)o0 * a.Kw, bytes),
                  [&](int r) {
                      const int o = (r >> 4) * 8 + (r & 7);
                      return o < no ? (unsigned)o * (unsigned)a.Kw * 2u : (unsigned)kTileSpan;
                  });
    } else {
        const auto rs = byte_buffer(seg.wa + (size_t)v0 * a.Kw, ((size_t)(n - 1) * a.Kw + a.K) * 2);
        g.weights(rs, rs, [&](int r) { return r < n ? (unsigned)r * (unsigned)a.Kw * 2u : (unsigned)kTileSpan; });
    }
    g.template prologue<0>();
    g.template loop<0>();

    const int lane = g.lane;
    const TileFinish& f = a.fin;
    if (t.S > 1 || f.epi == kTileStore) {
        float* out = seg.table + (size_t)split * seg.R * a.N;
#pragma unroll
        for (int x = 0; x < NXT; ++x) {
            const int row = row0 + g.xrow(x);
#pragma unroll
            for (int m = 0; m < WMT; ++m) {
                const int v = v0 + g.wrow(m);
                if (row < seg.R && v < a.N) *reinterpret_cast<f32x4*>(out + (size_t)row * a.N + v) = g.acc[m][x];
            }
        }
        return;
    }
#pragma unroll
    for (int x = 0; x < NXT; ++x) {
        const int row = row0 + g.xrow(x);
        const int state = state_of(f.rt, min(row, seg.R - 1));
        for (int q = 0; q < f.nhh; ++q) {
            const float* hrow = f.hh + ((size_t)q * f.states + state) * a.N;
            f32x4 hv[WMT];
#pragma unroll
            for (int m = 0; m < WMT; ++m) hv[m] = *reinterpret_cast<const f32x4*>(hrow + min(v0 + g.wrow(m), a.N - 4));
#pragma unroll
            for (int m = 0; m < WMT; ++m) g.acc[m][x] += hv[m];
        }
        if (f.epi == kTileSwiGLU) {
            // a 16-row tile holds 8 gate rows (lanes 0-31) and their up rows (lanes 32-63):
            // half-wave swaps give the lower lanes tile m's pairs, the upper lanes tile m + 1's
#pragma unroll
            for (int m = 0; m < WMT; m += 2) {
                const int m1 = m + 1 < WMT ? m + 1 : m;
                float v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_int(g.acc[m][x][j]),
                                                                    __float_as_int(g.acc[m1][x][j]), false, false);
                    v[j] = silu(__int_as_float(p[0])) * __int_as_float(p[1]);
                }
                const int up = lane >> 5;
                const int i = ((v0 + (g.wa * WMT + m + up) * 16) >> 1) + 4 * ((lane >> 4) & 1);
                if (row < seg.R && i < f.width && m + up < WMT) store_pairs(f.out, f.width, row, i, v);
            }
        } else {
#pragma unroll
            for (int m = 0; m < WMT; ++m) {
                const int v = v0 + g.wrow(m);
                if (row >= seg.R || v >= a.N) continue;
                if (f.epi == kTileSiLU) {
                    const float s[4] = {silu(g.acc[m][x][0]), silu(g.acc[m][x][1]), silu(g.acc[m][x][2]),
                                        silu(g.acc[m][x][3])};
                    store_pairs(f.out, f.width, row, v, s);
                } else {
                    store_residual(f, row, state, v, g.acc[m][x]);
                }
            }
        }
    }
}

// Rows' outputs from their tables, eight to a thread.
__global__ __launch_bounds__(256) void tile_finish_kernel(TileFinish f) {
    const int per = f.width >> 3;
    const long long id = (long long)blockIdx.x * 256 + threadIdx.x;
    if (id >= (long long)f.R * per) return;
    const int row = (int)(id / per), o = (int)(id % per) * 8;
    const int s = row / f.rt.Rs, rl = row - s * f.rt.Rs;
    const int state = s * f.rt.gamma + f.rt.depth(rl) - 1;
    const bool pair = f.epi == kTileSwiGLU;
    const int c = pair ? 2 * o : o;   // eight gate columns, then their eight up columns
    f32x4 y[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) y[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto add = [&](const float* table, size_t r) {
        const f32x4* p = reinterpret_cast<const f32x4*>(table + r * f.N + c);
        y[0] += p[0];
        y[1] += p[1];
        if (pair) {
            y[2] += p[2];
            y[3] += p[3];
        }
    };
    for (int q = 0; q < f.nown; ++q) add(f.own, (size_t)q * f.R + row);
    for (int q = 0; q < f.nhh; ++q) add(f.hh, (size_t)q * f.states + state);
    if (f.t1 != nullptr) {
        // token tables hold, per sequence, the context, the root, then every candidate of depths 1 .. gamma - 1
        const size_t base = (size_t)s * bigram_tokens(f.rt.gamma, f.rt.M);
        add(f.t1, base + f.rt.bigram_token(rl, 0));
        add(f.t2, base + f.rt.bigram_token(rl, 1));
    }
    if (f.epi == kTileResidual) {
        store_residual(f, row, state, o, y[0]);
        store_residual(f, row, state, o + 4, y[1]);
        return;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = pair ? silu(y[j][e]) * y[2 + j][e] : silu(y[j][e]);
        store_pairs(f.out, f.width, row, o + 4 * j, v);
    }
}

template <int WMT, int NXT, bool PAIRED, bool WIDE = false>
static hipError_t launch_shape(const TilePlan& p, const TileProductArgs& a, hipStream_t st) {
    using G = TileGemm<WMT, NXT, PAIRED, true, WIDE>;
    auto kern = tile_product_kernel<WMT, NXT, PAIRED, WIDE>;
    const hipError_t e =
        hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, G::SMEM);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(p.items() * a.nseg), dim3(G::NTH), G::SMEM, st, a,
                       TileGrid{p.nrb, p.ntw, p.S, p.per, p.nk});
    return hipGetLastError();
}

hipError_t launch_tile_product(const TilePlan& p, bool paired, const TileProductArgs& a, hipStream_t st) {
    if (p.wide)
        return paired ? launch_shape<kTileWideW, kTileWideX, true, true>(p, a, st)
                      : launch_shape<kTileWideW, kTileWideX, false, true>(p, a, st);
#define TF_TILE_SHAPE(W, X, P) \
    if (p.WMT == W && p.NXT == X && paired == P) return launch_shape<W, X, P>(p, a, st);
    TF_TILE_SHAPES(TF_TILE_SHAPE)
#undef TF_TILE_SHAPE
    return hipErrorInvalidValue;
}

hipError_t launch_tile_finish(const TileFinish& f, hipStream_t st) {
    const long long threads = (long long)f.R * (f.width >> 3);
    hipLaunchKernelGGL(tile_finish_kernel, dim3((unsigned)cdiv(threads, 256)), dim3(256), 0, st, f);
    return hipGetLastError();
}

}  // namespace tf
