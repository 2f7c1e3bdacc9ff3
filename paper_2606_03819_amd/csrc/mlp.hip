// The AR approximator of Eq. 1 for every conditional row:
//   h'_r = h_{depth(r)} + W_down( silu(W_gate x_r) * (W_up x_r) ),
//   x_r  = [ rms(h_{depth(r)}) * g_h ; rms(Embd(prev_r)) * g_e ],
// the w/ Linear ablation h'_r = h_{depth(r)} + W_lin x_r, and the w/ 2-prev
// ablation whose x_r appends the normalised embedding of the token before
// prev_r (Ablations, Model Design).  Rows follow the tables in rows.hpp.
#include "common.hpp"
#include "launch.hpp"
#include "mlp_dma.hpp"
#include "plan.hpp"
#include "rows.hpp"
#include "tile_product.hpp"

namespace tf {

__device__ __forceinline__ float load_elem(const uint16_t* p, size_t i) { return bf16_bits_to_f32(p[i]); }
__device__ __forceinline__ float load_elem(const float* p, size_t i) { return p[i]; }
__device__ __forceinline__ void store_elem(uint16_t* p, size_t i, float v) { p[i] = (uint16_t)f32_to_bf16_bits(v); }
__device__ __forceinline__ void store_elem(float* p, size_t i, float v) { p[i] = v; }

// RMSNorm of the b*gamma drafter states (into ht) and of the npre previous-
// token embeddings of each of the b*R rows (into et, [b*R, npre*d], the
// nearer token first); one workgroup per vector.  bf16 outputs are rounded to
// nearest even: they are the bf16 operand x of the products that follow.
template <class T>
__global__ __launch_bounds__(256) void rmsnorm_rows_kernel(const T* __restrict__ h, const int32_t* __restrict__ root,
                                                           const int32_t* __restrict__ context,
                                                           const int32_t* __restrict__ topk,
                                                           const T* __restrict__ emb, const T* __restrict__ gh,
                                                           const T* __restrict__ ge, int b, int d, int V, RowTable rt,
                                                           int npre, float eps, T* __restrict__ ht,
                                                           T* __restrict__ et, int* __restrict__ diag,
                                                           int* __restrict__ counters, int ncounters) {
    __shared__ float red[4];
    if (diag != nullptr && blockIdx.x == 0 && threadIdx.x == 0) diag[0] = 0;
    if (blockIdx.x == 0)   // arrival counters of the products that follow on this stream
        for (int i = threadIdx.x; i < ncounters; i += 256) counters[i] = 0;
    const int row = blockIdx.x;
    const T* src;
    const T* gain;
    T* dst;
    if (row < b * rt.gamma) {
        src = h + (size_t)row * d;
        gain = gh;
        dst = ht + (size_t)row * d;
    } else {
        const int e = row - b * rt.gamma;
        const int rr = e / npre, which = e - rr * npre;
        const int s = rr / rt.Rs;
        int prev = rt.prev_token(s, rr - s * rt.Rs, which, root, context, topk);
        prev = min(max(prev, 0), V - 1);   // ids are documented to be < V; never read out of bounds
        src = emb + (size_t)prev * d;
        gain = ge;
        dst = et + (size_t)rr * npre * d + (size_t)which * d;
    }
    float ss = 0.f;
#pragma unroll 4   // four loads in flight before the first use
    for (int k = threadIdx.x; k < d; k += 256) {
        const float x = load_elem(src, k);
        ss = fmaf(x, x, ss);
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    ss = (red[0] + red[1]) + (red[2] + red[3]);
    const float inv = 1.0f / sqrtf(ss / (float)d + eps);
    if (gain != nullptr) {
#pragma unroll 4
        for (int k = threadIdx.x; k < d; k += 256) store_elem(dst, k, load_elem(src, k) * inv * load_elem(gain, k));
    } else {
#pragma unroll 4
        for (int k = threadIdx.x; k < d; k += 256) store_elem(dst, k, load_elem(src, k) * inv);
    }
}

// bf16 with every row 16-byte aligned: one wave per vector; each lane keeps
// its 16-byte pieces (pieces lane, lane + 64, ...; at most MAXC of them) in
// registers between the sum of squares and the scaling, so the vector is
// read once and the reduction needs no barrier.
template <int MAXC>
__global__ __launch_bounds__(256) void rmsnorm_rows_bf16_kernel(const uint16_t* __restrict__ h,
                                                                const int32_t* __restrict__ root,
                                                                const int32_t* __restrict__ context,
                                                                const int32_t* __restrict__ topk,
                                                                const uint16_t* __restrict__ emb,
                                                                const uint16_t* __restrict__ gh,
                                                                const uint16_t* __restrict__ ge, int b, int d, int V,
                                                                RowTable rt, int npre, float eps,
                                                                uint16_t* __restrict__ ht, uint16_t* __restrict__ et,
                                                                int* __restrict__ diag, int* __restrict__ counters,
                                                                int ncounters) {
    if (diag != nullptr && blockIdx.x == 0 && threadIdx.x == 0) diag[0] = 0;
    if (blockIdx.x == 0)   // arrival counters of the products that follow on this stream
        for (int i = threadIdx.x; i < ncounters; i += 256) counters[i] = 0;
    const int lane = threadIdx.x & 63;
    const int vec = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int nvec = b * rt.gamma + b * rt.Rs * npre;
    if (vec >= nvec) return;
    const uint16_t* src;
    const uint16_t* gain;
    uint16_t* dst;
    if (vec < b * rt.gamma) {
        src = h + (size_t)vec * d;
        gain = gh;
        dst = ht + (size_t)vec * d;
    } else {
        const int e = vec - b * rt.gamma;
        const int rr = e / npre, which = e - rr * npre;
        const int s = rr / rt.Rs;
        int prev = rt.prev_token(s, rr - s * rt.Rs, which, root, context, topk);
        prev = min(max(prev, 0), V - 1);   // ids are documented to be < V; never read out of bounds
        src = emb + (size_t)prev * d;
        gain = ge;
        dst = et + (size_t)rr * npre * d + (size_t)which * d;
    }
    const int npc = d >> 3;   // 16-byte pieces
    u32x4 v[MAXC], gv[MAXC];
    // Every load is issued before the first use: the branch per piece is
    // uniform and a lane past the row re-reads its last piece (its values are
    // dropped below), so the row and its gains take one round trip.
#pragma unroll
    for (int c = 0; c < MAXC; ++c) {
        if (64 * c < npc) {
            const int pc = min(lane + 64 * c, npc - 1);
            v[c] = *reinterpret_cast<const u32x4*>(src + 8 * pc);
            gv[c] = gain != nullptr ? *reinterpret_cast<const u32x4*>(gain + 8 * pc)
                                    : u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};   // bf16 ones
        }
    }
    float ss = 0.f;
#pragma unroll
    for (int c = 0; c < MAXC; ++c) {
        if (64 * c < npc && lane + 64 * c < npc) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float lo = bf16_bits_to_f32(v[c][q] & 0xffffu), hi = bf16_bits_to_f32(v[c][q] >> 16);
                ss = fmaf(lo, lo, ss);
                ss = fmaf(hi, hi, ss);
            }
        }
    }
    ss = wave_sum(ss);
    const float inv = 1.0f / sqrtf(ss / (float)d + eps);
#pragma unroll
    for (int c = 0; c < MAXC; ++c) {
        const int pc = lane + 64 * c;
        if (pc < npc) {
            u32x4 o;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float lo = bf16_bits_to_f32(v[c][q] & 0xffffu) * inv * bf16_bits_to_f32(gv[c][q] & 0xffffu);
                const float hi = bf16_bits_to_f32(v[c][q] >> 16) * inv * bf16_bits_to_f32(gv[c][q] >> 16);
                o[q] = f32x2_to_bf16x2_bits(lo, hi);
            }
            *reinterpret_cast<u32x4*>(dst + 8 * pc) = o;
        }
    }
}

// ------------------------------------------------------------ fp32

// The approximator's fp32 products (small models): out[r, n] = epi( x_r . W[n] )
// with x_r = [x0 row of r's drafter state (d0 wide) ; x1 row r (K - d0 wide)],
// 16 rows x 16 output columns a workgroup.
//   GATE:  act = silu(x . W_gate[n]) * (x . W_up[n])  (W_up null: silu alone)
//   else:  out = h[r's drafter state, n] + x . W[n]   (down projection, linear)
// A handful of workgroups and one fmaf chain an output: what bounds it is the
// chain and the round trips to memory, so a chunk is 256 columns wide (all of x
// and W for the widths such models have, in one or two trips, the next chunk's in
// flight while one is multiplied) and LDS is read 16 bytes at a time.  31 rows, I = d = 256: gate/up 29.5 -> 10.3 us, down 9.6
// -> 4.9 us against 64-wide chunks and 4-byte reads.
template <bool GATE>
__global__ __launch_bounds__(256) void mlp_f32_kernel(const float* __restrict__ wa, const float* __restrict__ wb, int N,
                                                      int K, const float* __restrict__ x0, int d0,
                                                      const float* __restrict__ x1, int ld1, RowTable rt, int rows,
                                                      const float* __restrict__ h, float* __restrict__ out, int ldo) {
    constexpr int KC = 256, LD = KC + 4;
    constexpr int NW = GATE ? 2 : 1;
    __shared__ __align__(16) float xs[16 * LD];
    __shared__ __align__(16) float ws[NW][16 * LD];
    const int tid = threadIdx.x;
    const int n0 = blockIdx.x * 16, r0 = blockIdx.y * 16;
    const int tx = tid & 15, ty = tid >> 4;
    const bool two = GATE && wb != nullptr;
    auto state_of = [&](int r) {
        const int s = r / rt.Rs;
        return s * rt.gamma + rt.depth(r - s * rt.Rs) - 1;
    };
    // this thread's pieces of a chunk: rows tid / 64 + 4 j, k 4 (tid % 64)
    const int prow = tid >> 6, pk = (tid & 63) * 4;
    int xrow[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = r0 + prow + 4 * j;
        xrow[j] = r < rows ? state_of(r) : -1;
    }
    const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 px[4], pw[NW][4];
    auto fetch = [&](int k0) {
        const int k = k0 + pk;   // d0, K and the strides are multiples of 16
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = r0 + prow + 4 * j, n = n0 + prow + 4 * j;
            const float* xp = k < d0 ? x0 + (size_t)xrow[j] * d0 + k : x1 + (size_t)r * ld1 + (k - d0);
            px[j] = xrow[j] >= 0 && k < K ? *reinterpret_cast<const f32x4*>(xp) : zero;
            const bool in = n < N && k < K;
            pw[0][j] = in ? *reinterpret_cast<const f32x4*>(wa + (size_t)n * K + k) : zero;
            if constexpr (GATE) pw[1][j] = in && two ? *reinterpret_cast<const f32x4*>(wb + (size_t)n * K + k) : zero;
        }
    };
    float acc[NW];
#pragma unroll
    for (int q = 0; q < NW; ++q) acc[q] = 0.f;
    fetch(0);
    for (int k0 = 0; k0 < K; k0 += KC) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            *reinterpret_cast<f32x4*>(xs + (prow + 4 * j) * LD + pk) = px[j];
#pragma unroll
            for (int q = 0; q < NW; ++q) *reinterpret_cast<f32x4*>(&ws[q][(prow + 4 * j) * LD + pk]) = pw[q][j];
        }
        __syncthreads();
        if (k0 + KC < K) fetch(k0 + KC);
        const int kn = min(KC, K - k0);   // a multiple of 16
#pragma unroll 4
        for (int k = 0; k < kn; k += 4) {
            const f32x4 xv = *reinterpret_cast<const f32x4*>(xs + ty * LD + k);
#pragma unroll
            for (int q = 0; q < NW; ++q) {
                const f32x4 wv = *reinterpret_cast<const f32x4*>(&ws[q][tx * LD + k]);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[q] = fmaf(xv[e], wv[e], acc[q]);
            }
        }
        __syncthreads();
    }
    const int r = r0 + ty, n = n0 + tx;
    if (r >= rows || n >= N) return;
    if constexpr (GATE) {
        float a = acc[0] / (1.0f + expf(-acc[0]));
        if (two) a *= acc[1];
        out[(size_t)r * ldo + n] = a;
    } else {
        out[(size_t)r * ldo + n] = h[(size_t)state_of(r) * N + n] + acc[0];
    }
}

// ------------------------------------------------------------------ launcher

static bool aligned16p(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

template <class T>
static void launch_norms(const void* h, const int32_t* root, const int32_t* context, const int32_t* topk,
                         const void* emb, const void* gh, const void* ge, int b, int d, int V, const RowTable& rt,
                         int npre, float eps, void* ht, void* et, int* diag, int* counters, int ncounters,
                         hipStream_t stream) {
    const int nvec = b * rt.gamma + b * rt.Rs * npre;
    constexpr int kMaxPieces = 16;   // d <= 16 * 64 * 8 = 8192 in registers
    if constexpr (sizeof(T) == 2) {
        // h rows are 16-byte aligned (checked at the boundary); the embedding and gains are only
        // required to be 4-byte aligned, so this path is taken when they happen to be 16-byte aligned
        if (d <= kMaxPieces * 64 * 8 && aligned16p(emb) && (gh == nullptr || aligned16p(gh)) &&
            (ge == nullptr || aligned16p(ge))) {
            hipLaunchKernelGGL(rmsnorm_rows_bf16_kernel<kMaxPieces>, dim3(cdiv(nvec, 4)), dim3(256), 0, stream,
                               static_cast<const uint16_t*>(h), root, context, topk,
                               static_cast<const uint16_t*>(emb), static_cast<const uint16_t*>(gh),
                               static_cast<const uint16_t*>(ge), b, d, V, rt, npre, eps,
                               static_cast<uint16_t*>(ht), static_cast<uint16_t*>(et), diag, counters, ncounters);
            return;
        }
    }
    hipLaunchKernelGGL(rmsnorm_rows_kernel<T>, dim3(nvec), dim3(256), 0, stream, static_cast<const T*>(h), root,
                       context, topk, static_cast<const T*>(emb), static_cast<const T*>(gh),
                       static_cast<const T*>(ge), b, d, V, rt, npre, eps, static_cast<T*>(ht), static_cast<T*>(et),
                       diag, counters, ncounters);
}

// ------------------------------------------------ one row block (mlp_dma.hpp)

// Ring depths: SW - 1 weight stages in flight (TG tiles of 4 KiB each) and
// two activation chunks (four to six weight stages measured equal).
template <int NTE>
constexpr int mlp_dma_sw() {
    return NTE == 8 ? 4 : 5;
}
// activation stages: eight tiles' 32 KiB chunks leave room for one in flight
template <int NTE>
constexpr int mlp_dma_sx() {
    return NTE == 8 ? 2 : 3;
}

template <int TG, int NTE, int WMAP, int EPI>
static hipError_t launch_mlp_dma_nte(const MlpDmaArgs& a, hipStream_t st) {
    constexpr int SW = mlp_dma_sw<NTE>(), SX = mlp_dma_sx<NTE>();
    using T = MlpDmaTraits<TG, NTE, SW, SX>;
    static_assert(T::SMEM <= 152 * 1024, "LDS of one workgroup");
    auto kern = mlp_dma_kernel<TG, NTE, SW, SX, WMAP, EPI>;
    const hipError_t e =
        hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, T::SMEM);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(a.G), dim3(256), T::SMEM, st, a);
    return hipGetLastError();
}

template <int WMAP, int EPI>
static hipError_t launch_mlp_dma(const MlpDmaArgs& a, const MlpDmaPlan& p, hipStream_t st) {
    constexpr int TG = TF_MLP_DMA_TG_IN;
    if (p.TG != TG) return hipErrorInvalidValue;
    if (p.NTE == 1) return launch_mlp_dma_nte<TG, 1, WMAP, EPI>(a, st);
    if (p.NTE == 2) return launch_mlp_dma_nte<TG, 2, WMAP, EPI>(a, st);
    if constexpr (EPI != kMlpEpiResidual) {   // eight tiles: the input projections only
        if (p.NTE == 8) return launch_mlp_dma_nte<TG, 8, WMAP, EPI>(a, st);
    }
    if (p.NTE != 4) return hipErrorInvalidValue;
    return launch_mlp_dma_nte<TG, 4, WMAP, EPI>(a, st);
}

static MlpDmaArgs mlp_dma_args(const MlpDmaPlan& p, const uint16_t* w, const uint16_t* wu, int N, int Kw,
                               const uint16_t* xh, const uint16_t* xe, long lde, int Rh, int Re, uint16_t* out,
                               int Nout, const uint16_t* h, const RowTable& rt, float* partial, int* counter) {
    return MlpDmaArgs{w,     wu,    N,   Kw,   xh,   xe,   lde, Rh,   Re,      p.ntiles, p.items, p.nkh,
                      p.nke, p.G,   p.wh, p.we, out, Nout, h,  rt,   partial, counter};
}

// One product with its finished outputs: from the accumulators, or from the
// splits' tables.
static hipError_t tile_product_finished(const TilePlan& p, bool paired, const uint16_t* wa, const uint16_t* wb,
                                        const uint16_t* x, long ldx, int Kw, int K, float* tables, TileFinish f,
                                        hipStream_t st) {
    TileProductArgs a{};
    a.seg[0] = TileSegment{wa, wb, x, f.R, tables};
    a.nseg = 1;
    a.gateup = wb != nullptr;
    a.N = f.N;
    a.Kw = Kw;
    a.K = K;
    a.ldx = ldx;
    a.fin = f;
    const hipError_t e = launch_tile_product(p, paired, a, st);
    if (e != hipSuccess || p.S == 1) return e;
    f.own = tables;
    f.nown = p.S;
    return launch_tile_finish(f, st);
}

// Eq. 1 in bf16.  The down projection runs on the block-tiled kernel; so do the
// input projections that the one-row-block kernel does not take (more rows,
// more states, other widths), split at the h~ / e~ boundary of x (the h~ half
// once per drafter state); the
// bigram rows, which combine few distinct tokens in many pairs, have it split
// once more, at the previous token's boundary, and computed once per token
// (at 16 x 8 candidates 122 tokens for 905 rows, a seventh of the products).
static hipError_t launch_arapprox_tile(const void* h, const int32_t* root, const int32_t* context,
                                       const int32_t* topk_idx, const void* emb, const void* gain_h,
                                       const void* gain_e, const void* w_gate, const void* w_up, const void* w_down,
                                       int b, int d, int I, int V, const RowTable& rt, float eps, void* ht, void* et,
                                       void* act, void* hp, float* partial, int* counters, float* hh, int* diag,
                                       hipStream_t stream) {
    const bool swiglu = w_up != nullptr;
    const int rows = b * rt.Rs, states = b * rt.gamma;
    const int N = swiglu ? 2 * I : I;
    const int npre = rt.bigram ? 2 : 1, ew = npre * d;
    const uint16_t* hb = static_cast<const uint16_t*>(h);
    const uint16_t* htb = static_cast<const uint16_t*>(ht);
    const uint16_t* etb = static_cast<const uint16_t*>(et);
    const uint16_t* wg = static_cast<const uint16_t*>(w_gate);
    const uint16_t* wu = static_cast<const uint16_t*>(w_up);
    uint16_t* actb = static_cast<uint16_t*>(act);
    TileFinish f{};
    f.epi = swiglu ? kTileSwiGLU : kTileSiLU;
    f.R = rows;
    f.N = N;
    f.out = actb;
    f.width = I;
    f.hh = hh;
    f.states = states;
    f.rt = rt;
    const bool wide = tile_wide(d + (long long)ew);   // the input projections' rows
    hipError_t e;
    if (mlp_dma_gate_applies(b, rt.gamma, rt.Rs, d, I, ew, swiglu, rt.bigram)) {
        const MlpDmaPlan pg = mlp_dma_gate_plan(rows, d, ew, I, swiglu);
        launch_norms<uint16_t>(h, root, context, topk_idx, emb, gain_h, gain_e, b, d, V, rt, npre, eps, ht, et, diag,
                               counters, pg.items, stream);
        const MlpDmaArgs ag = mlp_dma_args(pg, wg, wu, I, d + ew, htb, etb, ew, states, rows, actb, I, hb, rt, partial,
                                           counters);
        e = swiglu ? launch_mlp_dma<kMlpWGateUp, kMlpEpiSwiGLU>(ag, pg, stream)
                   : launch_mlp_dma<kMlpWPlain, kMlpEpiSiLU>(ag, pg, stream);
    } else if (rt.bigram && !wide) {
        const RowTable tt = make_token_table(rt.gamma, rt.M);
        const int tokens = b * tt.Rs;
        launch_norms<uint16_t>(h, root, context, topk_idx, emb, gain_h, gain_e, b, d, V, tt, 1, eps, ht, et, diag,
                               counters, 0, stream);
        float* t1 = hh + (size_t)states * N;
        float* t2 = t1 + (size_t)tokens * N;
        TileProductArgs a{};
        a.seg[0] = TileSegment{wg, wu, htb, states, hh};
        a.seg[1] = TileSegment{wg + d, wu + d, etb, tokens, t1};
        a.seg[2] = TileSegment{wg + 2 * d, wu + 2 * d, etb, tokens, t2};
        a.nseg = 3;
        a.gateup = true;
        a.N = N;
        a.Kw = 3 * d;
        a.K = d;
        a.ldx = d;
        e = launch_tile_product(tile_token_plan(tokens, N, d), false, a, stream);
        if (e != hipSuccess) return e;
        f.nhh = 1;
        f.t1 = t1;
        f.t2 = t2;
        e = launch_tile_finish(f, stream);
    } else {
        launch_norms<uint16_t>(h, root, context, topk_idx, emb, gain_h, gain_e, b, d, V, rt, npre, eps, ht, et, diag,
                               counters, 0, stream);
        const TilePlan ph = tile_state_plan(states, N, d, wide);
        TileProductArgs a{};
        a.seg[0] = TileSegment{wg, wu, htb, states, hh};
        a.nseg = 1;
        a.gateup = swiglu;
        a.N = N;
        a.Kw = d + ew;
        a.K = d;
        a.ldx = d;
        e = launch_tile_product(ph, false, a, stream);
        if (e != hipSuccess) return e;
        f.nhh = ph.S;
        e = tile_product_finished(tile_input_plan(rows, N, ew, wide), false, wg + d, swiglu ? wu + d : nullptr, etb, ew,
                                  d + ew, ew, partial, f, stream);
    }
    if (e != hipSuccess) return e;
    TileFinish r{};
    r.epi = kTileResidual;
    r.R = rows;
    r.N = r.width = d;
    r.out = static_cast<uint16_t*>(hp);
    r.h = hb;
    r.states = states;
    r.rt = rt;
    return tile_product_finished(tile_down_plan(rows, d, I), true, static_cast<const uint16_t*>(w_down), nullptr, actb,
                                 2l * I, I, I, partial, r, stream);
}

hipError_t launch_arapprox(const void* h, const int32_t* root, const int32_t* context, const int32_t* topk_idx,
                           const void* emb, const void* gain_h, const void* gain_e, const void* w_gate,
                           const void* w_up, const void* w_down, int b, int gamma, int d, int I, int V, int k,
                           bool bigram, float eps, bool bf16, void* ht, void* et, void* act, void* hp,
                           float* mlp_partial, int* counters, float* hh, int* diag, hipStream_t stream) {
    const RowTable rt = make_row_table(gamma, k, bigram ? 1 : 0);
    const int npre = bigram ? 2 : 1;
    const int ew = npre * d;
    const int rows = b * rt.Rs;
    if (bf16)
        return launch_arapprox_tile(h, root, context, topk_idx, emb, gain_h, gain_e, w_gate, w_up, w_down, b, d, I, V, rt,
                                    eps, ht, et, act, hp, mlp_partial, counters, hh, diag, stream);
    launch_norms<float>(h, root, context, topk_idx, emb, gain_h, gain_e, b, d, V, rt, npre, eps, ht, et, diag, counters, 0,
                        stream);
    const float *xh = static_cast<const float*>(ht), *xe = static_cast<const float*>(et);
    float* ab = static_cast<float*>(act);
    hipLaunchKernelGGL(mlp_f32_kernel<true>, dim3(cdiv(I, 16), cdiv(rows, 16)), dim3(256), 0, stream,
                       static_cast<const float*>(w_gate), static_cast<const float*>(w_up), I, d + ew, xh, d, xe, ew, rt,
                       rows, nullptr, ab, I);
    hipLaunchKernelGGL(mlp_f32_kernel<false>, dim3(cdiv(d, 16), cdiv(rows, 16)), dim3(256), 0, stream,
                       static_cast<const float*>(w_down), nullptr, d, I, nullptr, 0, ab, I, rt, rows,
                       static_cast<const float*>(h), static_cast<float*>(hp), d);
    return hipGetLastError();
}

hipError_t launch_arapprox_linear(const void* h, const int32_t* root, const int32_t* topk_idx, const void* emb,
                                  const void* gain_h, const void* gain_e, const void* w_lin, int b, int gamma, int d,
                                  int V, int k, float eps, bool bf16, void* ht, void* et, void* hp,
                                  float* mlp_partial, int* counters, float* hh, int* diag, hipStream_t stream) {
    const RowTable rt = make_row_table(gamma, k, 0);
    const int rows = b * rt.Rs;
    if (mlp_dma_linear_applies(bf16, b, gamma, rt.Rs, d)) {
        // one row block: the h~ half once per drafter state, residual epilogue
        const MlpDmaPlan pl = mlp_dma_linear_plan(rows, d);
        launch_norms<uint16_t>(h, root, nullptr, topk_idx, emb, gain_h, gain_e, b, d, V, rt, 1, eps, ht, et, diag,
                               counters, pl.items, stream);
        const uint16_t* hb = static_cast<const uint16_t*>(h);
        const MlpDmaArgs al = mlp_dma_args(pl, static_cast<const uint16_t*>(w_lin), nullptr, d, 2 * d,
                                           static_cast<const uint16_t*>(ht), static_cast<const uint16_t*>(et), d,
                                           b * gamma, rows, static_cast<uint16_t*>(hp), d, hb, rt, mlp_partial,
                                           counters);
        return launch_mlp_dma<kMlpWPlain, kMlpEpiResidual>(al, pl, stream);
    }
    if (bf16) {
        const bool wide = tile_wide(2ll * d);
        // the h~ half once per drafter state, then the e~ half with the residual
        const int states = b * gamma;
        launch_norms<uint16_t>(h, root, nullptr, topk_idx, emb, gain_h, gain_e, b, d, V, rt, 1, eps, ht, et, diag,
                               counters, 0, stream);
        const uint16_t* wl = static_cast<const uint16_t*>(w_lin);
        TileProductArgs ah{};
        ah.seg[0] = TileSegment{wl, nullptr, static_cast<const uint16_t*>(ht), states, hh};
        ah.nseg = 1;
        ah.N = d;
        ah.Kw = 2 * d;
        ah.K = d;
        ah.ldx = d;
        const TilePlan ph = tile_state_plan(states, d, d, wide), pe = tile_input_plan(rows, d, d, wide);
        const hipError_t e = launch_tile_product(ph, false, ah, stream);
        if (e != hipSuccess) return e;
        TileFinish f{};
        f.epi = kTileResidual;
        f.R = rows;
        f.N = f.width = d;
        f.out = static_cast<uint16_t*>(hp);
        f.h = static_cast<const uint16_t*>(h);
        f.hh = hh;
        f.nhh = ph.S;
        f.states = states;
        f.rt = rt;
        return tile_product_finished(pe, false, wl + d, nullptr, static_cast<const uint16_t*>(et), d, 2 * d, d,
                                     mlp_partial, f, stream);
    }
    launch_norms<float>(h, root, nullptr, topk_idx, emb, gain_h, gain_e, b, d, V, rt, 1, eps, ht, et, diag, counters, 0,
                        stream);
    hipLaunchKernelGGL(mlp_f32_kernel<false>, dim3(cdiv(d, 16), cdiv(rows, 16)), dim3(256), 0, stream,
                       static_cast<const float*>(w_lin), nullptr, d, 2 * d, static_cast<const float*>(ht), d,
                       static_cast<const float*>(et), d, rt, rows, static_cast<const float*>(h), static_cast<float*>(hp),
                       d);
    return hipGetLastError();
}

}  // namespace tf
