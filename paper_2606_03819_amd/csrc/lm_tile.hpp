// LM-head epilogue of the block-tiled GEMM (tile_gemm.hpp): each wave holds
// 16 WMT vocabulary rows x 16 NXT activation rows, a lane 4 WMT logits of
// each of NXT activation rows, the four lanes of a quarter-stride
// (lane, lane ^ 16, lane ^ 32, ...) the same activation rows.
//
// Per lane and row: the L best logits as keys (the truncated value with a
// position in the cleared bits), the maximum and the sum of exponentials.
// The four lanes of a row then merge their lists in registers: gfx950's
// half-wave and row swaps turn two rows' lists into both lanes' lists of one
// row in one instruction per value, so every lane merges NXT / 2, then
// NXT / 4 pairs, and only 2 lists per row (one per wave) go through LDS
// instead of 8.  A position is the token's place among the wave's 16 WMT rows
// (7 bits), so merged keys still name their token.
//
// The partial's bound covers everything unlisted: what a lane did not list is
// at most its L-th best key, what a merge drops is at most the largest
// dropped key.
#pragma once

#include "common.hpp"
#include "tile_gemm.hpp"

namespace tf {

template <int WMT, int NXT, bool LONG>
struct EpiLmTile {
    static constexpr int KEEP = LONG ? kKeepLong : kKeep;
    static constexpr int L = LONG ? kLaneTileLong : kLaneTile;   // keys a lane ranks (its list; the last bounds the rest)
    static constexpr int P = KEEP;                               // merged list length, a power of two
    static constexpr int W = P + 2;                              // words of a wave's list in LDS: keys, bound, sum
    static constexpr int RSTRIDE = 2 * W + 1;                    // odd: the rows of a wave hit distinct banks
    static constexpr int SMEM = 32 * NXT * RSTRIDE * 4;
    static constexpr int TAG = (1 << kLogitTagBits) - 1;
    static_assert(WMT * 16 <= TAG + 1, "positions of a wave's rows fit the tag bits");
    static_assert(L <= P && 16 >= L, "list lengths");
    static_assert(NXT % 2 == 0, "row pairs");

    struct List {
        float k[P];   // keys in decreasing order, -inf when empty
        float u;      // at least every key not listed
        float s;      // sum of exponentials relative to the truncated best key
    };

    static __device__ __forceinline__ float exp2_diff(float a, float m, float sl2) {   // 2^((a - m) sl2), 0 for a = -inf
        return a == neg_inf() ? 0.f : __builtin_amdgcn_exp2f((a - m) * sl2);
    }

    // b merged into a
    static __device__ __forceinline__ void merge(List& a, const List& b, float sl2) {
        const float ma = logit_trunc(a.k[0]), mb = logit_trunc(b.k[0]);
        float drop = fmaxf(a.u, b.u);
        float t[P];
#pragma unroll
        for (int i = 0; i < P; ++i) {
            t[i] = fmaxf(a.k[i], b.k[P - 1 - i]);
            drop = fmaxf(drop, fminf(a.k[i], b.k[P - 1 - i]));
        }
        // t is bitonic: half-cleaners sort it
#pragma unroll
        for (int h = P / 2; h > 0; h >>= 1)
#pragma unroll
            for (int i = 0; i < P; ++i)
                if ((i & h) == 0) {
                    const float x = t[i], y = t[i + h];
                    t[i] = fmaxf(x, y);
                    t[i + h] = fminf(x, y);
                }
#pragma unroll
        for (int i = 0; i < P; ++i) a.k[i] = t[i];
        a.u = drop;
        const float m = fmaxf(ma, mb);
        a.s = a.s * exp2_diff(ma, m, sl2) + b.s * exp2_diff(mb, m, sl2);
    }

    template <int J>
    static __device__ __forceinline__ void swap_rows(float& x, float& y) {
        if constexpr (J == 32) {
            const auto p = __builtin_amdgcn_permlane32_swap(__float_as_int(x), __float_as_int(y), false, false);
            x = __int_as_float((int)p[0]);
            y = __int_as_float((int)p[1]);
        } else {
            const auto p = __builtin_amdgcn_permlane16_swap(__float_as_int(x), __float_as_int(y), false, false);
            x = __int_as_float((int)p[0]);
            y = __int_as_float((int)p[1]);
        }
    }
    // x: row i's list, y: row i + half's; after it, x holds the merged list of
    // row i in the lanes with bit J clear and of row i + half in the others
    template <int J>
    static __device__ __forceinline__ void fold(List& x, List& y, float sl2) {
#pragma unroll
        for (int i = 0; i < P; ++i) swap_rows<J>(x.k[i], y.k[i]);
        swap_rows<J>(x.u, y.u);
        swap_rows<J>(x.s, y.s);
        merge(x, y, sl2);
    }

    // The list of accumulator column n: the wave's tokens are v0 .. v0 + 16
    // WMT - 1, those before vend count.  One pass: groups of four tiles' 16
    // logits are ranked, then summed relative to the running maximum.
    template <class G>
    static __device__ __forceinline__ List lane_list(const G& g, int n, int v0, int vend, float sl2) {
        float k[L];
#pragma unroll
        for (int q = 0; q < L; ++q) k[q] = neg_inf();
        // +inf in a scalar register the compiler cannot see through: the
        // maximum as a median with it spares the quieting of every key
        float pinf;
        asm("s_mov_b32 %0, 0x7f800000" : "=s"(pinf));
        auto insert = [&](float key) {
            float r[L];
            r[0] = __builtin_amdgcn_fmed3f(k[0], key, pinf);
#pragma unroll
            for (int q = 1; q < L; ++q) r[q] = __builtin_amdgcn_fmed3f(k[q - 1], k[q], key);
#pragma unroll
            for (int q = 0; q < L; ++q) k[q] = r[q];
        };
        const int q4 = 4 * (g.lane >> 4);
        float m = neg_inf(), s = 0.f;
        constexpr int GM = 4;   // tiles per group
#pragma unroll
        for (int m0 = 0; m0 < WMT; m0 += GM) {
            if (v0 + 16 * m0 >= vend) continue;   // wave-uniform
            const int hi = m0 + GM < WMT ? m0 + GM : WMT;
            const bool full = v0 + 16 * hi <= vend;
            float xv[4 * GM];
#pragma unroll
            for (int i = 0; i < 4 * GM; ++i)
                if (m0 + i / 4 < WMT) xv[i] = g.acc[m0 + i / 4 < WMT ? m0 + i / 4 : 0][n][i % 4];
            // position 16 m + 4 q + j of the wave: its complement's m and j bits here, the q bits below
            auto key = [&](int i) {
                return __int_as_float((__float_as_int(xv[i]) & ~TAG) | (TAG - 12 - (16 * (m0 + i / 4) + i % 4)));
            };
            auto valid = [&](int i) { return v0 + 16 * (m0 + i / 4) + q4 + i % 4 < vend; };
            if (full) {
#pragma unroll
                for (int i = 0; i < 4 * GM; ++i)
                    if (m0 + i / 4 < WMT) insert(key(i));
            } else {
#pragma unroll
                for (int i = 0; i < 4 * GM; ++i)
                    if (m0 + i / 4 < WMT) insert(valid(i) ? key(i) : neg_inf());
            }
            const float mn = logit_trunc(k[0]);
            if (mn != neg_inf()) {
                const float ms = mn * sl2;
                float t = 0.f;
                if (full) {
#pragma unroll
                    for (int i = 0; i < 4 * GM; ++i)
                        if (m0 + i / 4 < WMT) t += __builtin_amdgcn_exp2f(fmaf(xv[i], sl2, -ms));
                } else {
#pragma unroll
                    for (int i = 0; i < 4 * GM; ++i)
                        if (m0 + i / 4 < WMT && valid(i)) t += __builtin_amdgcn_exp2f(fmaf(xv[i], sl2, -ms));
                }
                s = s * __builtin_amdgcn_exp2f((m - mn) * sl2) + t;   // m = -inf: s is still 0
                m = mn;
            }
        }
        List o;
        const int qbits = 12 - q4;   // the complement of the position's q bits
#pragma unroll
        for (int q = 0; q < P; ++q)
            o.k[q] = q < L && k[q < L ? q : 0] != neg_inf() ? __int_as_float(__float_as_int(k[q < L ? q : 0]) | qbits)
                                                            : neg_inf();
        o.u = o.k[L - 1];
        o.s = s;
        return o;
    }

    // Reduce the workgroup's logits to the partials of (row, slice): tokens
    // vbase + 32 WMT rows, those before vend count; activation rows row0 ...
    // below R.  `smem` holds SMEM bytes nobody else uses.
    template <class G>
    static __device__ __forceinline__ void apply(const G& g, unsigned char* smem, int vbase, int vend, int row0, int R,
                                                 int slice, int nslices, float sl2, float* part) {
        float* cm = reinterpret_cast<float*>(smem);
        const int v0 = vbase + g.wa * WMT * 16;
        constexpr int H = NXT / 2, H2 = (H + 1) / 2;
        List l[H];
#pragma unroll
        for (int i = 0; i < H; ++i) {
            l[i] = lane_list(g, i, v0, vend, sl2);
            List y = lane_list(g, i + H, v0, vend, sl2);
            fold<32>(l[i], y, sl2);
        }
        const bool b32 = (g.lane & 32) != 0, b16 = (g.lane & 16) != 0;
#pragma unroll
        for (int i = 0; i < H2; ++i) {
            const bool pair = i + H2 < H;
            List y = pair ? l[i + H2 < H ? i + H2 : i] : l[i];
            fold<16>(l[i], y, sl2);
            const int n = (b32 ? H : 0) + i + (pair && b16 ? H2 : 0);
            if (pair || !b16) {
                float* c = cm + ((g.wb * NXT + n) * 16 + (g.lane & 15)) * RSTRIDE + g.wa * W;
#pragma unroll
                for (int q = 0; q < P; ++q) c[q] = l[i].k[q];
                c[P] = l[i].u;
                c[P + 1] = l[i].s;
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        const int r = threadIdx.x;
        if (r < 32 * NXT && row0 + r < R) {
            // the two waves' lists of row r: value and token of the best KEEP
            const float* c = cm + r * RSTRIDE;
            float v[2][P];
            int id[2][P];
#pragma unroll
            for (int w = 0; w < 2; ++w)
#pragma unroll
                for (int q = 0; q < P; ++q) {
                    const float k = c[w * W + q];
                    v[w][q] = logit_trunc(k);
                    id[w][q] = k == neg_inf() ? -1 : vbase + w * WMT * 16 + TAG - (__float_as_int(k) & TAG);
                }
            float u = logit_trunc(fmaxf(c[P], c[W + P]));
            const float ma = v[0][0], mb = v[1][0], m = fmaxf(ma, mb);
            const float s = c[P + 1] * exp2_diff(ma, m, sl2) + c[W + P + 1] * exp2_diff(mb, m, sl2);
            float tv[P];
            int ti[P];
#pragma unroll
            for (int q = 0; q < P; ++q) {
                const bool first = v[0][q] >= v[1][P - 1 - q];
                tv[q] = first ? v[0][q] : v[1][P - 1 - q];
                ti[q] = first ? id[0][q] : id[1][P - 1 - q];
                u = fmaxf(u, first ? v[1][P - 1 - q] : v[0][q]);
            }
#pragma unroll
            for (int h = P / 2; h > 0; h >>= 1)
#pragma unroll
                for (int q = 0; q < P; ++q)
                    if ((q & h) == 0) {
                        const bool keep = tv[q] >= tv[q + h];
                        const float x = tv[q], y = tv[q + h];
                        const int xi = ti[q], yi = ti[q + h];
                        tv[q] = keep ? x : y;
                        ti[q] = keep ? xi : yi;
                        tv[q + h] = keep ? y : x;
                        ti[q + h] = keep ? yi : xi;
                    }
            int cnt = 0;
#pragma unroll
            for (int q = 0; q < P; ++q) cnt += tv[q] != neg_inf() ? 1 : 0;
            float* o = part + ((size_t)(row0 + r) * nslices + slice) * part_stride(KEEP);
            *reinterpret_cast<f32x4*>(o) = f32x4{m, s, u, __int_as_float(cnt)};
#pragma unroll
            for (int q = 0; q < P; q += 4) {
                *reinterpret_cast<f32x4*>(o + 4 + q) = f32x4{tv[q], tv[q + 1], tv[q + 2], tv[q + 3]};
                *reinterpret_cast<f32x4*>(o + 4 + KEEP + q) =
                    f32x4{__int_as_float(ti[q]), __int_as_float(ti[q + 1]), __int_as_float(ti[q + 2]),
                          __int_as_float(ti[q + 3])};
            }
        }
    }
};

}  // namespace tf
