// Block-tiled GEMM main loop for gfx950: Y[r, n] = sum_k X[r, k] * W[n, k]
// with enough activation rows (more than one 128-row block) that the matrix
// cores, not the weight stream, set the pace.
//
// What bounds it is power: at the 256 x 256 tile the card holds about 1.8 GHz
// against 2.4 nominal, so the shape is chosen for energy per product as much
// as for issue slots.
//  - MFMA 16x16x32 instead of 32x32x16: half the accumulator traffic per
//    product.  From registers alone, on random operands, it ran 2190 TFLOP/s
//    (2.1 GHz) against 1920 (1.8 GHz).
//  - Four waves, one per SIMD, in a 2 x 2 grid of (16 WMT) x (16 NXT) wave
//    tiles: a 128 x 128 wave tile reads 0.5 KiB of LDS per 32 K products,
//    eight 64 x 128 tiles read 0.75.
//  - One wave per SIMD hides nothing behind another wave, so the order of
//    issue is pinned (sched_barrier after every MFMA): the fragments of the
//    next 32-wide sub-step and the copies of later steps go out one by one
//    between the MFMAs of this one.  Left to the compiler, the fragment reads
//    sank to their first use and the loop ran at 0.39 of the MFMA rate.
// The main loop alone at 1936 x 151936 x 4096: 1845 us (1.31 PFLOP/s, 0.82 of
// the MFMA rate at the clock held), against 2400 us for eight waves of 2 x 4
// 32x32x16 tiles that waited for their fragments before every eight MFMAs
// (0.58), and 1950 us for the library GEMM of that shape.
//
// Copies go from memory straight into LDS, 1 KiB an instruction (8 rows of
// 128 bytes), through buffer descriptors: the row offsets are constant, the k
// step is a scalar offset (no address arithmetic in the loop, 1.5% faster
// than 64-bit addresses), and rows past the operand's end read as zeros
// without touching memory.  Weights go through a ring of three stages (copied
// two steps ahead), activations through two; DEEP: four and three where the
// LDS holds them, for tiles whose steps are shorter than a copy's latency.
// 16-byte slots are XOR-swizzled by row so that the 16 rows a quarter-wave
// reads cover all 64 banks.
//
// One barrier a step, a quarter into the second sub-step: by then this wave
// holds every fragment of step j, so the barrier both frees the stages of
// step j and publishes the copies of step j + 1, whose first fragments are
// read right after it, under the remaining MFMAs.
//
// PAIRED: the activation rows hold bf16 hi/lo pairs interleaved by 8 (256
// bytes a step), both multiplied by the same weight fragment.
//
// WIDE: rows too long for a descriptor's offsets (more than 2^20 elements).
// Copies go through 64-bit addresses, and what lies past an operand's end comes
// from a piece of zeros.
#pragma once

#include <utility>

#include "common.hpp"
#include "dma.hpp"

namespace tf {

// f(std::integral_constant<int, 0>) .. f(<N - 1>): a loop whose body sees its
// index as a constant (the unroller gives up on the main loop's size)
template <class F, int... I>
__device__ __forceinline__ void static_for_seq(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_seq(f, std::make_integer_sequence<int, N>{});
}
// The operation issued before MFMA q when `n` of them are spread over the
// MFMAs [q0, q0 + span), the t-th at q0 + (t + shift / 2) * span / n; -1: none.
constexpr int op_at(int q, int q0, int span, int n, int shift) {
    for (int t = 0; t < n; ++t)
        if (q == q0 + (2 * t + shift) * span / (2 * n)) return t;
    return -1;
}

__device__ __forceinline__ f32x4 mfma_16x16x32_bf16(const u32x4& a, const u32x4& b, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                   0, 0);
}

// a buffer descriptor over `bytes` bytes at `p` (loads past them give zeros)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t byte_buffer(const void* p, size_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)(bytes < kTileSpan ? bytes : kTileSpan),
                                             0x00020000);
}

template <int WMT, int NXT, bool PAIRED = false, bool DEEP = false, bool WIDE = false>
struct TileGemm {
    static constexpr int NTH = 256;
    static constexpr int WROWS = 32 * WMT;              // weight rows of a workgroup
    static constexpr int XROWS = 32 * NXT;              // activation rows of a workgroup
    static constexpr int NP = PAIRED ? 2 : 1;
    static constexpr int XROWB = 128 * NP;              // bytes of an activation row in one stage
    static constexpr unsigned kTailBit = 2 * kTileSpan;   // on a byte offset: past K
    static constexpr int WST = WROWS * 128;
    static constexpr int XST = XROWS * XROWB;
    // stages of the two rings
    static constexpr int SX = DEEP && 3 * WST + 3 * XST <= 160 * 1024 ? 3 : 2;
    static constexpr int SW = SX == 3 && 4 * WST + 3 * XST <= 160 * 1024 ? 4 : 3;
    static constexpr int XOFF = SW * WST;
    static constexpr int SMEM = XOFF + SX * XST;
    static constexpr int WI = WMT;                      // copies per wave and step
    static constexpr int XI = NXT * NP;
    static constexpr int MF = WMT * NXT * NP;           // MFMAs per sub-step
    static constexpr int NR = WMT + NXT * NP;           // fragment reads per sub-step
    static_assert(SMEM <= 160 * 1024, "LDS");
    static_assert((SW - 1) * WI + SX * XI < 64, "vmcnt range");
    static_assert(MF - MF / 4 >= NR, "at most one read per MFMA");

    // accumulator (m, n) register j: weight row wrow(m) + j, activation row xrow(n)
    f32x4 acc[WMT][NXT];

    unsigned char* lds;
    int lane, wave, wa, wb;
    __amdgpu_buffer_rsrc_t rw[2], rx;   // weight copy i reads through rw[i & 1]
    unsigned wof[WI], xof[XI];          // byte offsets of this lane's pieces
    const uint16_t *wp[WI], *xp[XI];    // WIDE: their addresses at step 0, `zeros` apart from the live ones
    const uint16_t* zeros;
    unsigned wlive, xlive;
    int krem;                           // columns of the last step, 64 where it is whole
    int step0, last;                    // first and last 64-wide step

    __device__ __forceinline__ int wrow(int m) const { return (wa * WMT + m) * 16 + 4 * (lane >> 4); }
    __device__ __forceinline__ int xrow(int n) const { return (wb * NXT + n) * 16 + (lane & 15); }

    __device__ __forceinline__ void init(unsigned char* smem) {
        lds = smem;
        lane = threadIdx.x & 63;
        wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        wa = wave & 1;
        wb = wave >> 1;
    }
    // tile rows of weight copy i: row0 .. row0 + 7, this lane row0 + lane / 8
    __device__ __forceinline__ int wcopy_row(int i) const { return (wave * WI + i) * 8 + (lane >> 3); }

    // Weights: row r of the tile at byte offset offset(r) behind descriptor
    // `even` (copies of rows 16 t .. 16 t + 7) or `odd` (the other eight).
    template <class RowOffset>
    __device__ __forceinline__ void weights(__amdgpu_buffer_rsrc_t even, __amdgpu_buffer_rsrc_t odd,
                                            const RowOffset& offset) {
        const bool flip = (wave * WI) & 1;
        rw[0] = flip ? odd : even;
        rw[1] = flip ? even : odd;
#pragma unroll
        for (int i = 0; i < WI; ++i) {
            const int row = wcopy_row(i);
            wof[i] = offset(row) + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
        }
    }
    // WIDE: row r of the tile at row(r), null past the operand's end; `z` is a piece of zeros.
    template <class RowAddress>
    __device__ __forceinline__ void weights(const uint16_t* z, const RowAddress& address) {
        zeros = z;
        wlive = 0;
#pragma unroll
        for (int i = 0; i < WI; ++i) {
            const int row = wcopy_row(i);
            const uint16_t* p = address(row);
            wp[i] = p != nullptr ? p + (((lane & 7) ^ ((row >> 1) & 7)) << 3) : z;
            wlive |= p != nullptr ? 1u << i : 0u;
        }
    }
    // Activations: rows [0, rows) of x, `ld` elements apart; the reduction
    // covers K weight columns.  Steps [s0, s1) of 64 columns.
    __device__ __forceinline__ void activations(const uint16_t* x, long ld, int rows, int K, int s0, int s1) {
        krem = s1 > (K - 1) / 64 ? K - (K - 1) / 64 * 64 : 64;
        if constexpr (!WIDE) rx = byte_buffer(x, ((size_t)(rows - 1) * ld + (size_t)K * NP) * 2);
        xlive = 0;
#pragma unroll
        for (int i = 0; i < XI; ++i) {
            const int row = PAIRED ? (wave * XI + i) * 4 + (lane >> 4) : (wave * XI + i) * 8 + (lane >> 3);
            const int ls = PAIRED ? (lane & 15) ^ (row & 15) : (lane & 7) ^ ((row >> 1) & 7);
            if constexpr (WIDE) {
                xp[i] = x + (size_t)(row < rows ? row : 0) * ld + ls * 8;
                xlive |= row < rows ? 1u << i : 0u;
            } else {
                xof[i] = row < rows ? (unsigned)((size_t)row * ld * 2) + ls * 16 : (unsigned)kTileSpan;
            }
        }
        step0 = s0;
        last = s1 - 1;
    }

    template <int CPOL>
    __device__ __forceinline__ void copy_w(int step, int slot, int i) const {
        unsigned char* const to = lds + slot * WST + (wave * WI + i) * 1024;
        if constexpr (WIDE)
            dma16((wlive >> i & 1) != 0 ? wp[i] + (size_t)step * 64 : zeros, to, CPOL);
        else
            buffer_dma16(rw[i & 1], wof[i], step * 128, to, CPOL);
    }
    __device__ __forceinline__ void copy_x(int step, int slot, int i) const {
        unsigned char* const to = lds + XOFF + slot * XST + (wave * XI + i) * 1024;
        if constexpr (WIDE)
            dma16((xlive >> i & 1) != 0 ? xp[i] + (size_t)step * (XROWB / 2) : zeros, to, 0);
        else
            buffer_dma16(rx, xof[i], step * XROWB, to, 0);
    }
    // Before the copies of the last step: pieces past K go out of range, the
    // weights' too (what lies there times a zero need not be a zero).
    __device__ __forceinline__ void enter_w(int step) {
        if (step != last || krem == 64) return;
#pragma unroll
        for (int i = 0; i < WI; ++i)
            if ((((lane & 7) ^ ((wcopy_row(i) >> 1) & 7)) << 3) >= krem) {
                if constexpr (WIDE)
                    wlive &= ~(1u << i);
                else
                    wof[i] |= kTailBit;
            }
    }
    __device__ __forceinline__ void enter_x(int step) {
        if (step != last || krem == 64) return;
#pragma unroll
        for (int i = 0; i < XI; ++i) {
            const int ls = PAIRED ? ((lane & 15) ^ (((wave * XI + i) * 4 + (lane >> 4)) & 15)) >> 1
                                  : (lane & 7) ^ ((((wave * XI + i) * 8 + (lane >> 3)) >> 1) & 7);
            if (ls * 8 >= krem) {
                if constexpr (WIDE)
                    xlive &= ~(1u << i);
                else
                    xof[i] |= kTailBit;
            }
        }
    }
    __device__ __forceinline__ void leave() {   // (WIDE: one loop an operand)
        if (WIDE || krem == 64) return;
#pragma unroll
        for (int i = 0; i < WI; ++i) wof[i] &= ~kTailBit;
#pragma unroll
        for (int i = 0; i < XI; ++i) xof[i] &= ~kTailBit;
    }

    // The copies of the first steps (the LDS rings must be free): SW - 1 of the
    // weights, SX of the activations, in the order of the steps.
    template <int CPOL>
    __device__ __forceinline__ void prologue() {
        static_assert(SW - 1 <= SX, "order of the first copies");
#pragma unroll
        for (int s = 0; s < SX; ++s) {
            const int step = min(step0 + s, last);
            if (s < SW - 1) {
                enter_w(step);
#pragma unroll
                for (int i = 0; i < WI; ++i) copy_w<CPOL>(step, s, i);
            }
            enter_x(step);
#pragma unroll
            for (int i = 0; i < XI; ++i) copy_x(step, s, i);
        }
    }

    // acc = the product over steps [step0, last], after prologue(); ends with
    // every copy landed and this wave's LDS reads done, but no barrier.
    template <int CPOL>
    __device__ __forceinline__ void loop() {
        u32x4 af[2][WMT], bf[2][NXT * NP];
        // fragment byte offsets within a stage, by 32-wide sub-step
        int wfo[2], xfo[2][NP];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int r = lane & 15, ls = 4 * s + (lane >> 4);
            wfo[s] = wa * WMT * 2048 + r * 128 + ((ls ^ ((r >> 1) & 7)) << 4);
            if constexpr (PAIRED) {
#pragma unroll
                for (int p = 0; p < 2; ++p) xfo[s][p] = XOFF + wb * NXT * 4096 + r * 256 + (((2 * ls + p) ^ r) << 4);
            } else {
                xfo[s][0] = XOFF + wb * NXT * 2048 + r * 128 + ((ls ^ ((r >> 1) & 7)) << 4);
            }
        }
        auto read = [&](int set, int sub, int wslot, int xslot, int t) {
            if (t < NXT * NP)
                bf[set][t] = *reinterpret_cast<const u32x4*>(lds + xslot * XST + xfo[sub][t % NP] + (t / NP) * 16 * XROWB);
            else
                af[set][t - NXT * NP] =
                    *reinterpret_cast<const u32x4*>(lds + wslot * WST + wfo[sub] + (t - NXT * NP) * 2048);
        };
#pragma unroll
        for (int m = 0; m < WMT; ++m)
#pragma unroll
            for (int n = 0; n < NXT; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
        wait_vmcnt<(SW - 2) * WI + (SX - 1) * XI>();   // step step0 has landed (this wave's copies; the barrier: everyone's)
        block_barrier();
#pragma unroll
        for (int t = 0; t < NR; ++t) read(0, 0, 0, 0, t);
        constexpr int QB = MF / 4;              // the second sub-step's MFMAs before the barrier
        constexpr int SPAN = MF - MF / 4;       // MFMAs the reads and copies are spread over
        int ws = 0, xs = 0;
        for (int j = step0; j <= last; ++j) {
            const int ws1 = ws == SW - 1 ? 0 : ws + 1, wfree = ws == 0 ? SW - 1 : ws - 1;
            const int xs1 = xs == SX - 1 ? 0 : xs + 1;
            // past the end the last step is copied again, into stages nobody reads
            const int jw = min(j + SW - 1, last), jx = min(j + SX, last);
            enter_w(jw);
            enter_x(jx);
            __builtin_amdgcn_sched_barrier(0);
            static_for<2 * MF>([&](auto idx) {
                constexpr int sub = idx.value / MF, q = idx.value % MF;
                constexpr int q0 = sub == 0 ? 0 : QB;
                constexpr int rt = op_at(q, q0, SPAN, NR, 0);
                constexpr int wi = sub == 0 ? op_at(q, q0, SPAN, WI, 1) : -1;
                constexpr int xi = sub == 1 ? op_at(q, q0, SPAN, XI, 1) : -1;
                if constexpr (sub == 1 && q == QB) {
                    // this wave holds all of step j, and its copies of step j + 1 have landed
                    // (weights of steps j + 2 .. j + SW - 1 and activations of j + 2 .. j + SX - 1 may be out)
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    wait_vmcnt<(SW - 2) * WI + (SX - 2) * XI>();
                    block_barrier();
                }
                if constexpr (rt >= 0) {
                    if constexpr (sub == 0)
                        read(1, 1, ws, xs, rt);
                    else
                        read(0, 0, ws1, xs1, rt);
                }
                if constexpr (wi >= 0) copy_w<CPOL>(jw, wfree, wi);
                if constexpr (xi >= 0) copy_x(jx, xs, xi);
                constexpr int m = q / (NXT * NP), qn = q % (NXT * NP);
                constexpr int nn = (m & 1) ? NXT * NP - 1 - qn : qn;   // back and forth along the activations
                acc[m][nn / NP] = mfma_16x16x32_bf16(af[sub][m], bf[sub][nn], acc[m][nn / NP]);
                __builtin_amdgcn_sched_barrier(0);
            });
            ws = ws1;
            xs = xs1;
        }
        leave();
        wait_vmcnt<0>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
};

}  // namespace tf
