// OPT-Tree selection in rounds (tree.hip): the arguments of a selection and the
// device function every kernel of 65 to 512 nodes tries first.  Apart from HIP's
// built-in names it needs nothing of the GPU, so that the tests run it on the host.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "plan.hpp"

namespace tf {

constexpr int kTreeThreads = 1024;  // all waves preload; wave 0 alone selects

// Row tables the selection expands into.  Single: a node whose token is
// candidate m of its depth i expands into row 1 + (i-1)*M + m.  Marginal:
// every node above depth gamma expands into the marginal row of the next
// depth.  Bigram (w/ 2-prev): row 1 + m at depth 1, else
// 1 + M + (i-2)*M*M + m2*M + m with m2 the parent's candidate index.
constexpr int kTreeSingle = 0;
constexpr int kTreeMarginal = 1;
constexpr int kTreeBigram = 2;

struct TreeArgs {
    const int32_t* cond_idx;
    const float* cond_lp;
    const int32_t* topk;
    int gamma, M, K2, B, Rs, P;   // P = leading ranks of each row cached in LDS
    int mode;                     // kTreeSingle, kTreeMarginal or kTreeBigram
    int rounds;                   // select in rounds where the rows allow it
    int32_t* tok;
    int32_t* par;
    int32_t* dep;
    float* score;
    int32_t* crow;
};

// ------------------------------------------------------- selection in rounds
//
// Popping one node at a time is a serial chain of about 1 us a node once the
// frontier spans several registers a lane (257 us for four trees of 256
// nodes).  Log-probs are at most 0 and rows are sorted, so a node never scores
// above its parent or its preceding sibling, and the popped nodes are simply
// the B first of the whole tree in the candidate order.  All threads therefore
// grow the tree in rounds: every node that may still belong to the B best and
// expands gets its children down to a threshold, then the threshold rises to
// (just below) the B-th best score found so far, by a histogram.  A round is a
// few dependent steps for the whole frontier, and there are about as many
// rounds as depths; at the end each node's place is the number of nodes before
// it (258 -> 66 us for those four trees).
//
// Rows that are not sorted or hold a positive or NaN log-prob have no such
// order (a later entry may beat an earlier one), and thousands of equal scores
// may not fit the pool: both are left to the serial selection.  Only what the
// serial selection could read matters, so a row is checked up to the last child
// taken from it, as it is taken.
constexpr int kPoolCap = 1536;      // nodes held at once
constexpr int kPoolList = 512;      // nodes expanded in one round
constexpr int kPoolBins = kTreeThreads;
constexpr size_t kPoolFixed =       // score, link, info; expansion list; bins; places; scan words; scalars
    (size_t)12 * kPoolCap + 8 * kPoolList + 4 * kPoolBins + 2 * kPoolCap + 4 * 48 + 64;
constexpr int kPoolLds = 159 * 1024;
// bits of a node's info word (crow + 1) << 16 | depth << 8 | state
constexpr uint32_t kSeen = 1, kDone = 2;

__host__ __device__ inline int pool_ranks(int Rs, int K2, int ncand) {
    const long long room = (long long)kPoolLds - (long long)kPoolFixed - 4ll * ncand;
    const long long P = room / (4ll * Rs);
    return (int)(P < K2 ? P : K2);
}
inline size_t pool_lds_bytes(int Rs, int K2, int ncand) {
    return kPoolFixed + (size_t)4 * ncand + (size_t)4 * Rs * pool_ranks(Rs, K2, ncand);
}

// Selection in rounds from 65 to 512 nodes.  One sequence of 121 rows, us, serial / rounds: peaked rows, 65 nodes
// 43 / 29, 96 63 / 38, 128 83 / 44, 256 256 / 47, 512 790 / 78 (48 25 / 34 and 64 32 / 31 while the first row's entries
// took a round of their own); star-shaped trees, 65 nodes 5.1 / 3.5, 128 7.1 / 4.0, 256 16 / 5.0, 512 30 / 9.0; one of
// 128 nodes with 13 below the first row's 9.9 / 10.7; rows of fewer entries than nodes, peaked, 32 entries and 128
// nodes 81 / 50, 16 and 256 202 / 58.  Flat rows one entry short of the budget are the worst left: 64 and 65 5.1 / 13.9.
constexpr int kPoolMinBudget = 65, kPoolMaxBudget = 512;
inline bool tree_takes_rounds(int B, int Rs, int K2, int ncand) {
    return B >= kPoolMinBudget && B <= kPoolMaxBudget && pool_ranks(Rs, K2, ncand) >= 1 && Rs < 65535;
}

struct Pool {
    float* score;
    uint32_t* link;    // parent << 16 | rank
    uint32_t* info;
    uint32_t* list;    // nodes to expand: node << 16 | children, then first child
    uint32_t* base;
    uint32_t* bins;    // histogram; reused for the renumbering
    uint16_t* place;
    uint32_t* tot;     // 3 x 16 wave totals
    int* word;         // [0] pool size, [1] bin, [2] rows in order so far, [3] nodes to expand, [4] rows to open
    int* tk;
    float* lp;         // [Rs][P]
};

__device__ __forceinline__ uint32_t wave_scan_u32(uint32_t v) {   // inclusive sums over the lanes
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);    // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);    // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);    // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);    // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);   // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);   // row_bcast:31
    return v;
}
// Inclusive sums over the workgroup's threads (one barrier); `tot` is not
// written again before another barrier.
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* tot, uint32_t& total) {
    const int wave = threadIdx.x >> 6;
    const uint32_t in = wave_scan_u32(v);
    if ((threadIdx.x & 63) == 63) tot[wave] = in;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kTreeThreads / 64; ++w) {
        const uint32_t x = tot[w];
        before += w < wave ? x : 0u;
        all += x;
    }
    total = all;
    return before + in;
}

// Is node x before node y in the candidate order, their scores being equal?
__device__ inline bool pool_tie_before(const Pool& p, int x, int y) {
    const int dx = (p.info[x] >> 8) & 255, dy = (p.info[y] >> 8) & 255;
    if (dx != dy) return dx < dy;
    uint32_t lx = p.link[x], ly = p.link[y];
    while ((lx >> 16) != (ly >> 16)) {   // equal depths: both reach the common ancestor together
        lx = p.link[lx >> 16];
        ly = p.link[ly >> 16];
    }
    return (lx & 0xffff) < (ly & 0xffff);
}

static_assert(kPoolMaxBudget <= kTreeThreads && kPoolMaxBudget < kPoolCap, "a thread an entry of the first row");

// Selects a sequence's tree; false (for the whole workgroup, nothing written)
// when the rows or their ties call for the serial selection.
__device__ bool tree_rounds(const TreeArgs& a, int seq, unsigned char* dyn) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int K2 = a.K2;
    const int ncand = a.mode == kTreeMarginal ? 0 : a.gamma * a.M;
    const int P = pool_ranks(a.Rs, K2, ncand);
    Pool p;
    {
        uint32_t* w = reinterpret_cast<uint32_t*>(dyn);
        p.bins = w; w += kPoolBins;
        p.score = reinterpret_cast<float*>(w); w += kPoolCap;
        p.link = w; w += kPoolCap;
        p.info = w; w += kPoolCap;
        p.list = w; w += kPoolList;
        p.base = w; w += kPoolList;
        p.place = reinterpret_cast<uint16_t*>(w); w += kPoolCap / 2;
        p.tot = w; w += 48;
        p.word = reinterpret_cast<int*>(w); w += 16;
        p.tk = reinterpret_cast<int*>(w); w += ncand;
        p.lp = reinterpret_cast<float*>(w);
    }
    const int nent = a.Rs * K2, ncache = a.Rs * P;
    const float* rlp = a.cond_lp + (size_t)seq * nent;
    const int32_t* ridx = a.cond_idx + (size_t)seq * nent;
    // the rows' leading log-probs (all of them where they fit) and the candidates
    if (tid == 0) {
        p.word[0] = K2 >= a.B ? 1 + a.B : 1;
        p.word[2] = 1;
        p.word[3] = 0;
        p.word[4] = 0;
        p.score[0] = 0.f;   // the root: entry 0
        p.link[0] = 0;
        p.info[0] = (1u << 16) | kSeen | (K2 >= a.B ? kDone : 0u);
    }
    const int tok0 = tid < min(K2, a.B) ? ridx[tid] : -1;
    for (int e = tid; e < ncand; e += kTreeThreads) p.tk[e] = a.topk[(size_t)seq * ncand + e];
    for (int e0 = tid; e0 < ncache; e0 += 8 * kTreeThreads) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int e = min(e0 + u * kTreeThreads, ncache - 1);
            const int r = P == K2 ? 0 : e / P;
            v[u] = rlp[P == K2 ? e : r * K2 + (e - r * P)];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (e0 + u * kTreeThreads < ncache) p.lp[e0 + u * kTreeThreads] = v[u];
        }
    }
    __syncthreads();
    auto get_lp = [&](int r, int c) -> float { return c < P ? p.lp[r * P + c] : rlp[(size_t)r * K2 + c]; };
    const uint32_t target = a.B + 1;   // with the root
    // the root alone has B entries: none below the B-th can be among the B best
    const float edge = get_lp(0, min(K2, a.B) - 1);
    // no such bound: at a threshold above the root's 0, or none, nothing would be taken and nothing checked
    if (K2 >= a.B && !(edge <= 0.f)) return false;
    float tau = K2 >= a.B ? 0.f + edge : neg_inf();
    int n = 1;
    // Where the first row bounds the tree, its first B entries are in play from the start.  A star-shaped tree is
    // those alone: none of them opens a row that starts above the B-th, by their tokens (random weights seldom rank
    // a candidate there) or by the scores.  It is written at once; the serial selection takes it in a few sibling
    // runs, and the rounds took twice as long.
    if (K2 >= a.B) {
        float s = 0.f;
        int crow = -1;
        if (tid < a.B) {
            const float v = get_lp(0, tid);
            s = 0.f + v;
            if (!(v <= (tid > 0 ? get_lp(0, tid - 1) : 0.f))) p.word[2] = 0;   // not in order
            if (a.mode == kTreeMarginal)
                crow = a.gamma > 1 ? 1 : -1;
            else if (a.gamma > 1)
                for (int m = a.M - 1; m >= 0; --m) crow = p.tk[m] == tok0 ? 1 + m : crow;
            const bool opens = crow >= 0 && !(s + get_lp(crow, 0) < tau);
            if (opens) p.word[4] = 1;
            p.score[1 + tid] = s;
            p.link[1 + tid] = (uint32_t)tid;
            p.info[1 + tid] = (uint32_t)(crow + 1) << 16 | 1u << 8 | kSeen | (opens ? 0u : kDone);
        }
        __syncthreads();
        if (p.word[2] == 0) return false;
        if (p.word[4] == 0) {
            if (tid < a.B) {
                const size_t o = (size_t)seq * a.B + tid;
                a.tok[o] = tok0;
                a.par[o] = -1;
                a.dep[o] = 1;
                a.score[o] = s;
                if (a.crow != nullptr) a.crow[o] = crow;
            }
            return true;
        }
        n = 1 + a.B;
    }
    float scale = 1000.f / fminf(fmaxf(-edge, 1e-3f), 1e6f);   // bins of the score, finer as tau rises
    // rows of fewer than B entries do not bound the B-th best, which lies rows deeper: left out of the bins it leaves
    // the threshold open, and the pool overflows with nodes of no use
    if (K2 < a.B) scale *= 0.0625f;
    bool packed = false;
    uint32_t total;

    // drops the nodes below tau and renumbers the rest
    auto pack = [&]() {
        uint16_t* remap = reinterpret_cast<uint16_t*>(p.bins);
        float sc[2];
        uint32_t lk[2], in[2];
        bool alive[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int e = tid + q * kTreeThreads;
            const bool have = e < n;
            sc[q] = have ? p.score[e] : 0.f;
            lk[q] = have ? p.link[e] : 0u;
            in[q] = have ? p.info[e] : 0u;
            alive[q] = have && sc[q] >= tau;
        }
        const uint32_t incl = block_scan((alive[0] ? 1u : 0u) + (alive[1] ? 1u : 0u), p.tot, total);
        int at = (int)(incl - (alive[0] ? 1u : 0u) - (alive[1] ? 1u : 0u));
        int to[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            to[q] = at;
            if (alive[q]) remap[tid + q * kTreeThreads] = (uint16_t)at++;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (alive[q]) {
                p.score[to[q]] = sc[q];
                p.link[to[q]] = ((uint32_t)remap[lk[q] >> 16] << 16) | (lk[q] & 0xffff);   // a parent scores no less
                p.info[to[q]] = in[q];
            }
        n = (int)total;
        if (tid == 0) p.word[0] = n;
        __syncthreads();
    };

    for (int round = 0;; ++round) {
        if (round > a.B) return false;   // more rounds than pops
        // every node in play: its child row, then how many of its children reach tau
        uint32_t cnt[2] = {0u, 0u};
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int e = tid + q * kTreeThreads;
            if (e >= n) continue;
            const float s = p.score[e];
            uint32_t in = p.info[e];
            if (!(s >= tau) || (in & kDone)) continue;
            if (!(in & kSeen)) {
                const uint32_t lk = p.link[e];
                const int row = (int)(p.info[lk >> 16] >> 16) - 1, depth = (in >> 8) & 255;
                int crow = -1;
                if (depth < a.gamma) {
                    if (a.mode == kTreeMarginal) {
                        crow = depth;
                    } else {
                        const int tok = ridx[(size_t)row * K2 + (lk & 0xffff)];
                        const int* tk = p.tk + (depth - 1) * a.M;
                        int mc = -1;
                        for (int m = a.M - 1; m >= 0; --m) mc = tk[m] == tok ? m : mc;
                        if (mc >= 0) {
                            if (a.mode == kTreeSingle) {
                                crow = 1 + (depth - 1) * a.M + mc;
                            } else if (depth == 1) {
                                crow = 1 + mc;
                            } else {
                                const int mp = depth == 2 ? row - 1 : (row - 1 - a.M) % a.M;
                                crow = 1 + a.M + (depth - 2) * a.M * a.M + mp * a.M + mc;
                            }
                        }
                    }
                }
                in |= kSeen | ((uint32_t)(crow + 1) << 16) | (crow < 0 ? kDone : 0u);
            }
            const int crow = (int)(in >> 16) - 1;
            if (crow >= 0) {
                int lo = 0, hi = K2;   // children [0, lo) reach tau
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (s + get_lp(crow, mid) >= tau)
                        lo = mid + 1;
                    else
                        hi = mid;
                }
                cnt[q] = (uint32_t)lo;
                // the first child below tau ends what the serial selection may pop, unless it is no number
                if (lo < K2 && !(get_lp(crow, lo) <= 0.f)) p.word[2] = 0;
                if (lo == 0) in |= kDone;   // tau only rises
            }
            p.info[e] = in;
        }
        // nodes (high bits) and children (low 21) of the prefix that fits the pool
        uint32_t v[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) v[q] = cnt[q] != 0u ? (1u << 21) | cnt[q] : 0u;
        const uint32_t incl = block_scan(v[0] + v[1], p.tot + 16, total);
        const uint32_t before[2] = {incl - v[0] - v[1], incl - v[1]};
        if (total >> 21 == 0u) break;
        auto fits = [&](uint32_t upto) { return (upto >> 21) <= kPoolList && (int)(upto & 0x1fffffu) <= kPoolCap - n; };
        if (!fits(total) && !packed) {
            __syncthreads();   // every info word is written
            pack();
            packed = true;
            continue;
        }
        p.bins[tid] = 0u;
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (v[q] != 0u && fits(before[q] + v[q])) {
                const int e = tid + q * kTreeThreads, at = before[q] >> 21;
                const int first = n + (int)(before[q] & 0x1fffffu);
                p.list[at] = ((uint32_t)e << 16) | cnt[q];
                p.base[at] = (uint32_t)first;
                p.info[e] |= kDone;
                atomicMax(&p.word[0], first + (int)cnt[q]);
                atomicMax(&p.word[3], at + 1);
            }
        __syncthreads();
        const int nlist = p.word[3];
        if (nlist == 0) return false;   // one node's children alone overflow the pool
        n = p.word[0];
        packed = false;
        // children, a wave per node
        for (int i = wave; i < nlist; i += kTreeThreads / 64) {
            const uint32_t l = p.list[i];
            const int e = (int)(l >> 16), c1 = (int)(l & 0xffff), first = (int)p.base[i];
            const uint32_t in = p.info[e];
            const float ps = p.score[e];
            const int row = (int)(in >> 16) - 1;
            const uint32_t depth = ((in >> 8) & 255) + 1;
            for (int c = lane; c < c1; c += 64) {
                const float v = get_lp(row, c);
                if (!(v <= (c > 0 ? get_lp(row, c - 1) : 0.f))) p.word[2] = 0;   // not in order
                p.score[first + c] = ps + v;
                p.link[first + c] = ((uint32_t)e << 16) | (uint32_t)c;
                p.info[first + c] = depth << 8;
            }
        }
        __syncthreads();
        if (p.word[2] == 0) return false;
        // tau to just below the bin of the B-th best
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int e = tid + q * kTreeThreads;
            if (e < n) {
                const float s = p.score[e];
                if (s >= tau) atomicAdd(&p.bins[(int)fminf(-s * scale, (float)(kPoolBins - 1))], 1u);
            }
        }
        if (tid == 0) {
            p.word[1] = kPoolBins - 1;
            p.word[3] = 0;
        }
        __syncthreads();
        const uint32_t own = p.bins[tid];
        const uint32_t upto = block_scan(own, p.tot + 32, total);
        if (upto >= target && upto - own < target) p.word[1] = tid;
        __syncthreads();
        const int bin = p.word[1];
        if (bin < kPoolBins - 1) {
            const float t = -((float)(bin + 1) / scale) * 1.000001f;
            tau = fmaxf(tau, t);
            if (tau < 0.f) scale = fminf(1000.f / -tau, 1e30f);
        } else if (total >= target) {
            scale *= 0.0625f;   // the B-th best lies past the bins
        }
    }

    __syncthreads();
    if (p.word[2] == 0) return false;

    // every node's place in the order: the nodes of the bins before its own,
    // then those of its bin that come before it
    p.bins[tid] = 0u;
    __syncthreads();
    uint16_t* order = reinterpret_cast<uint16_t*>(p.list);   // nodes by bin (list and base)
    int bin[2], at[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int e = tid + q * kTreeThreads;
        bin[q] = -1;
        at[q] = -1;
        if (e < 1 || e >= n || !(p.score[e] >= tau)) continue;
        bin[q] = (int)fminf(-p.score[e] * scale, (float)(kPoolBins - 1));
        at[q] = (int)atomicAdd(&p.bins[bin[q]], 1u);
    }
    __syncthreads();
    const uint32_t mine = p.bins[tid];
    const uint32_t last = block_scan(mine, p.tot, total);
    p.bins[tid] = last - mine;   // only this thread reads or writes it up to here
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (bin[q] >= 0) order[p.bins[bin[q]] + at[q]] = (uint16_t)(tid + q * kTreeThreads);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        if (bin[q] < 0) continue;
        const int e = tid + q * kTreeThreads;
        const float s = p.score[e];
        const int i0 = (int)p.bins[bin[q]], i1 = bin[q] + 1 < kPoolBins ? (int)p.bins[bin[q] + 1] : (int)total;
        int pos = i0;
        for (int i = i0; i < i1; ++i) {
            const int x = order[i];
            const float so = p.score[x];
            if (so > s || (so == s && x != e && pool_tie_before(p, x, e))) ++pos;
        }
        at[q] = pos;
        p.place[e] = (uint16_t)pos;
    }
    __syncthreads();
    const size_t o = (size_t)seq * a.B;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        if (at[q] < 0 || at[q] >= a.B) continue;
        const int e = tid + q * kTreeThreads;
        const uint32_t lk = p.link[e], in = p.info[e];
        const int parent = (int)(lk >> 16);
        const int row = (int)(p.info[parent] >> 16) - 1;
        a.tok[o + at[q]] = ridx[(size_t)row * K2 + (lk & 0xffff)];
        a.par[o + at[q]] = parent == 0 ? -1 : (int)p.place[parent];
        a.dep[o + at[q]] = (int)((in >> 8) & 255);
        a.score[o + at[q]] = p.score[e];
        if (a.crow != nullptr) a.crow[o + at[q]] = (int)(in >> 16) - 1;
    }
    // rows too short for B nodes: the rest get the empty values
    for (int i = (int)total + tid; i < a.B; i += kTreeThreads) {
        a.tok[o + i] = -1;
        a.par[o + i] = -1;
        a.dep[o + i] = 0;
        a.score[o + i] = neg_inf();
        if (a.crow != nullptr) a.crow[o + i] = -1;
    }
    return true;
}

}  // namespace tf
