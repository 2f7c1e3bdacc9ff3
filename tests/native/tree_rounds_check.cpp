// Host run of the tree selection in rounds (tree_rounds.hpp): the device
// function itself, its 1024 threads as fibers that switch at barriers and
// cross-lane moves, in an order that varies.  LDS and every array end at a page
// nothing may touch.  For each case: the LDS the launch reserves suffices; a
// selection that reports it finished wrote what a best-first walk pops one node
// at a time; rows that are sorted, at most 0 and not full of equal scores are
// finished here, not handed to the serial selection, and rows that hold a NaN
// or a positive entry where that selection would read it are handed over.
// Prints "<cases> cases, <finished> finished, <failures> failures".
#include <setjmp.h>
#include <sys/mman.h>
#include <ucontext.h>
#include <unistd.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <queue>
#include <random>
#include <vector>

#include <hip/hip_runtime.h>

#include "rows.hpp"

// ---------------------------------------------------------------- one workgroup

namespace emu {
constexpr int N = 1024;
enum State { kRun, kLane, kBarrier, kDone };
static ucontext_t home, ctx[N];   // a fiber's first entry; later switches are jumps, which spare the system calls
static jmp_buf home_at, at[N];
static bool entered[N];
static State state[N];
static int cur, posted[N], fetched[N], ctrl[N], barriers;
static std::vector<char> stacks((size_t)N * 49152);
static struct { int x; } tid;
static void yield(State s) {
    state[cur] = s;
    if (!_setjmp(at[cur])) _longjmp(home_at, 1);
}
static void resume(int t) {
    cur = tid.x = t;
    if (_setjmp(home_at)) return;
    if (entered[t]) _longjmp(at[t], 1);
    entered[t] = true;
    setcontext(&ctx[t]);
}
static int dpp(int, int v, int c, int row_mask, int, bool bound) {
    posted[cur] = v;
    ctrl[cur] = c | row_mask << 16 | (bound ? 1 << 24 : 0);
    yield(kLane);
    return fetched[cur];
}
// the moves the scans use: row_shr n, row_bcast 15 and 31; `old` is 0
static void lanes(int wave) {
    for (int l = 0; l < 64; ++l) {
        const int t = wave * 64 + l, c = ctrl[t] & 0xffff, mask = ctrl[t] >> 16 & 15;
        int src = -1;
        if (c > 0x110 && c < 0x120) src = (l & 15) >= (c & 15) ? l - (c & 15) : -1;
        else if (c == 0x142) src = l >= 16 ? (l & ~15) - 1 : -1;
        else if (c == 0x143) src = l >= 32 ? 31 : -1;
        else abort();
        fetched[t] = src >= 0 && (mask >> (l >> 4) & 1) ? posted[wave * 64 + src] : 0;
    }
}
static void (*body)();
static void entry() {
    body();
    yield(kDone);
}
static void run(void (*f)(), std::mt19937& rng) {
    body = f;
    barriers = 0;
    for (int t = 0; t < N; ++t) {
        getcontext(&ctx[t]);
        ctx[t].uc_stack.ss_sp = stacks.data() + (size_t)t * 49152;
        ctx[t].uc_stack.ss_size = 49152;
        ctx[t].uc_link = &home;
        makecontext(&ctx[t], entry, 0);
        state[t] = kRun;
        entered[t] = false;
    }
    for (;;) {
        int w[16];
        for (int i = 0; i < 16; ++i) w[i] = i;
        std::shuffle(w, w + 16, rng);
        for (int wave : w)
            for (;;) {   // the wave to its next barrier
                const bool up = rng() & 1;
                for (int i = 0; i < 64; ++i) {
                    const int t = wave * 64 + (up ? i : 63 - i);
                    if (state[t] != kRun) continue;
                    resume(t);
                }
                int nl = 0;
                for (int i = 0; i < 64; ++i) nl += state[wave * 64 + i] == kLane;
                if (nl == 0) break;
                if (nl != 64) {
                    std::printf("lanes part at a cross-lane move\n");
                    exit(1);
                }
                lanes(wave);
                for (int i = 0; i < 64; ++i) state[wave * 64 + i] = kRun;
            }
        int nb = 0, nd = 0;
        for (int t = 0; t < N; ++t) nb += state[t] == kBarrier, nd += state[t] == kDone;
        if (nd == N) return;
        if (nb != N) {
            std::printf("%d threads at a barrier, %d ended\n", nb, nd);
            exit(1);
        }
        ++barriers;
        for (int t = 0; t < N; ++t) state[t] = kRun;
    }
}
}   // namespace emu

#undef __syncthreads
#define threadIdx emu::tid
#define __syncthreads() emu::yield(emu::kBarrier)
#define __builtin_amdgcn_update_dpp emu::dpp
#define min std::min
static uint32_t atomicAdd(uint32_t* p, uint32_t v) { const uint32_t o = *p; *p += v; return o; }
static int atomicMax(int* p, int v) { const int o = *p; *p = std::max(o, v); return o; }
namespace tf {
static float neg_inf() { return -INFINITY; }
}
#include "tree_rounds.hpp"
#undef min
using namespace tf;

// ---------------------------------------------------------------- cases

// n bytes that end at a page without access
struct Guarded {
    char* page;
    size_t len, n;
    explicit Guarded(size_t bytes) : n(bytes) {
        const size_t p = 4096;
        len = (bytes + p - 1) / p * p + p;
        page = (char*)mmap(nullptr, len, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
        mprotect(page + len - p, p, PROT_NONE);
        std::memset(page, 0xa5, len - p);
    }
    ~Guarded() { munmap(page, len); }
    void* at() { return page + len - 4096 - n; }
    template <class T>
    T* as() { return (T*)at(); }
};

struct Case {
    int mode, gamma, M, K2, B, Rs;
    std::vector<int32_t> idx, topk;
    std::vector<float> lp;
};

struct Node { int tok, par, dep, crow; float score; };

static int child_row(const Case& c, int depth, int tok, int row) {
    if (depth >= c.gamma) return -1;
    if (c.mode == kTreeMarginal) return depth;
    for (int m = 0; m < c.M; ++m)
        if (c.topk[(depth - 1) * c.M + m] == tok) {
            if (c.mode == kTreeSingle) return 1 + (depth - 1) * c.M + m;
            if (depth == 1) return 1 + m;
            const int mp = depth == 2 ? row - 1 : (row - 1 - c.M) % c.M;
            return 1 + c.M + (depth - 2) * c.M * c.M + mp * c.M + m;
        }
    return -1;
}

static std::vector<Node> walk(const Case& c) {
    struct Q { float s, ps; int depth, row, rank, par; std::vector<int> path; };
    auto after = [](const Q& a, const Q& b) {
        if (a.s != b.s) return a.s < b.s;
        if (a.depth != b.depth) return a.depth > b.depth;
        return a.path > b.path;
    };
    std::priority_queue<Q, std::vector<Q>, decltype(after)> q(after);
    auto push = [&](float ps, int depth, int row, int rank, int par, std::vector<int> path) {
        if (rank >= c.K2) return;
        path.push_back(rank);
        q.push(Q{ps + c.lp[(size_t)row * c.K2 + rank], ps, depth, row, rank, par, path});
    };
    std::vector<Node> out;
    push(0.f, 1, 0, 0, -1, {});
    while (!q.empty() && (int)out.size() < c.B) {
        Q t = q.top();
        q.pop();
        const int tok = c.idx[(size_t)t.row * c.K2 + t.rank], crow = child_row(c, t.depth, tok, t.row);
        const int n = (int)out.size();
        out.push_back(Node{tok, t.par, t.depth, crow, t.s});
        if (crow >= 0) push(t.s, t.depth + 1, crow, 0, n, t.path);
        t.path.pop_back();
        push(t.ps, t.depth, t.row, t.rank + 1, t.par, t.path);
    }
    return out;
}

static std::mt19937 rng(7);
static float uniform(float a, float b) { return std::uniform_real_distribution<float>(a, b)(rng); }

static Case make(int mode, int gamma, int M, int K2, int B, const char* shape) {
    Case c{mode, gamma, mode == kTreeMarginal ? 0 : M, K2, B, 0, {}, {}, {}};
    c.Rs = mode == kTreeMarginal ? gamma : (int)cond_rows(gamma, M, mode == kTreeBigram);
    const std::string sh = shape;
    std::vector<std::vector<int>> cand(gamma);   // M candidates a depth
    std::vector<int> pool(4096);
    for (int i = 0; i < 4096; ++i) pool[i] = i;
    for (auto& d : cand) {
        std::shuffle(pool.begin(), pool.end(), rng);
        d.assign(pool.begin(), pool.begin() + M);
        if (mode != kTreeMarginal) c.topk.insert(c.topk.end(), d.begin(), d.end());
    }
    const RowTable rt = make_row_table(gamma, M, mode == kTreeBigram);
    for (int r = 0; r < c.Rs; ++r) {
        const int depth = mode == kTreeMarginal ? r : rt.depth(r) - 1;
        std::vector<int> toks = cand[depth];   // candidates lead most rows
        std::shuffle(toks.begin(), toks.end(), rng);
        for (int i = 0; i < K2; ++i) toks.push_back(5000 + i);
        toks.resize(K2);
        if (r % 3 == 0) std::shuffle(toks.begin(), toks.end(), rng);
        if (sh == "closed" && r == 0)   // the first candidates come past the B-th entry, or not at all
            for (int i = 0; i < std::min(K2, B); ++i) toks[i] = 9500 + i;
        c.idx.insert(c.idx.end(), toks.begin(), toks.end());
        std::vector<float> l(K2);
        const float slope = uniform(0.6f, 2.f);
        for (int i = 0; i < K2; ++i) {
            l[i] = std::min(-1.2f * std::log1p((float)i) * slope - 0.3f + uniform(-0.4f, 0.4f), -1e-3f);
            if (sh == "flat") l[i] = uniform(-10.f, -9.f);
            if (sh == "mixed") l[i] = r == 0 ? uniform(-4.f, -1.f) : uniform(-4.f, -2.f);
            if (sh == "ties") l[i] = std::round(l[i] * 2) / 2;
            if (sh == "zeros" && i < 3) l[i] = 0.f;
            if (sh == "allzero") l[i] = r % 2 ? 0.f : -0.f;
            if (sh == "edge") l[i] = r == 0 ? -1.f - (i >= B / 2) : -1.f;   // children tie with the first row's B-th
        }
        std::sort(l.rbegin(), l.rend());
        if (sh == "tail")
            for (int i = K2 / 5; i < K2; ++i) l[i] = -INFINITY;
        if (sh == "impossible") std::fill(l.begin(), l.end(), -INFINITY);
        c.lp.insert(c.lp.end(), l.begin(), l.end());
    }
    return c;
}

static int cases = 0, finished = 0, fails = 0;
static TreeArgs g_args;
static unsigned char* g_dyn;
static bool g_ret[emu::N];

// want: 2 must finish before the first round, 1 must finish, 0 must be handed over, -1 either
static void check(const Case& c, const char* shape, int want) {
    ++cases;
    const int ncand = c.mode == kTreeMarginal ? 0 : c.gamma * c.M;
    auto fail = [&](const char* what) {
        if (fails++ < 20)
            std::printf("FAIL %s mode %d gamma %d M %d K2 %d B %d: %s\n", shape, c.mode, c.gamma, c.M, c.K2, c.B, what);
    };
    if (!tree_takes_rounds(c.B, c.Rs, c.K2, ncand)) return fail("not selected in rounds");
    Guarded idx(c.idx.size() * 4), lp(c.lp.size() * 4), topk(c.topk.size() * 4), lds(pool_lds_bytes(c.Rs, c.K2, ncand));
    Guarded tok(4 * c.B), par(4 * c.B), dep(4 * c.B), score(4 * c.B), crow(4 * c.B);
    std::memcpy(idx.at(), c.idx.data(), c.idx.size() * 4);
    std::memcpy(lp.at(), c.lp.data(), c.lp.size() * 4);
    std::memcpy(topk.at(), c.topk.data(), c.topk.size() * 4);
    if (lds.n > 160 * 1024) return fail("more LDS than a workgroup has");
    g_args = TreeArgs{idx.as<int32_t>(), lp.as<float>(), topk.as<int32_t>(), c.gamma, c.M, c.K2, c.B, c.Rs, 0, c.mode, 1,
                      tok.as<int32_t>(), par.as<int32_t>(), dep.as<int32_t>(), score.as<float>(), crow.as<int32_t>()};
    g_dyn = lds.as<unsigned char>();
    emu::run([] { g_ret[emu::cur] = tree_rounds(g_args, 0, g_dyn); }, rng);
    for (int t = 1; t < emu::N; ++t)
        if (g_ret[t] != g_ret[0]) return fail("threads disagree");
    finished += g_ret[0];
    if (want >= 0 && g_ret[0] != (want >= 1)) return fail(want ? "handed over" : "not handed over");
    if (want == 2 && emu::barriers > 2) return fail("a star-shaped tree selected in rounds");
    if (!g_ret[0]) return;
    const std::vector<Node> w = walk(c);
    for (int i = 0; i < c.B; ++i) {
        const Node e = i < (int)w.size() ? w[i] : Node{-1, -1, 0, -1, -INFINITY};
        if (g_args.tok[i] != e.tok || g_args.par[i] != e.par || g_args.dep[i] != e.dep || g_args.crow[i] != e.crow ||
            g_args.score[i] != e.score)
            return fail("differs from the walk");
    }
}

int main() {
    struct { int gamma, M, K2, B; } sizes[] = {
        {16, 8, 256, 256}, {16, 8, 65, 65}, {9, 3, 40, 512}, {16, 30, 128, 128}, {1, 4, 300, 300}, {2, 5, 100, 90},
        {3, 2, 30, 150}, {12, 16, 300, 300}, {16, 8, 512, 400}, {5, 4, 512, 512}, {8, 4, 4096, 100}, {16, 8, 16, 256},
        {16, 8, 32, 65}, {16, 8, 32, 512}};
    for (auto s : sizes)
        for (int mode : {kTreeSingle, kTreeMarginal, kTreeBigram}) {
            if (mode == kTreeBigram && s.M > 16) continue;
            long long cap = 0, pw = s.K2;   // nodes the rows hold
            for (int j = 0; j < s.gamma && cap < s.B; ++j, pw *= mode == kTreeMarginal ? s.K2 : s.M) cap += pw;
            if (cap < s.B) continue;
            for (const char* sh : {"peaked", "flat", "mixed", "tail"}) {
                // rows of fewer than B entries give no threshold to start from, and may overflow the pool
                check(make(mode, s.gamma, s.M, s.K2, s.B, sh), sh, sh[0] != 't' ? 1 : -1);
            }
            // a first row that opens none, or bounds all, of the rows below
            if (s.K2 >= s.B) {
                check(make(mode, s.gamma, s.M, s.K2, s.B, "flat"), "flat", 2);
                if (mode != kTreeMarginal) check(make(mode, s.gamma, s.M, s.K2, s.B, "closed"), "closed", 2);
            }
            for (const char* sh : {"ties", "zeros", "allzero", "edge", "impossible"})
                check(make(mode, s.gamma, s.M, s.K2, s.B, sh), sh, -1);
            // what the serial selection reads first: the first row's leading entries, up to the B-th
            for (int at : {0, s.B / 2, s.B - 1}) {
                if (at >= s.K2) continue;
                Case c = make(mode, s.gamma, s.M, s.K2, s.B, "peaked");
                c.lp[at] = NAN;
                check(c, "nan", 0);
            }
            for (int upto : {1, s.K2}) {
                Case c = make(mode, s.gamma, s.M, s.K2, s.B, "peaked");
                for (int i = 0; i < upto; ++i) c.lp[i] += 60.f;
                check(c, "positive", 0);
            }
            for (int rep = 0; rep < 2; ++rep) {   // any entries out of order, positive or not
                Case c = make(mode, s.gamma, s.M, s.K2, s.B, "peaked");
                for (int i = 0; i < 1 + 4 * rep; ++i) c.lp[rng() % c.lp.size()] = uniform(-2.f, rep ? 1.f : 0.f);
                check(c, "disorder", -1);
            }
        }
    std::printf("%d cases, %d finished, %d failures\n", cases, finished, fails);
    return fails != 0;
}
