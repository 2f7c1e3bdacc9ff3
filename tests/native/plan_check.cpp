// Host-side check of the launch plans and the workspace layout (plan.hpp) over
// random shapes: every bf16 product gets a tile shape there is a kernel for and
// splits that are not empty; the LM head's slices cover the vocabulary once, with
// no more tiles than a workgroup's round takes; what each call keeps in the
// workspace fits its part of the layout; and a workspace is never smaller for a
// larger b, gamma or k, nor (what the linear layer relies on) for a larger I than
// for I = 16.
// Prints "<shapes> shapes, <failures> failures" and exits 1 on any failure.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>

#include "plan.hpp"

using namespace tf;

static int fails = 0;
#define CHECK(c, ...)                         \
    do {                                      \
        if (!(c)) {                           \
            if (fails++ < 20) {               \
                std::printf("FAIL %s: ", #c); \
                std::printf(__VA_ARGS__);     \
                std::printf("\n");            \
            }                                 \
        }                                     \
    } while (0)

struct Shape { int b, gamma, k, d, I, V; bool bf16, bigram; };

static void check_product(const TilePlan& p, bool paired, const char* what, const Shape& s) {
    bool known = false;
#define KNOWN(W, X, P) known = known || (p.WMT == W && p.NXT == X && paired == P);
    TF_TILE_SHAPES(KNOWN)
#undef KNOWN
    CHECK(p.wide || p.WMT * 64ll * (paired ? s.I : s.d) < (long long)kTileSpan, "%s: offsets", what);
    CHECK(known && (!p.wide || (p.WMT == kTileWideW && p.NXT == kTileWideX)), "%s %d x %d", what, p.WMT, p.NXT);
    CHECK(p.S >= 1 && (p.S - 1) * p.per < p.nk && p.S * p.per >= p.nk, "%s S %d per %d nk %d (b %d d %d I %d)", what, p.S,
          p.per, p.nk, s.b, s.d, s.I);
}

static void check_lm(int rows, int V, int d, bool bf16, bool lean) {
    const LmPlan p = lm_plan(rows, V, d, bf16, lean);
    const int most = p.tile ? p.WM : p.chunk;
    int next = 0;
    for (int s = 0; s < p.nsplit(); ++s) {
        int t0, t1;
        slice_tiles(p.map, s, t0, t1);
        if (t0 == t1) continue;
        CHECK(t0 == next && t1 - t0 <= most && t1 <= p.ntiles, "slice %d [%d, %d) after %d (rows %d V %d d %d)", s, t0, t1,
              next, rows, V, d);
        next = t1;
    }
    CHECK(next == p.ntiles, "%d of %d tiles (rows %d V %d d %d)", next, p.ntiles, rows, V, d);
    CHECK(p.nrb * (bf16 ? 32 * p.NT : 16) >= rows, "row blocks of %d rows", rows);
    if (p.tile) {
        bool known = false;
#define KNOWN(W, X, N) known = known || (p.WM == W && p.NT == X && p.wnt == N);
        TF_LM_TILE_SHAPES(KNOWN)
#undef KNOWN
        CHECK(known, "LM head %d x %d wnt %d", p.WM, p.NT, p.wnt);
    }
    CHECK(lm_scratch_bytes(p, rows, bf16) <= lm_reserve_bytes(rows, V, d, bf16) || lean, "LM scratch (rows %d V %d d %d)",
          rows, V, d);
}

// What the calls on this workspace keep in it, against the layout.
static void check_fits(const Shape& s) {
    const Workspace w = workspace_layout(s.b, s.gamma, s.d, s.I, s.V, s.k, s.bf16, s.bigram);
    const int R = (int)cond_rows(s.gamma, s.k, s.bigram), rows = s.b * R, states = s.b * s.gamma;
    const int npre = s.bigram ? 2 : 1, ew = npre * s.d;
    const size_t part = w.ht - w.mlp_part, hh = w.total - w.hh, es = s.bf16 ? 2 : 4;
    CHECK(w.ht - w.lm >= lm_scratch_bytes(rows, s.V, s.d, s.bf16) && w.ht - w.lm >= lm_scratch_bytes(states, s.V, s.d, s.bf16),
          "LM scratch");
    CHECK(w.et - w.ht >= (size_t)states * s.d * es && w.hp - w.act >= (size_t)rows * s.I * 4 &&
              w.counters - w.hp >= (size_t)rows * s.d * es,
          "rows");
    if (!s.bf16) return;
    const bool wide = tile_wide(s.d + (long long)ew);
    auto gate = [&](bool swiglu) { return mlp_dma_gate_applies(s.b, s.gamma, R, s.d, s.I, ew, swiglu, s.bigram); };
    const size_t erows = s.bigram && !gate(true) && !wide ? (size_t)s.b * bigram_tokens(s.gamma, s.k) : (size_t)rows * npre;
    CHECK(w.act - w.et >= erows * s.d * es, "embeddings (b %d gamma %d k %d)", s.b, s.gamma, s.k);
    auto tables = [&](const TilePlan& p, bool paired, int n, long long N, size_t room, const char* what) {
        check_product(p, paired, what, s);
        if (p.S > 1) CHECK((size_t)p.S * n * N * 4 <= room, "%s: S %d rows %d N %lld", what, p.S, n, N);
    };
    auto pieces = [&](const MlpDmaPlan& q) {
        CHECK(q.part_floats() * 4 <= part && q.items <= w.ncounters && w.hh - w.counters >= (size_t)q.items * 4,
              "pieces (rows %d d %d I %d)", rows, s.d, s.I);
    };
    for (int N : {2 * s.I, s.I}) {
        if (gate(N == 2 * s.I)) {
            pieces(mlp_dma_gate_plan(rows, s.d, ew, s.I, N == 2 * s.I));
        } else if (s.bigram && !wide) {
            if (N == s.I) continue;
            const int tokens = s.b * bigram_tokens(s.gamma, s.k);
            check_product(tile_token_plan(tokens, N, s.d), false, "token", s);
            CHECK(((size_t)states + 2 * (size_t)tokens) * N * 4 <= hh, "token tables");
        } else {
            const TilePlan ph = tile_state_plan(states, N, s.d, wide);
            check_product(ph, false, "state", s);
            CHECK((size_t)ph.S * states * N * 4 <= hh, "state tables (states %d N %d S %d)", states, N, ph.S);
            tables(tile_input_plan(rows, N, ew, wide), false, rows, N, part, "input");
        }
    }
    tables(tile_down_plan(rows, s.d, s.I), true, rows, s.d, part, "down");
    if (s.bigram) return;
    if (mlp_dma_linear_applies(true, s.b, s.gamma, R, s.d)) {
        pieces(mlp_dma_linear_plan(rows, s.d));
    } else {
        const bool lw = tile_wide(2ll * s.d);
        const TilePlan ph = tile_state_plan(states, s.d, s.d, lw);
        check_product(ph, false, "linear state", s);
        CHECK((size_t)ph.S * states * s.d * 4 <= hh, "linear state tables");
        tables(tile_input_plan(rows, s.d, s.d, lw), false, rows, s.d, part, "linear input");
    }
}

static std::mt19937 rng(11);
static int log_uniform(int lo, int hi) {
    return (int)std::exp(std::uniform_real_distribution<double>(std::log(lo), std::log(hi + 1.0))(rng));
}

int main() {
    long long shapes = 0;
    auto total = [](const Shape& s) {
        return workspace_layout(s.b, s.gamma, s.d, s.I, s.V, s.k, s.bf16, s.bigram).total;
    };
    for (int n = 0; n < 60000; ++n) {
        Shape s;
        s.bf16 = rng() % 8 != 0;
        s.bigram = rng() % 4 == 0;
        s.b = log_uniform(1, 64);
        s.gamma = 1 + rng() % 24;
        s.k = log_uniform(1, 64);
        const int unit = rng() % 3 ? 64 : 16;
        s.d = std::max(unit, log_uniform(16, 1 << (n % 50 == 0 ? 21 : 14)) / unit * unit);
        s.I = std::max(unit, log_uniform(16, 1 << (n % 50 == 1 ? 22 : 15)) / unit * unit);
        s.V = std::max(s.k, log_uniform(64, 400000));
        if ((long long)s.b * cond_rows(s.gamma, s.k, s.bigram) > 1 << 20) continue;
        ++shapes;
        check_fits(s);
        const int rows = s.b * (int)cond_rows(s.gamma, s.k, s.bigram);
        check_lm(rows, s.V, s.d, s.bf16, false);
        check_lm(rows, s.V, s.d, s.bf16, true);
        // any smaller call on the same weights
        Shape t = s;
        t.b = 1 + rng() % s.b;
        t.gamma = 1 + rng() % s.gamma;
        t.k = 1 + rng() % s.k;
        if (rng() % 2) t.gamma = s.gamma, t.k = s.k, t.b = std::max(1, s.b - 1);
        CHECK(total(t) <= total(s), "b %d gamma %d k %d needs %zu, b %d gamma %d k %d %zu (d %d I %d V %d %s%s)", t.b,
              t.gamma, t.k, total(t), s.b, s.gamma, s.k, total(s), s.d, s.I, s.V, s.bf16 ? "bf16" : "fp32",
              s.bigram ? " bigram" : "");
        t = s;
        t.I = 16;
        if (!s.bigram) CHECK(total(t) <= total(s), "I %d: %zu below %zu (d %d b %d)", s.I, total(s), total(t), s.d, s.b);
    }
    // every row count around the plans' steps, at widths of the 4B and 8B shapes
    for (int d : {2560, 4096, 2000})
        for (int V : {32000, 151936, 300000})
            for (int rows = 1; rows < 2600; rows += rows < 300 ? 1 : 37, ++shapes) {
                CHECK(lm_reserve_bytes(rows, V, d, true) <= lm_reserve_bytes(rows + 1, V, d, true), "rows %d", rows);
                CHECK(lm_reserve_bytes(rows, V, d, false) <= lm_reserve_bytes(rows + 1, V, d, false), "fp32 rows %d", rows);
                check_lm(rows, V, d, true, false);
                check_lm(rows, V, d, false, false);
            }
    // what the GPU tests of the lean plan and of its kernel's two row blocks take to reach them
    const LmPlan usual = lm_plan(256, 200001, 192, true), lean = lm_plan(256, 200001, 192, true, true);
    CHECK(usual.tile && 256 + lm_scratch_bytes(usual, 256, true) > 16u << 20, "usual plan");
    CHECK(lean.grid && lean.nrb == 2 && 256 + lm_scratch_bytes(lean, 256, true) <= 16u << 20, "lean plan");
    for (int V : {262209, 262176, 300007}) CHECK(lm_plan(200, V, 64, true).grid && lm_plan(200, V, 64, true).nrb == 2, "V %d", V);
    CHECK(!lm_plan(200, 262183, 80, true).tile && !lm_plan(200, 262183, 80, true).dma, "register-staged");
    std::printf("%lld shapes, %d failures\n", shapes, fails);
    return fails != 0;
}
