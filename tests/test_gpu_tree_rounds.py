"""Budgets that are selected in rounds (65 to 512 nodes) against a best-first
walk on the host, which pops one node at a time and so also defines the result
for rows that are not sorted or hold positive entries (the rounds must leave
those to the serial selection).  Trees are compared exactly."""
import heapq

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _walk(idx, lp, topk, gamma, k, B, marginal, bigram=False):
    """One pop at a time: score desc, depth asc, rank path asc; a node's next sibling follows it into the queue."""
    K2 = idx.shape[1]
    out = []

    def push(queue, ps, depth, row, path, rank, parent):
        if rank < K2:
            s = np.float32(ps) + lp[row, rank]
            heapq.heappush(queue, (-float(s), depth, path + (rank,), float(s), row, rank, parent, ps))
    queue = []
    push(queue, np.float32(0), 1, 0, (), 0, -1)
    while queue and len(out) < B:
        _, depth, path, s, row, rank, parent, ps = heapq.heappop(queue)
        tok = int(idx[row, rank])
        n = len(out)
        out.append((tok, parent, depth, s))
        push(queue, ps, depth, row, path[:-1], rank + 1, parent)
        if depth < gamma:
            child = None
            if marginal:
                child = depth
            else:
                hit = np.nonzero(topk[depth - 1] == tok)[0]
                if hit.size and bigram and depth > 1:
                    older = row - 1 if depth == 2 else (row - 1 - k) % k
                    child = 1 + k + (depth - 2) * k * k + older * k + int(hit[0])
                elif hit.size:
                    child = 1 + (depth - 1) * k + int(hit[0])
            if child is not None:
                push(queue, np.float32(s), depth + 1, child, path, 0, n)
    return out


def _case(shape, gamma, k, K2, seed, marginal, bigram=False):
    rng = np.random.default_rng(seed)
    R = gamma if marginal else 1 + (gamma - 1) * k
    depth = np.arange(R) if marginal else np.concatenate([[0], 1 + np.arange((gamma - 1) * k) // k])
    if bigram:
        depth = np.concatenate([[0], np.ones(k, int), 2 + np.arange(max(gamma - 2, 0) * k * k) // (k * k)])
        depth = depth[:1] if gamma == 1 else depth
        R = len(depth)
    topk = np.stack([rng.permutation(5000)[:k] for _ in range(gamma)])
    idx = np.empty((R, K2), np.int64)
    for r in range(R):   # the depth's candidates lead most rows
        rest = rng.permutation(np.arange(5000, 5000 + 2 * K2))[:K2]
        idx[r] = np.concatenate([rng.permutation(topk[depth[r]]), rest])[:K2]
        if r % 3 == 0:
            idx[r] = rng.permutation(idx[r])
    if shape == "closed":   # no candidate among the first row's entries: the tree is these alone
        idx[0] = np.arange(20000, 20000 + K2)
    lp = -1.2 * np.log1p(np.arange(K2))[None] * rng.uniform(0.6, 2.0, (R, 1)) - 0.3 + 0.3 * rng.standard_normal((R, K2))
    lp = np.minimum(lp, -1e-3)
    if shape == "flat":
        lp = -9.0 - rng.random((R, K2))
    if shape == "ties":
        lp = np.round(lp * 2) / 2
    if shape == "zeros":
        lp[:, :3] = 0.0
    lp = -np.sort(-lp, axis=1).astype(np.float32)
    if shape == "tail":   # a list whose rest is impossible
        lp[:, K2 // 5:] = -np.inf
    if shape == "unsorted":
        lp[1 + seed % (R - 1), 2] = 0.0
        lp[0, K2 // 2] = -0.5
    if shape == "positive":
        lp[2 % R, 0] = 1.5
    return idx.astype(np.int32), lp.astype(np.float32), topk.astype(np.int32)


@pytest.mark.parametrize("shape,gamma,k,K2,B", [
    ("peaked", 16, 8, 256, 256), ("peaked", 16, 8, 65, 65), ("peaked", 9, 3, 40, 512), ("peaked", 16, 40, 128, 128),
    ("peaked", 1, 4, 300, 300), ("peaked", 3, 2, 30, 150), ("peaked", 12, 16, 300, 300), ("peaked", 16, 8, 512, 400),
    ("flat", 16, 8, 256, 256), ("ties", 8, 4, 100, 100), ("ties", 16, 8, 256, 512), ("zeros", 6, 4, 80, 80),
    ("peaked", 16, 8, 16, 256), ("flat", 16, 8, 32, 128), ("peaked", 16, 8, 32, 512), ("flat", 4, 8, 64, 65),
    # star-shaped trees: the first row's entries alone
    ("flat", 16, 8, 65, 65), ("flat", 16, 8, 128, 128), ("flat", 1, 4, 100, 100), ("flat", 12, 40, 200, 130),
    ("closed", 16, 8, 65, 65), ("closed", 16, 8, 512, 512), ("closed", 3, 4, 200, 130),
    ("tail", 6, 4, 100, 300), ("unsorted", 8, 4, 100, 100), ("positive", 8, 4, 100, 100), ("unsorted", 16, 20, 70, 70),
])
@pytest.mark.parametrize("marginal", [False, True])
def test_rounds_pop_what_the_walk_pops(shape, gamma, k, K2, B, marginal):
    import torch
    from paper_2606_03819_amd import binding
    if marginal and shape in ("unsorted", "positive") and gamma < 3:
        pytest.skip("needs a second row")
    cases = [_case(shape, gamma, k, K2, seed, marginal) for seed in (1, 2)]
    idx, lp, topk = (torch.from_numpy(np.stack(x)).cuda() for x in zip(*cases))
    if marginal:
        got = binding.treeflash_build_tree_marginal(idx, lp, B)
    else:
        got = binding.treeflash_build_tree(idx, lp, topk, B)
    for s, (i, p, t) in enumerate(cases):
        want = _walk(i, p, t, gamma, k, B, marginal)
        n = len(want)
        for f, name in enumerate(("token", "parent", "depth", "score")):
            g = got[name][s].cpu().numpy()
            assert g[:n].tolist() == [w[f] for w in want], f"{name} differs"
        assert (got["token"][s, n:] == -1).all() and (got["depth"][s, n:] == 0).all()


# bigram rows: parents of depth 1, 2 and deeper, no and one level of children, rows of which LDS holds a part (905 x 128)
@pytest.mark.parametrize("shape,gamma,k,K2,B", [
    ("peaked", 8, 4, 100, 100), ("peaked", 16, 8, 128, 128), ("peaked", 1, 4, 300, 300), ("peaked", 2, 5, 100, 90),
    ("ties", 6, 4, 80, 80), ("peaked", 5, 12, 256, 512), ("flat", 7, 5, 65, 65), ("unsorted", 8, 4, 100, 100),
    ("closed", 8, 4, 100, 100),
])
def test_bigram_rounds_pop_what_the_walk_pops(shape, gamma, k, K2, B):
    import torch
    from paper_2606_03819_amd import binding
    cases = [_case(shape, gamma, k, K2, seed, False, bigram=True) for seed in (1, 2)]
    idx, lp, topk = (torch.from_numpy(np.stack(x)).cuda() for x in zip(*cases))
    got = binding.treeflash_build_tree_2prev(idx, lp, topk, B)
    for s, (i, p, t) in enumerate(cases):
        want = _walk(i, p, t, gamma, k, B, False, bigram=True)
        assert len(want) == B
        for f, name in enumerate(("token", "parent", "depth", "score")):
            assert got[name][s].cpu().numpy().tolist() == [w[f] for w in want], f"{name} differs"


def test_rounds_leave_nan_to_the_serial_selection():
    """A best-first tree's first 64 nodes are the tree of budget 64, which is always selected serially."""
    import torch
    from paper_2606_03819_amd import binding
    for at in ((0, 3), (2, 0), (5, 20)):
        i, p, t = _case("peaked", 8, 4, 100, 3, False)
        p[at] = np.nan
        idx, lp, topk = (torch.from_numpy(x[None]).cuda() for x in (i, p, t))
        small, large = (binding.treeflash_build_tree(idx, lp, topk, B) for B in (64, 100))
        for f in ("token", "parent", "depth"):
            assert torch.equal(small[f], large[f][:, :64]), f


@pytest.mark.parametrize("B", [65, 100, 300, 512])
@pytest.mark.parametrize("marginal", [False, True])
def test_a_first_row_out_of_order_up_to_its_last_entry(B, marginal):
    """The first row's B-th entry bounds the tree: NaN or positive there (every entry positive), it must not."""
    import torch
    from paper_2606_03819_amd import binding
    i, p, t = _case("peaked", 8, 4, B, 3, marginal)

    def build(lp, budget):
        idx, row, topk = (torch.from_numpy(x[None]).cuda() for x in (i, lp, t))
        got = (binding.treeflash_build_tree_marginal(idx, row, budget) if marginal
               else binding.treeflash_build_tree(idx, row, topk, budget))
        return {f: got[f][0].cpu().numpy() for f in ("token", "parent", "depth", "score")}
    positive = p.copy()
    positive[0] += np.float32(60)
    got, want = build(positive, B), _walk(i, positive, t, 8, 4, B, marginal)
    for f, name in enumerate(got):
        assert got[name].tolist() == [w[f] for w in want], name
    nan = p.copy()
    nan[0, B - 1] = np.nan
    large, small = build(nan, B), build(nan, 64)   # 64 nodes are always selected serially
    for name in ("token", "parent", "depth"):
        assert large[name][:64].tolist() == small[name].tolist() and (large["depth"] > 0).all(), name
