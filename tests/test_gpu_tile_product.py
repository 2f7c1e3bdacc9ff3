"""The approximator's block-tiled products (the down projection, and the input
projections of more rows than the one-row-block kernel takes, of widths that are
no multiple of 64, of many drafter states) against
plain torch in 64 bits, for every tile shape, with and without split
reductions, and with the bigram rows' products taken once per token.

The reference rounds the normalised inputs to bf16 as the kernels do and
nothing else; h' is then within one bf16 unit (the sum next to a rounding
boundary may round either way) plus 1e-3 (the activation's 16 significant
bits and the fp32 sums), and for the linear layer, which passes its input on
undamped, one input element rounded to its other neighbour: one unit of the
largest |x| times the largest |W|.
"""
import pytest

pytestmark = pytest.mark.gpu


def _rows(form, s, gamma, k, root, context, topk):
    """depth - 1 and previous tokens (nearer first) of the rows of sequence s"""
    depth, prev = [0], [(root[s], context[s])]
    for i in range(1, gamma):
        olds = [root[s]] if i == 1 else topk[s][i - 2]
        for old in olds if form == "2prev" else [0]:
            for tok in topk[s][i - 1]:
                depth.append(i)
                prev.append((tok, old))
    return depth, prev


def _inputs(form, b, gamma, k, d, I, seed, V=3000):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape, std):
        return (torch.randn(shape, generator=g, device="cuda") * std).to(torch.bfloat16)
    kin = (3 if form == "2prev" else 2) * d
    w = dict(h=normal(b, gamma, d, std=1.5), emb=normal(V, d, std=0.5), gh=(1 + normal(d, std=0.1)), ge=(1 + normal(d, std=0.1)))
    if form == "linear":
        w["lin"] = normal(d, kin, std=kin ** -0.5)
    else:
        w["gate"], w["up"], w["down"] = normal(I, kin, std=kin ** -0.5), normal(I, kin, std=kin ** -0.5), normal(d, I, std=I ** -0.5)
        if form == "silu":
            w["up"] = None

    def tokens(*shape):
        return torch.randint(0, V, shape, generator=g, device="cuda", dtype=torch.int32)
    w.update(root=tokens(b), context=tokens(b), topk=tokens(b, gamma, k))
    return w


def _gpu(form, w):
    from paper_2606_03819_amd import binding
    head = (w["h"], w["root"], w["topk"], w["emb"], w["gh"], w["ge"])
    if form == "linear":
        return binding.treeflash_arapprox_linear_hidden(*head, w["lin"])
    if form == "2prev":
        return binding.treeflash_arapprox_2prev_hidden(w["h"], w["context"], *head[1:], w["gate"], w["up"], w["down"])
    return binding.treeflash_arapprox_hidden(*head, w["gate"], w["up"], w["down"])


def _reference(form, w):
    import torch
    b, gamma, d = w["h"].shape
    k = w["topk"].shape[2]

    def rms(x, gain):
        x = x.float()
        return (x / (x.square().mean(-1, keepdim=True) + 1e-6).sqrt() * gain.float()).to(torch.bfloat16).double()
    root, context, topk = w["root"].tolist(), w["context"].tolist(), w["topk"].tolist()
    out = []
    for s in range(b):
        depth, prev = _rows(form, s, gamma, k, root, context, topk)
        h = w["h"][s][torch.tensor(depth, device="cuda")]
        x = [rms(h, w["gh"])]
        for j in range(2 if form == "2prev" else 1):
            x.append(rms(w["emb"][torch.tensor([p[j] for p in prev], device="cuda")], w["ge"]))
        x = torch.cat(x, 1)
        if form == "linear":
            out.append(h.double() + x @ w["lin"].double().t())
            continue
        a = torch.nn.functional.silu(x @ w["gate"].double().t())
        if w["up"] is not None:
            a = a * (x @ w["up"].double().t())
        out.append(h.double() + a @ w["down"].double().t())
    flip = 0.0
    if form == "linear":
        lin = w["lin"].float()
        flip = 2.0 ** -8 * 2 * float(x.abs().max()) * float(lin[lin.isfinite()].abs().max())
    return torch.stack(out), flip


def _check(form, w, rows=None):
    import torch
    got = _gpu(form, w).double()
    ref, flip = _reference(form, w)
    if rows is not None:
        got, ref = got[:, :, rows], ref[:, :, rows]
    ulp = torch.exp2(torch.floor(torch.log2(torch.maximum(got.abs(), ref.abs()).clamp_min(1e-30))) - 7)
    bad = ((got - ref).abs() > ulp + 1e-3 + flip) | got.isnan()
    assert not bad.any(), (int(bad.sum()), bad.nonzero()[:4].tolist())


# comments: tile shapes (16-row tiles of a wave, weights x rows) of the e~ half / the down projection
@pytest.mark.parametrize("form,b,gamma,k,d,I", [
    ("swiglu", 2, 9, 8, 64, 2048),      # 130 rows; 2 x 4 / 4 x 2 in eight splits
    ("swiglu", 5, 8, 8, 80, 48),        # ragged widths; 4 x 2 / 2 x 4
    ("swiglu", 16, 4, 2, 64, 64),       # few rows of many states (64)
    ("swiglu", 1, 16, 9, 208, 16),      # the narrowest SwiGLU
    ("swiglu", 3, 16, 11, 112, 9728),   # 5 x 8, 498 rows
    ("swiglu", 8, 16, 16, 80, 3008),    # 6 x 8, 1928 rows
    ("silu", 16, 16, 8, 64, 8176),      # 8 x 8, 1936 rows
    ("silu", 6, 7, 20, 1040, 1504),     # the state half in two splits; 4 x 4 in four
    ("swiglu", 16, 16, 8, 4096, 64),    # 2 x 4 in eight splits / 8 x 4
    ("swiglu", 1, 16, 16, 128, 6144),   # 241 rows of one sequence
    # the input projections on the one-row-block kernel, the down projection here: 17 to 128 rows, with and
    # without splits, and either side of the size from which 129 to 256 rows keep the one-row-block kernel
    ("swiglu", 1, 5, 4, 64, 4096), ("silu", 1, 32, 1, 192, 1024), ("swiglu", 1, 5, 8, 2560, 512),
    ("swiglu", 1, 16, 8, 128, 4160), ("swiglu", 4, 8, 4, 192, 64), ("silu", 2, 8, 9, 1088, 6208),
    ("swiglu", 1, 16, 16, 2048, 7296), ("swiglu", 1, 16, 16, 2048, 7360),
    ("silu", 1, 16, 16, 2048, 9728), ("silu", 1, 16, 16, 2048, 9792),
    # down projections of at most 64 rows: 2 x 2, one and eight splits
    ("silu", 1, 1, 1, 192, 64), ("swiglu", 1, 8, 9, 1024, 3072), ("silu", 2, 3, 4, 80, 2064),
    ("linear", 16, 16, 8, 96, 0),
    ("linear", 16, 16, 8, 2064, 0),     # 5 x 8 in two splits
    ("linear", 16, 16, 8, 4096, 0),     # 4 x 8
    ("2prev", 1, 10, 6, 96, 64), ("2prev", 2, 8, 8, 144, 2064), ("2prev", 1, 16, 8, 64, 4096),
    ("2prev", 3, 12, 1, 48, 32), ("2prev", 2, 1, 5, 80, 16), ("2prev", 2, 2, 5, 80, 16),
])
def test_block_tiled_products(form, b, gamma, k, d, I):
    print(f"[tile] {form} b{b} gamma{gamma} k{k} d{d} I{I}", flush=True)
    _check(form, _inputs(form, b, gamma, k, d, I, b * gamma + d))


def test_a_row_past_the_reduction_does_not_leak():
    """d % 64 != 0: the last step's pieces past a weight row's end lie in the next row, whose infinities must stay out."""
    import torch
    b, gamma, k, d, I = 3, 16, 8, 80, 96
    w = _inputs("linear", b, gamma, k, d, I, 5)
    w["lin"][8:24] = float("inf")
    w["lin"][40, ::3] = float("nan")
    keep = torch.ones(d, dtype=torch.bool, device="cuda")
    keep[8:24] = False
    keep[40] = False
    _check("linear", w, keep)


# weight rows of more than 2^20 columns, in the down projection or the input projections: whole and ragged last steps,
# one and many splits, more rows than one tile
@pytest.mark.parametrize("form,b,gamma,k,d,I", [
    ("swiglu", 2, 9, 8, 16, (1 << 20) + 16), ("silu", 1, 5, 4, 64, (1 << 20) + 64),
    ("swiglu", 1, 5, 4, (1 << 19) + 64, 64), ("swiglu", 1, 9, 9, (1 << 19) + 48, 48), ("silu", 2, 3, 2, (1 << 19) + 16, 16),
    ("2prev", 1, 4, 3, 349552, 32), ("2prev", 1, 3, 2, 16, (1 << 20) + 32),
])
def test_widths_past_the_tile_offsets(form, b, gamma, k, d, I):
    print(f"[wide] {form} b{b} gamma{gamma} k{k} d{d} I{I}", flush=True)
    _check(form, _inputs(form, b, gamma, k, d, I, b * gamma + 9, V=64))
