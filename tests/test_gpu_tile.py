"""The LM head's block-tiled kernel on small shapes.

Operands are small integers (and a power of two), so every logit is exact in
any order of the sums and carries many ties: the lists must equal a stable
sort by (value desc, id asc) entry by entry, which exercises the lane, wave
and workgroup merges, the bounds and the exact re-evaluation of the kernel's
own chain.
"""
import pytest

pytestmark = pytest.mark.gpu


def _case(rows, V, d, seed, spread):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    h = torch.randint(-2, 3, (1, rows, d), generator=g, device="cuda").to(torch.bfloat16)
    lm = torch.randint(-spread, spread + 1, (V, d), generator=g, device="cuda").to(torch.bfloat16) * 0.25
    return h, lm


def _check(h, lm, k, idx, lp, lse):
    import torch
    y = h[0].double() @ lm.double().t()
    want = torch.sort(y, dim=1, descending=True, stable=True)
    assert torch.equal(idx[0].long(), want.indices[:, :k]), "ids are not the stable sort's"
    ref_lse = torch.logsumexp(y, 1)
    # fp32 sums of at most V exponentials and one logarithm
    assert (lse[0].double() - ref_lse).abs().max() <= 1e-4
    assert (lp[0].double() - (want.values[:, :k] - ref_lse[:, None])).abs().max() <= 1e-4


# row blocks of 192 and 256 rows and their remainders; slices of 6, 7 and 8
# tiles, several rounds, a ragged last tile; k steps with a tail (d % 64) and
# fewer steps than the rings hold; short and long lists
@pytest.mark.parametrize("rows,V,d,k", [
    (129, 8193, 64, 8), (192, 20011, 16, 32), (193, 57344, 80, 32), (256, 65536 + 31, 128, 64),
    (241, 50021, 112, 100), (257, 5003, 192, 32), (384, 3001, 48, 64), (385, 9000, 1040, 16), (513, 300, 320, 300),
    (700, 33, 64, 5),
])
def test_lm_head_tile_is_the_stable_sort(rows, V, d, k):
    import torch
    from paper_2606_03819_amd import binding
    h, lm = _case(rows, V, d, rows + V, 2 if d < 512 else 1)
    lse = torch.empty((1, rows), dtype=torch.float32, device="cuda")
    idx, lp = binding.treeflash_marginal_topk(h, lm, k, lse=lse)
    _check(h, lm, k, idx, lp, lse)


# at most 128 rows: vocabularies of 2 to 8 tiles a CU (slices of 4, 6, 7 and 8
# tiles, ragged last tiles and CUs without one), and widths that are no multiple
# of 64 over several rounds
@pytest.mark.parametrize("rows,V,d,k", [
    (1, 8193, 64, 8), (16, 33000, 80, 16), (32, 57344, 128, 100), (33, 40961, 64, 32), (64, 65536, 192, 64),
    (65, 16384, 48, 32), (97, 50021, 320, 70), (128, 57345, 64, 16), (121, 70001, 112, 32),
])
def test_lm_head_tile_few_rows(rows, V, d, k):
    import torch
    from paper_2606_03819_amd import binding
    h, lm = _case(rows, V, d, rows + V, 2)
    lse = torch.empty((1, rows), dtype=torch.float32, device="cuda")
    idx, lp = binding.treeflash_marginal_topk(h, lm, k, lse=lse)
    _check(h, lm, k, idx, lp, lse)


def test_lm_head_tile_against_the_lean_plan():
    """The static-scratch call keeps fitting 16 MiB by the plan with fewer slices (two row blocks of the streaming
    kernel, from 196616 tokens on at 256 rows; plan_check.cpp holds that the usual plan does not fit here)."""
    import torch
    from paper_2606_03819_amd import binding
    rows, V, d, k = 256, 200001, 192, 32
    h, lm = _case(rows, V, d, 7, 2)
    lse = torch.empty((1, rows), dtype=torch.float32, device="cuda")
    idx, lp = binding.treeflash_marginal_topk_static(h, lm, k, lse=lse)
    _check(h, lm, k, idx, lp, lse)
    lse2 = torch.empty_like(lse)
    idx2, lp2 = binding.treeflash_marginal_topk(h, lm, k, lse=lse2)
    assert torch.equal(idx, idx2) and (lse - lse2).abs().max() <= 1e-4


# 129 to 256 rows over vocabularies past the tile kernel's slices (262176 tokens on): the streaming kernel's two row
# blocks, its register-staged form at widths that are no multiple of 64; short and long lists
@pytest.mark.parametrize("rows,V,d,k", [(129, 262209, 64, 8), (256, 262176, 192, 70), (193, 300007, 64, 33),
                                        (200, 262183, 80, 16)])
def test_lm_head_two_row_blocks(rows, V, d, k):
    import torch
    from paper_2606_03819_amd import binding
    h, lm = _case(rows, V, d, rows + V, 2)
    lse = torch.empty((1, rows), dtype=torch.float32, device="cuda")
    idx, lp = binding.treeflash_marginal_topk(h, lm, k, lse=lse)
    _check(h, lm, k, idx, lp, lse)


# either side of the widths below which many rows stay on the streaming kernels: 256-row blocks (up to 640 columns for
# two or three of them, 448 for more, 128 for one) and, at widths that are no multiple of 64, 128-row blocks
@pytest.mark.parametrize("rows,V,d,k", [
    (400, 3001, 64, 32), (512, 9001, 640, 70), (512, 9001, 704, 70), (1000, 5003, 448, 64), (1000, 5003, 512, 8),
    (256, 40001, 128, 16), (256, 40001, 192, 100), (300, 4099, 496, 16), (300, 4099, 528, 33), (600, 20003, 144, 64),
    (513, 8225, 80, 5), (385, 300, 48, 100),
])
def test_lm_head_narrow_widths(rows, V, d, k):
    import torch
    from paper_2606_03819_amd import binding
    h, lm = _case(rows, V, d, rows + V, 2 if d < 512 else 1)
    lse = torch.empty((1, rows), dtype=torch.float32, device="cuda")
    idx, lp = binding.treeflash_marginal_topk(h, lm, k, lse=lse)
    _check(h, lm, k, idx, lp, lse)
