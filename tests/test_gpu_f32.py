"""The fp32 LM head at the edges of its row blocks and vocabulary slices.

Small integer operands make every logit exact whatever the order of the sums,
with many ties: the lists must be a stable sort by (value desc, id asc).
"""
import pytest

pytestmark = pytest.mark.gpu


# one row, a row block and one more; slices of 1, 2 and 8 tiles; ragged last
# tiles; widths below, at and above a 128-wide chunk; lists longer than a slice keeps
@pytest.mark.parametrize("rows,V,d,k", [
    (1, 33, 16, 8), (16, 4096, 256, 16), (17, 4099, 144, 40), (29, 20000, 128, 64), (70, 9001, 48, 5),
    (600, 5000, 272, 33), (2, 200003, 32, 300),
])
def test_f32_lm_head_is_the_stable_sort(rows, V, d, k):
    import torch
    from paper_2606_03819_amd import binding
    g = torch.Generator(device="cuda").manual_seed(rows + V)
    h = torch.randint(-2, 3, (1, rows, d), generator=g, device="cuda").float()
    lm = torch.randint(-2, 3, (V, d), generator=g, device="cuda").float() * 0.25
    lse = torch.empty((1, rows), dtype=torch.float32, device="cuda")
    idx, lp = binding.treeflash_marginal_topk(h, lm, k, lse=lse)
    y = h[0].double() @ lm.double().t()
    want = torch.sort(y, dim=1, descending=True, stable=True)
    assert torch.equal(idx[0].long(), want.indices[:, :k]), "ids are not the stable sort's"
    # fp32 sums of at most V exponentials and one logarithm
    ref = torch.logsumexp(y, 1)
    assert (lse[0].double() - ref).abs().max() <= 1e-4
    assert (lp[0].double() - (want.values[:, :k] - ref[:, None])).abs().max() <= 1e-4
