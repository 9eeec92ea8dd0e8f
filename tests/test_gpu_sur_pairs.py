"""First-layer workgroups of two 32-row tiles: up to 2048 rows the input is cut
into the same 8 splits as for 1024 rows and fewer, whose workgroups take one
tile each, so the logits have to be the same bits."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1025, 1056, 1057, 1536, 1999, 2016, 2048])
def test_pairs_of_tiles_keep_the_bits(rows):
    import torch
    print("case: pairs of tiles", rows, flush=True)
    from paper_2306_07552_amd import gal
    g = torch.Generator(device="cuda").manual_seed(rows)
    x = torch.randn((rows, 2112), generator=g, device="cuda").to(torch.bfloat16).view(torch.int16)
    mlp = gal.Mlp(max_rows=2048, seed=3)
    z = torch.full((rows,), float("nan"), device="cuda")
    mlp.forward(x, z)
    want = torch.full((rows,), float("nan"), device="cuda")
    for k in range(0, rows, 992):
        mlp.forward(x[k:k + 992], want[k:k + 992])
    torch.cuda.synchronize()
    assert not torch.isnan(z).any() and torch.equal(z, want)
