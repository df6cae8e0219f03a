"""The one-sample Gram matrix with its diagonal tiles taken two at a time: even and odd numbers of 128-row tiles, a last tile that is
not full, token counts around slabs (64) and folds (512), added to what is there."""
import pytest
import torch

from paper_2405_14917_amd import binding

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def slim():
    s = binding.Slim("cuda:0")
    yield s
    s.close()


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("m,t", [(2568, 65), (4000, 300), (4096, 64), (4096, 2048), (4104, 1), (4104, 63), (4104, 65), (4224, 575), (4224, 576), (4232, 513), (4352, 2047)])
def test_diagonal_tiles_in_pairs(slim, m, t, dtype):
    gen = torch.Generator(device="cuda").manual_seed(m + t)
    X = torch.randn((m, (t + 7) // 8 * 8), generator=gen, device="cuda").to(dtype)[:, :t]
    G = torch.randn((m, m), generator=gen, device="cuda")
    G = G + G.T
    before = G.double()
    assert slim.hessian_accumulate(X, G, 5) == 5 + t
    x = X.double()
    want = before + x @ x.T
    # exact products; fp32 sums of at most 512 + 63 terms (the tokens behind the last whole slab are not folded), at most four of
    # those, and the addition to G
    bound = (min(t, 575) + 8) * 2.0 ** -24 * (x.abs() @ x.abs().T + before.abs())
    assert ((G.double() - want).abs() <= bound).all()
    assert torch.equal(G, G.T)
