"""The Gram matrix on row and token counts around the tiles (256 rows) and slabs (64 tokens) of its kernel: fewer than one,
whole ones, one more or less, several token ranges with a short last one, and tail tiles cut into pieces some of which are
empty.  Activations are small integers, so every sum is exact in fp32 and the result has to be equal; the padding behind the
tokens and the rows behind the matrix hold NaN, which must not get in."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("m,t", [(8, 1), (8, 63), (248, 64), (256, 65), (264, 127), (504, 200), (512, 1024), (1000, 3001),
                                 (1504, 4096), (2056, 777), (4096, 8229), (4104, 2048), (5120, 10007),
                                 (2568, 61), (2696, 2048), (3000, 1100), (4096, 2048), (5000, 513)])
def test_shapes(m, t, dtype):
    from paper_2405_14917_amd import binding
    ldx = (t + 7) // 8 * 8 + 8
    gen = torch.Generator(device="cuda").manual_seed(m + t)
    X = torch.full((m + 8, ldx), float("nan"), dtype=dtype, device="cuda")
    X[:m, :t] = torch.randint(-8, 9, (m, t), generator=gen, device="cuda").to(dtype)
    G = torch.ones((m, m), dtype=torch.float32, device="cuda")
    slim = binding.Slim("cuda:0")
    assert slim.hessian_accumulate(X[:m, :t], G, 5) == 5 + t
    ref = X[:m, :t].double() @ X[:m, :t].double().t().contiguous() + 1.0
    assert float(ref.max()) < 2 ** 24                # exact in fp32
    assert torch.equal(G.double(), ref), "m %d, t %d" % (m, t)
    slim.close()


@pytest.mark.parametrize("m,t", [(264, 130), (8, 61)])
def test_rows_far_apart(m, t):
    """Rows further apart than 32-bit offsets reach: the kernel with 64-bit row pointers."""
    from paper_2405_14917_amd import binding
    ldx = 2 ** 32 // (2 * 255) // 8 * 8 + 8
    X = torch.empty((m, ldx), dtype=torch.float16, device="cuda")[:, :t]
    X.copy_(torch.randint(-8, 9, (m, t), device="cuda"))
    G = torch.zeros((m, m), dtype=torch.float32, device="cuda")
    slim = binding.Slim("cuda:0")
    slim.hessian_accumulate(X, G, 0)
    Xc = X.double().contiguous()
    assert torch.equal(G.double(), Xc @ Xc.t().contiguous())
    slim.close()


@pytest.mark.parametrize("m,t,pad", [(2696, 130, 1), (2600, 2047, 2), (2568, 64, 3), (264, 100, 1)])
def test_a_leading_dimension_that_four_does_not_divide(m, t, pad):
    """Tiles that add to G themselves (and those that do not), where the rows of G are not aligned to 16 bytes; what lies
    beside the matrix stays as it is, and the tiles that add to G need no workspace."""
    from paper_2405_14917_amd import binding
    gen = torch.Generator(device="cuda").manual_seed(m)
    X = torch.zeros((m, (t + 7) // 8 * 8), dtype=torch.bfloat16, device="cuda")[:, :t]
    X.copy_(torch.randint(-8, 9, (m, t), generator=gen, device="cuda"))
    G = torch.full((m, m + pad), 3.0, dtype=torch.float32, device="cuda")
    slim = binding.Slim("cuda:0")
    slim.hessian_accumulate(X, G[:, :m], 0)
    Xc = X.double().contiguous()
    assert torch.equal(G[:, :m].double(), Xc @ Xc.t().contiguous() + 3.0)
    assert bool((G[:, m:] == 3.0).all())
    assert (slim.workspace_bytes() == 0) == (m > 2560)
    slim.close()
