"""The linear layer on the stored form for up to 64 tokens (its own kernel) against the float64 oracle: every tile (by the layer's
rows) at row counts that fill none, one and two token tiles and blocks of them, group sizes that 128, 64 and only 32 divide, every code width,
zero points outside the operand's form, more groups than one range of parameters holds, skipped groups, packed zeros."""
import numpy as np
import pytest
import torch

from test_gpu_linear_many_tokens import stored

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def slim():
    from paper_2405_14917_amd import binding
    s = binding.Slim("cuda:0")
    yield s
    s.close()


@pytest.mark.parametrize("t,n,m,beta,base,dtype,odd", [
    (1, 17, 32, 32, 1, torch.float16, False), (8, 300, 640, 128, 2, torch.float16, True),
    (9, 4096, 512, 64, 1, torch.bfloat16, True), (17, 1001, 13824, 32, 1, torch.float16, True),
    (16, 4097, 288, 96, 2, torch.bfloat16, True), (32, 8192, 256, 256, 1, torch.float16, False),
    (5, 8193, 3840, 32, 2, torch.float16, True), (64, 9001, 384, 128, 1, torch.bfloat16, True),
    (16, 16401, 3840, 32, 1, torch.bfloat16, True), (3, 16385, 256, 128, 2, torch.float16, False),
    (50, 16385, 192, 64, 2, torch.bfloat16, False)])
def test_few_tokens(slim, t, n, m, beta, base, dtype, odd):
    rng = np.random.default_rng(t + n)
    packed, gbits, row_off, scale, zero, What = stored(slim, rng, n, m, beta, base, odd)
    X = torch.from_numpy(rng.standard_normal((t, m))).to(dtype).cuda()
    Yw = torch.full((t, n + 5), -1.0, dtype=torch.float32, device="cuda")
    Y = slim.dequant_matmul(packed, gbits, row_off, scale, zero, beta, X, Y=Yw[:, :n], bit_base=base)
    Xn = X.double().cpu().numpy()
    # fp32 sums of exact products, m / 32 of them in a row at most: 1e-5 of the sum of magnitudes
    assert np.all(np.abs(Y.cpu().numpy() - Xn @ What.T) <= 1e-5 * (np.abs(Xn) @ np.abs(What).T) + 1e-30)
    assert bool((Yw[:, n:] == -1.0).all())
    # a token's outputs are the same bytes whichever other tokens share its call
    for part in (slice(0, 1), slice(t // 2, t)):
        assert torch.equal(Y[part], slim.dequant_matmul(packed, gbits, row_off, scale, zero, beta, X[part].contiguous(), bit_base=base))


def test_packed_zeros_and_skipped_groups(slim):
    rng = np.random.default_rng(3)
    for t, dtype in ((4, torch.float16), (20, torch.bfloat16)):
        packed, gbits, row_off, scale, zero, _ = stored(slim, rng, 333, 1152, 128, 1, False)
        zero = (zero * 2 + 1) / 2                      # halves too: a rest is left at widths above 1
        X = torch.from_numpy(rng.standard_normal((t, 1152))).to(dtype).cuda()
        zp, bad = slim.pack_zeros(zero, 7)
        assert bad == 0
        Y = slim.dequant_matmul(packed, gbits, row_off, scale, zero, 128, X)
        assert torch.equal(Y, slim.dequant_matmul_zp(packed, gbits, row_off, scale, zp, 7, 128, X))
        assert not bool(slim.dequant_matmul(packed, gbits, row_off, scale, zero, 128, X, bit_base=2).any())
