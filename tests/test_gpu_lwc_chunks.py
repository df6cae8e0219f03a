"""The clipping's integer products by chunk: one chunk, an even and an odd number of them, five to seven digits (columns of G that
span up to 2^53), weights of one to several digits, and workgroups of 128 rows that are not full; against the float64 oracle."""
import numpy as np
import pytest
import torch

from oracle import slim_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,beta,dtype,span", [
    (16, 128, 128, torch.float16, 0), (129, 96, 32, torch.float32, 4), (40, 160, 32, torch.bfloat16, 12),
    (300, 256, 64, torch.float32, 9), (31, 640, 128, torch.float16, 16)])
def test_chunks(n, m, beta, dtype, span):
    from paper_2405_14917_amd import binding
    g = torch.Generator().manual_seed(m + span)
    W = (torch.randn((n, m), generator=g) * 0.05).to(dtype)
    X = torch.randn((m, 2 * m), generator=g, dtype=torch.float64)
    X = X + 0.5 * X[torch.randperm(m, generator=g)]
    X *= 2.0 ** torch.linspace(-span, span, m, dtype=torch.float64)[torch.randperm(m, generator=g)][:, None]
    G = (X @ X.t()).to(torch.float32)
    k = m // beta
    bits = np.array(([2, 3, 1] * k)[:k], dtype=np.uint8)
    ref = orc.lwc_quantize(W.double().numpy(), G.double().numpy(), 2 * m, bits, beta, steps=4)
    slim = binding.Slim("cuda:0")
    try:
        out = slim.lwc_quantize(W.cuda(), G.cuda(), 2 * m, torch.from_numpy(bits).cuda(), beta, steps=4)
        # the bounds of the other tests of this entry point
        assert np.allclose(out["loss_curve"], ref["loss_curve"], rtol=1e-9)
        ok = ref["round_margin"].min(axis=1) > 1e-6
        assert np.array_equal(out["codes"].cpu().numpy()[ok], ref["codes"][ok])
        assert np.allclose(out["scale"].cpu().numpy(), ref["scale"], rtol=1e-9)
    finally:
        slim.close()


def few_digits(kind, m, g):
    """G whose chunks have few digits or none."""
    X = torch.randint(-2, 3, (m, 2 * m), generator=g).double()
    if kind == "diagonal":
        return torch.diag((X * X).sum(1))
    G = X @ X.t()
    if kind == "blocks":                                     # two digits near the diagonal, whole chunks without any
        i = torch.arange(m) // 96
        G = G * (i[:, None] == i[None, :])
    if kind == "mixed":                                      # most columns with five digits or more
        v = 2.0 ** (12.0 * torch.rand(m, generator=g).double())
        v[: m // 4] = 1.0
        G = v[:, None] * G * v[None, :]
    return G


@pytest.mark.parametrize("kind", ["diagonal", "blocks", "small", "mixed"])
@pytest.mark.parametrize("n,m,beta,dtype", [
    (70, 128, 128, torch.float16), (129, 288, 32, torch.bfloat16), (300, 640, 128, torch.float32), (33, 768, 256, torch.float32)])
def test_few_digits(kind, n, m, beta, dtype):
    """Sums by pairs of digits, with chunks passed over: rows far from zero (zeros outside int8) in groups without digits of their own,
    and weights of which whole chunks are zero."""
    from paper_2405_14917_amd import binding
    g = torch.Generator().manual_seed(n + m)
    W = torch.randn((n, m), generator=g) * 0.05
    if dtype == torch.float32:                               # (16-bit weights around 9 would sit on rounding ties)
        W[: n // 4] += 9.0
    W[:, m // 3: m // 3 + 64] = 0.0
    W = W.to(dtype)
    G = few_digits(kind, m, g).to(torch.float32)
    k = m // beta
    bits = np.array(([3, 2, 4] * k)[:k], dtype=np.uint8)
    ref = orc.lwc_quantize(W.double().numpy(), G.double().numpy(), 2 * m, bits, beta, steps=4)
    slim = binding.Slim("cuda:0")
    try:
        slim.profile_enable()
        out = slim.lwc_quantize(W.cuda(), G.cuda(), 2 * m, torch.from_numpy(bits).cuda(), beta, steps=4)
        assert ("lwc_grad_product@int_outputs_by_pairs" in slim.profile_collect()) == (kind != "mixed")
        assert np.allclose(out["loss_curve"], ref["loss_curve"], rtol=1e-9)
        ok = ref["round_margin"].min(axis=1) > 1e-6
        assert np.array_equal(out["codes"].cpu().numpy()[ok], ref["codes"][ok])
        assert np.allclose(out["scale"].cpu().numpy(), ref["scale"], rtol=1e-9)
    finally:
        slim.close()
