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
