"""The decoding of the linear layer for few tokens, width by width: every code value at every place of a chunk, whole and half zero
points up to the bounds of the operand, in groups whose codes are placed (64 and more) and shifted (32; 64 rows x 32 tokens a
wavefront, more than 8192 rows and 16 tokens)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,t", [(96, 1), (96, 17), (8448, 20), (16640, 3)])
@pytest.mark.parametrize("beta", [32, 64, 128])
@pytest.mark.parametrize("b", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_every_code_at_every_place(n, t, beta, b, dtype):
    from paper_2405_14917_amd import binding
    k = 3
    m, top = k * beta, 2 ** b
    base = 1 if b < 3 else 2
    rng = np.random.default_rng(b * beta + n)
    # row r, channel c: every value of a code passes every place of a chunk of 32
    codes = ((np.arange(n)[:, None] + np.arange(m)[None, :] // 32 + rng.integers(0, top, (1, m))) % top).astype(np.uint8)
    bits = torch.full((k,), b, dtype=torch.uint8, device="cuda")
    zero = np.rint(rng.uniform(0, top - 1, (n, k)))
    zero[:, 0] = 0.5 if b == 1 else np.rint(rng.uniform(-90, 90, n))
    zero[1::7, 1] += 0.5 if b == 1 else 3.0
    scale = rng.uniform(0.005, 0.02, (n, k))
    X = torch.from_numpy(rng.integers(-8, 9, (t, m)).astype(np.float32)).to(dtype)
    slim = binding.Slim("cuda:0")
    try:
        packed, gbits, row_off, _ = slim.pack(torch.from_numpy(codes).cuda(), bits, beta, bit_base=base)
        Y = slim.dequant_matmul(packed, gbits, row_off, torch.from_numpy(scale).cuda(), torch.from_numpy(zero).cuda(), beta, X.cuda(), bit_base=base)
    finally:
        slim.close()
    # integer activations: a group's sum is exact, so what is left is the scale rounded to fp32 and the sum of three groups in fp32
    exact, size = np.zeros((t, n)), np.zeros((t, n))
    for g in range(k):
        c = slice(g * beta, (g + 1) * beta)
        part = X[:, c].double().numpy() @ (codes[:, c].astype(np.float64) - zero[:, g:g + 1]).T * scale[:, g]
        exact += part
        size += np.abs(part)
    assert np.all(np.abs(Y.double().cpu().numpy() - exact) <= 4 * 2.0 ** -24 * size)
