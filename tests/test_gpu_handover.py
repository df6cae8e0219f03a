"""The hand-over between layers against the same steps in torch: clamp, rounding and transposition of what slim_dequant_matmul
gives, byte for byte, around the tiles of the layout kernels (64), both forms of the product (up to 64 tokens, more) and its split
over ranges of groups, with rows that are not aligned."""
import pytest
import torch

from paper_2405_14917_amd import binding, pipeline

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def slim():
    s = binding.Slim("cuda:0")
    yield s
    s.close()


def stored(slim, n, m, beta, gen):
    k = m // beta
    bits = torch.randint(1, 4, (k,), generator=gen, device="cuda").to(torch.uint8)
    codes = (torch.rand((n, m), generator=gen, device="cuda") * (2 ** bits.float()).repeat_interleave(beta)).floor().to(torch.uint8)
    packed, gbits, row_off, _ = slim.pack(codes, bits, beta)
    scale = torch.rand((n, k), generator=gen, device="cuda", dtype=torch.float64) * 0.2
    zero = torch.randint(0, 4, (n, k), generator=gen, device="cuda").double()
    return dict(packed=packed, gbits=gbits, row_off=row_off, scale=scale, zero=zero, bit_base=1)


@pytest.mark.parametrize("n,m,t,lead,dtype", [
    (64, 64, 1, 0, torch.float16), (65, 96, 63, 1, torch.float16), (130, 64, 66, 3, torch.float16), (257, 160, 131, 0, torch.bfloat16),
    (512, 256, 1000, 8, torch.float16), (4096, 256, 2050, 0, torch.float16), (4100, 128, 4096 + 77, 2, torch.float16)])
def test_handover_equals_its_steps(slim, n, m, t, lead, dtype):
    gen = torch.Generator(device="cuda").manual_seed(n + t)
    beta = 32
    r = stored(slim, n, m, beta, gen)
    buf = torch.randn((m, t + lead + 1), generator=gen, device="cuda").to(dtype)
    X = buf[:, lead:lead + t]
    if t > 2:
        X[:, 1] = 60000.0                                     # outputs beyond fp16's range
        X[0, 2] = float("nan")
    got = pipeline.next_layer_input(slim, r, beta, X, n)
    strided = pipeline.next_layer_input(slim, r, beta, X.t().contiguous().t(), n)      # tokens not contiguous
    want = torch.empty_like(got)
    for t0 in range(0, t, 4096):
        y = slim.dequant_matmul(r["packed"], r["gbits"], r["row_off"], r["scale"], r["zero"], beta,
                                X[:, t0:t0 + 4096].t().contiguous(), bit_base=1)
        want[:, t0:t0 + 4096] = y.clamp(-65504.0, 65504.0).to(torch.float16).t()
    for x in (got, strided):
        assert torch.equal(x.isnan(), want.isnan()) and torch.equal(x.nan_to_num(), want.nan_to_num())
