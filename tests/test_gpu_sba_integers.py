"""The bit allocation's integer products (digits of X_s and W, codes with one scale per row and group) where they can go
wrong: group sizes that are padded, that are cut into several chunks, and that give more chunks than the kernels describe in
LDS; token and row counts around the tiles; one to seven digits; weights and activations of every type; zero points outside
int8; all-zero channels; eight-bit codes; and inputs that are not finite.  Against the float64 oracle, with the bound of the
other tests of the objective (1e-9 relative)."""
import numpy as np
import pytest
import torch

from oracle import slim_oracle as orc
from paper_2405_14917_amd import binding

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def slim():
    s = binding.Slim("cuda:0")
    yield s
    s.close()


def layer(seed, n, m, ts, wt, xt, spread):
    g = torch.Generator().manual_seed(seed)
    # (outputs of a few hundred at most: the softmax of either side overflows beyond that)
    W = (torch.randn((n, m), generator=g) * 0.05 * 2.0 ** (-max(0, spread - 10) / 2)).to(wt)
    X = torch.randn((m, ts), generator=g) * torch.exp2(spread * (torch.rand((m, 1), generator=g) - 0.5))
    X = X.clamp(-60000.0, 60000.0).to(xt)
    X[m // 2] = 0
    if n > 8:
        W[3] = (W[3].abs() * 0.02 + W[4].abs().max()).to(wt)          # one sign, narrow range: zero points outside int8
        W[5] = 0
    return W, X, torch.rand(m, generator=g, dtype=torch.float64)


@pytest.mark.parametrize("n,m,beta,ts,N,wt,xt,spread,obj", [
    (1, 64, 32, 4, 2, torch.float16, torch.float16, 0, 0), (129, 288, 36, 36, 2, torch.float32, torch.float16, 6, 0),
    (257, 384, 96, 100, 3, torch.bfloat16, torch.bfloat16, 6, 0), (70, 640, 160, 68, 2, torch.float16, torch.bfloat16, 30, 0),
    (33, 1024, 512, 32, 7, torch.float16, torch.float16, 14, 0), (40, 512, 256, 260, 4, torch.float32, torch.bfloat16, 44, 0),
    (20, 4224, 4, 8, 2, torch.bfloat16, torch.float16, 4, 0), (300, 512, 64, 132, 7, torch.float16, torch.float16, 20, 1),
    (64, 256, 128, 64, 2, torch.float32, torch.float16, 28, 1)])
def test_integer_products(slim, n, m, beta, ts, N, wt, xt, spread, obj):
    W, X, d = layer(n + m + ts, n, m, ts, wt, xt, spread)
    gs = d[: m // beta].numpy().copy()
    Wn, Xn = W.double().numpy(), X.double().numpy()
    bits_o, p_o, obj_o, margin = orc.sba_allocate(Wn, gs, beta, N, Xn, objective=orc.OBJ_MSE if obj else orc.OBJ_KL)
    bits, p, curve = slim.sba_allocate(W.cuda(), torch.from_numpy(gs).cuda(), beta, N, X.cuda(), objective=obj)
    # 1e-9 relative; per token the divergence is a difference of terms of the size of the outputs, which fp64 holds to a few
    # times 2^-53 each (20 of them here), so that is what is left where it cancels (a single output: exactly zero)
    floor = ts * 20 * 2.0 ** -53 * (1.0 + np.max(np.abs(Wn @ Xn)))
    assert np.allclose(curve, obj_o, rtol=1e-9, atol=floor), np.max(np.abs(curve - obj_o) / (1e-9 * np.abs(obj_o) + floor))
    if margin > 1e-6:
        assert p == p_o and np.array_equal(bits.cpu().numpy(), bits_o)
    # prepared ahead: the same bytes
    slim.sba_prepare(W.cuda(), beta, N, X.cuda(), objective=obj)
    bits2, p2, curve2 = slim.sba_allocate(W.cuda(), torch.from_numpy(gs).cuda(), beta, N, X.cuda(), objective=obj)
    assert np.array_equal(curve, curve2) and p == p2 and torch.equal(bits, bits2)


@pytest.mark.parametrize("where", ["W", "X"])
def test_inputs_that_are_not_finite(slim, where):
    """Every candidate's objective is then not a number, and the widths stay at the target."""
    W, X, d = layer(3, 40, 256, 32, torch.float16, torch.float16, 4)
    (W if where == "W" else X)[7, 9] = float("nan")
    bits, p, curve = slim.sba_allocate(W.cuda(), d[:4].cuda(), 64, 2, X.cuda())
    assert np.isnan(curve).all() and p == 0 and bool((bits == 2).all())


@pytest.mark.parametrize("beta,groups", [(4096, 1), (2048, 2)])
def test_sums_of_wide_groups(slim, beta, groups):
    """A zero point outside int8 multiplies the sum of a group's activations: here thousands of integers of 54 bits."""
    g = torch.Generator().manual_seed(beta)
    n, m, ts = 6, beta * groups, 32
    W = (1.0 + torch.rand((n, m), generator=g) / 64).to(torch.float16)         # zero points of about -190
    X = (1.0 + torch.rand((m, ts), generator=g)).to(torch.bfloat16)
    X[5, 7] = 2.0 ** -53                                                       # the unit is its own digit
    gs = np.arange(groups, dtype=np.float64)
    _, _, obj_o, _ = orc.sba_allocate(W.double().numpy(), gs, beta, 2, X.double().numpy(), objective=orc.OBJ_MSE)
    _, _, curve = slim.sba_allocate(W.cuda(), torch.from_numpy(gs).cuda(), beta, 2, X.cuda(), objective=1)
    assert np.allclose(curve, obj_o, rtol=1e-9), (curve, obj_o)


@pytest.mark.parametrize("huge", ["X", "W", "row of W"])
def test_blocks_of_very_different_size(slim, huge):
    """Elements that are a hundred binary digits larger than the others, and that meet zeros: the others keep their digits."""
    n, m, beta, ts = 40, 512, 128, 96
    W, X, d = layer(9, n, m, ts, torch.float32, torch.bfloat16, 0)
    X[m // 2] = torch.randn(ts).to(torch.bfloat16)
    if huge == "row of W":                            # in the same channels as the others' weights
        W[7], X[beta: beta + 16] = 0.0, 0.0
        W[7, beta: beta + 16] = 2.0 ** 100
    else:
        W[:, beta: 2 * beta] = 0.0
        X[beta: 2 * beta] = 0.0
        (X if huge == "X" else W.t())[beta: 2 * beta] = 2.0 ** 100
    gs = d[: m // beta].numpy().copy()
    bits_o, p_o, obj_o, margin = orc.sba_allocate(W.double().numpy(), gs, beta, 2, X.double().numpy(), objective=orc.OBJ_MSE)
    bits, p, curve = slim.sba_allocate(W.cuda(), torch.from_numpy(gs).cuda(), beta, 2, X.cuda(), objective=1)
    assert obj_o.min() > 0.0 and np.allclose(curve, obj_o, rtol=1e-9), (curve, obj_o)
    if margin > 1e-6:
        assert p == p_o and np.array_equal(bits.cpu().numpy(), bits_o)
