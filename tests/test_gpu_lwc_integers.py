"""The integer products of the learnable weight clipping where they can go wrong: padded and chunked group sizes, rows and
columns around the tiles, columns of G that span many digits (outlier channels), eight-bit codes, zero points outside int8, and
every type of W; against the float64 oracle."""
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


@pytest.mark.parametrize("n,m,beta,dtype,outlier,widths", [
    (5, 64, 32, torch.float16, 1.0, (1, 2)), (257, 300, 100, torch.float32, 300.0, (2, 3, 8)),
    (70, 640, 160, torch.bfloat16, 50.0, (2, 4)), (33, 1024, 512, torch.float16, 1000.0, (8, 7)),
    (128, 144, 36, torch.float32, 1.0, (1, 5))])
def test_lwc_against_the_oracle(slim, n, m, beta, dtype, outlier, widths):
    g = torch.Generator().manual_seed(n + m)
    W = (torch.randn((n, m), generator=g) * 0.05).to(dtype)
    W[1, :beta] = (W[1, :beta].abs() * 0.05 + 0.4).to(dtype)              # one sign: a zero point outside int8
    W[2, :beta] = 0
    X = torch.randn((m, 2 * m), generator=g, dtype=torch.float64)
    X = X + 0.5 * X[torch.randperm(m, generator=g)]
    X[3:7] *= outlier
    G = (X @ X.t()).to(torch.float32)
    k = m // beta
    bits = np.array((list(widths) * k)[:k], dtype=np.uint8)
    steps = 6
    ref = orc.lwc_quantize(W.double().numpy(), G.double().numpy(), 2 * m, bits, beta, steps=steps)
    out = slim.lwc_quantize(W.cuda(), G.cuda(), 2 * m, torch.from_numpy(bits).cuda(), beta, steps=steps, want_what=torch.float64)
    # (the bounds of the other tests of this entry point)
    assert np.allclose(out["loss_curve"], ref["loss_curve"], rtol=1e-9)
    ok = ref["round_margin"].min(axis=1) > 1e-6
    assert ok.mean() > 0.7
    assert np.array_equal(out["codes"].cpu().numpy()[ok], ref["codes"][ok])
    assert np.allclose(out["scale"].cpu().numpy(), ref["scale"], rtol=1e-9)
    assert np.array_equal(out["zero"].cpu().numpy()[ok], ref["zero"][ok])
    again = slim.lwc_quantize(W.cuda(), G.cuda(), 2 * m, torch.from_numpy(bits).cuda(), beta, steps=steps)
    assert np.array_equal(again["loss_curve"], out["loss_curve"]) and torch.equal(again["codes"], out["codes"])


@pytest.mark.parametrize("n,m,beta,dtype,widths", [
    (3, 12, 6, torch.float16, (2, 3)), (17, 36, 1, torch.float32, (1, 2)), (18, 100, 2, torch.bfloat16, (2,)),
    (5, 132, 33, torch.float16, (3, 8)), (40, 2052, 18, torch.float32, (2, 5)), (16, 60, 5, torch.bfloat16, (4, 2))])
def test_groups_that_four_does_not_divide(slim, n, m, beta, dtype, widths):
    """A group takes in no weight of its neighbour, and nothing is written behind the last row."""
    g = torch.Generator().manual_seed(n * m)
    W = (torch.randn((n, m), generator=g) * 0.05).to(dtype)
    X = torch.randn((m, 2 * m), generator=g, dtype=torch.float64)
    G = (X @ X.t()).to(torch.float32)
    k, steps = m // beta, 5
    bits = np.array((list(widths) * k)[:k], dtype=np.uint8)
    ref = orc.lwc_quantize(W.double().numpy(), G.double().numpy(), 2 * m, bits, beta, steps=steps)
    Wd, Gd, bd = W.cuda(), G.cuda(), torch.from_numpy(bits).cuda()
    out = slim.lwc_quantize(Wd, Gd, 2 * m, bd, beta, steps=steps)
    assert np.allclose(out["loss_curve"], ref["loss_curve"], rtol=1e-9)
    ok = ref["round_margin"].min(axis=1) > 1e-6
    assert ok.mean() > 0.7
    assert np.array_equal(out["codes"].cpu().numpy()[ok], ref["codes"][ok])
    assert np.allclose(out["scale"].cpu().numpy(), ref["scale"], rtol=1e-9)
    assert np.array_equal(out["zero"].cpu().numpy()[ok], ref["zero"][ok])
    # the entry point itself, with guards behind its outputs
    codes = torch.full((n * m + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    what = torch.full((n * m + 64,), -7.0, dtype=torch.float64, device="cuda")
    scale, zero = torch.empty((n, k), dtype=torch.float64, device="cuda"), torch.empty((n, k), dtype=torch.float64, device="cuda")
    ptr = binding._ptr
    slim._check(slim.lib.slim_lwc_quantize(slim.ctx, ptr(Wd), binding._DT[dtype], n, m, m, ptr(Gd), m, 2 * m, ptr(bd), beta, steps,
                                           1e-2, 0.9, 0.999, 1e-8, 4.0, ptr(codes), ptr(scale), ptr(zero), ptr(what),
                                           binding._DT[torch.float64], None))
    assert torch.equal(codes[: n * m].view(n, m), out["codes"]) and bool((codes[n * m:] == 0xA5).all())
    assert bool((what[n * m:] == -7.0).all())
    expect = (codes[: n * m].view(n, k, beta).double() - zero[:, :, None]) * scale[:, :, None]
    assert torch.equal(what[: n * m].view(n, k, beta), expect)


@pytest.mark.parametrize("n,m,beta,bits,huge", [(3, 256, 64, 5, 1.0), (2, 512, 128, 4, 1.0), (5, 320, 32, 3, 1.0), (2, 640, 160, 8, 1.0),
                                                (3, 256, 64, 5, 2.0 ** 36), (3, 256, 64, 5, 2.0 ** 60)])
def test_the_difference_of_the_products_keeps_its_digits(slim, n, m, beta, bits, huge):
    """Weights of one sign, a thousand times their distance from W_hat and all of W_hat - W exact in fp64: the loss is then
    W_hat G - W G to its last digits, and the digits that the two products share must not cost it any; nor must a row whose
    weights are much larger (and lie on their quantiser's values)."""
    rng = np.random.default_rng(m)
    Q = 2 ** bits - 1
    W = 2.0 + rng.integers(0, 4 * Q + 1, (n, m)) * 2.0 ** -13
    W.reshape(n, m // beta, beta)[:, :, 0] = 2.0                             # delta = 4 * 2^-13, the zero point -2 / delta
    W.reshape(n, m // beta, beta)[:, :, 1] = 2.0 + 4 * Q * 2.0 ** -13
    if huge > 1.0:
        W[0] = (2.0 + np.rint((W[0] - 2.0) * 2.0 ** 11) * 2.0 ** -11) * huge
    X = rng.standard_normal((m, 2 * m)) * np.exp(rng.standard_normal((m, 1)))
    G = torch.from_numpy(X @ X.T).to(torch.float32)
    Wd = torch.from_numpy(W).to(torch.float32)
    widths = torch.full((m // beta,), bits, dtype=torch.uint8, device="cuda")
    # (sigmoid(60) = 1: the whole range, the loss before any step)
    out = slim.lwc_quantize(Wd.cuda(), G.cuda(), 2 * m, widths, beta, steps=0, init=60.0, want_what=torch.float64)
    D = out["What"].cpu().numpy() - W
    assert 0.0 < np.abs(D).max() <= 2.0 ** -12 and (huge == 1.0 or not D[0].any()) and np.array_equal(D * 2.0 ** 13, np.rint(D * 2.0 ** 13))
    L = np.longdouble
    DG = np.stack([(D[i].astype(L)[:, None] * G.numpy().astype(L)).sum(axis=0) for i in range(n)])
    exact, terms = (D.astype(L) * DG).sum(), float((np.abs(D).astype(L) * np.abs(DG)).sum())
    # one rounding per product and the additions of the n m terms in the kernels' order (at most 64 in a row)
    got = L(out["loss_curve"][0]) * n * 2 * m
    assert abs(float(got - exact)) <= 64 * 2.0 ** -53 * terms, float(got - exact) / terms


def test_what_the_sums_round_away_is_kept_over_many_chunks(slim):
    """Two thousand channels whose entries of G lie far below their column's largest, weights of one sign and on their quantiser's
    values but for one channel: the loss is that channel's squared distance times its diagonal entry, and the two products share
    everything else, also the sums over all chunks of the lowest digits."""
    n, m, beta, bits = 16, 4096, 128, 5
    rng = np.random.default_rng(m)
    Q, far, big = 2 ** bits - 1, 5, m // 2
    step, lowest = 3001, 2796                                                # delta = 3001 * 2^-22, the zero point -2796
    W = step * (lowest + rng.integers(0, Q + 1, (n, m)))
    W.reshape(n, m // beta, beta)[:, :, 0] = step * lowest
    W.reshape(n, m // beta, beta)[:, :, 1] = step * (lowest + Q)
    W[:, far] = step * (lowest + rng.integers(0, Q, n)) + step // 4
    # the small entries: 24 bits from bit 0 .. 7 of a column's unit 2^-53 on
    G = rng.integers(2 ** 23, 2 ** 24, (m, m)) * 2.0 ** rng.integers(-53, -45, (m, m))
    G[big:, :] = 1.0                                                         # the largest of their columns, 2^53 units ...
    G[:, big:] = 1.0
    G[-1, :-1] = G[:-1, -1] = 2.0 ** -60                                     # ... because some entry has a digit below 2^-53
    G = torch.from_numpy(np.triu(G) + np.triu(G, 1).T).to(torch.float32)
    widths = torch.full((m // beta,), bits, dtype=torch.uint8, device="cuda")
    # (sigmoid(60) = 1: the whole range, the loss before any step)
    out = slim.lwc_quantize(torch.from_numpy(W * 2.0 ** -22).to(torch.float32).cuda(), G.cuda(), 2 * m, widths, beta, steps=0,
                            init=60.0, want_what=torch.float64)
    D = out["What"].cpu().numpy() - W * 2.0 ** -22
    assert (D[:, far] == -(step // 4) * 2.0 ** -22).all() and not np.delete(D, far, axis=1).any()
    exact = float((D[:, far] ** 2).sum()) * float(G[far, far])
    # In units (of 2^-53): y starts from 1.5 * 2^80 and rounds by 2^27 at most, at each of the additions of 64 chunks, four pairs
    # of digits of G and three digits of W, and fewer for the codes.  lo gathers these remainders, and rounds by 2^-53 of what it
    # holds.  Remainders and roundings are uniform and independent: eight standard deviations.
    adds = 2 * 64 * 4 * 3
    lo = 2.0 ** 27 / 3 ** 0.5 * adds ** 0.5
    sigma = adds ** 0.5 * lo * 2.0 ** -53 / 3 ** 0.5 * 2.0 ** -53
    got = out["loss_curve"][0] * n * 2 * m
    bound = 8 * sigma * float((D[:, far] ** 2).sum()) ** 0.5 + 64 * 2.0 ** -53 * exact
    assert abs(got - exact) <= bound, (got - exact, bound, exact)


@pytest.mark.parametrize("m,beta", [(64, 32), (60, 6)])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_weights_that_are_not_finite(slim, m, beta, value):
    """Nothing can be learnt in the row of such a weight: the loss is not a number and the row's quantisers are those of a
    group without a range (scale 1, zero 0), in both forms of the product; the other rows are as without it."""
    g = torch.Generator().manual_seed(m)
    W = (torch.randn((5, m), generator=g) * 0.05).to(torch.float16)
    X = torch.randn((m, 2 * m), generator=g, dtype=torch.float64)
    G, bits = (X @ X.t()).to(torch.float32).cuda(), torch.full((m // beta,), 2, dtype=torch.uint8, device="cuda")
    good = slim.lwc_quantize(W.cuda(), G, 2 * m, bits, beta, steps=3)
    W[3, 7] = value
    out = slim.lwc_quantize(W.cuda(), G, 2 * m, bits, beta, steps=3)
    assert np.isnan(out["loss_curve"]).all()
    assert bool((out["scale"][3] == 1.0).all()) and bool((out["zero"][3] == 0.0).all())
    rest = [0, 1, 2, 4]
    assert torch.equal(out["codes"][rest], good["codes"][rest]) and torch.equal(out["scale"][rest], good["scale"][rest])
