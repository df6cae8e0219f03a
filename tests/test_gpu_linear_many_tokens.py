"""The linear layer on the stored form for more than 64 tokens (its own kernel) against the float64 oracle: token and row
counts around the tiles (128 or 64 tokens x 128 rows), one and several group ranges, both slab widths (group sizes that 64
divides and that it does not), every code width, both activation types, zero points outside the operand's form, groups
that are skipped, and activations the kernel cannot fetch (the sliced form takes those)."""
import numpy as np
import pytest
import torch

from oracle import slim_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def slim():
    from paper_2405_14917_amd import binding
    s = binding.Slim("cuda:0")
    yield s
    s.close()


def stored(slim, rng, n, m, beta, base, odd_zeros):
    k = m // beta
    bits = (base + np.arange(k) % (4 if base == 2 else 3)).astype(np.uint8)
    codes = np.concatenate([rng.integers(0, 2 ** int(b), (n, beta)) for b in bits], axis=1).astype(np.uint8)
    scale = rng.uniform(0.005, 0.02, (n, k))
    zero = np.stack([rng.integers(0, 2 ** int(b), n).astype(np.float64) for b in bits], axis=1)
    zero[:, bits == 1] = 0.5
    if odd_zeros:
        zero[: n // 3, 0] = -700.0                    # beyond the fp16 operand's form
        zero[n // 3: n // 2, -1] = 96.0               # beyond the bf16 operand's form
        zero[n // 2, k // 2] = 3.3                    # not a multiple of 1/2
    packed, gbits, row_off, _ = slim.pack(torch.from_numpy(codes).cuda(), torch.from_numpy(bits).cuda(), beta, bit_base=base)
    What = np.repeat(scale, beta, axis=1) * (codes - np.repeat(zero, beta, axis=1))
    return packed, gbits, row_off, torch.from_numpy(scale).cuda(), torch.from_numpy(zero).cuda(), What


@pytest.mark.parametrize("t,n,m,beta,base,dtype,odd", [
    (65, 77, 64, 64, 1, torch.float16, False), (128, 128, 512, 128, 1, torch.float16, True),
    (129, 300, 1024, 128, 2, torch.bfloat16, True), (200, 129, 320, 32, 1, torch.float16, True),
    (257, 260, 288, 96, 2, torch.bfloat16, False), (70, 1000, 2304, 128, 1, torch.bfloat16, False),
    (640, 9000, 256, 256, 1, torch.float16, True), (300, 130, 1024, 512, 2, torch.float16, False)])
def test_many_tokens(slim, t, n, m, beta, base, dtype, odd):
    rng = np.random.default_rng(t + n)
    packed, gbits, row_off, scale, zero, What = stored(slim, rng, n, m, beta, base, odd)
    X = torch.from_numpy(rng.standard_normal((t, m))).to(dtype).cuda()
    Yw = torch.full((t, n + 5), -1.0, dtype=torch.float32, device="cuda")
    Y = slim.dequant_matmul(packed, gbits, row_off, scale, zero, beta, X, Y=Yw[:, :n], bit_base=base)
    Xn = X.double().cpu().numpy()
    # the bound of the linear layer: fp32 sums of exact products, 1e-5 of the sum of magnitudes (m <= 2304 terms)
    assert np.all(np.abs(Y.cpu().numpy() - Xn @ What.T) <= 1e-5 * (np.abs(Xn) @ np.abs(What).T) + 1e-30)
    assert bool((Yw[:, n:] == -1.0).all())
    assert torch.equal(Y, slim.dequant_matmul(packed, gbits, row_off, scale, zero, beta, X, bit_base=base))
    # the entry point that allocates nothing: same kernel, same ranges, same bytes
    Yn = torch.empty((t, n), dtype=torch.float32, device="cuda")
    slim.dequant_matmul(packed, gbits, row_off, scale, zero, beta, X, Y=Yn, bit_base=base, noalloc=True)
    assert torch.equal(Y, Yn)


def test_skipped_groups_and_unaligned_activations(slim):
    rng = np.random.default_rng(5)
    n, m, beta, t = 200, 512, 64, 90
    packed, gbits, row_off, scale, zero, What = stored(slim, rng, n, m, beta, 1, False)
    X = torch.from_numpy(rng.standard_normal((t, m)).astype(np.float16)).cuda()
    assert not bool(slim.dequant_matmul(packed, gbits, row_off, scale, zero, beta, X, bit_base=2).any())
    Xo = torch.zeros((t, m + 12), dtype=torch.float16, device="cuda")       # a leading dimension that is no multiple of 8
    Xo[:, :m] = X
    Y = slim.dequant_matmul(packed, gbits, row_off, scale, zero, beta, Xo[:, :m])
    Xn = X.double().cpu().numpy()
    assert np.all(np.abs(Y.cpu().numpy() - Xn @ What.T) <= 1e-5 * (np.abs(Xn) @ np.abs(What).T))


def test_a_workspace_for_sixteen_tokens_serves_more():
    from paper_2405_14917_amd import binding
    rng = np.random.default_rng(11)
    n, m, beta = 512, 512, 32
    small = binding.Slim("cuda:0", workspace_bytes=binding.workspace_query(n, m, beta, t_x=16))
    packed, gbits, row_off, scale, zero, What = stored(small, rng, n, m, beta, 1, False)
    zp, bad = small.pack_zeros(zero, 4)
    assert bad == 0
    for t in (16, 70, 300, 700, 2500):
        X = torch.from_numpy(rng.standard_normal((t, m))).half().cuda()
        Y = small.dequant_matmul(packed, gbits, row_off, scale, zero, beta, X)
        Xn = X.double().cpu().numpy()
        assert np.all(np.abs(Y.cpu().numpy() - Xn @ What.T) <= 1e-5 * (np.abs(Xn) @ np.abs(What).T))
        assert torch.equal(Y, small.dequant_matmul_zp(packed, gbits, row_off, scale, zp, 4, beta, X))
    small.close()


@pytest.mark.parametrize("t,aligned", [(5, True), (90, True), (300, True), (5, False)])
def test_a_skipped_group_adds_nothing_whatever_its_activations(slim, t, aligned):
    """A group whose width disagrees with its rows is skipped by every kernel, also where its activations are infinite."""
    rng = np.random.default_rng(t)
    n, m, beta = 150, 512, 64
    packed, gbits, row_off, scale, zero, What = stored(slim, rng, n, m, beta, 1, False)
    gbits = gbits.clone()
    gbits[0] ^= 1 << (2 * 2)                          # group 2: another width than its rows hold
    What[:, 2 * beta: 3 * beta] = 0.0
    X = torch.zeros((t, m + (0 if aligned else 4)), dtype=torch.float16, device="cuda")[:, :m]
    X.copy_(torch.from_numpy(rng.standard_normal((t, m))).half())
    Xn = X.double().cpu().numpy()
    X[:, 2 * beta: 3 * beta] = float("inf")
    Y = slim.dequant_matmul(packed, gbits, row_off, scale, zero, beta, X)
    assert np.all(np.abs(Y.cpu().numpy() - Xn @ What.T) <= 1e-5 * (np.abs(Xn) @ np.abs(What).T) + 1e-30)


def test_more_groups_than_the_kernel_holds(slim):
    """Twice the groups of one launch's limit, and so many tokens that nothing is split: taken 64 tokens at a time."""
    n, beta, k, t = 544, 32, 36864, 3860
    m = beta * k
    gen = torch.Generator(device="cuda").manual_seed(1)
    codes = torch.randint(0, 4, (n, m), generator=gen, device="cuda", dtype=torch.uint8)
    packed, gbits, row_off, _ = slim.pack(codes, torch.full((k,), 2, dtype=torch.uint8, device="cuda"), beta)
    del codes
    scale = torch.full((n, k), 2.0 ** -10, dtype=torch.float64, device="cuda")
    zero = torch.full((n, k), 1.0, dtype=torch.float64, device="cuda")
    X = torch.zeros((t, m), dtype=torch.float16, device="cuda")
    X[:, ::64] = torch.randint(-1, 2, (t, m // 64), generator=gen, device="cuda").half()
    Y = slim.dequant_matmul(packed, gbits, row_off, scale, zero, beta, X)
    for t0 in (0, 1984, t - 40):                      # the same as in calls of few tokens, exactly (every sum is exact)
        part = X[t0: t0 + 40]
        assert torch.equal(Y[t0: t0 + 40], slim.dequant_matmul(packed, gbits, row_off, scale, zero, beta, part))
    assert float(Y.abs().max()) > 0.0


def plan(n, m, beta, t):
    """The kernel's rule: tokens per tile, and groups per workgroup."""
    cus, k, cdiv = torch.cuda.get_device_properties(0).multi_processor_count, m // beta, lambda a, b: (a + b - 1) // b
    tile = 64 if cdiv(n, 128) * cdiv(t, 128) < 2 * cus else 128
    want = min(k, max(1, 2 * cus // (cdiv(n, 128) * cdiv(t, tile))))
    return tile, cdiv(k, max(1, min(want, 2 ** 22 // (t * n))))


@pytest.mark.parametrize("t,n,m,beta,base,dtype,odd,tile,gper", [
    (2049, 4000, 2304, 128, 1, torch.float16, True, 128, 18),     # a fold at sixteen groups and two behind it, ragged tiles
    (2049, 4000, 2304, 128, 2, torch.bfloat16, True, 128, 18),
    (1153, 7200, 1088, 32, 1, torch.bfloat16, False, 128, 34),    # slabs of 32 channels, one a group
    (1200, 6700, 1536, 96, 2, torch.float16, True, 128, 16),      # three of them a group, exactly one fold
    (1000, 4100, 2176, 128, 1, torch.bfloat16, True, 64, 17),     # tiles of 64 tokens, several groups
    (700, 5900, 1024, 64, 2, torch.float16, False, 64, 16),
    (200, 1000, 2304, 128, 1, torch.float16, True, 64, 2)])       # several ranges of several groups
def test_groups_of_one_workgroup(slim, t, n, m, beta, base, dtype, odd, tile, gper):
    """The loop over a workgroup's groups of changing width, with either tile, against the product in fp64."""
    assert plan(n, m, beta, t) == (tile, gper)
    rng = np.random.default_rng(t + n)
    packed, gbits, row_off, scale, zero, What = stored(slim, rng, n, m, beta, base, odd)
    X = torch.from_numpy(rng.standard_normal((t, m))).to(dtype).cuda()
    Y = slim.dequant_matmul(packed, gbits, row_off, scale, zero, beta, X, bit_base=base)
    Xd, Wd = X.double(), torch.from_numpy(What).cuda()
    bound = 1e-5 * (Xd.abs() @ Wd.abs().t().contiguous()) + 1e-30
    assert bool(((Y.double() - Xd @ Wd.t().contiguous()).abs() <= bound).all())
