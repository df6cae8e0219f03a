"""The rank-512 products of the inverse and the sweep from residues on the int8 matrix cores, against the same calls with the
fp64 products (a caller's workspace without room for the residues takes those) and against the identity they solve, and the two
kernels by themselves against exact sums."""
import ctypes
import math
from fractions import Fraction

import pytest
import torch

pytestmark = pytest.mark.gpu

# the fp64 products' sums of K = 512 terms are off by up to about sqrt(K) roundings; the residues' by less
EPS = 2.0 ** -53


@pytest.fixture(scope="module")
def contexts():
    from paper_2405_14917_amd import binding
    made = []

    def make(nbytes=0):
        made.append(binding.Slim("cuda:0", nbytes))
        return made[-1]
    yield binding, make
    for c in made:
        c.close()


def gram(m, t, gen):
    """Correlated channels of very different scale, some of them outliers."""
    scale = torch.exp(0.5 * torch.randn(m, 1, generator=gen, device="cuda"))
    scale[100:108] *= 50.0
    X = scale * (torch.randn(m, t, generator=gen, device="cuda") + 0.3 * torch.randn(1, t, generator=gen, device="cuda"))
    X = X.half().float()
    return X @ X.t()


def base_inverse(m):
    up = lambda b: (b + 255) // 256 * 256
    return 2 * up(8 * m * m) + up(8 * -(-m // 256) * m) + 256


def base_sweep(n, m):
    up = lambda b: (b + 255) // 256 * 256
    return up(8 * n * m) + up(8 * n * 512) + up(16 * n) + up(8 * n)


def steps(s):
    """The launches of a profiled context, "<step>@<kernel>"."""
    return {name.split("#")[0] for name in s.profile_collect()}


# one far update that takes the path, of a whole group and of a last group of 386 channels; last groups of 504 and 510, and one whose
# 322 channels are left to the fp64 form; widths that fill no tile of 128 and no block of 64; the terms of one and of several groups
@pytest.mark.parametrize("m", [2946, 3072, 4096, 4480, 4600, 4930, 6400, 9214])
def test_inverse_from_residues(contexts, m):
    binding, make = contexts
    need = binding.workspace_query(0, m, 0)
    assert need > base_inverse(m)
    gen = torch.Generator(device="cuda").manual_seed(m)
    t = m + 512
    G = gram(m, t, gen)
    full, less = make(need), make(base_inverse(m))
    full.profile_enable()
    less.profile_enable()
    U, d = full.hessian_inverse(G, t, 0.01)
    U0, d0 = less.hessian_inverse(G, t, 0.01)
    assert "inv_syrk_dgemm@rgemm_kernel" in steps(full)
    assert ("inv_trtri_terms_dgemm@rgemm_kernel" in steps(full)) == (m >= 4096)
    assert not any("rgemm_kernel" in s for s in steps(less))
    H = (2.0 / t) * G.double()
    H += 0.01 * H.diagonal().mean() * torch.eye(m, dtype=torch.float64, device="cuda")
    off = lambda V: ((V @ H).mul_(1.0) @ V.t() - torch.eye(m, dtype=torch.float64, device="cuda")).norm().item()
    # U (H + lambda I) U^T = I: the residual of either form is condition times roundings; with the residues it is no larger
    # (1.2: the products of the check itself round too)
    a, b = off(U), off(U0)
    assert a <= 1.2 * b, (a, b)
    cond = (U.norm() ** 2 * H.norm()).item()
    assert ((U - U0).norm() / U0.norm()).item() <= 64 * EPS * cond
    assert ((d - d0).abs() / d0).max().item() <= 64 * EPS * cond
    assert not torch.tril(U, -1).any()


@pytest.mark.parametrize("n,m,beta", [(1024, 8704, 128), (2500, 4096, 64), (4099, 3072, 32), (9001, 2048, 512)])
def test_sweep_from_residues(contexts, n, m, beta):
    binding, make = contexts
    need = binding.workspace_query(n, m, beta)
    gen = torch.Generator(device="cuda").manual_seed(n)
    t = 2 * m
    G = gram(m, t, gen)
    W = (0.02 * torch.randn(n, m, generator=gen, device="cuda")).half()
    W[:, 40:44] *= 8
    bits = torch.randint(1, 4, (m // beta,), generator=gen, device="cuda", dtype=torch.uint8)
    full, less = make(need), make(base_sweep(n, m))
    U, _ = make().hessian_inverse(G, t, 0.01)
    full.profile_enable()
    less.profile_enable()
    a, b = full.gptq_quantize(W, U, bits, beta), less.gptq_quantize(W, U, bits, beta)
    assert "gptq_trailing_dgemm@rgemm_kernel" in steps(full) and not any("rgemm_kernel" in s for s in steps(less))
    # A weight within 1e-12 of a rounding tie may go the other way, and the rest of its row with it: of these layers' 9 to 18
    # million normal weights none is expected to be; one row is allowed.  (Outliers that alone decide a group's losses meet exact
    # ties of the calibration's candidates, 7 tau_18 = 6 tau_96 among them.)  Where the codes agree, the continuous values do.
    rows = (a["codes"] != b["codes"]).any(dim=1)
    assert int(rows.sum()) <= 1
    for key in ("scale", "zero"):
        x, y = a[key][~rows], b[key][~rows]
        assert ((x - y).abs() <= 1e-11 * (y.abs() + y.abs().mean())).all(), key


def test_rows_that_are_not_finite_stay_alone(contexts):
    """With the 3-sigma rule by row, a row of W with an infinity or a NaN changes no other row, through the residues too."""
    binding, make = contexts
    n, m, beta = 2500, 4096, 128
    gen = torch.Generator(device="cuda").manual_seed(5)
    G = gram(m, 2 * m, gen)
    s = make()
    U, _ = s.hessian_inverse(G, 2 * m, 0.01)
    W = (0.02 * torch.randn(n, m, generator=gen, device="cuda")).half()
    bits = torch.full((m // beta,), 2, dtype=torch.uint8, device="cuda")
    params = binding.SlimParams()
    params.mask_scope = 1
    s.profile_enable()
    a = s.gptq_quantize(W, U, bits, beta, params=params)
    W[37, 300] = float("inf")
    W[700, 1000] = float("nan")
    b = s.gptq_quantize(W, U, bits, beta, params=params)
    assert "gptq_trailing_dgemm@rgemm_kernel" in steps(s)
    keep = torch.ones(n, dtype=torch.bool, device="cuda")
    keep[37] = keep[700] = False
    for key in ("codes", "scale", "zero"):
        assert torch.equal(a[key][keep], b[key][keep]), key


@pytest.mark.parametrize("m,g0", [(6144, 3072), (6400, 2560)])
def test_columns_of_a_group_beside_a_large_channel(contexts, m, g0):
    """H = [[I + B B^T, B], [B^T, I]] over all integers, B one group's columns in the rows of the group above: U = [[I, -B], [0, I]],
    every step of it exact in fp64.  One channel of B is 2^10 times the others, which must not cost the columns before it digits."""
    binding, make = contexts
    s = make(binding.workspace_query(0, m, 0))
    B = torch.zeros((512, 512), dtype=torch.float64, device="cuda")
    B[:, :8] = torch.arange(512 * 8, device="cuda").reshape(512, 8) % 15 - 7
    B[:, 300] = 1024.0
    H = torch.eye(m, dtype=torch.float64, device="cuda")
    H[g0 - 512:g0, g0 - 512:g0] += B @ B.t()
    H[g0 - 512:g0, g0:g0 + 512] = B
    H[g0:g0 + 512, g0 - 512:g0] = B.t()
    G = H.float()
    assert torch.equal(G.double(), H)
    s.profile_enable()
    U, _ = s.hessian_inverse(G, 2, 0.0)
    assert "inv_trtri_terms_dgemm@rgemm_kernel" in steps(s)
    assert ((U[g0 - 512:g0, g0:g0 + 512] + B).abs() <= 4 * EPS * B.abs()).all()


class Operand(ctypes.Structure):
    _fields_ = [("planes", ctypes.c_void_p), ("scale", ctypes.c_void_p)]


class Product(ctypes.Structure):
    _fields_ = [("A", Operand), ("B", Operand), ("rowsA", ctypes.c_int), ("rowsB", ctypes.c_int), ("C", ctypes.c_void_p),
                ("ldc", ctypes.c_int64), ("M", ctypes.c_int), ("N", ctypes.c_int), ("alpha", ctypes.c_double), ("upper", ctypes.c_bool),
                ("beside", ctypes.c_bool)]


def product(s, A, B, C, M, N, alpha, upper=False, beside=False):
    """C[:M, :N] += alpha A B by the library's own two kernels; A rows x K, B K x cols (views of wider matrices)."""
    residues = s.lib._Z16slim_rg_residuesP8slim_ctxPKcRK15slim_rg_operandPKdliib
    rgemm = s.lib._Z10slim_rgemmP8slim_ctxPKcRK12slim_rg_desc
    keep, ops = [], []
    for X, rows, columns in ((A, A.shape[0], False), (B, B.shape[1], True)):
        padded = -(-rows // 128) * 128
        planes = torch.full((padded * 512 * 14,), 77, dtype=torch.uint8, device="cuda")
        scale = torch.full((padded,), 3.0, dtype=torch.float64, device="cuda")
        keep += [planes, scale]
        ops.append(Operand(planes.data_ptr(), scale.data_ptr()))
        assert residues(s.ctx, b"inv_panel_residues", ctypes.byref(ops[-1]), ctypes.c_void_p(X.data_ptr()), ctypes.c_int64(X.stride(0)),
                        ctypes.c_int(rows), ctypes.c_int(A.shape[1]), ctypes.c_bool(columns)) == 0
    d = Product(ops[0], ops[1], A.shape[0], B.shape[1], C.data_ptr(), C.stride(0), M, N, alpha, upper, beside)
    assert rgemm(s.ctx, b"gptq_trailing_dgemm", ctypes.byref(d)) == 0
    torch.cuda.synchronize()


# a tile and less, one row or column more than tiles, ranks from the least to the most with every kind of remainder of 16 and 128, more
# than one tile per workgroup, results narrower than the operands
@pytest.mark.parametrize("M,N,K,extra,beside", [
    (1, 2, 2, 0, False), (128, 128, 512, 0, False), (129, 257, 386, 0, True), (40, 300, 510, 0, False), (700, 130, 130, 0, False),
    (257, 64, 16, 200, False), (2304, 2176, 100, 0, False), (2050, 2300, 504, 130, True)])
def test_product_against_exact_sums(contexts, M, N, K, extra, beside):
    binding, make = contexts
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    rnd = lambda *shape: torch.randn(*shape, generator=gen, device="cuda", dtype=torch.float64)
    # rows and columns of very different size, channels of different size in each; rows and columns of zeros, of tiny and of whole
    # numbers, and of equal ones (the largest sums of residues)
    A = rnd(M + extra, K + 2)[:, :K] * 2.0 ** (40.0 * rnd(M + extra, 1)) * 2.0 ** (4.0 * rnd(1, K))
    B = rnd(K, N + extra) * 2.0 ** (40.0 * rnd(1, N + extra)) * 2.0 ** (4.0 * rnd(K, 1))
    for r in range(5, M, 97):
        A[r] = 0.0
    if M > 30:
        A[11] = torch.randint(-5, 6, (K,), generator=gen, device="cuda").double() * 2.0 ** -500
        A[12] = 1.0
        A[13] = -1.0
    if N > 30:
        B[:, 7] = 0.0
        B[:, 8] = 1.0
        B[:, 9] = torch.arange(K, device="cuda").double()
    A = torch.nn.functional.pad(A, (0, K % 4 + 2))[:, :K]                        # an even leading dimension, 16-byte rows
    old = rnd(M + 3, N + 5)
    C = old.clone()
    product(make(), A, B, C, M, N, -1.0, beside=beside)
    assert torch.equal(C[M:], old[M:]) and torch.equal(C[:, N:], old[:, N:])
    pick = lambda size, some: sorted({x for x in some if x < size} | {int(x) for x in torch.randint(0, size, (12,), generator=gen, device="cuda")})
    rows, cols = pick(M, (0, 5, 11, 12, 13, M - 1)), pick(N, (0, 7, 8, 9, N - 1))
    a, b = A[rows].tolist(), B[:, cols].t().tolist()
    got, was = C[rows][:, cols].tolist(), old[rows][:, cols].tolist()
    square = []
    for i, x in enumerate(a):
        fx = [Fraction(v) for v in x]
        nx = math.sqrt(sum(v * v for v in fx)) if any(x) else 0.0
        for j, y in enumerate(b):
            ny = math.sqrt(sum(Fraction(v) ** 2 for v in y))
            err = abs(float(Fraction(was[i][j]) - sum(p * Fraction(q) for p, q in zip(fx, y)) - Fraction(got[i][j])))
            # an operand is rounded to half a unit of norm / 2^54.5 per channel, after a rounding of its own by 2^-53; the sum's fraction,
            # the scales and the last fma round by 2^-53 each, the fma relative to the result
            bound = nx * ny * ((math.sqrt(K) + 6.0) * 2.0 ** -54.5 + 4 * EPS) + EPS * abs(got[i][j])
            assert err <= bound, (rows[i], cols[j], err, bound)
            if nx * ny > 1e3 * abs(was[i][j]):
                square.append((err / (nx * ny)) ** 2)
    # over many elements: every rounding (of an element, of its scaled value, and the four of the sum) is off by 0.29 of its step
    assert len(square) < 50 or math.sqrt(sum(square) / len(square)) <= EPS


def test_product_of_the_upper_triangle(contexts):
    """Only tiles that reach the diagonal, on which every element is right; those below it stay as they are."""
    binding, make = contexts
    n, K = 1100, 512
    gen = torch.Generator(device="cuda").manual_seed(1)
    A = torch.randint(-9, 10, (n, K), generator=gen, device="cuda").double()
    C = torch.randint(-99, 100, (n, n), generator=gen, device="cuda").double()
    want = C + 2.0 * (A @ A.t())
    old = C.clone()
    product(make(), A, A.t().contiguous(), C, n, n, 2.0, upper=True, beside=True)
    tile = torch.arange(n, device="cuda") // 128
    upper = tile[:, None] <= tile[None, :]
    assert ((C - want)[upper].abs() <= 1e-9).all()
    assert torch.equal(C[~upper], old[~upper])
