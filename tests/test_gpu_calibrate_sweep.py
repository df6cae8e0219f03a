"""Calibration, sweep and window update in one launch (layers of up to 16 rows per compute unit) against the kernels that take larger
layers: with the unweighted loss no row depends on another, so the first rows of a layer that is too large for the one launch are,
byte for byte, those rows alone."""
import numpy as np
import pytest
import torch

from oracle import slim_oracle as orc
from paper_2405_14917_amd import binding

pytestmark = pytest.mark.gpu
UNIFORM = 1


@pytest.fixture(scope="module")
def slim():
    s = binding.Slim("cuda:0")
    yield s
    s.close()


def layer(n, m, seed):
    rng = np.random.default_rng(seed)
    W = (0.02 * rng.standard_normal((n, m))).astype(np.float32)
    W[0] = 0.25                                            # a constant row, one of zeros, one with a single value
    if n > 2:
        W[1], W[2] = 0.0, 0.0
        W[2, 5] = -1.0
    A = rng.standard_normal((m, 2 * m))
    U = np.linalg.cholesky(A @ A.T / m + 0.1 * np.eye(m)).T
    return torch.from_numpy(W).cuda(), torch.from_numpy(np.ascontiguousarray(U)).cuda()


@pytest.mark.parametrize("beta,groups,ncand", [(32, 4, 1), (32, 20, 100), (32, 1, 113), (32, 16, 129), (64, 4, 1), (64, 10, 100), (64, 4, 129),
                                               (128, 4, 1), (128, 7, 100), (128, 2, 113), (128, 5, 129)])
def test_one_launch_equals_several(slim, beta, groups, ncand):
    """(windows of 512 columns: whole, several, a last one that is not full, a single block)"""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    m = groups * beta
    W, U = layer(16 * cus + 1, m, beta + ncand)
    bits = torch.tensor(([1, 2, 3, 5] * groups)[:groups], dtype=torch.uint8, device="cuda")
    tau = 0.9 + 0.2 * torch.arange(ncand, dtype=torch.float64, device="cuda") / ncand
    prm = binding.SlimParams(sqc_weight_mode=UNIFORM)
    whole = slim.gptq_quantize(W, U, bits, beta, params=prm, tau=tau, want_what=torch.float64)
    # the smallest, and the edges of 4, 8 and 16 rows per workgroup
    for n in (1, 3, 4 * cus - 1, 4 * cus, 4 * cus + 1, 8 * cus, 8 * cus + 5, 16 * cus):
        part = slim.gptq_quantize(W[:n], U, bits, beta, params=prm, tau=tau, want_what=torch.float64)
        for key in ("scale", "zero", "codes", "What"):
            assert torch.equal(part[key], whole[key][:n]), (n, key)


@pytest.mark.parametrize("n", [5, 1024, 1030, 4096])
@pytest.mark.parametrize("scope", [0, 1])
def test_first_group_equals_the_calibration_alone(slim, n, scope):
    """3-sigma rule over the block or the row: scales and zeros of the first group as slim_sqc_calibrate gives them (the block's
    sums run in another order there, 1e-15 of the threshold, which no weight here is that close to)."""
    beta = 64
    W, U = layer(n, 2 * beta, n)
    W[:, :3] *= 12.0
    prm = binding.SlimParams(mask_scope=scope)
    for b in (1, 2, 4):
        bits = torch.full((2,), b, dtype=torch.uint8, device="cuda")
        out = slim.gptq_quantize(W, U, bits, beta, params=prm)
        scale, zero, _ = slim.sqc_calibrate(W[:, :beta].double().contiguous(), b, params=prm)
        assert torch.equal(out["scale"][:, 0], scale.reshape(-1)) and torch.equal(out["zero"][:, 0], zero.reshape(-1))


@pytest.mark.parametrize("rows,extra,groups", [(0, 7, 4), (4, 3, 4), (8, 5, 4), (8, 9, 18)])
def test_the_sums_of_the_next_block(slim, rows, extra, groups):
    """3-sigma rule over the block, every group against the oracle: the sums go from launch to launch, about each workgroup's own
    shift and weighted by its rows, of which the last one has fewer (4, 8 and 16 rows per workgroup; the last case goes over a
    window of 512).  The last rows lie far from the others, so that one of their number more or less moves the threshold."""
    n, beta = rows * torch.cuda.get_device_properties(0).multi_processor_count + extra, 32
    per = 4 if rows == 0 else 2 * rows
    m = groups * beta
    rng = np.random.default_rng(n)
    W = 0.01 + 0.02 * rng.standard_t(4, (n, m))
    W[n - n % per:] += 0.3
    W = W.astype(np.float32).astype(np.float64)
    A = rng.standard_normal((m, 2 * m))
    U = np.ascontiguousarray(np.linalg.cholesky(A @ A.T / m + 0.1 * np.eye(m)).T)
    bits, tau = np.array(([2, 3, 1, 2] * groups)[:groups], dtype=np.uint8), orc.tau_grid()
    ref = orc.gptq_quantize(W, U, bits, beta, tau)
    # a count of whole workgroups would be seen: group 1 under the threshold that it gives
    Wc = W[:, beta:2 * beta] - ref["E"][:, :beta] @ U[:beta, beta:2 * beta]
    full, first = per * -(-n // per) * beta, Wc[n - n % per:, 0].mean()
    s1, s2 = Wc.sum() + (full - Wc.size) * first, (Wc ** 2).sum() + (full - Wc.size) * first ** 2
    mu, sigma = s1 / Wc.size, np.sqrt(max(s2 / Wc.size - (s1 / Wc.size) ** 2, 0.0))
    mask = np.abs(Wc - mu) > 3.0 * sigma
    omega = np.stack([orc.sqc_weights(Wc[i], mask[i], orc.WEIGHT_MASK_MEAN) for i in range(n)])
    assert n < 100 or (orc._sqc_rows_fast(Wc, int(bits[1]), tau, omega, orc.Q1_SIGN)[2] != ref["cand_idx"][:, 1]).sum() > 20
    out = slim.gptq_quantize(torch.from_numpy(W).to(torch.float32).cuda(), torch.from_numpy(U).cuda(), torch.from_numpy(bits).cuda(), beta)
    # rows whose weights and losses leave the rounding and the choice to no last digit
    ok = (ref["round_margin"].min(axis=1) > 1e-8) & (ref["sqc_margin"].min(axis=1) > 1e-9)
    assert ok.mean() > 0.9
    assert np.array_equal(out["codes"].cpu().numpy()[ok], ref["codes"][ok])
    assert np.array_equal(out["zero"].cpu().numpy()[ok], ref["zero"][ok])
    assert np.allclose(out["scale"].cpu().numpy()[ok], ref["scale"][ok], rtol=1e-9, atol=0.0)
