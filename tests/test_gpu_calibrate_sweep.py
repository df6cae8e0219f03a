"""Calibration, sweep and window update in one launch (layers of up to 16 rows per compute unit) against the kernels that take larger
layers: with the unweighted loss no row depends on another, so the first rows of a layer that is too large for the one launch are,
byte for byte, those rows alone."""
import numpy as np
import pytest
import torch

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
