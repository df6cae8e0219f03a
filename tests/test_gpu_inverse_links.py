"""The factorisation's chain where it can go wrong: widths around the tiles of a diagonal block (16), the blocks (64) and the
groups of blocks (512), and pivots that fail in each tile."""
import numpy as np
import pytest
import torch

from paper_2405_14917_amd import binding

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def slim():
    s = binding.Slim("cuda:0")
    yield s
    s.close()


@pytest.mark.parametrize("m", [2, 16, 18, 34, 62, 64, 66, 126, 130, 446, 510, 512, 514, 574, 578, 642, 1022, 1026, 1090, 1538, 1600])
def test_inverse_at_the_edges_of_tiles_blocks_and_groups(slim, m):
    rng = np.random.default_rng(m)
    X = rng.standard_normal((m, 3 * m)) * np.exp(0.5 * rng.standard_normal((m, 1)))
    G = (X @ X.T).astype(np.float32)
    U, d = slim.hessian_inverse(torch.from_numpy(G).cuda(), 3 * m, 0.01)
    U, d = U.cpu().numpy(), d.cpu().numpy()
    H = np.triu(G).astype(np.float64) * (2.0 / (3 * m))
    H = H + np.triu(H, 1).T
    H += 0.01 * np.mean(np.diag(H)) * np.eye(m)
    assert np.array_equal(np.tril(U, -1), np.zeros((m, m))) and (np.diag(U) > 0).all()
    # U^-1 = R has R R^T = H up to the rounding of a Cholesky factorisation, m eps |H|, and the triangular inverse adds
    # m eps |U| |R|: with cond(H) = k the residual of U H U^T = I stays below m eps k (measured: below 0.01 of it)
    k = np.linalg.cond(H)
    res = np.linalg.norm(U @ H @ U.T - np.eye(m), 2)
    assert res <= m * 2.0 ** -53 * k, (res, k)
    assert np.allclose(d, (U * U).sum(axis=0), rtol=1e-13)


@pytest.mark.parametrize("m,fails", [(64, (0,)), (64, (15,)), (64, (16,)), (64, (31, 5)), (64, (47,)), (64, (48, 63)), (130, (129,)),
                                     (130, (63, 64)), (200, (70, 3)), (576, (512,)), (576, (511, 40))])
def test_the_first_pivot_that_fails_is_named(slim, m, fails):
    """Pivots go from the last column to the first: the highest failing column of the first failing block is reported."""
    h = np.full(m, 4.0)
    for j in fails:
        h[j] = -1000.0
    G = torch.from_numpy(np.diag(h).astype(np.float32)).cuda()
    with pytest.raises(binding.SlimError) as err:
        slim.hessian_inverse(G, 2, 0.0)
    assert err.value.status == binding.ERR_NOT_PD and "pivot at column %d)" % (max(fails) + 1) in str(err.value)
    # the context is as good as before
    U, _ = slim.hessian_inverse(torch.eye(m, device="cuda") * 4.0, 2, 0.0)
    assert torch.equal(U, torch.eye(m, dtype=torch.float64, device="cuda") * 0.5)
