"""The fill at the sizes where its launches change: near blocks in tiles of 16, 32 and 64 points (leaves of
1 to 33).

Near field of the exponential kernel as in the other fill tests (entries to 2e-14, symmetric bit for
bit) and of the Helmholtz kernel (relative to the largest entry 1e-14).
"""
import numpy as np
import pytest

from paper_2509_17257_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _h2x():
    import paper_2509_17257_amd as h2x
    return h2x


@pytest.mark.parametrize("leaf,p", [(1, 1), (7, 2), (16, 2), (17, 2), (32, 3), (33, 3)])
def test_near_tiles(leaf, p):
    h2x = _h2x()
    n = 500
    P = W.sphere_points(n, 440 + leaf)
    D = np.sqrt(((P[:, None] - P[None]) ** 2).sum(2))
    eye = torch.eye(n, dtype=torch.float64, device="cuda")
    # (a tiny eta: only pairs of single points, whose interpolation is exact, are admissible)
    A = h2x.H2Matrix(P, ell=0.5, shift=1.5, eta=1e-9, leaf=leaf, p=p)
    assert A.plan.n_adm == 0 or leaf == 1
    K = h2x.h2_matmul(A, eye).cpu().numpy()
    assert np.array_equal(K, K.T)
    assert np.abs(K / (np.exp(-D / 0.5) + 1.5 * np.eye(n)) - 1).max() <= 2e-14
    A = h2x.H2Matrix(P, kernel="helmholtz", ell=3.0, shift=1.5, eta=1e-9, leaf=leaf, p=p)
    K = h2x.h2_matmul(A, eye.to(torch.complex128)).cpu().numpy()
    with np.errstate(divide="ignore", invalid="ignore"):
        ref = np.exp(3j * D) / (n * D)
    np.fill_diagonal(ref, 1.5)
    assert np.abs(K - ref).max() <= 1e-14 * np.abs(ref).max()
