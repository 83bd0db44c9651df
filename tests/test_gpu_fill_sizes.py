"""The fill at the sizes where its launches change: near blocks in tiles of 16, 32 and 64 points (leaves of
1 to 33), and FP32 / BF16 coupling matrices of orders 5 to 8, pairs of blocks at once up to 6.

* Near field of the exponential kernel as in the other fill tests (entries to 2e-14, symmetric bit for
  bit) and of the Helmholtz kernel (relative to the largest entry 1e-14).
* FP32 products against the oracle's emulation (1e-5, the bar of the FP32 products), and for both
  storages a refill gives the bits of an operator created with that length scale.
"""
import numpy as np
import pytest

import oracle
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


@pytest.mark.parametrize("p,leaf,n", [(5, 64, 1500), (6, 70, 1200), (7, 70, 1100), (8, 70, 1100)])
@pytest.mark.parametrize("prec", ["f32", "bf16"])
def test_lowp_orders(p, leaf, n, prec):
    h2x = _h2x()
    P = W.line_points(n, 450 + p) + 0.05 * W.cube_points(n, 451 + p)
    prm = dict(shift=1.0, eta=1.0, leaf=leaf, p=p)
    X = W.rhs(n, 5, 452)
    Xd = torch.from_numpy(X).cuda()
    A = h2x.H2Matrix(P, ell=0.3, storage=prec, **prm)
    assert A.plan.n_adm > 4
    Y = h2x.h2_matmul(A, Xd)
    if prec == "f32":
        ref = oracle.OracleH2(P, ell=0.3, **prm).matmul_lowp(X, prec)
        assert (np.linalg.norm(Y.cpu().numpy() - ref, axis=0) / np.linalg.norm(ref, axis=0)).max() <= 1e-5
    A.set_ell(0.7)
    assert torch.equal(h2x.h2_matmul(A, Xd), h2x.h2_matmul(h2x.H2Matrix(P, ell=0.7, storage=prec, **prm), Xd))
    A.set_ell(0.3)
    assert torch.equal(h2x.h2_matmul(A, Xd), Y)
