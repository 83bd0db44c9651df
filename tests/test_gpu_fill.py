"""The operator's entries as the device writes them (exponential kernel, FP64).

* Every coupling matrix, at each Chebyshev order, against exp(-|x - y| / ell) at the nodes in
  numpy: relative 2e-14 (an argument of up to 13 carries its relative rounding of a few 2^-53
  into the exponential, and the nodes' own rounding adds |dx| / ell of 2^-52).
* S_(s,t) = S_(t,s)^T and N_(s,t) = N_(t,s)^T bit for bit (one of the two is evaluated).
* A refill at another length scale and back gives the first matrices bit for bit.
* Distances beyond the range of the fast square root (a cloud scaled by 2^480) give the product
  of the unscaled cloud.
"""
import numpy as np
import pytest

from paper_2509_17257_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _h2x():
    import paper_2509_17257_amd as h2x
    return h2x


@pytest.mark.parametrize("p,leaf,n", [(1, 8, 500), (2, 16, 900), (3, 32, 1500), (4, 64, 2500), (5, 64, 2000),
                                      (6, 70, 1500), (8, 70, 1100)])
def test_coupling_entries(p, leaf, n):
    h2x = _h2x()
    P = W.line_points(n, 400 + p) + 0.05 * W.cube_points(n, 410 + p)
    ell = 0.3
    A = h2x.H2Matrix(P, ell=ell, shift=1.0, eta=1.0, leaf=leaf, p=p)
    pl = A.plan
    S = A.coupling().cpu().numpy()
    cl, b = pl.clusters(), pl.blocks()
    Q = P[pl.perm()]
    ch = np.cos((2 * np.arange(p) + 1) * np.pi / (2 * p))
    nu = np.arange(p ** 3)
    dig = [nu % p, nu // p % p, nu // (p * p)]

    def nodes(c):
        q = Q[cl["first"][c]:cl["first"][c] + cl["size"][c]]
        lo, hi = q.min(0), q.max(0)
        return np.stack([0.5 * (lo[d] + hi[d]) + 0.5 * (hi[d] - lo[d]) * ch[dig[d]] for d in range(3)], 1)

    at = {(t, s): i for i, (t, s) in enumerate(zip(b["adm_t"], b["adm_s"]))}
    assert len(at) > 10
    for (t, s), i in at.items():
        r = np.sqrt(((nodes(t)[:, None] - nodes(s)[None]) ** 2).sum(2))
        ref = np.exp(-r / ell)
        assert np.abs(S[i] / ref - 1).max() <= 2e-14
        assert np.array_equal(S[i], S[at[(s, t)]].T)
    A.set_ell(0.7)
    assert not np.array_equal(A.coupling().cpu().numpy(), S)
    A.set_ell(ell)
    assert np.array_equal(A.coupling().cpu().numpy(), S)


@pytest.mark.parametrize("leaf,p", [(17, 3), (64, 4), (130, 4), (200, 5)])
def test_near_field_is_symmetric(leaf, p):
    """With a tiny eta no block is admissible: the operator is the kernel matrix itself."""
    h2x = _h2x()
    n = 700
    P = W.sphere_points(n, 420 + leaf)
    A = h2x.H2Matrix(P, ell=0.5, shift=1.5, eta=1e-9, leaf=leaf, p=p)
    assert A.plan.n_adm == 0
    K = h2x.h2_matmul(A, torch.eye(n, dtype=torch.float64, device="cuda")).cpu().numpy()
    assert np.array_equal(K, K.T)
    ref = np.exp(-np.sqrt(((P[:, None] - P[None]) ** 2).sum(2)) / 0.5) + 1.5 * np.eye(n)
    assert np.abs(K / ref - 1).max() <= 2e-14


def test_scaled_cloud():
    h2x = _h2x()
    n, sc = 1500, 2.0 ** 480
    P, X = W.cube_points(n, 430), torch.from_numpy(W.rhs(n, 5, 431)).cuda()
    prm = dict(shift=1.0, eta=1.0, leaf=32, p=3)
    Y = h2x.h2_matmul(h2x.H2Matrix(P, ell=0.5, **prm), X)
    Z = h2x.h2_matmul(h2x.H2Matrix(P * sc, ell=0.5 * sc, **prm), X)
    assert torch.isfinite(Z).all()
    assert (torch.linalg.norm(Z - Y, dim=0) / torch.linalg.norm(Y, dim=0)).max().item() <= 1e-12
