"""Ranks above 64 where their other tests do not reach.

* A table of near rows too large for LDS (few points a block row, large leaves, on both sides of
  32 columns): the leaf stage runs on the generic tiles; products against the oracle (1e-12 per
  column, as the other FP64 products), and a system of a merged plan that has stopped is left
  alone by the products of the others.
* Kernels other than the exponential, whose coupling matrices are filled entry by entry with
  their padding: the product against the kernel matrix itself, which interpolation of order 3
  and above reproduces (1e-11: rounding of order 5 and 7 interpolation, Lebesgue constants
  below 3 per axis).
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


def _rel(a, b):
    return (np.linalg.norm(a - b, axis=0) / np.linalg.norm(b, axis=0)).max()


def _segment(n):
    """n evenly spaced points of a segment: four leaves of n / 4, neighbours near, others admissible"""
    P = np.zeros((n, 3))
    P[:, 0] = np.arange(n) / n
    return P


# near rows of an inner leaf 3 n / 4: above 12,144 for up to 32 columns, above 8,048 for more
LARGE = [(16800, 20), (11200, 40)]


@pytest.mark.parametrize("n,m", LARGE, ids=[f"m{c[1]}" for c in LARGE])
def test_large_near_tables(n, m):
    h2x = _h2x()
    prm = dict(ell=0.5, shift=1.0, eta=1.0, leaf=n // 4, p=5)
    P = _segment(n)
    A, o = h2x.H2Matrix(P, **prm), oracle.OracleH2(P, **prm)
    assert A.plan.n_adm > 0 and o.n_adm == A.plan.n_adm
    X, Y0 = W.rhs(n, m, 801), W.rhs(n, m, 802)
    ref = o.matmul(X)
    Xd, out = torch.from_numpy(X).cuda(), torch.from_numpy(Y0.copy()).cuda()
    assert _rel(h2x.h2_matmul(A, Xd).cpu().numpy(), ref) <= 1e-12
    h2x.h2_matmul(A, Xd, alpha=-1.5, beta=0.5, out=out)
    assert _rel(out.cpu().numpy(), 0.5 * Y0 - 1.5 * ref) <= 1e-12
    q = A.plan.perm()
    Yt = h2x.h2_matmul(A, torch.from_numpy(X[q]).cuda(), tree_order=True)
    assert _rel(Yt.cpu().numpy(), ref[q]) <= 1e-12


@pytest.mark.parametrize("n,m", LARGE, ids=[f"m{c[1]}" for c in LARGE])
def test_stopped_system_is_left_alone(n, m):
    """A zero right-hand side stops its system before the first iteration; the iterations' products
    then write nothing of it: its rows of A P (the fifth n x m block of the workspace) stay as
    they were, and the other system's solve is the one it has alone, bit for bit."""
    h2x = _h2x()
    n2 = 400
    prm = dict(ell=0.5, shift=1.0, eta=1.0, leaf=n // 4, p=5)
    small = dict(prm, leaf=100)
    A1 = h2x.H2Matrix(_segment(n), **prm)
    B1 = torch.from_numpy(W.rhs(n, m, 803)).cuda()
    X1, _ = h2x.block_cg_solve(A1, B1, rtol=1e-12, max_iter=2)
    del A1
    A = h2x.H2Matrix(h2x.Plan.merge([h2x.Plan(_segment(n), **prm), h2x.Plan(W.sphere_points(n2, 804), **small)]))
    B = torch.cat([B1, torch.zeros(n2, m, dtype=torch.float64, device="cuda")])
    ws = A.workspace(m, "cg")
    ws[:ws.numel() // 8 * 8].view(torch.float64).fill_(1.25)
    X, _ = h2x.block_cg_solve(A, B, rtol=1e-12, max_iter=2)
    block = (n + n2) * m * 8
    at = 4 * ((block + 255) // 256 * 256)
    AP = ws[at:at + block].view(torch.float64).view(n + n2, m)
    assert torch.equal(X[:n], X1) and torch.all(X[n:] == 0.0)
    assert not torch.any(AP[:n] == 1.25)
    assert torch.all(AP[n:] == 1.25)


@pytest.mark.parametrize("p,leaf,m", [(5, 64, 9), (7, 100, 3)])
@pytest.mark.parametrize("kernel", ["poly", "const"])
def test_other_kernels(p, leaf, m, kernel):
    h2x = _h2x()
    n = 1500
    P = W.line_points(n, 810 + p) + 0.05 * W.cube_points(n, 811 + p)
    A = h2x.H2Matrix(P, kernel=kernel, ell=0.5, shift=1.5, eta=1.0, leaf=leaf, p=p)
    assert A.plan.n_adm > 0
    K = (1.0 + P @ P.T) ** 2 if kernel == "poly" else np.ones((n, n))
    K += 1.5 * np.eye(n)
    X = W.rhs(n, m, 812)
    assert _rel(h2x.h2_matmul(A, torch.from_numpy(X).cuda()).cpu().numpy(), K @ X) <= 1e-11
    S = A.coupling()
    A.set_coupling(2.0 * S)
    assert torch.equal(A.coupling(), 2.0 * S)


def test_a_million_columns():
    """2^20 and more columns at rank 512: a cluster's rows of y-hat take more than 4 GiB.  The first,
    the middle and the last columns against the oracle."""
    h2x = _h2x()
    n, m, w = 200, (1 << 20) + 4096, 20
    P = 0.1 * W.cube_points(n, 820)
    P[n // 2:, 0] += 0.9
    prm = dict(ell=0.5, shift=1.0, eta=1.0, leaf=n // 2, p=8)
    A, o = h2x.H2Matrix(P, **prm), oracle.OracleH2(P, **prm)
    assert A.plan.n_adm == 2
    X = torch.randn(n, m, dtype=torch.float64, device="cuda", generator=torch.Generator(device="cuda").manual_seed(821))
    Y = h2x.h2_matmul(A, X)
    for a in (0, m // 2, m - w):
        ref = o.matmul(X[:, a:a + w].cpu().numpy())
        assert _rel(Y[:, a:a + w].cpu().numpy(), ref) <= 1e-12, a
