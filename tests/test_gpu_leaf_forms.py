"""Leaf stage at the edges of its tiles: one to four column tiles of 16 and narrow last slabs, chunks
of a leaf of 1 to 64 rows (two, three or four row tiles; leaves above 64 points take several chunks).
"""
import numpy as np
import pytest

import oracle
from paper_2509_17257_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

COLS = (1, 2, 15, 16, 17, 32, 33, 45, 48, 49, 64, 65, 96, 97)
# leaf sizes 16 and 28: two row tiles, 45: three, 64: four, 100: a second chunk
LEAVES = [(16, 2), (28, 3), (45, 4), (64, 4), (100, 4)]


def _rel(a, b):
    return (np.linalg.norm(a - b, axis=0) / np.linalg.norm(b, axis=0)).max()


@pytest.mark.parametrize("leaf,p", LEAVES)
@pytest.mark.parametrize("prec", ["f32", "bf16"])
def test_lowp_leaf(leaf, p, prec):
    """Against the form with a 64-row tile per wave and term (leaf_kind 1): both start from the same
    bits of X and y_t, so only the order of the FP32 sums of the leaf stage differs, for BF16 as for
    FP32; FP32 also against the oracle (BF16 intermediates of the earlier stages can round to
    neighbours there, which is not the leaf stage's)."""
    import paper_2509_17257_amd as h2x
    P = W.cube_points(2600, 700 + leaf)
    prm = dict(ell=0.4, shift=1.0, eta=1.0, leaf=leaf, p=p)
    A = h2x.H2Matrix(P, storage=prec, **prm)
    X = W.rhs(2600, max(COLS), 701)
    emu = oracle.OracleH2(P, **prm).matmul_lowp(X, prec) if prec == "f32" else None
    for m in COLS:
        Xd = torch.from_numpy(np.ascontiguousarray(X[:, :m])).cuda()
        A.set_tune(m, leaf_kind=1)
        ref = h2x.h2_matmul(A, Xd).cpu().numpy()
        A.set_tune(m)
        Y = h2x.h2_matmul(A, Xd)
        assert _rel(Y.cpu().numpy(), ref) <= 1e-5, m
        assert emu is None or _rel(Y.cpu().numpy(), emu[:, :m]) <= 1e-5, m
        # alpha and beta, and a wider row stride of the result
        out = torch.ones(2600, m + 3, dtype=torch.float64, device="cuda")
        h2x.h2_matmul(A, Xd, alpha=2.0, beta=3.0, out=out[:, :m])
        assert torch.equal(out[:, :m], 3.0 + 2.0 * Y) and torch.all(out[:, m:] == 1.0)


@pytest.mark.parametrize("leaf", [45, 64])
@pytest.mark.parametrize("prec", ["f32", "bf16"])
def test_lowp_many_leaves(leaf, prec):
    """More than 2048 work-groups on leaves above 32 points: two waves each."""
    import paper_2509_17257_amd as h2x
    n = 130000
    A = h2x.H2Matrix(W.sphere_points(n, 710), storage=prec, ell=0.5, shift=1.0, eta=1.0, leaf=leaf, p=2)
    X = torch.from_numpy(W.rhs(n, 64, 711)).cuda()
    for m in (7, 16, 31, 48, 64):
        Xm = X[:, :m].contiguous()
        A.set_tune(m, leaf_kind=1)
        ref = h2x.h2_matmul(A, Xm)
        A.set_tune(m)
        Y = h2x.h2_matmul(A, Xm)
        assert _rel(Y.cpu().numpy(), ref.cpu().numpy()) <= 1e-5, m


@pytest.mark.parametrize("leaf,p", LEAVES)
@pytest.mark.parametrize("cplx", [False, True], ids=["real", "complex"])
def test_fp64_leaf(leaf, p, cplx):
    """Against the oracle at FP64 rounding, and column by column the same bits whatever the slab."""
    import paper_2509_17257_amd as h2x
    n, top = 2600, 100 if not cplx else 50
    P = W.cube_points(n, 720 + leaf)
    prm = dict(ell=0.8, shift=1.0, eta=1.0, leaf=leaf, p=p)
    if cplx:
        prm["kernel"] = "helmholtz"
    A, o = h2x.H2Matrix(P, **prm), oracle.OracleH2(P, **prm)
    X = W.rhs(n, top, 721)
    if cplx:
        X = X + 1j * W.rhs(n, top, 722)
    ref = o.matmul_complex(X) if cplx else o.matmul(X)
    Xd = torch.from_numpy(X).cuda()
    Y = h2x.h2_matmul(A, Xd)
    assert _rel(Y.cpu().numpy(), ref) <= 1e-12
    for m in ((1, 7, 8, 9, 16, 17, 24, 25, 32, 33, 41) if cplx else COLS):
        Xm = Xd[:, :m].contiguous()
        Ym = h2x.h2_matmul(A, Xm)
        assert torch.equal(Ym, Y[:, :m]), m
        out = torch.ones_like(Ym)
        h2x.h2_matmul(A, Xm, alpha=2.0, beta=3.0, out=out)
        assert torch.equal(out, 3.0 + 2.0 * Ym), m


@pytest.mark.parametrize("leaf", [45, 64, 100])
def test_fp64_many_leaves(leaf):
    """17 to 32 columns on more than 1024 leaves above 32 points take two waves per leaf; the same bits
    as the first columns of a wider product, which takes four."""
    import paper_2509_17257_amd as h2x
    n = 130000
    A = h2x.H2Matrix(W.sphere_points(n, 730), ell=0.5, shift=1.0, eta=1.0, leaf=leaf, p=2)
    assert (A.plan.C + 1) // 2 >= 1024
    X = torch.from_numpy(W.rhs(n, 40, 731)).cuda()
    Y = h2x.h2_matmul(A, X)
    for m in (16, 17, 31, 32):
        assert torch.equal(h2x.h2_matmul(A, X[:, :m].contiguous()), Y[:, :m]), m
