"""The contraction at r_p <= 64, both products on three-term bf16 splits, against fp64 with the bounds
of fp32 arithmetic, and beside what plain fp32 products give."""

import numpy as np
import pytest
import torch

import paper_2608_21607_amd as nmd
from workloads import gen

pytestmark = pytest.mark.gpu


def _inputs(rows, blk, r, kind):
    g = np.random.default_rng(1000 * rows + 10 * blk + r)
    X = g.standard_normal((rows, r))
    P = g.standard_normal((blk, r))
    if kind == "thin":  # few positive entries
        X[:, -1], P[:, -1] = 2.0, -1.25 * r**0.5
    elif kind == "wide":  # rows of X and of the panel far apart in magnitude
        X *= 2.0 ** g.integers(-30, 30, (rows, 1))
        P *= 2.0 ** g.integers(-20, 20, (blk, 1))
    elif kind == "growing":  # every panel row larger than those before
        P *= 2.0 ** (np.arange(blk)[:, None] * (40.0 / blk))
    elif kind == "panel columns":  # the rank's columns far apart, in the panel alone
        P *= 2.0 ** -np.linspace(0, 40, r).round()
    elif kind == "balanced columns":  # the same in X and inversely in the panel: L as it was
        d = 2.0 ** np.linspace(-32, 32, r).round()
        X, P = X * d, P / d
    elif kind == "one column":  # one small column of X against a large one of the panel
        X[:, 3] *= 2.0**-40
        P[:, 3] *= 2.0**40
    elif kind == "constant":  # a constant column that cancels most of the others
        X[:, 2], P[:, 2] = 40.0, -40.0
        X[:, 5], P[:, 5] = 40.0 + X[:, 5], 40.0 + P[:, 5]
    return X.astype(np.float32), P.astype(np.float32)


def _bound(X, P):
    """Reference and elementwise bound: an fp32 sum of k products is off by k 2^-24 of the sum of
    their magnitudes; the matrix unit aligns sixteen products and cuts or rounds seventeen times; four
    more for the products' own rounding, the terms a split leaves out and the last additions."""
    X, P = X.astype(np.float64), P.astype(np.float64)
    r, blk = X.shape[1], P.shape[0]
    aX, aP = np.abs(X), np.abs(P)
    Z = np.maximum(X @ P.T, 0)
    eL = (17 / 16 * r + 4) * 2.0**-24 * (aX @ aP.T)
    return Z @ P, eL @ aP + (17 / 16 * blk + blk / 256 + 4) * 2.0**-24 * (Z @ aP)


KINDS = ["half", "thin", "wide", "growing", "panel columns", "balanced columns", "one column", "constant"]


@pytest.mark.parametrize("r", [16, 32, 48, 64])
@pytest.mark.parametrize("rows,blk", [(1, 1), (31, 17), (256, 128), (257, 333), (700, 2049)])
@pytest.mark.parametrize("kind", KINDS)
def test_small_contraction(r, rows, blk, kind):
    X, P = _inputs(rows, blk, r, kind)
    Y = nmd.rectified_contraction(torch.from_numpy(X).cuda(), torch.from_numpy(P).cuda()).cpu().numpy()
    want, bound = _bound(X, P)
    worst = (np.abs(Y - want) / np.maximum(bound, 1e-300)).max()
    print(f"r = {r}, {rows} x {blk}, {kind}: {worst:.3f} of the bound")
    assert worst <= 1.0


def _column_errors(Y, want):
    scale = np.linalg.norm(want, axis=0)
    return np.linalg.norm(Y - want, axis=0) / np.where(scale > 0, scale, 1)


@pytest.mark.parametrize("r", [16, 32, 48, 64])
@pytest.mark.parametrize("kind", ["half", "panel columns", "balanced columns", "one column"])
def test_each_column_as_close_as_fp32_products(r, kind):
    """Column by column no further from fp64 than twice what fp32 products and sums give."""
    X, P = _inputs(500, 900, r, kind)
    Y = nmd.rectified_contraction(torch.from_numpy(X).cuda(), torch.from_numpy(P).cuda()).cpu().numpy()
    want, _ = _bound(X, P)
    got, plain = _column_errors(Y, want), _column_errors(np.maximum(X @ P.T, 0) @ P, want)
    print(f"r = {r}, {kind}: worst column {got.max():.1e}, with fp32 products {plain.max():.1e}")
    assert (got <= 2 * plain + 2.0**-24).all()


def test_identity_factors_that_cancel():
    """The exact rank-3 factors of the identity: a constant column cancels the other two, so W H is
    what is left of terms up to 1e6 times larger."""
    W, H = gen.identity_exact_factors(2048)
    X, P = np.zeros((2048, 16), np.float32), np.zeros((2048, 16), np.float32)
    X[:, :3], P[:, :3] = W, H.T
    Y = nmd.rectified_contraction(torch.from_numpy(X).cuda(), torch.from_numpy(P).cuda()).cpu().numpy()
    want, _ = _bound(X, P)
    got = np.linalg.norm(Y - want) / np.linalg.norm(want)
    plain = np.linalg.norm(np.maximum(X @ P.T, 0) @ P - want) / np.linalg.norm(want)
    print(f"identity: {got:.1e}, with fp32 products {plain:.1e}")
    assert got <= 1.5 * plain


@pytest.mark.parametrize("r", [16, 48, 64])
@pytest.mark.parametrize("where", ["X", "P"])
@pytest.mark.parametrize("value", [2.0**-140, 2.0**-112, 1.5 * 2.0**127, 2.0**70])
def test_values_outside_the_splits_range(r, where, value):
    """Magnitudes that bf16 terms cannot hold, or whose products overflow, against plain fp32."""
    rows, blk = 300, 70
    X, P = _inputs(rows, blk, r, "half")
    if value > 1:  # one sign: what overflows is +infinity in any order
        X, P = np.abs(X), np.abs(P)
    if where == "X":
        X[5] = 0.0
        X[5, 3] = value
    else:
        P[5] = 0.0
        P[5, 3] = value
    if value == 2.0**70:
        (P if where == "X" else X)[:, 3] *= np.float32(2.0**70)  # L overflows
    Y = nmd.rectified_contraction(torch.from_numpy(X).cuda(), torch.from_numpy(P).cuda()).cpu().numpy()
    with np.errstate(all="ignore"):
        L = (X.astype(np.float64) @ P.astype(np.float64).T).astype(np.float32).astype(np.float64)
        terms = [(l[l > 0][:, None] * P[l > 0].astype(np.float64)) for l in L]
        want = np.stack([t.sum(0) for t in terms])
        mag = np.stack([np.abs(t).sum(0) for t in terms])
        want = want.astype(np.float32).astype(np.float64)
    inf = np.isinf(want)
    assert np.array_equal(np.isnan(Y), np.isnan(want)) and np.array_equal(Y[inf], want[inf])
    ok = np.isfinite(want)
    A = np.abs(X.astype(np.float64)) @ np.abs(P.astype(np.float64)).T
    slack = (r + blk + 8) * 2.0**-24 * (A @ np.abs(P.astype(np.float64)) + mag)
    slack += r * 2.0**-150 * np.abs(P.astype(np.float64)).sum(0) + blk * 2.0**-150  # subnormal roundings
    assert (np.abs(Y - want)[ok] <= slack[ok]).all()


@pytest.mark.parametrize("r", [16, 48, 64])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("where", ["X", "P"])
def test_small_contraction_not_finite(r, bad, where):
    """Entries of L that are not above zero add nothing, the others what fp32 products give."""
    rows, blk = 300, 70
    X, P = _inputs(rows, blk, r, "half")
    (X if where == "X" else P)[5, 3] = bad
    Y = nmd.rectified_contraction(torch.from_numpy(X).cuda(), torch.from_numpy(P).cuda()).cpu().numpy()
    with np.errstate(invalid="ignore", over="ignore"):
        L = X.astype(np.float64) @ P.astype(np.float64).T
        want = np.stack([(l[l > 0][:, None] * P[l > 0].astype(np.float64)).sum(0) for l in L])
    assert np.array_equal(np.isnan(Y), np.isnan(want))
    assert np.array_equal(np.isposinf(Y), np.isposinf(want))
    assert np.array_equal(np.isneginf(Y), np.isneginf(want))
    ok = np.isfinite(want)
    keep = np.isfinite(X).all(1)
    Xf, Pf = X[keep], P[np.isfinite(P).all(1)]
    _, bound = _bound(Xf, Pf)
    # rows computed again in fp32 round once per product: r + blk roundings of 2^-24
    slack = np.abs(Xf.astype(np.float64)) @ np.abs(Pf.T.astype(np.float64)) @ np.abs(Pf.astype(np.float64))
    bound = bound + (r + blk) * 2.0**-24 * slack
    m = ok[keep]
    assert (np.abs(Y[keep][m] - want[keep][m]) <= bound[m]).all()
