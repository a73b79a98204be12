"""The split dense kernel (r_p >= 128) through single update steps, against the fp64 oracle.

A step's result is W + V with V = Delta B_J (B_J^T B_J)^-1 (eta = 1, no momentum).  Row by row the
error may be what fp32 storage of the result costs (2^-23 of the row) plus TOL of the step:
products and sums of at most 512 + 1100 terms at 2^-23 each, random in sign, amplified by the
solve's condition (below 100 for these Gaussian panels): 2^-23 sqrt(1612) 100 / 5 ~ 1e-4.
"""

import numpy as np
import pytest
import torch

from oracle import salsa

import paper_2608_21607_amd as nmd

pytestmark = pytest.mark.gpu

TOL = 1e-4


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda()


def one_entry_per_row(m, n, g):
    return (np.arange(m + 1, dtype=np.int64), g.integers(0, n, m).astype(np.int32),
            g.uniform(0.5, 2.0, m).astype(np.float32))


def check_step(m, n, r, block_n, W, H, seed, d=None):
    """d: powers of two the rank's columns of W are scaled by, and the rows of H inversely; W H and the
    scaled step are what they were, and the oracle takes them unscaled."""
    g = np.random.default_rng(seed)
    S_arrays = one_entry_per_row(m, n, g)
    ctx = nmd.Context(m, n, r, m, block_n, seed=1, mode="stochastic")
    ctx.set_sparse_csr(*S_arrays)
    cb = ctx.block_bounds(0)
    S = salsa.csr_matrix(m, n, *S_arrays)
    d = np.ones(r) if d is None else d
    for k in range(len(cb) - 1):
        Wg, Hg = dev(W * d), dev(H / d[:, None])
        ctx.reset()
        ctx.run_steps(Wg, Hg, [k + 1])
        got = Wg.cpu().numpy().astype(np.float64) / d
        assert np.array_equal(Hg.cpu().numpy(), (H / d[:, None]).astype(np.float32))
        X = W.astype(np.float64)
        want, V = salsa.factor_step(S, X, H.astype(np.float64).T, cb[k], cb[k + 1], 1.0, 0.0,
                                    np.zeros_like(X))
        err = np.linalg.norm(got - want, axis=1)
        bar = TOL * np.linalg.norm(V, axis=1) + 2.0 ** -23 * np.linalg.norm(want, axis=1)
        print(f"r={r} block {k} ({cb[k + 1] - cb[k]} rows): worst row at {np.max(err / bar):.3f} of its bar")
        assert np.all(err <= bar)
        by_column = np.linalg.norm(got - want, axis=0)
        assert np.all(by_column <= TOL * np.linalg.norm(V, axis=0) + 2.0**-23 * np.linalg.norm(want, axis=0))
    return ctx


def factors(m, n, r, kind):
    g = np.random.default_rng(m * 7 + n)
    W = g.standard_normal((m, r)).astype(np.float32)
    H = g.standard_normal((r, n)).astype(np.float32)
    if kind != "half":  # L positive on about half a percent, in scattered places
        W[:, -1] = np.sqrt(2.6) * r ** 0.25
        H[-1] = -np.sqrt(2.6) * r ** 0.25
    if kind == "mixed":  # and on half of every other tile's rows (64 of them at r_p > 128, else 128)
        W[(np.arange(m) // (64 if r > 128 else 128)) % 2 == 0, -1] = 0.0
    return W, H


# rows at the edges of the 32-row groups and 64- and 128-row workgroups; panels of whole 32-row
# blocks, one row more, one less; every padded rank, with and without padding columns
@pytest.mark.parametrize("m,n,r,block_n", [
    (129, 258, 65, 129), (257, 383, 100, 383), (255, 642, 128, 321), (384, 352, 128, 352),
    (256, 512, 192, 256), (257, 451, 180, 226), (320, 1026, 256, 513), (383, 575, 250, 288),
    (352, 641, 320, 641), (385, 1100, 300, 1100), (448, 832, 384, 416), (449, 801, 330, 401),
    (513, 1023, 448, 512), (640, 1057, 512, 1057), (527, 1090, 500, 545)])
@pytest.mark.parametrize("kind", ["half", "thin"])
def test_step_edges(m, n, r, block_n, kind):
    print("[case]", m, n, r, block_n, kind, flush=True)
    check_step(m, n, r, block_n, *factors(m, n, r, kind), seed=m)


# panels long enough that a workgroup can find L dense and leave its rows to the fp32 kernel
@pytest.mark.parametrize("m,n,r", [(400, 2100, 128), (330, 2079, 180), (321, 2048, 256), (390, 2500, 320),
                                   (460, 2111, 384), (500, 2300, 448), (530, 2200, 512)])
@pytest.mark.parametrize("kind", ["half", "thin", "mixed"])
def test_step_dense_rows(m, n, r, kind):
    print("[case] dense rows", m, n, r, kind, flush=True)
    ctx = check_step(m, n, r, n, *factors(m, n, r, kind), seed=m)
    slices = ctx.dense_blocks()[0]
    if -(-r // 64) * 64 not in (256, 512):  # where the fp32 kernel counts slices, the split one entries
        assert (slices > 0) == (kind != "thin")


@pytest.mark.parametrize("r", [100, 128, 192, 256, 320, 384, 448, 512])
@pytest.mark.parametrize("thin", [False, True])
def test_step_columns_of_very_different_scale(r, thin):
    """Columns of W scaled over 2^-18 .. 2^18 and the rows of H inversely: each column of the step as
    exact as unscaled."""
    print("[case] columns", r, thin, flush=True)
    m, n = r + 67, 2 * r + 45
    g = np.random.default_rng(r + 1)
    W = g.standard_normal((m, r)).astype(np.float32)
    H = g.standard_normal((r, n)).astype(np.float32)
    if thin:
        W[:, -1], H[-1] = np.sqrt(2.6) * r**0.25, -np.sqrt(2.6) * r**0.25
    check_step(m, n, r, n, W, H, seed=r, d=2.0 ** np.linspace(-18, 18, r).round())


@pytest.mark.parametrize("r", [128, 192, 256, 320, 512])
@pytest.mark.parametrize("where", ["W", "H"])
@pytest.mark.parametrize("value", [2.0**-112, 2.0**-140])
def test_step_values_the_splits_cannot_hold(r, where, value):
    """A row of W (a column of H) with one value, which bf16 terms would cut short: the step is the
    oracle's in every row."""
    print("[case] range", r, where, value, flush=True)
    m, n = r + 130, 3 * r + 33
    g = np.random.default_rng(r + 2)
    W = g.standard_normal((m, r)).astype(np.float32)
    H = g.standard_normal((r, n)).astype(np.float32)
    W[:, -1], H[-1] = np.sqrt(2.6) * r**0.25, -np.sqrt(2.6) * r**0.25
    if where == "W":
        W[70] = 0.0
        W[70, 5] = value
    else:
        H[:, 7] = 0.0
        H[5, 7] = value
    check_step(m, n, r, n, W, H, seed=r)


@pytest.mark.parametrize("r", [128, 256, 320])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_step_not_finite_is_rejected(r, bad):
    """An entry of W or H that is not finite makes the step fail, and W and H come back as they were."""
    print("[case] not finite", r, bad, flush=True)
    m, n = r + 40, 2 * r + 9
    g = np.random.default_rng(r + 3)
    ctx = nmd.Context(m, n, r, m, n, seed=1, mode="stochastic")
    ctx.set_sparse_csr(*one_entry_per_row(m, n, g))
    for where, code in (("W", -6), ("H", -4)):
        W = g.standard_normal((m, r)).astype(np.float32)
        H = g.standard_normal((r, n)).astype(np.float32)
        (W if where == "W" else H)[3, 4] = bad
        Wg, Hg = dev(W), dev(H)
        with pytest.raises(nmd.NmdError) as e:
            ctx.run_steps(Wg, Hg, [1])
        assert e.value.code == code
        assert np.array_equal(Wg.cpu().numpy(), W, equal_nan=True)
        assert np.array_equal(Hg.cpu().numpy(), H, equal_nan=True)


@pytest.mark.parametrize("r", [128, 192, 256, 320, 512])
def test_step_rows_of_very_different_scale(r):
    """Rows of W scaled by 2^-60 .. 2^30, a third of the columns of H by 2^-8 or 2^-20, one row and
    one column zero: the step stays as exact in every row.  (The
    2 r unscaled Gaussian columns keep the Gram matrix's condition below 100.)"""
    print("[case] scales", r, flush=True)
    m, n = r + 129, 3 * r + 35
    g = np.random.default_rng(r)
    W = g.standard_normal((m, r)) * 2.0 ** g.integers(-60, 31, (m, 1))
    H = g.standard_normal((r, n))
    small = g.permutation(n)[: r]
    H[:, small] *= 2.0 ** np.where(np.arange(r) % 2, -8, -20)
    W[5] = 0.0
    H[:, 7] = 0.0
    check_step(m, n, r, n, W.astype(np.float32), H.astype(np.float32), seed=r)
