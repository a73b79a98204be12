"""The objective and the two measures at r_p >= 64 (L on three-term bf16 splits), against the fp64
oracle, at the edges of their tiles: column blocks that start and end inside 32-column blocks, ranges
of a few columns, rows short of a workgroup, rows with many adjacent entries, empty rows and columns.

Bar: an entry of L is within 2^-23 of its terms' sum of magnitudes (about sqrt(r) |L| here), random in
sign, and the sums run over 8000 entries and more: the relative error of a sum is below
2^-23 sqrt(512) / sqrt(8000) = 3e-8.
"""

import numpy as np
import pytest
import torch

from oracle import salsa
from workloads import gen

import paper_2608_21607_amd as nmd

pytestmark = pytest.mark.gpu

TOL = 3e-8


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda()


@pytest.mark.parametrize("m,n,r,block_n,density", [
    (127, 65, 64, 65, 0.5), (129, 1000, 64, 333, 0.02), (300, 257, 100, 128, 0.1),
    (128, 2001, 128, 1999, 0.01), (193, 400, 192, 397, 0.2), (257, 901, 250, 300, 0.05),
    (320, 330, 320, 330, 0.9), (385, 1025, 333, 513, 0.03), (449, 470, 448, 470, 0.1),
    (600, 1055, 512, 1055, 0.02)])
def test_metrics_edges(m, n, r, block_n, density):
    print("[case]", m, n, r, block_n, density, flush=True)
    g = np.random.default_rng(m + n)
    S = gen.random_sparse(m, n, density, r, empty_rows=3, empty_cols=5)
    W = (0.3 * g.standard_normal((m, r))).astype(np.float32)
    H = (0.3 * g.standard_normal((r, n))).astype(np.float32)
    ctx = nmd.Context(m, n, r, m, block_n)
    ctx.set_sparse_csr(*S)
    Wd, Hd = dev(W), dev(H)
    got, f = ctx.metrics(Wd, Hd), ctx.objective(Wd, Hd)
    L = W.astype(np.float64) @ H.astype(np.float64)
    Sd = salsa.csr_matrix(m, n, *S).toarray()
    want = {"objective": np.sqrt(salsa.squared_loss_dense(Sd, L)) / np.linalg.norm(Sd),
            "rmse": salsa.rmse_dense(Sd, np.maximum(L, 0)), "wjd": salsa.wjd_dense(Sd, np.maximum(L, 0))}
    print({k: f"{abs(got[k] / want[k] - 1):.1e}" for k in want}, f"{abs(f / want['objective'] - 1):.1e}")
    assert all(abs(got[k] - want[k]) <= TOL * want[k] for k in want)
    assert abs(f - want["objective"]) <= TOL * want["objective"]


@pytest.mark.parametrize("r", [64, 100, 128, 192, 256, 320, 384, 448, 512])
@pytest.mark.parametrize("tiny", [False, True])
def test_columns_of_very_different_scale(r, tiny):
    """Columns of W over 2^-30 .. 2^30 and the rows of H inversely: W H, and so the three numbers, as
    unscaled.  `tiny`: with an entry of H that bf16 terms cut short, so that L is formed in fp32."""
    print("[case] columns", r, tiny, flush=True)
    m, n = r + 75, 3 * r + 50
    g = np.random.default_rng(r)
    S = gen.random_sparse(m, n, 0.05, r)
    d = 2.0 ** np.linspace(-30, 30, r).round()
    W, H = 0.3 * g.standard_normal((m, r)), 0.3 * g.standard_normal((r, n))
    W, H = W.astype(np.float32), H.astype(np.float32)
    if tiny:
        H[:, 11] = 0.0
        H[3, 11] = 2.0**-80
        d[3] = 2.0**35  # 2^-115 after the division
    ctx = nmd.Context(m, n, r, m, n)
    ctx.set_sparse_csr(*S)
    got = ctx.metrics(dev(W * d), dev(H / d[:, None]))
    L = W.astype(np.float64) @ H.astype(np.float64)
    Sd = salsa.csr_matrix(m, n, *S).toarray()
    want = {"objective": np.sqrt(salsa.squared_loss_dense(Sd, L)) / np.linalg.norm(Sd),
            "rmse": salsa.rmse_dense(Sd, np.maximum(L, 0)), "wjd": salsa.wjd_dense(Sd, np.maximum(L, 0))}
    print({k: f"{abs(got[k] / want[k] - 1):.1e}" for k in want})
    assert all(abs(got[k] - want[k]) <= (4 * TOL if tiny else TOL) * want[k] for k in want)


@pytest.mark.parametrize("r", [64, 256])
@pytest.mark.parametrize("bad", [np.inf, -np.inf])
def test_infinite_factor_gives_no_finite_objective(r, bad):
    """An infinite entry of W whose row of W H holds +infinity makes the objective infinite (a row
    of -infinity rectifies to zero where S is zero, and is infinite at the row's entry)."""
    print("[case] infinity", r, bad, flush=True)
    m, n = r + 5, r + 40
    g = np.random.default_rng(r)
    S = gen.random_sparse(m, n, 0.1, 3)
    W = np.abs(g.standard_normal((m, r))).astype(np.float32)
    H = np.abs(g.standard_normal((r, n))).astype(np.float32)
    W[0, 1] = bad
    ctx = nmd.Context(m, n, r, m, n)
    ctx.set_sparse_csr(*S)
    assert not np.isfinite(ctx.objective(dev(W), dev(H)))
