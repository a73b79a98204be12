"""The kernels of small ranks (r_p <= 64) at the edges of their tiles, against the fp64 oracle: the
one-launch solve (chunks of 512, 160 and 64 panel rows, sixteen at most), the 16-row apply, and the
full steps' sparse correction in one launch.  W and H within the 1e-4 bar of the sweeps."""

import numpy as np
import pytest
import torch

from oracle import salsa
from workloads import gen

import paper_2608_21607_amd as nmd
from paper_2608_21607_amd import nmd as binding

pytestmark = pytest.mark.gpu

TOL = 1e-4


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda()


def run(m, n, r, bm, bn, arrays, mode, seed, sweeps=1):
    W0, H0 = gen.sign_constrained_init(m, n, r, float(arrays[2].mean()), seed)
    ctx = nmd.Context(m, n, r, bm, bn, seed=3, mode=mode, eta=0.5, momentum=0.5)
    ctx.set_sparse_csr(*arrays)
    W, H = dev(W0), dev(H0)
    ctx.sweep(W, H, sweeps)
    S = salsa.csr_matrix(m, n, *arrays)
    st = salsa.State(W0, H0)
    for _ in range(sweeps):
        salsa.sweep(S, S.T.tocsr(), st, bm, bn, 3, mode=mode, eta=0.5, gamma=0.5)
    ew, eh = rel(W.cpu().numpy(), st.W), rel(H.cpu().numpy(), st.H)
    print(f"m={m} n={n} r={r} {mode}: rel err W {ew:.1e} H {eh:.1e}")
    assert ew < TOL and eh < TOL


# panels of one chunk, of a chunk and a row, of more rows than sixteen chunks of one round
@pytest.mark.parametrize("m,n,r,bm,bn", [
    (17, 16, 1, 17, 16), (513, 1025, 8, 513, 1025), (1024, 512, 16, 512, 512),
    (161, 319, 17, 161, 160), (2721, 480, 32, 2721, 160), (129, 64, 33, 65, 64),
    (1100, 193, 48, 1100, 65), (128, 1030, 49, 64, 1030), (200, 2100, 64, 100, 2100)])
@pytest.mark.parametrize("mode", ["stochastic", "deterministic"])
def test_small_rank_sweep(m, n, r, bm, bn, mode):
    print("[case]", m, n, r, bm, bn, mode, flush=True)
    run(m, n, r, bm, bn, gen.random_sparse(m, n, 0.06, m + n + r), mode, m)


@pytest.mark.parametrize("r", [8, 40, 100, 320])
@pytest.mark.parametrize("heavy", [0.0, 0.5])
def test_full_step_sparse_rows(r, heavy):
    """Deterministic sweep over several blocks with empty rows and columns; with `heavy`, a row
    longer than one wave takes (700 entries), so that side goes block by block."""
    m, n = 900, 1300
    print("[case]", m, n, r, heavy, flush=True)
    S = gen.random_sparse(m, n, 0.01, 5 + r, empty_rows=40, empty_cols=70, heavy_row_frac=heavy)
    counts = np.diff(S[0])
    assert (counts.max() > 512) == (heavy > 0)
    run(m, n, r, 330, 400, S, "deterministic", 7)


# many rows without entries; a few entries in every row; many entries a row against a long panel
@pytest.mark.parametrize("m,n,r,blocks,per,by_rows", [
    (300_000, 200, 20, 4, 0.01, False), (300_000, 200, 20, 4, 3.0, True), (3000, 900, 20, 3, 0.01, True),
    (3000, 900, 150, 30, 5.0, True), (3000, 900, 150, 33, 5.0, False), (700, 30_000, 128, 4, 100.0, False)])
def test_full_step_sparse_route(m, n, r, blocks, per, by_rows):
    """One launch for all blocks only where it is the faster: the W-step's corrections are one launch by
    rows and one per block otherwise, and the sweep is the oracle's either way."""
    print("[case]", m, n, r, blocks, per, flush=True)
    g = np.random.default_rng(m + r)
    keys = np.unique(np.concatenate([g.integers(0, m * n, int(m * per)), (np.arange(n) % m) * n + np.arange(n)]))
    row_ptr = np.zeros(m + 1, np.int64)
    row_ptr[1:] = np.cumsum(np.bincount(keys // n, minlength=m))
    S = (row_ptr, (keys % n).astype(np.int32), g.uniform(0.5, 2.0, keys.size).astype(np.float32))
    bn = -(-n // blocks)
    run(m, n, r, m, bn, S, "deterministic", 5)
    ctx = nmd.Context(m, n, r, m, bn, seed=3, mode="deterministic", eta=0.5, flags=binding.FLAG_TIMING)
    ctx.set_sparse_csr(*S)
    W0, H0 = gen.sign_constrained_init(m, n, r, 1.0, 5)
    ctx.sweep(dev(W0), dev(H0), 1)
    # the H-step has one block
    assert ctx.kernel_timing(1)["launches"] == 1 + (1 if by_rows else blocks)
