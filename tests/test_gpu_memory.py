"""The copies that only make a step or the objective faster are left out where memory is short."""

import numpy as np
import pytest
import torch

import paper_2608_21607_amd as nmd

pytestmark = pytest.mark.gpu


def test_little_memory_left():
    """With all but the last 300 MB of what a context takes, which its panel's split copy (600 MB)
    does not fit, a step and the objective come out as with it; so they do once there is room."""
    m, n, r = 1000, 200_000, 512
    g = np.random.default_rng(1)
    S = (np.arange(m + 1, dtype=np.int64), g.integers(0, n, m).astype(np.int32), np.ones(m, np.float32))
    W0 = torch.randn((m, r), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    H0 = torch.randn((r, n), generator=torch.Generator(device="cuda").manual_seed(2), device="cuda")
    W0[:, -1], H0[-1] = 7.0, -7.0

    def run(then=lambda: None):
        ctx = nmd.Context(m, n, r, m, n, seed=1, mode="stochastic")
        ctx.set_sparse_csr(*S)
        W.copy_(W0)
        H.copy_(H0)
        before = torch.cuda.mem_get_info()[0]
        ctx.run_steps(W, H, [1])
        used = before - torch.cuda.mem_get_info()[0]
        f = ctx.objective(W, H)
        then()
        again = ctx.objective(W, H)
        ctx.close()
        return W.clone(), f, again, used

    W, H = W0.clone(), H0.clone()
    run()  # what is allocated once (code objects, streams) is there when the second run is measured
    W1, f, _, used = run()
    room = used - 300_000_000
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    print(f"[case] a context takes {used >> 20} MB, {room >> 20} MB are left", flush=True)
    filler = []
    for _ in range(8):  # a first piece may find cached memory that the free count does not hold
        over = torch.cuda.mem_get_info()[0] - room
        if over < 16_000_000:
            break
        filler.append(torch.empty(over, dtype=torch.uint8, device="cuda"))
    if torch.cuda.mem_get_info()[0] > room + 16_000_000:
        filler.clear()
        torch.cuda.empty_cache()
        pytest.skip("the free memory does not stay at its mark: the device is shared")

    def free():
        filler.clear()
        torch.cuda.empty_cache()

    W2, f2, f3, used2 = run(free)
    assert used2 < used - 200_000_000  # the copy was left out
    assert float((W2 - W1).norm() / W1.norm()) < 1e-5
    assert abs(f2 / f - 1) < 1e-7 and abs(f3 / f - 1) < 1e-7
