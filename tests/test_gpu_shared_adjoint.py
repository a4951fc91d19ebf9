"""blp_backward_shared's sums over the LPs (GPU) at the edges of its 16 x 16
tiles, groups of four tiles and steps of four LPs, against float64 products on
the CPU; NaN in LPs that are not OPTIMAL stays out."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [(1, 1), (15, 16), (16, 15), (17, 17), (100, 100), (33, 63), (5, 64), (16, 65), (112, 48)])
@pytest.mark.parametrize("count", [1, 3, 5, 17, 1025, 2500])
def test_sums(m, n, count):
    import torch

    import paper_1609_08114_amd as blp
    rng = np.random.default_rng(m * 1000 + n + count)
    x, y, g = rng.normal(size=(count, n)), rng.normal(size=(count, m)), rng.normal(size=count)
    st = np.where(rng.random(count) < 0.2, 3, 0).astype(np.int32)
    w = np.where(st == 0, g, 0.0)
    ref = w[:, None] * y
    ref_a, ref_b = -ref.T @ x, ref.sum(0)
    # every sum: count products and additions, each rounded (and the
    # reference's own), against the sum of the magnitudes
    tol = 2 * (count + 2) * 2.0 ** -53
    lim_a, lim_b = tol * (np.abs(ref).T @ np.abs(x)), tol * np.abs(ref).sum(0)
    x[st != 0] = np.nan
    y[st != 0] = np.nan
    dev = [torch.from_numpy(t).cuda() for t in (st, x, y, g)]
    dC = torch.empty(count * n, dtype=torch.float64, device="cuda")
    db = torch.full((m,), 7.0, dtype=torch.float64, device="cuda")
    dA = torch.full((m * n,), 7.0, dtype=torch.float64, device="cuda")
    s = blp.Solver()
    print(f"[shared adjoint] {count} LPs {m} x {n}", flush=True)
    blp.blp_backward_shared(s.h, m, n, count, *[blp._ptr(t) for t in dev], blp._ptr(dC), blp._ptr(db), blp._ptr(dA),
                            torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    s.close()
    assert (np.abs(dA.cpu().numpy().reshape(m, n) - ref_a) <= lim_a).all()
    assert (np.abs(db.cpu().numpy() - ref_b) <= lim_b).all()
