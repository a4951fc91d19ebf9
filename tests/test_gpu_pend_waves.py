"""The pending-pivot kernel's tiles of two, four and eight waves where the waves
exchange more than a candidate (GPU): pivots with non-finite entries, which any
wave may see and which are flushed before the next pivot, and the random
entering rule's ranks over all waves.  The kernels that update at every pivot
keep the same tableau, so the bits agree."""
import numpy as np
import pytest

import lpgen
import oracle
from solve_util import crafted_batch, gpu_solve

pytestmark = pytest.mark.gpu


def _eager(waves):
    """The 160 x 160 block tile, or, for LPs beyond it, the kernel that streams at every pivot."""
    import torch  # noqa: F401  (its HIP runtime before the library's)

    import paper_1609_08114_amd as blp
    if waves < 8:
        return dict(variant=[x[0] for x in blp.variants()].index("b8_r160_c160"))
    return dict(variant=-2, layout=blp.BLP_LAYOUT_ROW)


def _same(a, b):
    for k in ("status", "iters"):
        assert np.array_equal(a[k], b[k]), k
    for k in ("obj", "x", "y"):
        assert np.array_equal(np.isnan(a[k]), np.isnan(b[k])), k
        assert np.array_equal(np.nan_to_num(a[k], nan=7.0), np.nan_to_num(b[k], nan=7.0)), k


@pytest.mark.parametrize("waves,m,n", [(2, (70, 120), (20, 60)), (4, (130, 150), (30, 100)), (8, (257, 300), (10, 60))])
def test_non_finite_pivots(waves, m, n):
    rng = np.random.default_rng(waves)
    lps = []
    for t in range(60):
        mk, nk = int(rng.integers(*m)), int(rng.integers(*n))
        mag = (40, 160, 300)[t % 3]
        A = rng.uniform(-1, 10, size=(mk, nk)) * 10.0 ** rng.uniform(-mag, mag, size=(mk, nk))
        b = rng.uniform(1, 10, size=mk) * 10.0 ** rng.uniform(-mag, mag, size=mk)
        c = rng.uniform(1, 10, size=nk) * 10.0 ** rng.uniform(-mag / 2, mag / 2, size=nk)
        lps.append(dict(A=A, b=b, c=c, sense=(rng.random(mk) < 0.15).astype(np.int8)))
    hb = crafted_batch(lps)
    print(f"[pend waves] non-finite pivots, {waves} waves", flush=True)
    ref = gpu_solve(hb, max_iter=60, **_eager(waves))
    assert ref["bins"][-2] == (hb.count if waves == 8 else 0)  # (the tile holds them all)
    got = gpu_solve(hb, max_iter=60, variant=-2)
    assert ref["iters"].max() > 10
    # overflowing tableaux end as NUMERICAL, or without a row to leave
    assert (ref["status"] == oracle.NUMERICAL).sum() >= 3, np.bincount(ref["status"])
    _same(ref, got)


@pytest.mark.parametrize("waves,m,n,ty", [(2, 100, 70, 1), (4, 140, 60, 2), (4, 150, 150, 1), (8, 260, 40, 2)])
def test_random_rule(waves, m, n, ty):
    import paper_1609_08114_amd as blp
    K = 10
    hb = lpgen.make_batch(95, np.arange(K), np.full(K, ty, np.int32), np.full(K, m, np.int32), np.full(K, n, np.int32))
    kw = dict(pivot_rule=blp.BLP_RULE_RPC, seed=11)
    print(f"[pend waves] random rule, {waves} waves", flush=True)
    a, b = gpu_solve(hb, **_eager(waves), **kw), gpu_solve(hb, variant=-2, **kw)
    assert a["iters"].min() > 3
    _same(a, b)
