"""The streaming kernel with pending pivots (simplex_pend.hip), every LP forced
through the streaming bin: shapes at the edges of its row and slot ownership
(512 rows, 1,024 slots), of its 4 x 4 blocks and of the 16 x 16 matrix-core
tiles, more pivots than one flush, and entries whose pivots overflow."""
from __future__ import annotations

import numpy as np
import pytest

import lpgen
from solve_util import compare, crafted_batch, gpu_solve, oracle_solve

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,ty", [
    (1, 1, 1), (1, 3, 2), (3, 5, 2), (4, 4, 2), (5, 1, 2), (15, 17, 2), (16, 16, 2), (17, 33, 1), (31, 30, 2),
    (63, 65, 2), (64, 64, 2), (65, 63, 2), (100, 129, 2), (200, 201, 2), (255, 90, 2), (256, 300, 1),
    (510, 6, 2), (512, 512, 1), (512, 9, 2), (20, 1004, 2), (300, 600, 2),
    (513, 7, 2), (20, 1005, 2),  # just past the shape: the kernel that streams at every pivot
])
def test_shapes_strict(m, n, ty):
    K = 5
    hb = lpgen.make_batch(4000 + m, np.arange(K), np.full(K, ty, np.int32), np.full(K, m, np.int32),
                          np.full(K, n, np.int32))
    # up to 90 pivots (three flushes) of the large ones, to bound the oracle
    cap = 0 if m * n <= 12_000 else 90
    print(f"[pend] {m} x {n} type {ty}", flush=True)
    g = gpu_solve(hb, variant=-2, max_iter=cap)
    compare(hb, g, oracle_solve(hb, max_iter=cap), strict=True, tag=f"pend-{m}x{n}")


def test_both_streaming_kernels_in_one_batch():
    """LPs of both streaming kernels in one batch: each takes its own."""
    m = np.array([40, 513, 70, 520, 5, 512, 600], np.int32)
    n = np.array([50, 8, 1000, 12, 7, 9, 3], np.int32)
    hb = lpgen.make_batch(77, np.arange(7), np.array([2, 2, 1, 1, 2, 2, 2], np.int32), m, n)
    for mode in (0, 1, 2):
        print(f"[pend] both kernels, mode {mode}", flush=True)
        g = gpu_solve(hb, variant=-2, mode=mode)
        compare(hb, g, oracle_solve(hb), strict=True, tag=f"pend-both-{mode}")


def test_extreme_magnitudes_match_the_register_kernel():
    """Entries of wildly different magnitude: quotients outside the fast
    division's range, pivots that overflow to inf and NaN (flushed at once).
    The eager register kernel keeps the same tableau, so the bits agree."""
    import paper_1609_08114_amd as blp
    rng = np.random.default_rng(5)
    lps = []
    for t in range(120):
        m, n = int(rng.integers(2, 40)), int(rng.integers(2, 40))
        mag = (40, 160, 300)[t % 3]
        A = rng.uniform(-1, 10, size=(m, n)) * 10.0 ** rng.uniform(-mag, mag, size=(m, n))
        b = rng.uniform(1, 10, size=m) * 10.0 ** rng.uniform(-mag, mag, size=m)
        lps.append(dict(A=A, b=b, c=rng.uniform(1, 10, size=n) * 10.0 ** rng.uniform(-mag / 2, mag / 2, size=n),
                        sense=(rng.random(m) < 0.3).astype(np.int8)))
    hb = crafted_batch(lps)
    v = [x[0] for x in blp.variants()].index("b8_r160_c160")
    ref = gpu_solve(hb, variant=v, max_iter=80)
    g = gpu_solve(hb, variant=-2, max_iter=80)
    assert ref["iters"].max() > 3
    for k in ("status", "iters"):
        assert np.array_equal(ref[k], g[k]), k
    for k in ("obj", "x", "y"):
        a, b = ref[k], g[k]
        assert np.array_equal(np.isnan(a), np.isnan(b)), k
        assert np.array_equal(np.nan_to_num(a, nan=7.0), np.nan_to_num(b, nan=7.0)), k


def test_random_rule_draws_the_same_pivots():
    """The random entering rule ranks the slots in slot order, as the register
    kernels do."""
    import paper_1609_08114_amd as blp
    K = 12
    hb = lpgen.make_batch(91, np.arange(K), np.full(K, 2, np.int32), np.full(K, 60, np.int32), np.full(K, 70, np.int32))
    v = [x[0] for x in blp.variants()].index("b8_r160_c160")
    kw = dict(pivot_rule=blp.BLP_RULE_RPC, seed=11)
    a, b = gpu_solve(hb, variant=v, **kw), gpu_solve(hb, variant=-2, **kw)
    for k in ("status", "iters"):
        assert np.array_equal(a[k], b[k]), k
    for k in ("obj", "x", "y"):
        assert np.array_equal(a[k].view(np.int64), b[k].view(np.int64)), k


@pytest.mark.parametrize("m,n,K,name", [
    (33, 20, 1700, "p1_r64_s128"), (64, 64, 1700, "p1_r64_s128"), (64, 65, 1700, "b4_r112_c112"),
    (65, 63, 2600, "p2_r128_s256"), (30, 100, 2600, "p2_r128_s256"), (128, 128, 2600, "p2_r128_s256"),
    (33, 20, 1000, "w2_r64_c64"), (129, 60, 40, "p4_r256_s512"), (256, 256, 40, "p4_r256_s512"), (257, 20, 40, "streaming"),
])
def test_size_classes(m, n, K, name):
    """The automatic choice at the edges of the pending-pivot classes and of
    the batch sizes from which they come before the register tiles."""
    import paper_1609_08114_amd as blp
    hb = lpgen.make_batch(600 + m, np.arange(K), np.full(K, 2, np.int32), np.full(K, m, np.int32),
                          np.full(K, n, np.int32))
    cap = 40 if m * n > 3000 else 0
    print(f"[pend] class of {m} x {n} x {K}", flush=True)
    g = gpu_solve(hb, max_iter=cap)
    names = [v[0] for v in blp.variants()] + ["streaming"]
    assert g["bins"][names.index(name)] == K, [(a, b) for a, b in zip(names, g["bins"]) if b]
    compare(hb, g, oracle_solve(hb, max_iter=cap), strict=True, tag=name)
