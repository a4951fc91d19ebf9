"""Which class takes an LP goes by how many LPs run at a time (GPU): one in the
one-LP-per-launch mode, the workgroups of a launch in the grid mode, and few in
a batch of few LPs, whatever the batch's count."""
import numpy as np
import pytest

import lpgen
from solve_util import compare, gpu_solve, oracle_solve

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,ty,m,n,K,name", [
    (2, 1, 100, 100, 2600, "b4_r112_c112"), (2, 2, 47, 61, 1700, "b4_r112_c112"), (2, 2, 120, 60, 600, "b8_r128_c128"),
    (2, 2, 129, 60, 40, "b8_r160_c160"), (2, 2, 150, 100, 20, "p4_r256_s512"),  # (no tile holds the last)
    (1, 1, 100, 100, 2600, "b4_r112_c112"), (1, 1, 30, 30, 9000, "w1_r32_c32"), (1, 2, 47, 61, 1700, "p1_r64_s128"),
    (1, 2, 120, 60, 600, "p2_r128_s256"),
    (0, 2, 120, 60, 1, "b8_r128_c128"), (0, 2, 120, 60, 256, "b8_r128_c128"), (0, 2, 120, 60, 257, "p2_r128_s256"),
    (0, 2, 129, 60, 31, "b8_r160_c160"), (0, 2, 129, 60, 32, "p4_r256_s512"),
])
def test_class_by_mode_and_count(mode, ty, m, n, K, name):
    import paper_1609_08114_amd as blp
    hb = lpgen.make_batch(640 + m, np.arange(K), np.full(K, ty, np.int32), np.full(K, m, np.int32), np.full(K, n, np.int32))
    cap = 30 if m * n > 3000 else 0
    print(f"[class lines] mode {mode}, {K} of {m} x {n}", flush=True)
    g = gpu_solve(hb, mode=mode, max_iter=cap)
    names = [v[0] for v in blp.variants()] + ["streaming"]
    assert g["bins"][names.index(name)] == K, [(a, b) for a, b in zip(names, g["bins"]) if b]
    compare(hb, g, oracle_solve(hb, max_iter=cap), strict=True, tag=f"{name} mode {mode}")
