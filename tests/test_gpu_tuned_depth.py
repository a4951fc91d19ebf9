"""The autotuner chooses the streaming kernel's loads in flight from the LPs
that this kernel gets (GPU); where the pending-pivot kernel takes all streamed
LPs, the depth stays what it is untuned (deep: no tile holds them)."""
import json

import numpy as np
import pytest

import lpgen
import oracle
from solve_util import compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,own", [([257] * 9, [3] * 9, False), ([300] * 20, [40] * 20, False), ([260] * 6, [5] * 6, False),
                                     ([300] * 20 + [600] * 3, [40] * 20 + [7] * 3, True)])
def test_depth_from_its_own_lps(m, n, own, tmp_path):
    import torch

    import paper_1609_08114_amd as blp
    K = len(m)
    hb = lpgen.make_batch(17, np.arange(K), np.full(K, 2, np.int32), np.array(m, np.int32), np.array(n, np.int32))
    db = blp.DeviceBatch.from_host(hb, uniform=False)
    s = blp.Solver()
    path = str(tmp_path / "tuned.json")
    print(f"[tuned depth] {K} LPs", flush=True)
    s.autotune(db, sample=8, cache_path=path)
    deep = json.load(open(path))["streaming_deep"]
    assert deep in (0, 1) and (own or deep == 1)
    out = s.solve(db)
    torch.cuda.synchronize()
    g = {k: v.cpu().numpy() for k, v in out.items()}
    compare(hb, g, oracle.solve_batch(hb), strict=True, tag="tuned")
    s.close()


def test_no_time_on_lps_of_the_other_kernel():
    """Nothing to choose: the tuner runs no solve of the streamed LPs (it ran
    four, each some ten times as long as their solve)."""
    import time

    import torch

    import paper_1609_08114_amd as blp
    K = 40
    hb = lpgen.make_batch(18, np.arange(K), np.full(K, 2, np.int32), np.full(K, 270, np.int32), np.full(K, 200, np.int32))
    db = blp.DeviceBatch.from_host(hb, uniform=False)
    s = blp.Solver()
    s.autotune(db, sample=2)  # sizes the buffers
    s.solve(db)
    times = []
    for call in (lambda: s.solve(db), lambda: s.autotune(db, sample=K)):
        torch.cuda.synchronize()
        t = time.perf_counter()
        call()
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t)
    print(f"[tuned depth] solve {times[0]:.4f} s, tuner {times[1]:.4f} s", flush=True)
    assert times[1] < 4 * times[0]
    s.close()
