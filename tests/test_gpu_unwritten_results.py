"""Results without entries (GPU): y of a batch without rows, the sums over no
objectives.  No kernel writes them, so they must not hold what the allocator's
last owner left there."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu


def _leave_nan(dev):
    """Freed blocks of the allocator's smallest sizes that hold NaN."""
    import torch
    t = [torch.full((n,), float("nan"), dtype=torch.float64, device=dev) for n in (1, 6, 42, 512, 4096) for _ in range(12)]
    torch.cuda.synchronize()
    del t


@pytest.mark.parametrize("uniform", [True, False])
def test_y_of_boxes(uniform):
    import torch

    import paper_1609_08114_amd as blp
    db = blp.DeviceBatch.from_host(lpgen.config(5, range(70), part="box28"), uniform=uniform)
    s = blp.Solver()
    for stream in (None, None, torch.cuda.Stream()):
        _leave_nan("cuda")
        out = s.solve(db, stream=stream)
        torch.cuda.synchronize()
        assert out["y"].shape == (1,) and out["y"].item() == 0.0
    s.close()


def test_no_objectives():
    import torch

    import paper_1609_08114_amd as blp
    dev = torch.device("cuda")
    lp = lpgen.config(1, [0]).lp(0)
    A, b, sense = (torch.from_numpy(np.ascontiguousarray(lp[k])).to(dev) for k in ("A", "b", "sense"))
    m, n = lp["A"].shape
    s = blp.Solver()
    _leave_nan(dev)
    out = s.solve_shared(A, b, sense, torch.empty(0, n, dtype=torch.float64, device=dev))
    grad = s.backward_shared(out, m, n, torch.empty(0, dtype=torch.float64, device=dev))
    torch.cuda.synchronize()
    for k, v in {**out, **grad}.items():
        assert not v.any(), k
    s.close()
