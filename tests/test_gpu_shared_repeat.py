"""Repeated shared-constraint solves (GPU): the warm starts run along chunks of
objectives, more of them than workgroups, and equal calls give the same bits."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,count,turns", [(100, 100, 10_000, 1 / 18), (100, 100, 50_000, 1.0), (36, 78, 5_000, 1.0),
                                             (20, 15, 30_000, 1 / 40)])
def test_equal_calls_give_equal_bits(m, n, count, turns):
    import torch

    import paper_1609_08114_amd as blp
    hb = lpgen.make_batch(60 + m, [0], np.ones(1, np.int32), np.array([m], np.int32), np.array([n], np.int32))
    lp = hb.lp(0)
    A, b, sense = (torch.from_numpy(np.ascontiguousarray(lp[k])).cuda() for k in ("A", "b", "sense"))
    u, v = np.random.default_rng(m).normal(size=(2, n))
    t = np.arange(count)[:, None] * (turns * 2 * np.pi / count)
    C = torch.from_numpy(np.cos(t) * u + np.sin(t) * v).cuda()
    g = torch.rand(count, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    print(f"[shared repeat] {count} objectives on {m} x {n}", flush=True)
    s = blp.Solver()
    first = None
    for rep in range(6):
        out = s.solve_shared(A, b, sense, C)
        out.update(s.backward_shared(out, m, n, g))
        out = {k: w.clone().view(torch.int32) for k, w in out.items()}
        first = first or out
        for k, w in out.items():
            assert torch.equal(w, first[k]), (rep, k)
    s.close()
    assert not torch.any(first["status"])


def test_infeasible_constraints():
    """Phase 1 ends every objective: also then the outputs do not depend on who took which chunk."""
    import torch

    import paper_1609_08114_amd as blp
    m, n, count = 12, 9, 9_000
    rng = np.random.default_rng(4)
    A = torch.from_numpy(rng.uniform(1, 2, size=(m, n))).cuda()
    b = torch.from_numpy(np.where(np.arange(m) < m // 2, 1.0, 50.0)).cuda()
    sense = torch.from_numpy((np.arange(m) >= m // 2).astype(np.int8)).cuda()
    t = np.arange(count)[:, None] * 1e-4
    C = torch.from_numpy(np.cos(t) * rng.normal(size=n) + np.sin(t) * rng.normal(size=n)).cuda()
    s = blp.Solver()
    first = None
    for rep in range(6):
        out = {k: w.clone().view(torch.int32) for k, w in s.solve_shared(A, b, sense, C).items()}
        first = first or out
        for k, w in out.items():
            assert torch.equal(w, first[k]), (rep, k)
    s.close()
    assert torch.all(first["status"] == 1)
