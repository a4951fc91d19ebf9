"""A shared-constraint solve whose count and shape do not exceed an earlier
one's allocates nothing (GPU): captured across the number of objectives and
the shapes at which the route and its tile change."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu


def _set(m, n):
    import torch
    hb = lpgen.make_batch(970 + m, [0], np.ones(1, np.int32), np.array([m], np.int32), np.array([n], np.int32))
    lp = hb.lp(0)
    return [torch.from_numpy(np.ascontiguousarray(lp[k])).cuda() for k in ("A", "b", "sense")]


@pytest.mark.parametrize("large,small", [
    ((96, 96, 2600), (96, 96, 2500)), ((112, 100, 2600), (112, 100, 2559)),  # the class, then the streaming route
    ((129, 129, 800), (128, 128, 800)),                                      # a tile with more workgroups
    ((30, 120, 2000), (30, 60, 2000)),                                       # a register tile, then the class
])
def test_no_larger_call_in_a_capture(large, small):
    import torch

    import paper_1609_08114_amd as blp
    rng = np.random.default_rng(7)
    Cl, Cs = (torch.from_numpy(rng.normal(size=(c, n))).cuda() for _, n, c in (large, small))
    L, S = _set(*large[:2]), _set(*small[:2])
    print(f"[shared workspace] {large} then {small}", flush=True)
    sv = blp.Solver()
    eager = {k: v.clone() for k, v in sv.solve_shared(*S, Cs).items()}
    sv.close()
    sv = blp.Solver()
    sv.solve_shared(*L, Cl)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    st, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    st.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(g, stream=st):
        out = sv.solve_shared(*S, Cs, stream=st)
    for _ in range(3):
        for v in out.values():
            v.fill_(-7)
        sv.solve_shared(*S, Cs)  # eager work on the same handle between the replays
        g.replay()
        torch.cuda.synchronize()
        for k in eager:
            assert torch.equal(torch.nan_to_num(out[k]), torch.nan_to_num(eager[k])), k
    assert free - torch.cuda.mem_get_info()[0] < 64 << 20  # (results and the graph, no workspace)
    del g
    sv.close()
