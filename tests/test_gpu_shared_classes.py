"""The cold solves of a shared constraint set in a pending-pivot class (GPU):
the bits of the same LPs solved as a batch, on both sides of the number of
objectives from which the class is taken, and a smaller call allocates nothing
after a larger one."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu


def _set(ty, m, n, seed):
    hb = lpgen.make_batch(seed, [0], np.array([ty], np.int32), np.array([m], np.int32), np.array([n], np.int32))
    return hb.lp(0)


@pytest.mark.parametrize("ty,m,n,count", [(1, 40, 30, 1535), (1, 40, 30, 1536), (2, 60, 50, 1700), (1, 100, 100, 2600),
                                          (2, 100, 90, 2559), (2, 100, 90, 2600)])
def test_cold_solves(ty, m, n, count):
    import torch

    import paper_1609_08114_amd as blp
    lp = _set(ty, m, n, 900 + m)
    C = np.random.default_rng(count).normal(size=(count, n))
    A, b, s = (torch.from_numpy(np.ascontiguousarray(lp[k])).cuda() for k in ("A", "b", "sense"))
    Cd = torch.from_numpy(C).cuda()
    sv = blp.Solver()
    print(f"[shared classes] {count} objectives on {m} x {n}", flush=True)
    got = sv.solve_shared(A, b, s, Cd)
    db = blp.DeviceBatch(m=np.full(count, m, np.int32), n=np.full(count, n, np.int32), kind=np.zeros(count, np.int32),
                         a_off=np.arange(count) * m * n, row_off=np.arange(count) * m, col_off=np.arange(count) * n,
                         A=A.reshape(-1).repeat(count), b=b.repeat(count), sense=s.repeat(count), c=Cd.reshape(-1),
                         l=None, u=None, uniform=True)
    db._count = count
    ref = sv.solve(db)
    torch.cuda.synchronize()
    for k in ("status", "iters", "obj", "x", "y"):
        a, r = got[k].reshape(-1), ref[k].reshape(-1)
        assert torch.equal(a.isnan(), r.isnan()) and torch.equal(torch.nan_to_num(a), torch.nan_to_num(r)), k
    sv.close()


@pytest.mark.parametrize("m,n,large,small", [(40, 30, 3073, 3072), (100, 100, 2600, 2560), (130, 60, 769, 768)])
def test_smaller_call_in_a_capture(m, n, large, small):
    """Fewer LPs may run more workgroups per CU (whole rounds): the workspace
    of the larger call still holds them."""
    import torch

    import paper_1609_08114_amd as blp
    lp = _set(1, m, n, 950 + m)
    A, b, s = (torch.from_numpy(np.ascontiguousarray(lp[k])).cuda() for k in ("A", "b", "sense"))
    C = torch.from_numpy(np.random.default_rng(3).normal(size=(large, n))).cuda()
    sv = blp.Solver()
    sv.solve_shared(A, b, s, C)
    eager = {k: v.clone() for k, v in sv.solve_shared(A, b, s, C[:small].contiguous()).items()}
    sv.close()
    sv = blp.Solver()
    sv.solve_shared(A, b, s, C)
    torch.cuda.synchronize()
    Cs, st, g = C[:small].contiguous(), torch.cuda.Stream(), torch.cuda.CUDAGraph()
    st.wait_stream(torch.cuda.current_stream())
    print(f"[shared classes] capture {small} after {large}, {m} x {n}", flush=True)
    with torch.cuda.graph(g, stream=st):
        out = sv.solve_shared(A, b, s, Cs, stream=st)
    for _ in range(3):
        for v in out.values():
            v.zero_()
        g.replay()
        torch.cuda.synchronize()
        for k in eager:
            assert torch.equal(torch.nan_to_num(out[k]), torch.nan_to_num(eager[k])), k
    del g
    sv.close()
