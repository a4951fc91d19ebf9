"""Gradient tensors that blp_backward fills get no zeros first; every other
one does (GPU).  The allocator's memory holds NaN before each call."""
import pytest

import lpgen

pytestmark = pytest.mark.gpu


def _batch(blp, torch, case):
    if case == "uniform":
        hb = lpgen.config(2, range(40))
        return blp.DeviceBatch.from_host(hb, uniform=True)
    if case == "uniform longer":  # the data tensors go on past the batch
        db = blp.DeviceBatch.from_host(lpgen.config(2, range(40)), uniform=True)
        for k in ("A", "b", "sense", "c"):
            t = getattr(db, k)
            setattr(db, k, torch.cat([t, torch.ones(7, dtype=t.dtype, device=t.device)]))
        return db
    if case == "box":
        return blp.DeviceBatch.from_host(lpgen.config(5, range(300), part="box5"), uniform=True)
    if case == "sizes":
        hb = lpgen.config(5, range(60), part="simplex")
        assert hb.A.size >= 4096 * hb.count  # the offsets are looked at
        return blp.DeviceBatch.from_host(hb, uniform=False)
    if case == "sizes with a gap":
        db = blp.DeviceBatch.from_host(lpgen.config(5, range(60), part="simplex"), uniform=False)
        for k, off, at in (("A", "a_off", 3), ("c", "col_off", 5), ("b", "row_off", 59)):
            o, t = getattr(db, off).copy(), getattr(db, k)
            cut = int(o[at])
            o[at:] += 11
            setattr(db, off, o)
            ext = [t[:cut], torch.ones(11, dtype=t.dtype, device=t.device), t[cut:]]
            setattr(db, k, torch.cat(ext))
            if k == "b":
                db.sense = torch.cat([db.sense[:cut], torch.zeros(11, dtype=torch.int8, device="cuda"), db.sense[cut:]])
        return db
    return blp.DeviceBatch.from_host(lpgen.config(4, range(200)), uniform=False)  # hyperboxes among them


@pytest.mark.parametrize("case", ["uniform", "uniform longer", "box", "sizes", "sizes with a gap", "mixed"])
def test_unwritten_elements_are_zero(case):
    import torch

    import paper_1609_08114_amd as blp
    db = _batch(blp, torch, case)
    s = blp.Solver()
    out = s.solve(db)
    g = torch.linspace(0.5, 1.5, db.count, dtype=torch.float64, device="cuda")
    keys = [k for k, t in (("dc", db.c), ("db", db.b), ("dA", db.A), ("dl", db.l), ("du", db.u)) if t is not None]
    src = {"dc": db.c, "db": db.b, "dA": db.A, "dl": db.l, "du": db.u}
    want = {k: torch.zeros_like(src[k]) for k in keys}
    blp.blp_backward(s.h, blp._ptr(g), *[blp._ptr(want.get(k)) for k in ("dc", "db", "dA", "dl", "du")],
                     torch.cuda.current_stream().cuda_stream)
    for k in keys:  # leave NaN where the allocator will take the gradients from
        torch.full_like(src[k], float("nan"))
    got = s.backward(g, want=keys)
    torch.cuda.synchronize()
    assert bool((out["status"][:db.count] == 0).any())
    for k in keys:
        assert torch.equal(got[k], want[k]), k
    s.close()


def test_which_gradients_get_no_zeros():
    import torch

    import paper_1609_08114_amd as blp
    fills = {case: [k for k in ("dc", "db", "dA", "dl", "du")
                    if (t := {"dc": "c", "db": "b", "dA": "A", "dl": "l", "du": "u"}[k])
                    and getattr(db, t) is not None and blp._backward_fills(db, k, getattr(db, t))]
             for case in ("uniform", "uniform longer", "box", "sizes", "sizes with a gap", "mixed")
             for db in [_batch(blp, torch, case)]}
    assert fills == {"uniform": ["dc", "db", "dA"], "uniform longer": [], "box": ["dc", "dl", "du"],
                     "sizes": ["dA"], "sizes with a gap": [], "mixed": []}
