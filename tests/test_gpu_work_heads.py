"""The sharded work-list heads (GPU): every LP of a batch is taken exactly
once, whatever the number of workgroups and LPs."""
import numpy as np
import pytest

import lpgen
import oracle
from solve_util import compare, gpu_solve, oracle_solve

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", ["w1_r16_c16", "l64_r8_c8", "b4_r112_c112", "p1_r64_s128", "streaming"])
@pytest.mark.parametrize("count", [1, 7, 255, 257, 2049])
def test_every_lp_once(variant, count):
    """256 workgroups: fewer LPs than heads, than workgroups, one more, many."""
    import torch

    import paper_1609_08114_amd as blp
    names = [v[0] for v in blp.variants()]
    hb = lpgen.config(1, range(count))
    ref = oracle.solve_batch(hb)
    s = blp.Solver(variant=-2 if variant == "streaming" else names.index(variant), workers_per_cu=1)
    db = blp.DeviceBatch.from_host(hb)
    out = s.solve(db)
    for t in out.values():  # whatever is not written again shows
        t.fill_(-7)
    s.solve(db, outputs=out)
    torch.cuda.synchronize()
    assert np.array_equal(out["status"][:count].cpu().numpy(), ref["status"])
    assert np.array_equal(out["iters"][:count].cpu().numpy(), ref["iters"])
    assert np.array_equal(out["obj"][:count].cpu().numpy(), ref["obj"])
    s.close()


@pytest.mark.parametrize("ty,m,n,count,name", [
    (1, 6, 6, 17_000, "l64_r8_c8"),     # the class depends on the artificial rows: binned
    (2, 20, 20, 8_300, "p1_r64_s128"),  # one class whatever their number, from 32 LPs per CU
    (1, 20, 20, 8_100, "w1_r32_c32"),
    (2, 70, 40, 2_600, "p2_r128_s256"),
])
def test_uniform_batches_and_binning(ty, m, n, count, name):
    import paper_1609_08114_amd as blp
    hb = lpgen.make_batch(700 + m, np.arange(count), np.full(count, ty, np.int32), np.full(count, m, np.int32),
                          np.full(count, n, np.int32))
    names = [v[0] for v in blp.variants()]
    print(f"[heads] {count} of {m} x {n}", flush=True)
    for kw in ({}, {"graph": True}, {"layout": 1}):
        g = gpu_solve(hb, **kw)
        assert g["bins"][names.index(name)] == count, (kw, [(a, b) for a, b in zip(names, g["bins"]) if b])
        compare(hb, g, oracle_solve(hb), strict=True, tag=f"{name} {kw}")


@pytest.mark.parametrize("count", [900, 9_000])
def test_autotune_of_a_uniform_batch(count):
    """The tuner launches every class, also where a solve would take one
    launch without binning."""
    import torch

    import paper_1609_08114_amd as blp
    hb = lpgen.make_batch(31, np.arange(count), np.full(count, 2, np.int32), np.full(count, 20, np.int32),
                          np.full(count, 20, np.int32))
    s = blp.Solver()
    db = blp.DeviceBatch.from_host(hb)
    s.autotune(db, sample=64)
    out = s.solve(db)
    torch.cuda.synchronize()
    assert np.array_equal(out["obj"][:count].cpu().numpy(), oracle.solve_batch(hb)["obj"])
    s.close()


@pytest.mark.parametrize("m,n,count", [(1, 1, 20_000), (5, 5, 150_001), (6, 6, 17_000), (8, 20, 9_000), (9, 3, 9_001),
                                       (31, 10, 7_000), (32, 10, 7_000), (33, 10, 7_000)])
def test_classification_of_small_rows(m, n, count):
    """One LP per lane up to 32 rows, around the groups of 8 rows: the same
    bins as the batch classified LP by LP."""
    hb = lpgen.make_batch(800 + m, np.arange(count), np.where(np.arange(count) % 3 == 0, 1, 2).astype(np.int32),
                          np.full(count, m, np.int32), np.full(count, n, np.int32))
    print(f"[heads] classify {count} of {m} x {n}", flush=True)
    a, b = gpu_solve(hb, uniform=True, mode=1), gpu_solve(hb, uniform=False, mode=1)
    assert np.array_equal(a["bins"], b["bins"])
    assert np.array_equal(a["obj"], b["obj"]) and np.array_equal(a["iters"], b["iters"])
