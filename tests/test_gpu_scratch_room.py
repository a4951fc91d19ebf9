"""The allocation-free entry point where the scratch has room for one workspace
slot of the kernel that streams at every pivot, but not for one of the
pending-pivot kernel (GPU): the batch is solved, with the bits of
blp_solve_batch."""
import ctypes

import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu


def test_room_for_the_smaller_slot_only():
    import torch

    import paper_1609_08114_amd as blp
    room = 3 << 20
    # the largest slots: 512 x 511 doubles (500 x 10), and 512 x 908 for the rows of one and the columns of the other
    assert 512 * 511 * 8 < room - 65536 and room < 512 * 908 * 8
    K = (blp.blp_static_scratch_bytes() - room) // 48
    m, n = np.ones(K, np.int32), np.ones(K, np.int32)
    m[100], n[100], m[7000], n[7000] = 500, 10, 5, 900
    hb = lpgen.make_batch(5, np.arange(K), np.ones(K, np.int32), m, n)
    db = blp.DeviceBatch.from_host(hb, uniform=False)
    s = blp.Solver()
    print(f"[scratch room] {K} LPs", flush=True)
    ref = s.solve(db)
    got = {k: torch.full_like(v, -7) for k, v in ref.items()}
    o = blp.blp_outputs(*[ctypes.c_void_p(got[k].data_ptr()) for k in ("status", "iters", "obj", "x", "y")])
    st = db.c_struct()
    blp.blp_solve_batch_static(s.h, st, o, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    for k in ref:
        assert torch.equal(ref[k].view(torch.int32), got[k].view(torch.int32)), k
    assert blp.blp_last_bins(s.h)[len(blp.variants())] == 2
    s.close()
