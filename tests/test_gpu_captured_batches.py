"""A batch of mixed sizes captured by the caller (GPU): its classes fork inside
the capture from 2,048 LPs and run one after another below, and every replay
gives the eager bits."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [600, 2600])
def test_mixed_batch_in_a_caller_capture(count):
    import torch

    import paper_1609_08114_amd as blp
    hb = lpgen.config(5, range(count), part="simplex")
    db = blp.DeviceBatch.from_host(hb)
    e = blp.Solver()
    ref = {k: v.clone() for k, v in e.solve(db).items()}
    e.close()
    s = blp.Solver()
    out = s.solve(db)  # sizes the buffers
    torch.cuda.synchronize()
    st, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    st.wait_stream(torch.cuda.current_stream())
    print(f"[captured] {count} LPs", flush=True)
    with torch.cuda.graph(g, stream=st):
        s.solve(db, stream=st, outputs=out)
    for _ in range(3):
        for v in out.values():
            v.fill_(-7)
        torch.randn(1 << 16, device="cuda").sum().item()  # eager work between the replays
        g.replay()
        torch.cuda.synchronize()
        for k in ref:
            n = count if k in ("status", "iters", "obj") else ref[k].numel()
            assert torch.equal(out[k][:n].view(torch.int32), ref[k][:n].view(torch.int32)), k
    del g
    s.close()
