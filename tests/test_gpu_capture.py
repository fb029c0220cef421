"""A call recorded into a caller's graph leaves the context as the call does:
nothing that later calls read is put off to the graph's replay."""
import numpy as np
import pytest

from paper_1205_6872_amd import quapi as Q
from paper_1205_6872_amd import workloads as W


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["c128", "c64", "c64f64"])
@pytest.mark.parametrize("L", [4, 5, 6, 7])
def test_eager_call_after_a_recorded_first_call(L, dtype):
    # the persistent path: the context's first call is recorded, the graph is
    # dropped, and the state restored; the eager call gives a fresh context's bits
    import torch
    w = W.spin_boson_l7().with_(L=L)
    p = Q.params_from(w, dtype=dtype)
    n = 2 * (L + 3)
    with Q.create(p) as c:
        want = c.propagate(n)
    nbytes = Q.footprint(p)
    ws = torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda:0")      # NaN where nothing is written
    out = torch.zeros((n, 4, 2), dtype=torch.float64, device="cuda:0")
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    with Q.create(p, stream=st.cuda_stream, workspace=ws.data_ptr(), ws_bytes=nbytes) as c:
        state = c.checkpoint()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st, capture_error_mode="thread_local"):
            c.propagate_async(n, None, out.data_ptr())
        del g
        c.restore(*state)
        got = c.propagate(n)
    assert np.array_equal(got, want)
