"""A batch of every memory length of the persistent path (M = 2): the contexts
below L = 5 run in the launch of the others' full-window steps."""
import numpy as np
import pytest

from paper_1205_6872_amd import quapi as Q
from paper_1205_6872_amd import workloads as W


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["c128", "c64", "c64f64"])
@pytest.mark.parametrize("Ls", [(1, 2, 3, 4, 5), (4, 6), (3, 4, 5, 6, 7)])
def test_batch_of_mixed_lengths_equals_its_own_calls(Ls, dtype):
    import torch
    w = W.spin_boson_l7().with_(H=W.random_hermitian(np.random.default_rng(3), 2), xi=0.3,
                                rho0=np.array([[0.7, 0.2 - 0.1j], [0.2 + 0.1j, 0.3]]))
    ws = [w.with_(L=Ls[k % len(Ls)], kT=0.1 + 0.02 * k) for k in range(35)]       # two launches' worth
    parts = [[x.L + 1 + k % 5, 1 + k % 3, 0 if k % 4 == 0 else 9] for k, x in enumerate(ws)]
    modes = [k % 3 for k in range(35)]
    print(f"case Ls={Ls} {dtype}", flush=True)
    ctxs = [Q.create(Q.params_from(x, dtype=dtype)) for x in ws]
    own = [Q.create(Q.params_from(x, dtype=dtype)) for x in ws]
    try:
        for call in range(3):
            n = [p[call] for p in parts]
            outs = [torch.zeros((max(1, k), 4, 2), dtype=torch.float64, device="cuda:0") for k in n]
            torch.cuda.synchronize()
            Q.propagate_batch(ctxs, n, modes, [b.data_ptr() for b in outs])
            torch.cuda.synchronize()
            for c, o, k, mode, b in zip(ctxs, own, n, modes, outs):
                sel = [None, None, [o.step_count() + k]][mode] if k else []
                want = o.propagate(k, sel=[] if mode == 0 else sel)
                got = b.cpu().numpy().view(np.complex128).reshape(-1, 2, 2)[:len(want)]
                assert np.array_equal(got, want), (c.L, k, mode)
        for c, o in zip(ctxs, own):
            assert np.array_equal(c.read_tensor(0, c.tensor_size()), o.read_tensor(0, o.tensor_size())), c.L
    finally:
        for c in ctxs + own:
            c.destroy()
