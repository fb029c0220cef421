"""complex64 with FP32 arithmetic, M = 2: what a step rounds.

A state with one entry that is not zero gives an off-diagonal rho of one term,
factor * row coefficient * entry.  The coefficient of the oldest point is held in
FP32 and its product with the entry is rounded in FP32; the factor and the term
are FP64.  With unit roundoff u = 2^-24 a term's relative error is then at most
3 u (coefficient, product, and the sum of the two real products of a component),
and an error uniform in +-u 2^e has an rms of 0.42 u relative to values spread
evenly over a binade's logarithm, sqrt(3) 0.42 u = 0.73 u for the three.  A factor
rounded in parts and multiplied in FP32 brings about nine more of them, 1.45 u.
The line between is drawn at 1.0 u."""
import numpy as np
import pytest

from paper_1205_6872_amd import quapi as Q
from paper_1205_6872_amd import workloads as W

U32 = 2.0 ** -24


@pytest.mark.gpu
@pytest.mark.parametrize("L,driven", [(5, False), (7, False), (8, False), (11, False), (8, True)])
def test_offdiagonal_rho_terms_round_the_row_only(L, driven):
    rng = np.random.default_rng(L)
    H = W.random_hermitian(rng, 2)
    w = W.spin_boson_l7().with_(L=L, H=H, xi=0.3, rho0=np.array([[0.7, 0.4j], [0.2, 0.3]]))
    if driven:
        w = w.with_(H_t=np.stack([H + 0.1 * k * np.array([[0, 1], [1, 0]]) for k in range(2 * L)]))
    n_ent = 4 ** L
    rel = []
    with Q.create(Q.params_from(w, dtype="c64")) as c32, Q.create(Q.params_from(w, dtype="c128")) as c64:
        assert c32.mirror() == 0 and c64.mirror() == 0         # one entry has no mirror
        for k in range(60):
            step = L + k % 4                                    # every place in a group
            t = np.zeros(n_ent, dtype=np.complex128)
            t[rng.integers(n_ent)] = complex(np.complex64(rng.normal() + 1j * rng.normal()))
            rho = []
            for c in (c32, c64):
                c.restore(step, t)
                rho.append(c.propagate(1)[0])
            for a, b in ((0, 1), (1, 0)):
                rel.append(abs(rho[0][a, b] - rho[1][a, b]) / abs(rho[1][a, b]))
    rel = np.array(rel) / U32
    print(f"L={L} driven={driven}: rms {np.sqrt((rel ** 2).mean()):.2f} u, max {rel.max():.2f} u", flush=True)
    assert rel.max() <= 3.0
    assert np.sqrt((rel ** 2).mean()) <= 1.0
