"""The four-step tile kernel (M = 2, L >= 8, no pinned launch width): against
the oracle, against the one-step kernels, and however a run is split into
calls.  The tile enumeration and the store rule of mirror mode are modelled on
the CPU."""
import numpy as np
import pytest

from oracle.run import oracle_run
from paper_1205_6872_amd import quapi as Q
from paper_1205_6872_amd import workloads as W


def _mirror(x):
    """Swap the digits 1 and 2 of every base-4 digit."""
    m = 0x5555555555555555
    return ((x & m) << 1) | ((x >> 1) & m)


def _tile_hi(idx, k):
    """The kernel's map from a tile index to (high-digit value, own mirror)."""
    def diag(x):
        return sum(3 * ((x >> b) & 1) << (2 * b) for b in range(k))
    for p in range(k - 1, -1, -1):
        cnt = 1 << (k - 1 + p)
        if idx < cnt:
            return diag(idx >> (2 * p)) << (2 * (p + 1)) | 1 << (2 * p) | (idx & ((1 << (2 * p)) - 1)), False
        idx -= cnt
    return diag(idx), True


@pytest.mark.parametrize("k", [1, 2, 3, 5])
def test_tile_index_covers_the_kept_half_once(k):
    n = (4 ** k + 2 ** k) // 2
    got = [_tile_hi(i, k) for i in range(n)]
    assert sorted(h for h, _ in got) == [h for h in range(4 ** k) if h <= _mirror(h)]
    assert all(own == (h == _mirror(h)) for h, own in got)


@pytest.mark.parametrize("k", [1, 2])
def test_tile_stores_cover_the_kept_entries_once(k):
    # outputs (m, c), flat index m + 4^(k+2) c, m = 16 hi + w: a tile below its
    # mirror stores every output, at the mirrored address when it is above its
    # mirror; a tile that is its own mirror only those not above it
    mc = 4 ** (k + 2)
    seen = np.zeros(mc * 256, dtype=int)
    for i in range((4 ** k + 2 ** k) // 2):
        hi, own = _tile_hi(i, k)
        for w in range(16):
            for c in range(256):
                m, ub, r = 16 * hi + w, c % 16, c // 16
                rm, ubm = _mirror(r), _mirror(ub)
                direct = r < rm or (r == rm and ub <= ubm)
                if own and (not direct or (r == rm and ub == ubm and w > _mirror(w))):
                    continue
                seen[m + mc * c if direct else _mirror(m) + mc * _mirror(c)] += 1
    kept = np.array([x <= _mirror(x) for x in range(seen.size)])
    assert np.array_equal(seen, kept.astype(int))


# tolerances: the library's (complex128 1e-12 of rho's scale per step; the
# complex64 tiers 1e-5 and 1e-6 absolute)
TOL = {"c128": 1e-12, "c64": 1e-5, "c64f64": 1e-6}


def _run(w, dtype, parts, mirror=1, **kw):
    with Q.create(Q.params_from(w, dtype=dtype)) as c:
        if mirror != c.mirror():
            c.set_mirror(mirror)
        rho = np.concatenate([c.propagate(k, **kw) for k in parts])
        return rho, c.read_tensor(0, c.tensor_size())


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["c128", "c64", "c64f64"])
@pytest.mark.parametrize("hermitian", [True, False])
@pytest.mark.parametrize("L", [8, 11])            # no top table digit; one
def test_tile_passes_against_oracle_and_splits(L, hermitian, dtype):
    rho0 = np.array([[0.7, 0.2 - 0.1j], [0.2 + 0.1j if hermitian else 0.4j, 0.3]])
    w = W.spin_boson_l7().with_(L=L, H=W.random_hermitian(np.random.default_rng(L), 2), xi=0.3, rho0=rho0)
    n = L + 11
    print(f"case L={L} hermitian={hermitian} {dtype}", flush=True)
    mir = 1 if hermitian else 0
    one, tens = _run(w, dtype, [n], mir)
    o = oracle_run(w, n)[1:]
    assert np.abs(one - o).max() <= TOL[dtype] * (np.abs(o).max() if dtype == "c128" else 1.0)
    # any split gives the same bits; complex64 storage with FP64 arithmetic
    # rounds at the ends of a call, so there splits at whole pairs do
    splits = [[L, 2, 4, 2, 3], [L, 6, 5]] + ([] if dtype == "c64f64" else [[L, 1, 3, 1, 1, 5], [L + 3, 8], [1] * n])
    for parts in splits:
        rho, t = _run(w, dtype, parts, mir)
        assert np.array_equal(rho, one) and np.array_equal(t, tens), parts
    last, t = _run(w, dtype, [n], mir, sel=[L + 2, L + 7])   # passes with no, one and every rho
    assert np.array_equal(last, one[[L + 1, L + 6]]) and np.array_equal(t, tens)
    if hermitian:
        # the full tensor, and the one-step kernels, to rounding
        off, t0 = _run(w, dtype, [n], 0)
        assert np.abs(off - one).max() <= {"c128": 1e-13, "c64": 1e-5, "c64f64": 1e-6}[dtype]
        assert np.abs(t0 - tens).max() <= {"c128": 1e-13, "c64": 1e-5, "c64f64": 1e-6}[dtype] * np.abs(t0).max()
        with Q.create(Q.params_from(w, dtype=dtype)) as c:
            c.set_fused_steps(1)
            assert np.abs(c.propagate(n) - one).max() <= {"c128": 1e-13, "c64": 1e-5, "c64f64": 1e-6}[dtype]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["c128", "c64", "c64f64"])
@pytest.mark.parametrize("L", [8, 11])            # the newest outer digit in the middle table; in the top one
def test_driven_tile_passes_against_oracle_and_splits(L, dtype):
    rng = np.random.default_rng(L + 20)
    n = L + 11
    H_t = np.stack([0.7 * W.random_hermitian(rng, 2) for _ in range(L + 6)])     # held past step L + 6
    rho0 = np.array([[0.7, 0.2 - 0.1j], [0.2 + 0.1j, 0.3]])
    w = W.spin_boson_l7().with_(L=L, H=H_t[0].copy(), H_t=H_t, xi=0.3, rho0=rho0)
    print(f"case driven L={L} {dtype}", flush=True)
    one, tens = _run(w, dtype, [n])
    o = oracle_run(w, n)[1:]
    assert np.abs(one - o).max() <= TOL[dtype] * (np.abs(o).max() if dtype == "c128" else 1.0)
    # one step per group: any split gives the same bits at every tier
    for parts in ([L, 1, 3, 1, 1, 5], [L + 3, 8], [1] * n):
        rho, t = _run(w, dtype, parts)
        assert np.array_equal(rho, one) and np.array_equal(t, tens), parts
    last, t = _run(w, dtype, [n], sel=[n])
    assert np.array_equal(last, one[[n - 1]]) and np.array_equal(t, tens)
    if dtype != "c64":      # one Hamiltonian at every step is the static system (FP32 rounds its pairs otherwise)
        ws = w.with_(H_t=None)
        wd = w.with_(H_t=np.stack([w.H] * 3))
        d = np.abs(_run(ws, dtype, [n])[0] - _run(wd, dtype, [n])[0]).max()
        assert d == 0.0 if dtype == "c128" else d <= 1e-6
