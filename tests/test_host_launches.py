"""The launches of the library's host code, on the CPU: the library runs in a
process of its own on a HIP runtime that only logs kernel names
(tests/fake_hip.c); no kernel runs, so nothing here looks at values."""
import os
import subprocess
import sys
import textwrap
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent
LIB = ROOT / "paper_1205_6872_amd" / "_lib" / "libquapi.so"


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    """run(code): code as a program with `Q`, `W`, `np`, launched(call) -- the
    kernels that call() launches, as (name, blocks, threads) -- and fake, the
    runtime."""
    d = tmp_path_factory.mktemp("fake_hip")
    (d / "v.map").write_text("hip_4.2 { global: *; };\nhip_4.3 { global: hipGraph*; hipStreamBeginCapture; "
                             "hipStreamEndCapture; } hip_4.2;\n")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", str(d / "libamdhip64.so.7"), "-Wl,-soname,libamdhip64.so.7",
                    f"-Wl,--version-script={d / 'v.map'}", str(ROOT / "tests" / "fake_hip.c")], check=True)
    head = textwrap.dedent(f"""
        import ctypes, re, sys
        import numpy as np
        sys.path.insert(0, {str(ROOT)!r})
        fake = ctypes.CDLL({str(d / 'libamdhip64.so.7')!r})
        fake.fake_log.restype = ctypes.c_char_p
        from paper_1205_6872_amd import quapi as Q, workloads as W
        def short(name):
            m = re.match(r"_ZN5quapi(?:12_GLOBAL__N_1)?(\\d+)", name)
            k = int(m.group(1))
            return name[m.end():m.end() + k]
        def launched(call):
            fake.fake_reset()
            call()
            return [(short(l.split()[0]), int(l.split()[1]), int(l.split()[2]))
                    for l in fake.fake_log().decode().splitlines()]
        def names(call):
            return [n for n, _, _ in launched(call)]
        """)

    def go(code):
        if not LIB.exists():
            pytest.skip("the library is not built")
        env = dict(os.environ, LD_LIBRARY_PATH=str(d))
        r = subprocess.run([sys.executable, "-c", head + textwrap.dedent(code)], env=env, capture_output=True,
                           text=True, timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr
    return go


def test_first_call_launches_what_later_calls_launch(run):
    # the persistent path: everything a call needs beyond its own kernels is
    # formed at create (a batch of fresh contexts, as the server's, would pay for
    # it context by context)
    run("""
        for L in range(2, 8):
            w = W.spin_boson_l7().with_(L=L)
            ctxs = [Q.create(Q.params_from(w, dtype="c64")) for _ in range(24)]
            buf = np.zeros((24, 40, 8))
            call = lambda: Q.propagate_batch(ctxs, [30] * 24, [1] * 24, [b.ctypes.data for b in buf])
            first = names(call)
            assert set(first) <= {"small_kernel", "small_reg_kernel"} and len(first) <= 2, (L, first)
            with Q.create(Q.params_from(w)) as c:
                assert set(names(lambda: c.propagate(L + 9))) <= {"small_kernel", "small_reg_kernel"}
        """)


def test_mixed_batch_is_one_launch_after_the_growth_steps(run):
    # contexts of every memory length side by side: the growth steps (a launch for
    # each of the persistent path's two modes), then one launch for all the rest
    run("""
        for Ls in ((5, 6), (4, 5), (1, 2, 3, 4, 5, 6), (6, 7), (2, 4, 5, 6, 7)):
            ctxs = [Q.create(Q.params_from(W.spin_boson_l7().with_(L=Ls[k % len(Ls)]))) for k in range(24)]
            n = [30] * 23 + [0]
            buf = np.zeros((24, 30, 8))
            call = lambda: Q.propagate_batch(ctxs, n, [1] * 24, [b.ctypes.data for b in buf])
            got = launched(call)
            assert [g[0] for g in got] == ["small_kernel"] * (1 + (7 in Ls)) + ["small_reg_kernel"], (Ls, got)
            assert got[-1][1] == 23
            assert names(call) == ["small_reg_kernel"]                   # past the growth steps
        # one length, or none that keeps its tensor in registers: as it was
        for Ls in ((4,), (3, 4)):
            ctxs = [Q.create(Q.params_from(W.spin_boson_l7().with_(L=Ls[k % len(Ls)]))) for k in range(40)]
            buf = np.zeros((40, 30, 8))
            got = launched(lambda: Q.propagate_batch(ctxs, [30] * 40, [1] * 40, [b.ctypes.data for b in buf]))
            assert [g[:2] for g in got] == [("small_kernel", 32), ("small_kernel", 8)], got
        """)


@pytest.mark.parametrize("M,L", [(3, 7), (2, 8)])        # rho left to the next step's launch; to the next pass
def test_a_failed_call_leaves_no_rho_to_later_ones(run, M, L):
    # launches fail from the n-th of a call on: no sum of its rho runs after it
    run(f"""
        M, L = {M}, {L}
        w = W.spin_boson_l7().with_(M=M, L=L, s=np.linspace(-1, 1, M), H=np.diag(np.arange(1.0, M + 1)),
                                    rho0=np.eye(M) / M, H_t=np.stack([np.diag(np.arange(1.0, M + 1))] * 3))
        rho0 = np.zeros(M * M, dtype=complex)
        sums = lambda ns: [n for n in ns if n.startswith(("rho_", "tile_rho"))]
        with Q.create(Q.params_from(w)) as c:
            total = len(names(lambda: c.propagate(L + 6)))
        for n in range(total):
            with Q.create(Q.params_from(w)) as c:
                fake.fake_fail_after(n)
                try:
                    c.propagate(L + 6)
                    raise SystemExit("the call did not fail")
                except Q.QuapiError as e:
                    assert e.status == Q.ERR_DEVICE
                fake.fake_fail_after(-1)
                assert not sums(names(lambda: (c.restore(0, rho0), c.read_tensor(0, 1)))), n
                got = launched(lambda: c.propagate(L + 6))
                assert all(b in (M * M, 256, 1, 2, 3, 4) for k, b, _ in got if k.startswith(("rho_", "tile_rho")))
        """)


def test_static_calls_at_the_limit_of_their_scratch(run):
    # 64 MiB without the four-step kernel's tables and rho rows and the
    # quadrature's parts: the longest stacks of Hamiltonians that are taken
    run("""
        for M, L, dtype, most in ((2, 10, "c128", 254604), (2, 10, "c64", 385624), (2, 8, "c128", 505940),
                                  (2, 6, "c64", 522144), (2, 3, "c128", 523348), (3, 6, "c128", 170739),
                                  (4, 4, "c64", 127134), (4, 5, "c128", 63706)):
            for n, taken in ((most, True), (most + 1, False)):
                p = Q.params(M=M, s=np.arange(M), H=np.eye(M), rho0=np.eye(M) / M, kT=0.2, dt=0.1, L=L, dtype=dtype,
                             xi=0.1, omega_c=5.0, H_t=np.broadcast_to(np.eye(M), (n, M, M)))
                try:
                    Q.propagate_static(p, 1, [], 0)
                    assert taken, (M, L, dtype, n)
                except Q.QuapiError as e:
                    assert not taken and e.status == Q.ERR_INVALID, (M, L, dtype, n)
        """)


def test_server_chunks_are_whole_passes(run):
    # chunks that end on the server's group of steps take no part of a pass
    run("""
        from paper_1205_6872_amd import serve
        for L, dtype, driven in ((8, "c128", False), (13, "c64", False), (9, "c64f64", True), (8, "c128", True)):
            H_t = np.stack([np.diag([1.0, -1.0])] * 3) if driven else None
            w = W.spin_boson_l7().with_(L=L, dtype=dtype, H_t=H_t)
            with Q.create(Q.params_from(w)) as c:
                k = serve._group_steps(w, c)
                c.propagate(L, sel=[])
                got = names(lambda: [c.propagate(n, sel=[]) for n in (k, 2 * k, k)])
                assert got.count("tile_kernel") == k, (L, dtype, driven, k, got)
        for M, L, dtype in ((2, 7, "c128"), (2, 6, "c64"), (3, 8, "c128")):
            w = W.spin_boson_l7().with_(M=M, L=L, dtype=dtype, s=np.arange(M), H=np.eye(M), rho0=np.eye(M) / M)
            with Q.create(Q.params_from(w)) as c:
                assert serve._group_steps(w, c) == c.fused_steps()
        """)


def test_timing_counts_the_launches_that_run(run):
    # step_launches and step_steps are launches and their steps; the split by width
    # shares a four-step pass out over groups of quapi_fused_steps and the rest,
    # so its sums are those of the totals, and its counts only where no pass ran
    run("""
        kernels = ("step_kernel", "step_mirror_kernel", "step2_kernel", "step3_kernel", "tile_kernel")
        for L, dtype, pin, n, launches in ((13, "c128", 0, 8, 3), (13, "c64", 0, 12, 4), (9, "c64f64", 0, 8, 3),
                                           (13, "c128", 3, 7, 3), (12, "c64", 2, 7, 4), (9, "c128", 1, 5, 5)):
            w = W.spin_boson_l7().with_(L=L)
            with Q.create(Q.params_from(w, dtype=dtype)) as c:
                c.set_fused_steps(pin)
                c.propagate(L - 1, sel=[])
                c.set_timing(True)
                c.get_timing()
                got = [k for k in names(lambda: c.propagate(n, sel=[])) if k in kernels]
                t = c.get_timing()
                assert (t["step_launches"], t["step_steps"]) == (launches, n), (L, dtype, pin, t)
                if pin == 0:
                    assert got == ["step_kernel" if L < 12 else "step_mirror_kernel"] + ["tile_kernel"] * (launches - 1)
                k = t["width_launches"]
                assert sum(i * k[i] for i in range(4)) == n, (L, dtype, pin, t)
                assert abs(sum(t["width_ms"]) - t["step_ms"]) < 1e-9, (L, dtype, pin, t)
                assert pin == 0 or sum(k) == launches, (L, dtype, pin, t)
        """)
