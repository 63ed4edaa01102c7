"""CPU runs of the HIP kernels through the host emulation in tests/emu (no GPU needed).

The unchanged library source is compiled with g++ against a small HIP-runtime emulation in which
the threads of a workgroup are fibers switched at barriers, shuffles, ballots and sleeps. These
tests check kernel indexing, the solver's control flow (every thread of a workgroup must pass the
same barriers; a barrier that can never release is reported) and the whole pipeline against the
oracle, on small inputs: each check once in the default schedule, the whole sweep again under
AddressSanitizer, and again with the fibers scheduled at random."""
import os
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.join(HERE, "emu"))

import build as emu_build  # noqa: E402
import runner  # noqa: E402


@pytest.fixture(scope="module")
def emu_lib():
    return emu_build.build(asan=False)


def test_emulated_special_batched_overflow_unaligned(emu_lib):
    assert runner.run_extra(emu_lib, verbose=False)


def test_emulated_hybrid_coding(emu_lib):
    assert runner.check_hybrid(runner.load(emu_lib), verbose=False)


def test_emulated_capped_ties(emu_lib):
    assert runner.check_ties(runner.load(emu_lib), verbose=False)


def test_emulated_candidate_band(emu_lib):
    assert runner.check_candidates(runner.load(emu_lib), verbose=False)


def test_emulated_answer_inside_the_lowest_binade(emu_lib):
    assert runner.check_lowest_binade(runner.load(emu_lib), verbose=False)


def test_emulated_full_range_rows(emu_lib):
    assert runner.check_full_range(runner.load(emu_lib), verbose=False)


def test_emulated_random_rows_batches_segments(emu_lib):
    assert runner.check_random(runner.load(emu_lib), verbose=False)


def test_emulated_capped_values_past_the_lane_rows(emu_lib):
    assert runner.check_lane_rows(runner.load(emu_lib), verbose=False)


def test_emulated_band_region_overflow(emu_lib):
    assert runner.check_band_region_overflow(runner.load(emu_lib), verbose=False)


def test_emulated_variance_solver(emu_lib):
    assert runner.check_variance(runner.load(emu_lib), verbose=False)


def test_emulated_segmented(emu_lib):
    assert runner.check_segmented(runner.load(emu_lib), verbose=False)


def test_emulated_aggregate(emu_lib):
    assert runner.check_aggregate(runner.load(emu_lib), verbose=False)


def test_emulated_parity_subset(emu_lib):
    L = runner.load(emu_lib)
    import oracle
    import workloads as W
    from oracle.compare import compare_sample

    for name, mk in [("spiked", lambda: np.concatenate([W.normal(37, 9) * np.float32(40), W.normal(20000, 0)])),
                     ("tmix", lambda: W.t_mixture(30001, 2)), ("ties", lambda: W.integer_ties(12001, 3))]:
        g = np.ascontiguousarray(mk(), np.float32)
        for solver in ("greedy", "exact"):
            for rho in (0.01, 0.5):
                sol = oracle.solve(g, rho, solver, 2)
                idx, val, n, lam, k, fl = runner.sample_row(L, g, rho, solver, 77)
                assert fl == 0
                compare_sample(g, sol.p, 77, idx, val, n, lam, sol.lam)
                if solver == "exact":
                    assert lam == sol.lam and k == sol.k


@pytest.mark.parametrize("scale", [1e-42, 1e-36, 1e-24, 1e20, 1e36])
def test_emulated_selection_at_extreme_scales(emu_lib, scale):
    """Whole tiles at scales where lambda * 2^32 lies inside, below and beyond the range in which fp32
    decides a coordinate (and subnormal magnitudes), plus a ragged tail."""
    L = runner.load(emu_lib)
    import oracle
    import workloads as W
    from oracle.compare import compare_sample

    g = np.ascontiguousarray(W.t_mixture(2 * 16384 + 37, 31).astype(np.float64) * scale)
    g = np.clip(g, -3e38, 3e38).astype(np.float32)
    for solver, rho in (("exact", 0.05), ("greedy", 0.2), ("exact", 1.0)):
        sol = oracle.solve(g, rho, solver, 2)
        idx, val, n, lam, k, fl = runner.sample_row(L, g, rho, solver, 78)
        assert fl == 0
        compare_sample(g, sol.p, 78, idx, val, n, lam, sol.lam)


def test_emulated_full_sweep(emu_lib):
    assert runner.run_all(emu_lib, verbose=False) == 64


def test_emulated_asan_subset():
    """Kernel indexing under AddressSanitizer: a padded batch ending in partial groups with a
    candidate band, unaligned rows, the variance budget, segments on and off 16-byte boundaries with
    the hybrid coding, and aggregation (the whole sweep under ASan is below)."""
    lib = emu_build.build(asan=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0", LD_PRELOAD=emu_build.asan_runtime())
    r = subprocess.run([sys.executable, os.path.join(HERE, "emu", "runner.py"), lib, "asan_subset"], env=env,
                       capture_output=True, text=True, timeout=1200)
    assert r.returncode == 0 and "AddressSanitizer" not in r.stderr, r.stderr[-2000:]
    assert "asan subset ok" in r.stdout, r.stdout[-2000:]


def test_emulated_under_asan():
    """Every emulated check (edge cases, batching, overflow, the unaligned path, hybrid coding,
    ties, the candidate band and its overflows, aggregation, the variance budget, segments and the
    parity sweep) under AddressSanitizer."""
    lib = emu_build.build(asan=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0", LD_PRELOAD=emu_build.asan_runtime())
    r = subprocess.run([sys.executable, os.path.join(HERE, "emu", "runner.py"), lib, "all"], env=env,
                       capture_output=True, text=True, timeout=1200)
    assert r.returncode == 0 and "AddressSanitizer" not in r.stderr, r.stderr[-2000:]
    assert "checked 64" in r.stdout, r.stdout[-2000:]


def test_emulated_random_schedule(emu_lib):
    """Every emulated check again with the fibers of each workgroup scheduled at random, so that
    lanes run in another order after each barrier: a read of shared state that no barrier
    separates from another lane's write sees the wrong value in some workgroup."""
    env = dict(os.environ, EMU_SHUFFLE="1")
    r = subprocess.run([sys.executable, os.path.join(HERE, "emu", "runner.py"), emu_lib, "all"], env=env,
                       capture_output=True, text=True, timeout=1200)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-2000:])
    assert "checked 64" in r.stdout, r.stdout[-2000:]


def test_emulated_lookback_fallback():
    """Hide every published tile status so each look-back counts its predecessors itself."""
    lib = emu_build.build(asan=False)
    env = dict(os.environ, EMU_HIDE_STATUS="1", EMU_STALL_SECONDS="300")
    r = subprocess.run([sys.executable, os.path.join(HERE, "emu", "runner.py"), lib, "extra_lite"], env=env,
                       capture_output=True, text=True, timeout=1200)
    assert r.returncode == 0 and "extra cases ok" in r.stdout, (r.stdout[-2000:], r.stderr[-2000:])
    r = subprocess.run([sys.executable, os.path.join(HERE, "emu", "runner.py"), lib, "ties"], env=env,
                       capture_output=True, text=True, timeout=1200)
    assert r.returncode == 0 and "tie cases ok" in r.stdout, (r.stdout[-2000:], r.stderr[-2000:])


def test_emulated_two_tiles_per_workgroup():
    """The sampling pass's two-tiles-per-workgroup path (taken on the GPU by grids larger than the
    resident set) forced on the small emulated inputs: edge cases, batching, overflow, the
    unaligned path and the hybrid coding, with tile counts odd and even (segmented rows with two
    tiles per workgroup run on the GPU, in tests/test_gpu_segmented.py)."""
    env = dict(os.environ, GSPAR_EMU_RESIDENT="1", GSPAR_EMU_CAND_MIN_ROW=str(1 << 22))
    lib = subprocess.run([sys.executable, "-c", "import sys; sys.path.insert(0, %r); import build; print(build.build())"
                          % os.path.join(HERE, "emu")], env=env, capture_output=True, text=True, check=True).stdout.strip()
    r = subprocess.run([sys.executable, os.path.join(HERE, "emu", "runner.py"), lib, "extra_lite"], env=env,
                       capture_output=True, text=True, timeout=1200)
    assert r.returncode == 0 and "extra cases ok" in r.stdout, (r.stdout[-2000:], r.stderr[-2000:])
    r = subprocess.run([sys.executable, os.path.join(HERE, "emu", "runner.py"), lib, "hybrid"], env=env,
                       capture_output=True, text=True, timeout=1200)
    assert r.returncode == 0 and "hybrid cases ok" in r.stdout, (r.stdout[-2000:], r.stderr[-2000:])


@pytest.mark.parametrize("cap", [1, 40, 1500])
def test_emulated_solver_windows(cap):
    """The solver's window and count requests, which rows of many keys take, forced on the small
    emulated inputs by listing at most `cap` keys of a range: every emulated check."""
    env = dict(os.environ, GSPAR_EMU_LIST=str(cap))
    lib = subprocess.run([sys.executable, "-c", "import sys; sys.path.insert(0, %r); import build; print(build.build())"
                          % os.path.join(HERE, "emu")], env=env, capture_output=True, text=True, check=True).stdout.strip()
    r = subprocess.run([sys.executable, os.path.join(HERE, "emu", "runner.py"), lib, "all"], env=env,
                       capture_output=True, text=True, timeout=1200)
    assert r.returncode == 0 and "checked 64" in r.stdout, (r.stdout[-2000:], r.stderr[-2000:])


@pytest.mark.parametrize("d", [4095, 4096, 4097, 8193, 40003])
def test_emulated_listed_binade(emu_lib, d):
    """Rows whose keys all lie in one binade that a threshold cuts, so that one request lists all of
    them: up to the keys that the solver's leader holds in LDS, past them, and past whole batches.
    The exact solvers' lambda and capped count are the oracle's."""
    L = runner.load(emu_lib)
    import oracle
    from oracle.compare import compare_sample

    r = np.random.default_rng(d)
    g = ((1.0 + r.random(d)) * r.choice([-1.0, 1.0], d)).astype(np.float32)
    g = np.where(np.abs(g) >= 2.0, np.float32(1.5), g).astype(np.float32)
    for solver, rho in (("exact", 0.9), ("greedy", 0.9), ("variance", 0.02)):
        sol = oracle.solve(g, rho, solver, 2)
        idx, val, n, lam, k, fl = runner.sample_row(L, g, rho, solver, 79, cap=d)
        assert fl == 0
        compare_sample(g, sol.p, 79, idx, val, n, lam, sol.lam)
        if solver != "greedy":
            assert lam == sol.lam and 0 < sol.k < d


@pytest.mark.parametrize("rho", [0.12, 0.126, 0.25, 0.49, 0.51])
@pytest.mark.parametrize("tail", [0, 1, 4 * 64 * 8 + 3, 16383])
def test_emulated_staged_emission(emu_lib, rho, tail):
    """Survivor counts of a wave (of 4,096 coordinates) just below and above one staging round of 512,
    several rounds, and on both sides of the limit of the staged path, with capped coordinates of both
    signs alone in their group and two or more to a group, in whole tiles and in a row's last tile of 0,
    1 or nearly all coordinates: the compaction is the oracle's sample and the hybrid coding the same
    survivors."""
    L = runner.load(emu_lib)
    import oracle
    from oracle.compare import compare_sample

    d = 2 * 16384 + tail
    r = np.random.default_rng(1000 + tail)
    g = (r.choice([-1.0, 1.0], d) * (1.0 + 0.01 * r.random(d))).astype(np.float32)
    g[r.integers(0, d, d // 300)] *= np.float32(50.0)
    g[40:46] = [-300.0, 300.0, 200.0, -200.0, 100.0, -100.0]
    sol = oracle.solve(g, rho, "exact", 2)
    idx, val, n, lam, k, fl = runner.sample_row(L, g, rho, "exact", 80, cap=d)
    assert fl == 0 and lam == sol.lam and k == sol.k and k > 0
    compare_sample(g, sol.p, 80, idx, val, n, lam, sol.lam)
    big = np.abs(g[idx]) > 40.0
    assert np.array_equal(val[big], g[idx][big])
    ia, va, na, cb, nb, inv, q, lam2, fl2 = runner.hybrid_batched(L, g[None, :], [rho], [80], "exact")
    a, b = int(na[0]), int(nb[0])
    bi = cb[0, :b] & 0x7FFFFFFF
    assert not fl2.any() and a + b == n and a == k
    assert np.array_equal(np.sort(np.concatenate([ia[0, :a], bi])), idx) and np.all(np.diff(bi) > 0)
    assert np.array_equal(va[0, :a], g[ia[0, :a]]) and np.array_equal(cb[0, :b] < 0, g[bi] < 0)


@pytest.mark.parametrize("segs", [1, 255, 256, 257, 700])
def test_emulated_many_segments(emu_lib, segs):
    """Segment maps filled by several workgroups, of fewer and more rows than one scan holds, lengths
    around a histogram chunk and a tile (and empty ones) among them: every segment's sample is that of
    a row of its own."""
    L = runner.load(emu_lib)
    import workloads as W

    r = np.random.default_rng(segs)
    lens = r.integers(0, 40, segs)
    for at, n in ((0, 16385), (segs // 2, 8193), (segs - 1, 40001)):
        lens[at] = n
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    g = np.ascontiguousarray(W.t_mixture(int(off[-1]), 90 + segs), np.float32)
    seeds = np.arange(segs) + 5
    idx, val, nnz, lam, k, fl = runner.segmented(L, g, off, np.full(segs, 0.1), seeds, "exact")
    for i in {0, 1 % segs, segs // 2, segs - 2 if segs > 1 else 0, segs - 1}:
        row = g[off[i]:off[i + 1]]
        if row.size == 0:
            assert nnz[i] == 0
            continue
        ri, rv, n, rl, rk, rf = runner.sample_row(L, row, 0.1, "exact", int(seeds[i]))
        assert nnz[i] == n and fl[i] == rf and k[i] == rk and lam[i] == rl
        assert np.array_equal(idx[i][:n], ri) and np.array_equal(val[i][:n], rv)


def _exact_row(L, g, rho, solver, seed=5):
    """The compaction of one row, with lambda and the capped count equal to the oracle's bit for bit."""
    import oracle
    from oracle.compare import compare_sample

    g = np.ascontiguousarray(g, np.float32)
    sol = oracle.solve(g, rho, solver, 2)
    idx, val, n, lam, k, fl = runner.sample_row(L, g, rho, solver, seed, cap=g.size)
    assert fl == sol.flags and lam == sol.lam and k == sol.k, (solver, rho, lam, sol.lam, k, sol.k, fl)
    compare_sample(g, sol.p, seed, idx, val, n, lam, sol.lam)
    return n, k


_HALVES = np.concatenate([np.full(10, 0.5), [1.0, 1.5]])


@pytest.mark.parametrize("g, rho, solver", [
    (np.concatenate([np.ones(8), np.full(3, 2.0), np.zeros(89)]), 0.07, "exact"),
    (np.concatenate([np.zeros(88), _HALVES]), 0.07, "exact"),
    (_HALVES, 7 / 12 * (1 + 1e-14), "exact"),
    (np.concatenate([[2.0 ** -40], np.full(100, 1.25), [1.5]]), 2.2e-16, "variance"),
], ids=["ones_twos", "halves_zeros", "halves", "variance"])
def test_emulated_failing_tie_above_the_answer(emu_lib, g, rho, solver):
    """A value within rounding of Algorithm 2's criterion that fails it, alone in its window, above an
    answer that a higher level gave: lambda comes from the answer's own sums."""
    _exact_row(runner.load(emu_lib), g, rho, solver)


@pytest.mark.parametrize("solver", ["exact", "variance"])
def test_emulated_quantised_rows(emu_lib, solver):
    """Integer and fixed-point rows, whose budgets lie on an integer or a few ulps off it (variance
    budget: whose eps is about the rounding error of the sums), so that values meet the criterion with
    equality up to rounding: lambda and k are the oracle's bit for bit."""
    L = runner.load(emu_lib)
    r = np.random.default_rng(7)
    for _ in range(1500):
        d = int(np.exp(r.uniform(0.0, np.log(160.0))))
        top = int(r.choice([2, 3, 8]))
        g = r.integers(-top, top + 1, d) / float(r.choice([1, 2, 128]))
        if r.random() < 0.3:
            g = np.full(d, 1.0 + r.random())
            g[0] = 10.0 ** r.uniform(-14.0, 0.0)
        if r.random() < 0.4:
            g[r.random(d) < r.random()] = 0.0
        if solver == "exact":
            rho = int(r.integers(1, d + 1)) / d
            for _ in range(int(r.integers(0, 3))):
                rho = float(np.nextafter(rho, r.choice([0.0, 1.0])))
        else:
            rho = float(r.choice([10.0 ** r.uniform(-17.0, -15.0), 10.0 ** r.uniform(-15.0, 0.0), 0.25, 0.5, 1.0]))
        _exact_row(L, g, rho, solver)


@pytest.mark.parametrize("d", [8000, 16384, 2 * 16384 + 100])
def test_emulated_capped_below_one(emu_lib, d):
    """The variance budget with an eps of about the sums' rounding error: the criterion makes the run of
    equal magnitudes capped although fl(lambda |g_i|) lies well below 1. The capped set is kept whole, in
    a row's whole tiles and in its last one, by the compaction, the probabilities and the hybrid coding."""
    import oracle

    L = runner.load(emu_lib)
    r = np.random.default_rng(d)
    capped = np.arange(339, d)
    for _ in range(500):  # such a row: the rounding of the sums decides, so it is looked for
        g = np.full(d, r.uniform(1.0, 2.0), np.float32)
        g[0] = 0.55 * np.spacing(capped.size * float(g[1]))  # moves the sum of the rest by an ulp
        g[1:339] = 0
        eps = float(r.uniform(0.9e-16, 2.2e-16))
        sol = oracle.solve(g, eps, "variance", 2)
        if sol.k == capped.size and sol.lam * float(g[-1]) < 0.9:
            break
    else:
        pytest.fail("no such row")
    _, k = _exact_row(L, g, eps, "variance")
    idx, val, n, _, _, _ = runner.sample_row(L, g, eps, "variance", 5, cap=d)
    assert n == k == capped.size and np.array_equal(idx, capped) and np.array_equal(val, g[capped])
    p, lam, kp, fl = runner.probs_row(L, g, eps, "variance")
    assert kp == k and np.all(p[capped] == 1.0)
    ia, va, na, cb, nb, inv, q, lam, fl = runner.hybrid_batched(L, g[None, :], [eps], [5], "variance")
    assert na[0] == k and nb[0] == 0 and not fl.any()
    assert np.array_equal(ia[0, :k], capped) and np.array_equal(va[0, :k], g[capped])
    assert np.array_equal(np.flatnonzero(q[0]), capped) and np.all(q[0][capped] == 2)


@pytest.mark.parametrize("solver", ["greedy", "exact"])
@pytest.mark.parametrize("d, scale, rho", [(1000, 1e30, 1e-300), (3, 100.0, 5e-324), (16384 + 7, 1e36, 1e-310)])
def test_emulated_lambda_underflows(emu_lib, solver, d, scale, rho):
    """A positive budget so small that lambda = B / sum |g_i| rounds to zero: nothing is capped and
    nothing sampled, by the compaction, the hybrid coding and the probabilities."""
    L = runner.load(emu_lib)
    r = np.random.default_rng(d)
    g = (r.choice([-1.0, 1.0], d) * (1.0 + r.random(d)) * scale).astype(np.float32)
    idx, val, n, lam, k, fl = runner.sample_row(L, g, rho, solver, 5, cap=d)
    assert (n, lam, k, fl) == (0, 0.0, 0, 0)
    ia, va, na, cb, nb, inv, q, lam2, fl2 = runner.hybrid_batched(L, g[None, :], [rho], [5], solver)
    assert na[0] == nb[0] == 0 and lam2[0] == 0.0 and not fl2.any() and not q.any()
    p, lam3, k3, fl3 = runner.probs_row(L, g, rho, solver)
    assert not p.any() and (lam3, k3, fl3) == (0.0, 0, 0)


def _build_emu(concurrent=False, **env):
    """The emulation built with the given variables (see emu/build.py), in a process of its own."""
    r = subprocess.run([sys.executable, "-c", "import sys; sys.path.insert(0, %r); import build; "
                        "print(build.build(concurrent=%r))" % (os.path.join(HERE, "emu"), concurrent)],
                       env=dict(os.environ, **env), capture_output=True, text=True, check=True)
    return r.stdout.strip()


_CONCURRENT = """
import ctypes, sys
sys.path.insert(0, sys.argv[3])
import numpy as np
import runner
import workloads as W

A, B = runner.load(sys.argv[1]), runner.load(sys.argv[2])
same = lambda x, y: all(np.array_equal(np.asarray(u), np.asarray(v)) for u, v in zip(x, y))
buf = (ctypes.c_ulong * 4096)()


def helped(rows, call):
    # whether a workgroup past the rows' leaders finished a chunk of a request
    B.emu_waits(buf, ctypes.c_ulong(4096))
    out = call(B)
    B.emu_waits(buf, ctypes.c_ulong(4096))
    return out, sum(buf[rows:4096])


n = 0
for d, seed in ((100003, 3), (65536, 4)):
    g = np.ascontiguousarray(W.t_mixture(d, seed), np.float32)
    for solver, rho in (("exact", 0.05), ("greedy", 0.1), ("variance", 1.0)):
        f = lambda L: runner.sample_row(L, g, rho, solver, 5)
        b, h = helped(1, f)
        assert same(f(A), b), (d, solver)
        n += h
g2 = np.stack([W.t_mixture(40003, 30 + r) for r in range(3)])
for solver, rho in (("exact", 0.05), ("greedy", 0.1), ("variance", 1.0)):
    f = lambda L: runner.batched(L, g2, [rho] * 3, [1, 2, 3], solver)
    b, h = helped(3, f)
    assert same(f(A), b), solver
    n += h
off = np.cumsum([0, 30001, 5, 0, 70001]).astype(np.int64)
g = np.ascontiguousarray(W.t_mixture(int(off[-1]), 8), np.float32)
f = lambda L: runner.segmented(L, g, off, np.full(4, 0.1), [1, 2, 3, 4], "exact")
b, h = helped(4, f)
x, y = f(A), b
assert same(x[2:], y[2:]) and all(same(u, v) for u, v in zip(x[:2], y[:2]))
n += h
print("helped", n)
assert n > 0
"""


@pytest.mark.parametrize("resident, seed", [(2, 1), (4, 3), (8, 5)])
@pytest.mark.parametrize("listed, helpers", [(None, None), (40, None), (40, 3)])
def test_emulated_leader_and_helpers(emu_lib, listed, helpers, resident, seed):
    """The solver's leader and helpers resident at once, at random speeds (helpers that take chunks,
    lose them to the leader, hold an old request while the leader is at the next one, or start after
    the row is solved), for list requests and, with at most 40 keys listed, windows and counts, also
    with fewer helpers than chunks: all results are those of the leader working alone, bit for bit."""
    env = {} if listed is None else {"GSPAR_EMU_LIST": str(listed)}
    alone = emu_lib if listed is None else _build_emu(**env)
    if helpers is not None:
        env["GSPAR_EMU_HELPERS"] = str(helpers)
    conc = _build_emu(concurrent=True, **env)
    r = subprocess.run([sys.executable, "-c", _CONCURRENT, alone, conc, os.path.join(HERE, "emu")],
                       env=dict(os.environ, EMU_RESIDENT=str(resident), EMU_SHUFFLE_SEED=str(seed)),
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-2000:])


_SHARE = """
import ctypes, sys
sys.path.insert(0, sys.argv[2])
import numpy as np
import runner
import workloads as W

L = runner.load(sys.argv[1])
buf = (ctypes.c_ulong * 4096)()
lead = helped = 0
for solver, rho in (("exact", 0.05), ("greedy", 0.1), ("variance", 1.0)):
    g = np.ascontiguousarray(W.t_mixture(200003, 3), np.float32)
    L.emu_waits(buf, ctypes.c_ulong(4096))
    runner.sample_row(L, g, rho, solver, 5)
    L.emu_waits(buf, ctypes.c_ulong(4096))
    lead += buf[0]
    helped += sum(buf[1:4096])
print("leader", lead, "helpers", helped)
assert helped >= 0.4 * (lead + helped)
"""


@pytest.mark.parametrize("helpers", [2, None])
def test_emulated_more_chunks_than_helpers(helpers):
    """A row of 25 chunks with a leader and two helpers resident at even speeds, because no more are
    launched or because the others find no place: the two take most of what is not the leader's, where
    helpers bound to one chunk each left all but two of a request's chunks to the leader."""
    lib = _build_emu(concurrent=True, **({} if helpers is None else {"GSPAR_EMU_HELPERS": str(helpers)}))
    r = subprocess.run([sys.executable, "-c", _SHARE, lib, os.path.join(HERE, "emu")],
                       env=dict(os.environ, EMU_RESIDENT="3", EMU_EVEN="1"), capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-2000:])


@pytest.mark.parametrize("caps, rho", [(188, 0.1), (188, 0.3), (196, 0.084), (196, 0.088), (196, 0.3), (196, 0.55),
                                       (520, 0.13)])
@pytest.mark.parametrize("room", [1.0, 0.6])
def test_emulated_waves_that_cannot_be_staged(emu_lib, caps, rho, room):
    """Waves some of whose lanes have more capped values than their LDS rows hold, on both sides of the
    capped and of the total survivor counts at which their emission goes by groups, with room for every
    survivor and with a capacity that ends inside a wave: the compaction is the oracle's sample, the
    hybrid coding has the same survivors, and what the capacity cuts off is the tail."""
    L = runner.load(emu_lib)
    import oracle
    from oracle.compare import compare_sample

    # each wave (4,096 coordinates) has `caps` large magnitudes: 12 on its first lane, the rest anywhere
    r = np.random.default_rng(caps)
    g = (r.standard_normal(2 * 16384 + 123) * 1e-3).astype(np.float32)
    for w in range(8):
        at = 4096 * w + np.concatenate([256 * np.arange(3)[:, None] + np.arange(4)]).reshape(-1)
        rest = np.setdiff1d(np.arange(4096 * w, 4096 * (w + 1)), at)
        at = np.concatenate([at, r.choice(rest, caps - 12, replace=False)])
        g[at] = (100.0 + 8.0 * r.random(caps)) * r.choice([-1.0, 1.0], caps)
    rho = max(rho, caps / 4096.0 + 1e-4)
    sol = oracle.solve(g, rho, "exact", 2)
    idx, val, n, lam, k, fl = runner.sample_row(L, g, rho, "exact", 17, cap=g.size)
    assert fl == 0 and k >= 8 * caps
    compare_sample(g, sol.p, 17, idx, val, n, lam, sol.lam)
    cap = int(n * room)
    i2, v2, n2, _, _, f2 = runner.sample_row(L, g, rho, "exact", 17, cap=cap)
    assert n2 == n and f2 == (0 if cap == n else 2)
    assert np.array_equal(i2, idx[:cap]) and np.array_equal(v2, val[:cap])
    big = np.abs(g) * lam >= 1.0
    ia, va, na, cb, nb, inv, q, _, f3 = runner.hybrid_batched(L, g[None, :], [rho], [17], "exact", cap=cap)
    a, b = min(int(na[0]), cap), min(int(nb[0]), cap)
    assert na[0] + nb[0] == n and na[0] == k and f3[0] == (0 if max(na[0], nb[0]) <= cap else 2)
    qa, qb = idx[big[idx]], idx[~big[idx]]
    assert np.array_equal(ia[0, :a], qa[:a]) and np.array_equal(va[0, :a], g[qa[:a]])
    assert np.array_equal(cb[0, :b] & 0x7FFFFFFF, qb[:b]) and np.array_equal(cb[0, :b] < 0, g[qb[:b]] < 0)
