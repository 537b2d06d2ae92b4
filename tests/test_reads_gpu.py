"""Reading results back: through pinned blocks that the chains share, in pieces where a row is wider
than a block, by several threads at once, and schedules longer than a block."""
import statistics
import threading
import time

import numpy as np
import pytest

import oracle
from paper_2307_01236_amd import rk
from paper_2307_01236_amd.chaingen import Chain, make_config_chain, make_random_chain
from test_parity_gpu import check_same_schedule, full_parity, say

pytestmark = pytest.mark.gpu


def test_first_reads_of_a_chain_cost_what_later_ones_do():
    """No read allocates: over 24 new chains the first trade-off curve and the first row take the
    median time of the second ones (with a buffer of its own per chain, 2.5 to 15 times that)."""
    chains = [make_config_chain(0, rep) for rep in range(24)]
    solvers = [rk.Solver(c) for c in chains]
    try:
        for s in solvers:
            s.solve()
        times = {}
        for turn in ("first", "second"):
            for name, read in (("curve", lambda s: s.tradeoff_curve()), ("row", lambda s: s.row(0, s.L - 1))):
                for s in solvers:
                    t = time.perf_counter()
                    read(s)
                    times.setdefault((turn, name), []).append(time.perf_counter() - t)
        med = {k: statistics.median(v) for k, v in times.items()}
        say("  " + ", ".join(f"{a} {b} {v * 1e6:.0f} us" for (a, b), v in med.items()))
        assert med["first", "curve"] < 2 * med["second", "curve"]
        assert med["first", "row"] < 2 * med["second", "row"]
    finally:
        for s in solvers:
            s.close()


def test_many_chains_alive_and_gone():
    """1100 chains at once (more than one block of their pinned words), some destroyed and made again in
    between: every answer and schedule is the chain's own."""
    chains = [make_random_chain(60 + k, 2 + k, 2, xmax=5, amax=12, tmax=5) for k in range(10)]
    want = [(sol.answer, oracle.schedule(sol)) for sol in map(oracle.solve, chains)]
    solvers = []
    try:
        for k in range(1100):
            s = rk.Solver(chains[k % 10])
            assert s.solve() == want[k % 10][0]
            solvers.append(s)
            if k % 7 == 6:  # a chain in the middle goes, and comes back
                j = (k * 31) % len(solvers)
                solvers[j].close()
                solvers[j] = rk.Solver(chains[j % 10])
                assert solvers[j].solve() == want[j % 10][0]
        for k, s in enumerate(solvers):
            assert s.result() == want[k % 10][0], k
            if k % 11 == 0:
                ops, nf = s.schedule()
                assert np.array_equal(ops, want[k % 10][1][0]) and nf == want[k % 10][1][1], k
    finally:
        for s in solvers:
            s.close()


@pytest.mark.parametrize("M", [174719, 174720, 262143, 262144, 400000])
def test_rows_wider_than_a_block(M):
    """Rows of values and choices in pieces of 174720 columns, of values alone of 262144."""
    ch = make_random_chain(52, 3, 3, xmax=9000, amax=90000, tmax=3000, tmin=0)
    sol = full_parity(ch, M)
    s = rk.Solver(ch)
    try:
        s.solve(M)
        assert np.array_equal(s.rows(want_arg=False)[0], sol.rows()[0])
        assert np.array_equal(s.tradeoff_curve(), oracle.tradeoff_curve(sol))
    finally:
        s.close()


def test_readers_in_several_threads():
    """Twenty threads, each with a chain of its own, read at the same time (more than the blocks kept)."""
    chains = [make_random_chain(900 + k, 6 + k, 3, xmax=9, amax=20, tmax=9) for k in range(20)]
    want = [oracle.solve(c) for c in chains]
    bad = []

    def work(c, sol):
        s = rk.Solver(c)
        try:
            for _ in range(3):
                ops, nf = oracle.schedule(sol)
                g_opt, g_arg = (s.solve(), s.rows())[1]
                g_ops, g_nf = s.schedule()
                if not (np.array_equal(g_opt, sol.rows()[0]) and np.array_equal(g_arg, sol.rows()[1])
                        and np.array_equal(s.tradeoff_curve(), oracle.tradeoff_curve(sol))
                        and np.array_equal(g_ops, ops) and g_nf == nf):
                    bad.append(c.name)
        except Exception as e:  # noqa: BLE001 (a thread's failure is the test's)
            bad.append(repr(e))
        finally:
            s.close()

    threads = [threading.Thread(target=work, args=a) for a in zip(chains, want)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad


def test_schedule_longer_than_a_block():
    """A budget that holds one activation besides a block's own data: the forwards run again from the
    start for every block, about L^2 steps, more than the 87381 that a block holds."""
    L = 320
    one = lambda *n: np.ones(n, np.int32)  # noqa: E731
    zero = lambda *n: np.zeros(n, np.int32)  # noqa: E731
    ch = Chain(L=L, K=1, x=one(L + 1), fn_time=one(L), fn_tmp=zero(L), fwd=one(L, 1), bwd=one(L, 1), mem=one(L, 1),
               tmp_fwd=zero(L, 1), tmp_bwd=zero(L, 1), M=4, name="one_activation")
    sol = oracle.solve(ch)
    s = rk.Solver(ch)
    try:
        for M in (4, 4, 40, 4):
            sol = oracle.solve(ch, M)
            assert s.solve(M) == sol.answer
            check_same_schedule(s, sol, ch, M)
            assert M > 4 or len(s.schedule()[0]) > 87381
    finally:
        s.close()
