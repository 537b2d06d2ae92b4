"""The tiled fill (16 x 16 spans, 64 budgets per workgroup) at the sizes where it can go wrong,
full tables against the oracle: chains around multiples of 16 blocks, budgets around multiples
of 64 columns, and activation sizes and options that read up to just below, at and above the
columns staged in LDS (0, 64, 128 and 192; unstaged beyond)."""
import numpy as np
import pytest

import oracle
from paper_2307_01236_amd import rk
from paper_2307_01236_amd.chaingen import make_random_chain, store_all_bound
from test_parity_gpu import full_parity, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,M", [(1, 63), (2, 64), (15, 127), (16, 128), (17, 191), (31, 62), (32, 130), (33, 65),
                                 (47, 256), (48, 100), (49, 320), (81, 200)])
def test_tile_and_chunk_edges(L, M):
    """Both triangular and square tiles, whole and cut; the last chunk full and ragged."""
    ch = make_random_chain(600 + L, L, 1 + L % 6, allow_zero=L % 2 == 0, xmax=5, amax=9, tmax=4, tmin=0,
                           small_times=L % 3 == 0)
    full_parity(ch, M)


@pytest.mark.parametrize("L", [18, 19, 20, 23, 27, 30, 34, 37, 41, 44, 50, 53, 61, 65, 66, 97, 129, 170])
def test_tile_sides(L):
    """Chains cut into equal tiles of 9 to 16 blocks, the last one smaller or not; windows of LDS and
    none, and from 97 blocks on products of 40 splits and more."""
    M = 150 if L < 100 else 90
    for seed, xmax, amax in ((0, 5, 9), (1, 80, 160)):
        full_parity(make_random_chain(1300 + 2 * L + seed, L, 1 + L % 4, allow_zero=L % 2 == 0, xmax=xmax if L < 100 else 3,
                                      amax=amax if L < 100 else 5, tmax=4, tmin=0, small_times=L % 3 == 0), M + 250 * seed)


@pytest.mark.parametrize("reach", [0, 1, 63, 64, 65, 128, 129, 192, 193])
def test_reach_of_case_1(reach):
    """The largest x + mem of an option decides how many columns left of a chunk are staged."""
    ch = make_random_chain(700 + reach, 36, 5, xmax=max(1, reach // 3), amax=2 * reach // 3 + 1, tmax=9, tmin=0,
                           allow_zero=True)
    if reach == 0:
        ch.x[:], ch.mem[:] = 0, 0
    else:
        ch.mem[:] = np.minimum(ch.mem, np.maximum(reach - ch.x[1:, None], 0))
        s = int(np.argmin(ch.x[1:]))
        ch.mem[s, 0] = reach - ch.x[s + 1]
        assert int((ch.x[1:, None] + ch.mem).max()) == reach and ch.x.max() <= reach
    full_parity(ch, 900)


@pytest.mark.parametrize("L,K,xmax,amax", [(1, 2, 4, 9), (16, 3, 0, 0), (17, 1, 3, 9), (33, 4, 30, 90), (40, 3, 60, 190), (50, 2, 2, 4)])
def test_budgets_past_storing_everything(L, K, xmax, amax):
    """Columns where a tile and all that it reads are in closed form, next to ones where they are not:
    budgets past storing everything, each span's own bound plus the largest shift among them; launches of
    up to 256 workgroups, which take the row loop there, too, and of more."""
    ch = make_random_chain(950 + L, L, K, xmax=max(xmax, 1), amax=max(amax, 1), tmax=7, tmin=0, allow_zero=True)
    if xmax == 0:
        ch.x[:], ch.mem[:] = 0, 0
    bound = store_all_bound(ch) + int((ch.x[1:, None] + ch.mem).max())
    for M in (bound, bound + 64, bound + 133, bound + 64 * 256 + 1):
        full_parity(ch, M)


@pytest.mark.parametrize("L,M,xmax,amax", [(16, 200, 70, 20), (21, 90, 9, 30), (33, 260, 30, 90), (36, 500, 90, 170), (20, 900, 5, 20), (20, 20000, 5, 20)])
def test_operand_tables(L, M, xmax, amax):
    """The operands of the splits beside Opt: Opt(s, t, m - x_s), infinite for m < x_s, and
    P(s, t+1) + Opt(s, t, m), infinite where the sweep does not fit; staged and unstaged shifts."""
    import torch
    ch = make_random_chain(900 + L, L, 3, M=M, xmax=xmax, amax=amax, tmax=9, tmin=0, allow_zero=True)
    s = rk.Solver(ch)
    try:
        n = s.workspace_bytes(M)
        ws = torch.zeros(n // 4, dtype=torch.int32, device="cuda:0")
        s.solve_async(M, ws.data_ptr(), n, torch.cuda.Stream().cuda_stream)
        s.result()
        rows = L * (L + 1) // 2 + 65
        opt, ap, os = ws.cpu().numpy().astype(np.int64).reshape(3, rows, -1)[:, 32:]
        padl, inf = opt.shape[1] - (M + 1 + 63) // 64 * 64, (1 << 30) - 1
        r = 0
        for a in range(L):
            need = total = 0
            for b in range(a, L):
                row = opt[r, padl : padl + M + 1] & inf
                want = np.full(M + 1, inf)
                want[ch.x[a] :] = row[: max(M + 1 - ch.x[a], 0)]
                assert np.array_equal(os[r, padl : padl + M + 1], want), ("right", a, b)
                total += int(ch.fn_time[b])
                need = max(need, (int(ch.x[b]) if b > a else 0) + int(ch.x[b + 1]) + int(ch.fn_tmp[b]))
                if b + 1 < L:
                    want = np.minimum(total + row, inf)
                    want[:need] = inf
                    assert np.array_equal(ap[r, padl : padl + M + 1], want), ("left", a, b)
                r += 1
    finally:
        s.close()


def test_splits_sorted_out_in_pieces():
    """330 blocks: products of up to 305 splits, whose list of splits that matter is made in
    three pieces.  The fill by levels of diagonals (profiled solves) on the other side."""
    ch = make_random_chain(8123, 330, 2, M=420, xmax=2, amax=4, tmax=2, tmin=0)
    s, t = rk.Solver(ch), rk.Solver(ch)
    try:
        a = s.solve()
        ops, _ = s.schedule()
        ok, tm, pk, _ = oracle.simulate(ch, ops)
        assert ok and tm == a and pk <= ch.M
        t.set_profiling(1)  # the fill by levels of diagonals
        assert t.solve() == a
        assert np.array_equal(s.tradeoff_curve(), t.tradeoff_curve())
        for i in (0, 100, 250, 329):
            for j in range(i, 330, 13):
                for x, y in zip(s.row(i, j), t.row(i, j)):
                    assert np.array_equal(x, y), (i, j)
    finally:
        s.close()
        t.close()


def test_two_chains_at_once_on_two_streams():
    """Two fills in flight at the same time, each waiting for its own workgroups only."""
    import torch
    chains = [make_random_chain(31, 70, 4, xmax=9, amax=30, tmax=9), make_random_chain(32, 90, 3, xmax=7, amax=20, tmax=5)]
    want = [oracle.solve(c) for c in chains]
    solvers = [rk.Solver(c) for c in chains]
    try:
        ws = [torch.empty(s.workspace_bytes(c.M), dtype=torch.uint8, device="cuda:0") for s, c in zip(solvers, chains)]
        st = [torch.cuda.Stream() for _ in chains]
        for rep in range(5):
            say(f"  round {rep}")
            for s, c, w, q in zip(solvers, chains, ws, st):
                s.solve_async(c.M, w.data_ptr(), w.numel(), q.cuda_stream)
            for s, sol in zip(solvers, want):
                assert s.result() == sol.answer
        for s, sol in zip(solvers, want):
            assert np.array_equal(s.rows(want_arg=False)[0], sol.rows()[0])
    finally:
        for s in solvers:
            s.close()


def test_many_workgroups_of_two_fills_at_once():
    """Two fills of more workgroups per launch than the chip holds, on two streams: each waits
    only for workgroups of its own that have started.  The fill by diagonals on the other side."""
    import torch
    ch = make_random_chain(77, 128, 3, M=9000, xmax=60, amax=300, tmax=9)
    solvers = [rk.Solver(ch) for _ in range(2)]
    try:
        solvers[0].set_profiling(1)  # the fill by levels of diagonals
        want = solvers[0].solve()
        curve = solvers[0].tradeoff_curve()
        rows = {(i, j): solvers[0].row(i, j) for i, j in ((0, 127), (0, 63), (40, 127), (31, 80))}
        solvers[0].set_profiling(0)
        n = solvers[0].workspace_bytes(ch.M)
        ws = [torch.empty(n, dtype=torch.uint8, device="cuda:0") for _ in solvers]
        st = [torch.cuda.Stream() for _ in solvers]
        for rep in range(3):
            say(f"  round {rep}")
            for s, w, q in zip(solvers, ws, st):
                s.solve_async(ch.M, w.data_ptr(), n, q.cuda_stream)
            for s in solvers:
                assert s.result() == want
                assert np.array_equal(s.tradeoff_curve(), curve)
                for (i, j), (opt, arg) in rows.items():
                    g_opt, g_arg = s.row(i, j)
                    assert np.array_equal(g_opt, opt) and np.array_equal(g_arg, arg), (i, j)
    finally:
        for s in solvers:
            s.close()


def test_answer_of_the_last_solve_after_a_replay():
    """A captured fill at one budget, replayed after a solve at another: the answer asked for
    is the last solve's."""
    import torch
    ch = make_random_chain(41, 20, 3, M=120, xmax=5, amax=12, tmax=9)
    full = oracle.solve(ch).answer
    low, less = next((m, v) for m in range(ch.M - 1, 0, -1) for v in [oracle.solve(ch, m).answer] if v != full)
    s = rk.Solver(ch)
    try:
        n = s.workspace_bytes(ch.M)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda:0")
        st = torch.cuda.Stream()
        assert s.solve() == full
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            s.solve_async(ch.M, ws.data_ptr(), n, st.cuda_stream)
        for rep in range(3):
            assert s.solve(low) == less
            g.replay()
            torch.cuda.synchronize()
            say(f"  replay {rep}")
            assert s.result() == less
    finally:
        s.close()


def test_failure_belongs_to_the_table_it_happened_in():
    """A wait that gives up marks the table that was being filled (here the mark is planted: word
    256 of the workspace).  Reads of that table are refused until it is filled again, whatever
    replays of a captured fill do in another table; a mark in that other one means nothing to them."""
    import torch
    ch = make_random_chain(41, 20, 3, M=120, xmax=5, amax=12, tmax=9)
    s = rk.Solver(ch)
    try:
        n = s.workspace_bytes(ch.M)
        captured, last = (torch.empty(n // 4, dtype=torch.int32, device="cuda:0") for _ in range(2))
        st = torch.cuda.Stream()
        full = s.solve()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            s.solve_async(ch.M, captured.data_ptr(), n, st.cuda_stream)
        g.replay()
        torch.cuda.synchronize()
        s.solve_async(ch.M, last.data_ptr(), n, st.cuda_stream)
        assert s.result() == full
        last[256] = 1
        for rep in range(2):
            torch.cuda.synchronize()
            for read in (s.result, s.schedule, s.tradeoff_curve, lambda: s.row(0, 3)):
                with pytest.raises(rk.RKError) as e:
                    read()
                assert e.value.code == rk.RK_E_INTERNAL
            g.replay()  # a fill that does not fail, into the other table
        torch.cuda.synchronize()
        s.solve_async(ch.M, last.data_ptr(), n, st.cuda_stream)
        captured[256] = 1
        torch.cuda.synchronize()
        assert s.result() == full
        s.schedule(), s.tradeoff_curve(), s.row(0, 3)
        assert int(last[256]) == 0
    finally:
        s.close()


@pytest.mark.parametrize("L,first", [(17, 100000), (20, 150000), (24, 250000)])
def test_very_wide_budgets_by_diagonals(L, first):
    """17-24 blocks: from `first` columns on (as far as storing everything does not fit) the fill runs by
    diagonals, replayed from a captured graph; both sides of the line, and back, in one chain."""
    ch = make_random_chain(1700 + L, L, 2, xmax=2 * first // L, amax=8 * first // L, tmax=first // L, tmin=0)
    xbar = ch.x[1:, None].astype(np.int64) + ch.mem
    need, cost = xbar + np.maximum(ch.tmp_fwd, ch.tmp_bwd), ch.fwd + ch.bwd
    fits = 0  # the smallest budget in which the cheapest options of all blocks fit
    for i in range(L - 1, -1, -1):
        cheap = cost[i] == cost[i].min()
        fits = min(max(int(n), int(x) + fits if i < L - 1 else 0) for n, x in zip(need[i][cheap], xbar[i][cheap]))
    assert fits > first
    sols = {M: oracle.solve(ch, M) for M in (first - 1, first - 2)}
    s = rk.Solver(ch)
    try:
        for M in (first - 1, first - 2, first - 1, first - 1):  # M + 1 columns
            sol = sols[M]
            assert s.solve(M) == sol.answer
            assert (s.fill_ms()[1] == 3) == (M + 1 < first)
            assert np.array_equal(s.tradeoff_curve(), oracle.tradeoff_curve(sol))
            for i, j in ((0, L - 1), (0, L // 2), (L // 2, L - 1), (3, 4)):
                for x, y in zip(s.row(i, j), (sol.opt_row(i, j), sol.arg_row(i, j))):
                    assert np.array_equal(x, y), (i, j)
            ops, nf = s.schedule()
            exp = oracle.schedule(sol, M)
            assert np.array_equal(ops, exp[0]) and nf == exp[1]
    finally:
        s.close()
