"""The fill by levels of diagonals (band products, mid products, a finalize per span length) of
chains without the saving sweep, which profiled solves and some very wide ones run: full tables,
choices and schedules against the oracle at the sizes where its kernels have edges."""
import numpy as np
import pytest

import oracle
from paper_2307_01236_amd import rk
from paper_2307_01236_amd.chaingen import make_grid_chain, make_random_chain, store_all_bound
from test_parity_gpu import full_parity, fuzz_chains, sub_rows_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("idx", range(0, 24, 3))
def test_small_chains(idx):
    ch, M = fuzz_chains()[idx]
    full_parity(ch, M, diagonals=True)


@pytest.mark.parametrize("L,K", [(65, 3), (80, 9), (97, 2), (100, 16)])
def test_bands_and_mids(L, K):
    """Band products at spans 32, 64 and 96, both mid widths, folds into stored partials."""
    ch = make_random_chain(9100 + L, L, K, xmax=L % 40 + 1, amax=L % 60 + 1, tmax=L % 20, tmin=0, small_times=L % 2 == 1)
    full_parity(ch, min(store_all_bound(ch) // 2, 700), diagonals=True)


def test_option_sizes_beyond_the_staged_halo():
    """Shifts of more than the 256 columns that the finalize stages in LDS."""
    ch = make_random_chain(4242, 40, 4, xmax=40, amax=700, tmax=60, tmin=0)
    assert int(ch.mem.max()) + int(ch.x.max()) > 256
    full_parity(ch, 3000, diagonals=True)


def test_mid_levels_at_large_budgets():
    """64 blocks at 24 999 budget columns."""
    full_parity(make_random_chain(6464, 64, 3, xmax=50, amax=400, tmax=100, tmin=0), 24998, diagonals=True)


def test_several_bands_at_large_tables():
    """78 blocks x 21 000 columns, shifts of a few hundred."""
    full_parity(make_random_chain(97003, 78, 1, xmax=200, amax=900, tmax=100, tmin=0), 21000, diagonals=True)


def test_wide_budget():
    """200 001 columns: a left pad of about 2000 columns, 1 563 column chunks per cell in the finalize."""
    full_parity(make_random_chain(777, 12, 3, xmax=2000, amax=9000, tmax=3000, tmin=0), 200000, diagonals=True)


def test_grid_options_unpruned():
    full_parity(make_grid_chain(5, 24, 10, 10, types=3), prune=False, diagonals=True)


def test_longest_chain():
    """2000 blocks (1999 finalize launches after the first diagonal's): sub-chains at both ends exactly; the
    whole schedule replayed."""
    L = rk.RK_MAX_L
    ch = make_random_chain(2024, L, 2, M=600, xmax=3, amax=4, tmax=2, small_times=True)
    s, t = rk.Solver(ch), rk.Solver(ch)
    try:
        s.set_profiling(1)
        ans = s.solve()
        assert ans == t.solve()  # by tiles
        for s0 in (0, L - 14):
            sub_rows_parity(s, ch, s0, 14)
        rng = np.random.default_rng(1)
        for _ in range(200):
            a = int(rng.integers(0, L))
            b = int(rng.integers(a, L))
            for x, y in zip(s.row(a, b), t.row(a, b)):
                assert np.array_equal(x, y), (a, b)
        ops, nfwd = s.schedule()
        assert np.array_equal(ops, t.schedule()[0])
        ok, tm, pk, bad = oracle.simulate(ch, ops)
        assert ok and tm == ans and pk <= ch.M, bad
    finally:
        s.close()
        t.close()
