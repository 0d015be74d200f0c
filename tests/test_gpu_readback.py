"""Read-back of the queries: the device reorders the state into the caller's
order and the host widens it in chunks; every value must come back exactly, at
sizes on both sides of a chunk's and of the pinned ring's edges."""
import numpy as np
import pytest

from paper_1811_05474_amd import rwpt, workloads as W

pytestmark = pytest.mark.gpu

CHUNK = 2 << 20  # bytes per pinned slot; 16 slots


def sizes(ts):
    per = CHUNK // ts // 2  # particles whose two coordinates fill one chunk
    return [1, 63, per - 1, per, per + 1, 2 * per + 1, 16 * per, 17 * per + 3]


CASES = [(p, n) for p, ts in ((rwpt.RWPT_FP32, 4), (rwpt.RWPT_FP64, 8)) for n in sizes(ts)]


@pytest.mark.parametrize("prec,n", CASES)
def test_queries_return_the_state_exactly_in_the_callers_order(prec, n):
    x = W.positions(n, 2, 3)
    M = W.masses(n, 2, 3)
    if prec == rwpt.RWPT_FP32:
        x = x.astype(np.float32).astype(np.float64)
        M = M.astype(np.float32).astype(np.float64)
    # about four neighbours: the sort permutes the particles, the walk is off
    D = 4.0 / (np.pi * n) / 7.2
    with rwpt.Ensemble(dim=2, n_species=2, react=None, rw_ratio=0.0, precision=prec) as ens:
        ens.init([n], x, M)
        assert np.array_equal(ens.masses(), M)
        assert np.array_equal(ens.positions(), x)
        ens.step(0.1, D, 1)
        assert np.array_equal(ens.positions(), x)
        first = ens.masses()
        # the query's scratch is none of the state's: the next steps agree with a run that never queried
        ens.step(0.1, D, 2)
        after = ens.masses()
    with rwpt.Ensemble(dim=2, n_species=2, react=None, rw_ratio=0.0, precision=prec) as ens:
        ens.init([n], x, M)
        ens.step(0.1, D, 3)
        assert np.array_equal(ens.masses(), after)
    assert np.all(np.isfinite(first)) and abs(first.sum() - M.sum()) < 1e-5 * M.sum()


@pytest.mark.parametrize("dim,S", [(1, 1), (3, 3), (3, 5), (2, 8)])
def test_queries_with_unused_species_slots_and_several_realisations(dim, S):
    counts = [700, 0, 1, 2049]
    n = sum(counts)
    x = W.positions(n, dim, 5)
    M = W.masses(n, S, 5)
    with rwpt.Ensemble(dim=dim, n_species=S, react=None, precision=rwpt.RWPT_FP64, seed=5) as ens:
        ens.init(counts, x, M)
        assert np.array_equal(ens.masses(), M) and np.array_equal(ens.positions(), x)
        ens.step(0.1, 1e-5, 2)
        a, p = ens.masses(), ens.positions()
        ens.step(0.1, 1e-5, 2)
        b = ens.masses()
    with rwpt.Ensemble(dim=dim, n_species=S, react=None, precision=rwpt.RWPT_FP64, seed=5) as ens:
        ens.init(counts, x, M)
        ens.step(0.1, 1e-5, 4)
        assert np.array_equal(ens.masses(), b)
    assert np.isfinite(a).all() and ((p >= 0) & (p <= 1)).all()
