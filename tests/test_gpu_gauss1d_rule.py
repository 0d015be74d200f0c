"""The rule that takes a 1-D cutoff to the expansions (1152 expected neighbours,
2.4e7 pairs a step): which side each size falls on, as the cells per cutoff say,
neighbour sets, masses against the oracle, uneven positions, and the
allocation-free call.  Bars as in test_gpu_gauss1d: 1e-6 normwise per step of
the expansions, 1e-5 of the tiles."""
import numpy as np
import pytest

import oracle
from paper_1811_05474_amd import rwpt, workloads as W

pytestmark = pytest.mark.gpu

DT = 0.1
SYM, ROW = rwpt.RWPT_NORM_SYM, rwpt.RWPT_NORM_ROW


def D_for(n, nb):
    rc = nb / (2.0 * n)
    return rc * rc / (72.0 * DT)


def f32(a):
    return np.asarray(a, dtype=np.float32).astype(np.float64)


def ensemble(S, norm, rw=0.0):
    return rwpt.Ensemble(dim=1, n_species=S, react=(0, 1) if S > 1 else None, kappa=3.0, rw_ratio=rw, norm=norm, seed=4)


# sizes around the blocks of 128 particles; one, two and three groups of columns
@pytest.mark.parametrize("n,nb,S,norm,expand", [
    (16385, 1900.0, 2, SYM, True), (20097, 1600.0, 8, SYM, True), (26240, 1200.0, 1, SYM, True),
    (25729, 1180.0, 5, ROW, True), (16511, 2500.0, 3, SYM, True), (33023, 1160.0, 2, ROW, True),
    (8009, 3010.0, 2, SYM, True), (16385, 1400.0, 2, SYM, False), (40001, 1100.0, 2, SYM, False),
    (9000, 2600.0, 2, ROW, False)])
def test_either_side(n, nb, S, norm, expand):
    D = D_for(n, nb)
    x, M = f32(W.positions(n, 1, n)), f32(W.masses(n, S, n))
    ens = ensemble(S, norm)
    ens.init([n], x, M)
    rp, _ = oracle.neighbors(x, 3.0, D, DT, 32)
    assert np.array_equal(ens.rowsums(DT, D, unit_weights=True), np.diff(rp))
    ens.step(DT, D, 1)
    assert rwpt.rwpt_get_tiling(ens.ctx)[1][0] == (32.0 if expand else 16.0)
    ref = oracle.transfer(x, M, D, DT, kappa=3.0, prec=32, norm=oracle.NORM_SYM if norm == SYM else oracle.NORM_ROW,
                          react=(0, 1) if S > 1 else None)
    assert np.abs(ens.masses() - ref).max() < (1e-6 if expand else 1e-5) * np.abs(ref).max()
    ens.close()


@pytest.mark.parametrize("kind", ["one point", "two ends", "walls", "band"])
def test_uneven_positions(kind):
    n = 17001
    D = D_for(n, 2000.0)
    g = np.random.default_rng(5)
    x = 0.05 * g.random((n, 1))
    if kind == "one point":
        x[:] = 0.3
    elif kind == "two ends":
        x = np.where(g.random((n, 1)) < 0.5, 0.01, 0.98) * (1.0 + 0.01 * g.random((n, 1)))
    elif kind == "walls":
        x = g.choice([0.0, 1.0, 0.5, 1e-7], (n, 1))
    else:  # a dense band and a thin tail of isolated particles
        x[: n // 50] = g.random((n // 50, 1))
    x, M = f32(x), f32(W.masses(n, 2, 5))
    ens = ensemble(2, SYM)
    ens.init([n], x, M)
    ens.step(DT, D, 1)
    assert rwpt.rwpt_get_tiling(ens.ctx)[1][0] == 32.0
    ref = oracle.transfer(x, M, D, DT, kappa=3.0, prec=32, react=(0, 1))
    assert np.abs(ens.masses() - ref).max() < 1e-6 * np.abs(ref).max()
    ens.close()


@pytest.mark.parametrize("n,nb,S,norm", [(20003, 1700.0, 2, SYM), (100001, 1200.0, 8, ROW), (16601, 2000.0, 3, SYM)])
def test_allocation_free_call_equals_the_step(n, nb, S, norm):
    import torch

    D = D_for(n, nb)
    x, M = f32(W.positions(n, 1, n)), f32(W.masses(n, S, n))
    ens = ensemble(S, norm)
    ens.init([n], x, M)
    ens.step(DT, D, 1)
    assert rwpt.rwpt_get_tiling(ens.ctx)[1][0] == 32.0
    cfg = rwpt.rwpt_config_default()
    cfg.dim, cfg.n_species, cfg.norm = 1, S, norm
    xd, md = (torch.from_numpy(a).to("cuda", torch.float32) for a in (x, M))
    out = torch.empty_like(md)
    for _ in range(2):
        rwpt.rwpt_transfer_noalloc(cfg, n, xd.data_ptr(), md.data_ptr(), out.data_ptr(), DT, D)
    assert np.array_equal(out.double().cpu().numpy(), ens.masses())
    ens.close()


def test_with_the_walk_split_calls_and_graphs_agree_bitwise():
    n = 18000
    D = D_for(n, 1800.0)
    x, M = f32(W.positions(n, 1, 3)), f32(W.masses(n, 2, 3))
    out = []
    for calls in ((10,), (1, 9)):
        ens = ensemble(2, SYM, rw=1.0)
        ens.init([n], x, M)
        for k in calls:
            ens.step(DT, D, k)
        assert rwpt.rwpt_get_tiling(ens.ctx)[1][0] == 32.0
        out.append((ens.masses(), ens.positions(), ens.audit()))
        ens.close()
    assert all(np.array_equal(a, b) for a, b in zip(*out))
