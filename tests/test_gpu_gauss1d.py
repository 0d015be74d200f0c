"""Expansion kernels of dense 1-D neighbourhoods against the oracle.

Bars, normwise per step: the expansions are binary64 with a truncation below
2e-9 of a weight; 1 / r and the masses are rounded to binary32 (6e-8 each) and
the pairs at the cutoff's edge use binary32 weights (argument rounding
9 * 2^-24 * 2 = 1e-6 relative of weights below 3e-4): 3e-7, bar 1e-6.
Neighbour sets must be exact: unit-weight row sums are the oracle's counts.
"""
import math

import numpy as np
import pytest

import oracle
from paper_1811_05474_amd import rwpt, workloads as W

pytestmark = pytest.mark.gpu

F32 = rwpt.RWPT_FP32
SYM, ROW = rwpt.RWPT_NORM_SYM, rwpt.RWPT_NORM_ROW


def f32(a):
    return np.asarray(a, dtype=np.float32).astype(np.float64)


def D_for(n, nb, dt=0.1, kappa=3.0):
    rc = nb / (2.0 * (n - 1))
    return rc * rc / (kappa * kappa * 8.0 * dt)


def make(kappa=3.0, S=2, norm=SYM, rw=0.0, seed=4, hi=1.0):
    return rwpt.Ensemble(dim=1, n_species=S, react=(0, 1) if S > 1 else None, kappa=kappa, rw_ratio=rw, precision=F32,
                         norm=norm, seed=seed, box_hi=(hi, 1.0, 1.0))


def bar(got, ref, steps):
    err = np.abs(got - ref).max() / np.abs(ref).max()
    print("normwise error %.2e" % err)
    assert err < 1e-6 * steps


# sizes around the tiles of 16 and the blocks of 128 particles; plans of 32
# (>= 512 neighbours) and 16 (>= 256) cells per cutoff and, below, the pair
# tiles; one, two and three groups of columns
@pytest.mark.parametrize("n,nb,S,norm", [(1023, 700.0, 2, SYM), (2049, 900.0, 2, SYM), (4000, 300.0, 1, SYM),
                                         (4111, 520.0, 8, SYM), (4111, 290.0, 5, ROW), (3000, 600.0, 3, SYM),
                                         (20001, 1000.0, 8, ROW), (20001, 200.0, 2, SYM), (5000, 280.0, 2, ROW)])
def test_cutoff_sums(n, nb, S, norm):
    dt, D = 0.1, D_for(n, nb)
    x, M = f32(W.positions(n, 1, n)), f32(W.masses(n, S, n))
    ens = make(S=S, norm=norm)
    ens.init([n], x, M)
    rp, _ = oracle.neighbors(x, 3.0, D, dt, 32)
    assert np.array_equal(ens.rowsums(dt, D, unit_weights=True), np.diff(rp))
    onorm = oracle.NORM_SYM if norm == SYM else oracle.NORM_ROW
    ref = M
    for _ in range(2):
        ref = oracle.transfer(x, ref, D, dt, kappa=3.0, prec=32, norm=onorm, react=(0, 1) if S > 1 else None)
    ens.step(dt, D, 2)
    bar(ens.masses(), ref, 2)
    ens.close()


@pytest.mark.parametrize("n,S,norm", [(4100, 2, SYM), (9001, 8, SYM), (6000, 4, ROW)])
def test_full_matrix(n, S, norm):
    dt, D = 0.1, D_for(n, 700.0)
    x, M = f32(W.positions(n, 1, n)), f32(W.masses(n, S, n))
    ens = make(kappa=None, S=S, norm=norm)
    ens.init([n], x, M)
    ens.step(dt, D, 1)
    ref = oracle.transfer(x, M, D, dt, kappa=math.inf, prec=32, norm=oracle.NORM_SYM if norm == SYM else oracle.NORM_ROW,
                          react=(0, 1))
    bar(ens.masses(), ref, 1)
    ens.close()


def clustered(kind, n, seed):
    g = np.random.default_rng(seed)
    if kind == "one point":
        return np.full((n, 1), 0.3)
    if kind == "two ends":
        return np.where(g.random((n, 1)) < 0.5, 0.01, 0.98) * (1.0 + 0.01 * g.random((n, 1)))
    if kind == "walls":
        return g.choice([0.0, 1.0, 0.5, 1e-7], (n, 1))
    x = 0.05 * g.random((n, 1))          # a dense band and a thin tail of isolated particles
    x[: n // 50] = g.random((n // 50, 1))
    return x


@pytest.mark.parametrize("kappa", [3.0, None])
@pytest.mark.parametrize("kind", ["one point", "two ends", "walls", "band"])
def test_uneven_positions(kind, kappa):
    n, dt = 3001, 0.1
    D = D_for(n, 700.0)
    x, M = f32(clustered(kind, n, 5)), f32(W.masses(n, 2, 5))
    ens = make(kappa=kappa)
    ens.init([n], x, M)
    if kappa:
        rp, _ = oracle.neighbors(x, kappa, D, dt, 32)
        assert np.array_equal(ens.rowsums(dt, D, unit_weights=True), np.diff(rp))
    ens.step(dt, D, 1)
    bar(ens.masses(), oracle.transfer(x, M, D, dt, kappa=kappa or math.inf, prec=32, react=(0, 1)), 1)
    ens.close()


def test_realisations_of_unequal_size_one_without_diffusion():
    sizes, scale = [2500, 0, 1, 900, 3000], [1.0, 1.0, 1.0, 0.0, 0.6]
    dt, D = 0.1, D_for(2500, 900.0)
    n = sum(sizes)
    x, M = f32(W.positions(n, 1, 8)), f32(W.masses(n, 2, 8))
    ens = make()
    ens.init(sizes, x, M, d_scale=np.array(scale))
    ens.step(dt, D, 2)
    got, off = ens.masses(), np.concatenate([[0], np.cumsum(sizes)])
    for r, m in enumerate(sizes):
        if m == 0:
            continue
        a, b = off[r], off[r + 1]
        ref = M[:, a:b]
        for _ in range(2):
            ref = oracle.transfer(x[a:b], ref, D * scale[r], dt, kappa=3.0, prec=32, react=(0, 1))
        bar(got[:, a:b], ref, 2)
    total = ens.audit()[:, :2].sum(0)
    assert np.allclose(total, got.sum(1), rtol=1e-9)
    ens.close()


def test_with_the_walk_split_calls_and_graphs_agree_bitwise():
    n, dt = 6000, 0.1
    D = D_for(n, 600.0)
    x, M = f32(W.positions(n, 1, 3)), f32(W.masses(n, 2, 3))
    out = []
    for calls in ((6,), (1, 2, 3)):
        ens = make(rw=1.0)
        ens.init([n], x, M)
        for k in calls:
            ens.step(dt, D, k)
        out.append((ens.masses(), ens.positions(), ens.audit()))
        ens.close()
    assert all(np.array_equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("n,nb,S,norm", [(5003, 800.0, 2, SYM), (150001, 300.0, 8, ROW), (1500, 600.0, 3, SYM)])
def test_allocation_free_call_equals_the_step(n, nb, S, norm):
    import torch

    dt, D = 0.1, D_for(n, nb)
    x, M = f32(W.positions(n, 1, n)), f32(W.masses(n, S, n))
    ens = make(S=S, norm=norm)
    ens.init([n], x, M)
    ens.step(dt, D, 1)
    cfg = rwpt.rwpt_config_default()
    cfg.dim, cfg.n_species, cfg.precision, cfg.norm = 1, S, F32, norm
    cfg.react_a, cfg.react_b = 0, 1
    xd, md = (torch.from_numpy(a).to("cuda", torch.float32) for a in (x, M))
    out = torch.empty_like(md)
    for _ in range(2):
        rwpt.rwpt_transfer_noalloc(cfg, n, xd.data_ptr(), md.data_ptr(), out.data_ptr(), dt, D)
    assert np.array_equal(out.double().cpu().numpy(), ens.masses())
    ens.close()
