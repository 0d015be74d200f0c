"""The one-launch sort of small realisations against the oracle's steps: on
either side of its limit of 4096 particles (16384 cells), with empty and
one-particle realisations, walks, clusters in one cell, and the allocation-free
call, whose masses are the step's."""
import math

import numpy as np
import pytest

import oracle
from paper_1811_05474_amd import rwpt, workloads as W

import _oracle_steps as OS

pytestmark = pytest.mark.gpu

F32, F64 = rwpt.RWPT_FP32, rwpt.RWPT_FP64


def D_for(n, nb, dim, dt=0.1):
    unit = {1: 2.0, 2: math.pi, 3: 4.0 * math.pi / 3.0}[dim]
    rc = (nb / (n * unit)) ** (1.0 / dim)
    return rc * rc / (72.0 * dt)


# one cell row of the 2-D grids is 16 cells per cutoff, so few neighbours give many cells (at most 4 per particle)
@pytest.mark.parametrize("dim,n,nb,S", [(1, 1, 1.0, 2), (1, 4096, 30.0, 2), (1, 4097, 30.0, 2), (2, 4095, 3.0, 2),
                                        (2, 4096, 3.0, 5), (2, 1025, 40.0, 8), (3, 4096, 0.7, 8), (3, 2047, 5.0, 3)])
def test_walked_steps(dim, n, nb, S):
    dt, seed = 0.1, 21
    D = D_for(n, nb, dim)
    x, M = W.positions(n, dim, seed), W.masses(n, S, seed)
    ens = rwpt.Ensemble(dim=dim, n_species=S, react=(0, 1), kappa=3.0, rw_ratio=1.0, precision=F64, seed=seed)
    ens.init([n], x, M)
    for xr, mr in OS.steps(x, M, 3, D, dt, seed, (0,) * dim, (1,) * dim, False):
        ens.step(dt, D, 1)
        assert np.abs(ens.positions() - xr).max() <= 2 * np.spacing(1.0)
        bar = 1e-12 + 0.3 * 12.0 * np.spacing(1.0) / math.sqrt(8.0 * D * dt)
        assert np.abs(ens.masses() - mr).max() <= bar * np.abs(mr).max()
    ens.close()


def test_both_sorts_give_the_same_bits():
    # three grids in turn; the realisations come first in both runs, so their ids and walks are the same
    sizes = [0, 1, 4096, 37, 0, 2000, 900]
    n, dt, seed = sum(sizes), 0.1, 33
    x, M = W.positions(n, 2, 6), W.masses(n, 2, 6)
    out = []
    for order in (sizes, sizes + [5000]):  # a larger realisation: every step takes the general sort
        m = sum(order)
        xx, MM = W.positions(m, 2, 6), W.masses(m, 2, 6)
        xx[:n], MM[:, :n] = x, M
        ens = rwpt.Ensemble(dim=2, n_species=2, react=(0, 1), rw_ratio=1.0, precision=F64, seed=seed)
        ens.init(order, xx, MM)
        for D in (1e-4, 1e-5, 3e-4):
            ens.step(dt, D, 2)
        out.append((ens.positions()[:n], ens.masses()[:, :n]))
        ens.close()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("prec", [F32, F64])
@pytest.mark.parametrize("dim,n,S,norm", [(2, 4096, 2, rwpt.RWPT_NORM_SYM), (2, 4099, 2, rwpt.RWPT_NORM_SYM),
                                          (3, 1000, 8, rwpt.RWPT_NORM_ROW), (1, 777, 5, rwpt.RWPT_NORM_SYM),
                                          (2, 1, 1, rwpt.RWPT_NORM_SYM)])
def test_allocation_free_call_and_clusters(dim, n, S, norm, prec):
    import torch

    dt, D = 0.1, D_for(n, 12.0, dim)
    x, M = W.positions(n, dim, n), W.masses(n, S, n)
    x[: n // 4] = 0.25  # one cell
    x, M = x.astype(np.float32).astype(np.float64), M.astype(np.float32).astype(np.float64)
    react = (0, 1) if S > 1 else None
    ens = rwpt.Ensemble(dim=dim, n_species=S, react=react, rw_ratio=0.0, precision=prec, norm=norm)
    ens.init([n], x, M)
    ens.step(dt, D, 1)
    want = ens.masses()
    ens.close()
    cfg = rwpt.rwpt_config_default()
    cfg.dim, cfg.n_species, cfg.precision, cfg.norm = dim, S, prec, norm
    cfg.react_a, cfg.react_b = react or (-1, -1)
    t = torch.float32 if prec == F32 else torch.float64
    xd, md = torch.from_numpy(x).to("cuda", t), torch.from_numpy(M).to("cuda", t)
    out = torch.empty_like(md)
    for _ in range(2):
        rwpt.rwpt_transfer_noalloc(cfg, n, xd.data_ptr(), md.data_ptr(), out.data_ptr(), dt, D)
    assert np.array_equal(out.double().cpu().numpy(), want)
    ref = oracle.transfer(x, M, D, dt, kappa=3.0, prec=32 if prec == F32 else 64, react=react,
                          norm=oracle.NORM_SYM if norm == rwpt.RWPT_NORM_SYM else oracle.NORM_ROW)
    assert np.abs(want - ref).max() <= (1e-5 if prec == F32 else 1e-12) * np.abs(ref).max()
