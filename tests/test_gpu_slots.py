"""Neighbour slots of the one-lane-per-particle kernels (more than 1.5 expected
neighbours) against the oracle: 16 and 32 slots, the last sparse and the first
slotted density, particles with more neighbours than slots, with a walk."""
import math

import numpy as np
import pytest

import oracle
from paper_1811_05474_amd import rwpt, workloads as W

import _oracle_steps as OS

pytestmark = pytest.mark.gpu

F32, F64 = rwpt.RWPT_FP32, rwpt.RWPT_FP64
SYM, ROW = rwpt.RWPT_NORM_SYM, rwpt.RWPT_NORM_ROW
# normwise bars per step of these kernels in binary32 / binary64 (see test_gpu_parity)
BAR = {F32: 1e-5, F64: 1e-12}


def D_for(n, nb, dim, dt=0.1):
    unit = {1: 2.0, 2: math.pi, 3: 4.0 * math.pi / 3.0}[dim]
    rc = (nb / (n * unit)) ** (1.0 / dim)
    return rc * rc / (72.0 * dt)


@pytest.mark.parametrize("prec", [F32, F64])
@pytest.mark.parametrize("dim,n,nb,S,norm,clustered", [
    (3, 20003, 1.45, 2, SYM, False), (3, 20003, 1.55, 2, SYM, False), (3, 20003, 5.9, 8, SYM, False),
    (3, 20003, 6.1, 8, ROW, False), (3, 6401, 25.0, 3, SYM, False), (2, 9999, 4.0, 2, SYM, False),
    (3, 8000, 3.0, 8, SYM, True), (3, 8000, 10.0, 2, ROW, True)])
def test_against_the_oracle(dim, n, nb, S, norm, clustered, prec):
    dt, D = 0.1, D_for(n, nb, dim)
    x, M = W.positions(n, dim, n + S), W.masses(n, S, n)
    if clustered:  # a sixteenth of the particles within a cutoff or so: hundreds of neighbours
        x[::16] = 0.4 + math.sqrt(72.0 * D * dt) * x[::16]
    if prec == F32:
        x, M = (a.astype(np.float32).astype(np.float64) for a in (x, M))
    bits = 32 if prec == F32 else 64
    ens = rwpt.Ensemble(dim=dim, n_species=S, react=(0, 1), kappa=3.0, rw_ratio=0.0, precision=prec, norm=norm,
                        tile_lanes=-1)
    ens.init([n], x, M)
    rp, _ = oracle.neighbors(x, 3.0, D, dt, bits)
    assert np.array_equal(ens.rowsums(dt, D, unit_weights=True), np.diff(rp))
    ens.step(dt, D, 2)
    ref = M
    for _ in range(2):
        ref = oracle.transfer(x, ref, D, dt, kappa=3.0, prec=bits, norm=oracle.NORM_SYM if norm == SYM else
                              oracle.NORM_ROW, react=(0, 1))
    assert np.abs(ens.masses() - ref).max() <= 2.0 * BAR[prec] * np.abs(ref).max()
    ens.close()


def test_walk_in_three_dimensions():
    n, dt, seed = 20000, 0.1, 12
    D = D_for(n, 4.0, 3)
    x, M = W.positions(n, 3, seed), W.masses(n, 2, seed)
    ens = rwpt.Ensemble(dim=3, n_species=2, react=(0, 1), kappa=3.0, rw_ratio=1.0, precision=F64, seed=seed)
    ens.init([n], x, M)
    for xr, mr in OS.steps(x, M, 3, D, dt, seed, (0, 0, 0), (1, 1, 1), False):
        ens.step(dt, D, 1)
        assert np.abs(ens.positions() - xr).max() <= 2 * np.spacing(1.0)
        # a position's ulp changes a weight by up to 6 ulp / sigma
        bar = BAR[F64] + 0.3 * 12.0 * np.spacing(1.0) / math.sqrt(8.0 * D * dt)
        assert np.abs(ens.masses() - mr).max() <= bar * np.abs(mr).max()
    ens.close()
