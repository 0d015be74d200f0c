"""Binary64 pair kernels of the 8- and 16-lane tiles against the oracle: one
and two tiles per wave on either side of 8192 tiles, odd numbers of tiles and
particles, one and three realisations, and cutoffs on either side of the
largest the fast weight takes (kappa^2 = 700)."""
import math

import numpy as np
import pytest

import oracle
from paper_1811_05474_amd import rwpt, workloads as W

pytestmark = pytest.mark.gpu

F64 = rwpt.RWPT_FP64
SYM, ROW = rwpt.RWPT_NORM_SYM, rwpt.RWPT_NORM_ROW


# (dim, sizes, lanes, neighbours, species, normalisation, kappa)
CASES = [(2, [65529], 0, 20.0, 2, SYM, 3.0), (2, [65537], 0, 20.0, 2, SYM, 3.0), (2, [65544], 8, 9.0, 3, ROW, 3.0),
         (2, [40001, 7, 30003], 0, 15.0, 8, SYM, 3.0), (1, [32773], 0, 30.0, 2, SYM, 3.0),
         (1, [9001], 16, 30.0, 5, ROW, 3.0), (3, [70001], 8, 6.0, 2, SYM, 2.5), (2, [1], 0, 1.0, 2, SYM, 3.0),
         (2, [66000], 0, 12.0, 2, SYM, 26.4), (2, [66000], 0, 12.0, 2, SYM, 26.5)]


@pytest.mark.parametrize("dim,sizes,lanes,nb,S,norm,kappa", CASES)
def test_against_the_oracle(dim, sizes, lanes, nb, S, norm, kappa):
    dt, n = 0.1, sum(sizes)
    unit = {1: 2.0, 2: math.pi, 3: 4.0 * math.pi / 3.0}[dim]
    rc = (nb / (max(sizes) * unit)) ** (1.0 / dim)
    D = rc * rc / (kappa * kappa * 8.0 * dt)
    x, M = W.positions(n, dim, n), W.masses(n, S, n)
    ens = rwpt.Ensemble(dim=dim, n_species=S, react=(0, 1), kappa=kappa, rw_ratio=0.0, precision=F64, norm=norm,
                        tile_lanes=lanes)
    ens.init(sizes, x, M)
    counts = ens.rowsums(dt, D, unit_weights=True)
    ens.step(dt, D, 1)
    got, off = ens.masses(), np.concatenate([[0], np.cumsum(sizes)])
    for a, b in zip(off[:-1], off[1:]):
        rp, _ = oracle.neighbors(x[a:b], kappa, D, dt, 64)
        assert np.array_equal(counts[a:b], np.diff(rp))
        ref = oracle.transfer(x[a:b], M[:, a:b], D, dt, kappa=kappa, prec=64,
                              norm=oracle.NORM_SYM if norm == SYM else oracle.NORM_ROW, react=(0, 1))
        # binary64 weights within 2^-53 (2 * 9 + 1.2) and sums of some tens of terms
        assert np.abs(got[:, a:b] - ref).max() <= 1e-14 * np.abs(ref).max()
    ens.close()
