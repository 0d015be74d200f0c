"""1-D expansions over several realisations: unequal sizes, one without
diffusion, one of few particles, and many realisations of few cells each; the
plan in use is asserted through the cells per cutoff.  Bars as for one
realisation (binary64 expansions truncated below 2e-9 of a weight, masses
rounded to binary32): 1e-6 normwise per step."""
import numpy as np
import pytest

import oracle
from paper_1811_05474_amd import rwpt, workloads as W

pytestmark = pytest.mark.gpu

DT = 0.1
SYM, ROW = rwpt.RWPT_NORM_SYM, rwpt.RWPT_NORM_ROW


def D_for(n, nb):
    rc = nb / (2.0 * (n - 1))
    return rc * rc / (72.0 * DT)


def f32(a):
    return np.asarray(a, dtype=np.float32).astype(np.float64)


@pytest.mark.parametrize("sizes,scale,D,S,norm", [
    ([20000, 700, 16000, 18000], [1.0, 1.0, 0.0, 0.6], D_for(20000, 2200.0), 2, SYM),
    ([18000, 16000, 700, 20000], [0.6, 0.0, 1.0, 1.0], D_for(20000, 2200.0), 5, ROW),
    ([1500 + 7 * k for k in range(40)], None, D_for(1500, 1300.0), 2, SYM)])
def test_realisations(sizes, scale, D, S, norm):
    n = sum(sizes)
    scale = scale or [1.0] * len(sizes)
    x, M = f32(W.positions(n, 1, 8)), f32(W.masses(n, S, 8))
    ens = rwpt.Ensemble(dim=1, n_species=S, react=(0, 1), kappa=3.0, rw_ratio=0.0, norm=norm, seed=4)
    ens.init(sizes, x, M, d_scale=np.array(scale))
    ens.step(DT, D, 2)
    assert rwpt.rwpt_get_tiling(ens.ctx) == (4, (32.0, 1.0, 1.0))
    got, counts = ens.masses(), ens.rowsums(DT, D, unit_weights=True)
    onorm = oracle.NORM_SYM if norm == SYM else oracle.NORM_ROW
    off = np.concatenate([[0], np.cumsum(sizes)])
    for r, Dr in enumerate(D * np.array(scale)):
        a, b = off[r], off[r + 1]
        if Dr > 0.0:
            rp, _ = oracle.neighbors(x[a:b], 3.0, Dr, DT, 32)
            assert np.array_equal(counts[a:b], np.diff(rp))
        ref = M[:, a:b]
        for _ in range(2):
            ref = oracle.transfer(x[a:b], ref, Dr, DT, kappa=3.0, prec=32, norm=onorm, react=(0, 1))
        assert np.abs(got[:, a:b] - ref).max() < 2e-6 * np.abs(ref).max()
    assert np.allclose(ens.audit()[:, :2].sum(0), got.sum(1)[:2], rtol=1e-9)
    ens.close()
