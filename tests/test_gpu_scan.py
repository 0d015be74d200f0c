"""Cell scan at the edges of its chunks of 4096 cells: one chunk, exact
multiples, one cell more, and the last grid of the one-launch form (256 chunks)
against the first of the three-launch form, each by the pairs found and the
masses after two steps."""
import numpy as np
import pytest

from paper_1811_05474_amd import rwpt, workloads as W

pytestmark = pytest.mark.gpu

# cells per axis
GRIDS = [(64, 64), (4097, 1), (128, 64), (1023, 1024), (1024, 1024), (1025, 1024)]


def test_cell_scan_chunk_edges():
    n, dt, rc = 300_001, 0.1, 1.0 / 256.0
    D = rc * rc / 72.0 / dt
    x = W.positions(n, 2, 91)
    M = W.masses(n, 2, 91)
    out = []
    for nc in GRIDS:
        # cells per cutoff length; half a cell over, so that the floor gives nc
        refine = tuple((c + 0.5) * rc * (1.0 + 1e-5) for c in nc) + (0.0,)
        ens = rwpt.Ensemble(dim=2, n_species=2, react=(0, 1), kappa=3.0, rw_ratio=1.0, seed=9,
                            precision=rwpt.RWPT_FP64, cell_refine=refine)
        ens.init([n], x, M)
        ens.step(dt, D, 1)
        ens.step(dt, D, 1)
        assert ens.stats()["n_cells"] == nc[0] * nc[1]
        out.append((ens.count_pairs(dt, D)[0], ens.positions(), ens.masses()))
        ens.close()
    for pairs, pos, mass in out[1:]:
        assert pairs == out[0][0]
        assert np.array_equal(pos, out[0][1])
        # binary64 sums of about 14 terms in another order
        assert np.abs(mass - out[0][2]).max() <= 1e-14 * np.abs(out[0][2]).max()
