"""Cells of many particles in the one-launch sort, whose in-cell order comes from
bitmaps of the ids beyond 64 particles: the order is the general sort's, bit for
bit, after steps that leave the particles where they are and after walked ones."""
import numpy as np
import pytest

from paper_1811_05474_amd import rwpt, workloads as W

pytestmark = pytest.mark.gpu


def positions(kind, n, g):
    x = g.random((n, 2))
    if kind == "one point":
        x[:] = 0.4
    elif kind == "edges":  # cells of 63 to 66 particles, one of 1000
        at = 0
        for k, c in enumerate((63, 64, 65, 66, 1000)):
            x[at:at + c] = 0.1 + 0.15 * k
            at += c
    elif kind == "many":  # 62 cells of 66
        x = 0.05 + 0.9 * np.stack([np.arange(n) // 66 % 8, np.arange(n) // 66 // 8], 1) / 8.0
    return x[g.permutation(n)]


@pytest.mark.parametrize("rw", [0.0, 0.05])
@pytest.mark.parametrize("kind,n", [("one point", 4096), ("one point", 65), ("edges", 2000), ("many", 4092),
                                    ("spread", 4096)])
def test_order_is_the_general_sorts(kind, n, rw):
    g = np.random.default_rng(n)
    x, M = positions(kind, n, g), W.masses(n, 2, 6)
    # the realisations come second, so that their ids do not start at zero
    first = 33
    out = []
    for extra in (0, 5000):  # a larger realisation at the end: every step takes the general sort
        sizes = [first, n, n] + ([extra] if extra else [])
        xx = np.concatenate([W.positions(first, 2, 6), x, x, W.positions(extra, 2, 7)])
        MM = np.concatenate([W.masses(first, 2, 6), M, M, W.masses(extra, 2, 7)], 1)
        ens = rwpt.Ensemble(dim=2, n_species=2, react=(0, 1), rw_ratio=rw, precision=rwpt.RWPT_FP64, seed=33)
        ens.init(sizes, xx, MM)
        for D in (1e-5, 1e-4):
            ens.step(0.1, D, 2)
        rows = slice(0, first + 2 * n)
        out.append((ens.positions()[rows], ens.masses()[:, rows], ens.rowsums(0.1, 1e-4)[rows]))
        ens.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("n", [64, 4095])
def test_allocation_free_call_in_one_cell(n):
    import torch

    x, M = W.positions(n, 2, n), W.masses(n, 2, n)
    cfg = rwpt.rwpt_config_default()
    cfg.precision, cfg.kappa, cfg.path = rwpt.RWPT_FP64, float("inf"), rwpt.RWPT_PATH_SPARSE
    xd, md = torch.from_numpy(x).to("cuda"), torch.from_numpy(M).to("cuda")
    out = torch.empty_like(md)
    for _ in range(2):
        rwpt.rwpt_transfer_noalloc(cfg, n, xd.data_ptr(), md.data_ptr(), out.data_ptr(), 0.1, 1e-3)
    ens = rwpt.Ensemble(dim=2, n_species=2, react=(0, 1), kappa=None, rw_ratio=0.0, precision=rwpt.RWPT_FP64,
                        path=rwpt.RWPT_PATH_SPARSE)
    ens.init([n, 5000], np.concatenate([x, W.positions(5000, 2, 1)]), np.concatenate([M, W.masses(5000, 2, 1)], 1))
    ens.step(0.1, 1e-3, 1)
    assert np.array_equal(out.cpu().numpy(), ens.masses()[:, :n])
    ens.close()
