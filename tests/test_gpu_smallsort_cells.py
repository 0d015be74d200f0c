"""Cells of many particles in the one-launch sort, whose in-cell order comes from
bitmaps of the ids beyond 128 particles: the order is the general sort's, bit for
bit, after steps that leave the particles where they are and after walked ones."""
import numpy as np
import pytest

from paper_1811_05474_amd import rwpt, workloads as W

pytestmark = pytest.mark.gpu


def positions(kind, n, g):
    x = g.random((n, 2))
    if kind == "one point":
        x[:] = 0.4
    elif kind == "edges":  # cells of 127 to 130 particles, one of 1000
        at = 0
        for k, c in enumerate((127, 128, 129, 130, 1000)):
            x[at:at + c] = 0.1 + 0.15 * k
            at += c
    elif kind == "many":  # 31 cells of 132
        x = 0.05 + 0.9 * np.stack([np.arange(n) // 132 % 8, np.arange(n) // 132 // 8], 1) / 8.0
    return x[g.permutation(n)]


@pytest.mark.parametrize("rw", [0.0, 0.05])
@pytest.mark.parametrize("kind,n", [("one point", 4096), ("one point", 129), ("edges", 2000), ("many", 4092),
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


@pytest.mark.parametrize("n", [128, 4095])
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


# (dimension, realisations, particles each, species): either side of 768 realisations, of 700
# particles on average beyond, of 2048 single particles, and of 2048 particles in 3-D with eight
# species slots in binary64
@pytest.mark.parametrize("dim,n_real,n,S", [(2, 768, 20, 2), (2, 769, 20, 2), (2, 800, 699, 2), (2, 800, 700, 2),
                                            (2, 2048, 1, 2), (2, 2049, 1, 2), (3, 3, 2048, 8), (3, 3, 2049, 5),
                                            (2, 3, 2049, 8)])
def test_limits(dim, n_real, n, S):
    dt, seed = 0.1, 11
    D = 2e-5 * 400.0 / n if dim == 2 else 1e-4
    x, M = W.positions(n_real * n, dim, n), W.masses(n_real * n, S, n)
    ens = rwpt.Ensemble(dim=dim, n_species=S, react=(0, 1), rw_ratio=1.0, precision=rwpt.RWPT_FP64, seed=seed)
    ens.init([n] * n_real, x, M)
    ens.step(dt, D, 2)
    ens.step(dt, D, 1)
    got, pos = ens.masses(), ens.positions()
    assert np.allclose(ens.audit()[:, :S].sum(0), got.sum(1), rtol=1e-12)
    ens.close()
    # the realisations do not see each other, so the middle one is the same with a larger one beside it,
    # under the general sort (its ids, hence its walk, are the same)
    r = n_real // 2
    rows = slice(r * n, (r + 1) * n)
    bar = 1e-12 * np.abs(got).max() if dim == 3 else 0.0  # other cells, by the mean neighbours of all realisations
    ens = rwpt.Ensemble(dim=dim, n_species=S, react=(0, 1), rw_ratio=1.0, precision=rwpt.RWPT_FP64, seed=seed)
    ens.init([r * n, n, 5000], np.concatenate([x[:(r + 1) * n], W.positions(5000, dim, 1)]),
             np.concatenate([M[:, :(r + 1) * n], W.masses(5000, S, 1)], 1))
    ens.step(dt, D, 3)
    assert np.array_equal(ens.positions()[rows], pos[rows])
    assert np.abs(ens.masses()[:, rows] - got[:, rows]).max() <= bar
    ens.close()
