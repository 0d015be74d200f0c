"""The allocation-free call on arrays that begin one element into a larger one:
aligned to their elements and to no vector.  The masses are those of the call on
arrays of their own, bit for bit."""
import numpy as np
import pytest

from paper_1811_05474_amd import rwpt, workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [rwpt.RWPT_FP32, rwpt.RWPT_FP64])
@pytest.mark.parametrize("dim,n,S", [(1, 501, 1), (1, 5001, 3), (2, 501, 2), (2, 5001, 2), (2, 5001, 5), (3, 501, 8),
                                     (3, 5001, 3)])
def test_offset_arrays(dim, n, S, prec):
    import torch

    t = torch.float32 if prec == rwpt.RWPT_FP32 else torch.float64
    cfg = rwpt.rwpt_config_default()
    cfg.dim, cfg.n_species, cfg.precision = dim, S, prec
    cfg.react_a, cfg.react_b = (0, 1) if S > 1 else (-1, -1)
    D = (20.0 / n) ** (2.0 / dim) / 72.0 / 4.0
    x, M = (torch.from_numpy(a).to("cuda", t) for a in (W.positions(n, dim, 1), W.masses(n, S, 1)))
    out = []
    for off in (0, 1):
        xs, ms = torch.zeros(x.numel() + 1, dtype=t, device="cuda"), torch.zeros(M.numel() + 1, dtype=t, device="cuda")
        xs[off:off + x.numel()] = x.reshape(-1)
        ms[off:off + M.numel()] = M.reshape(-1)
        res = torch.full((M.numel() + 2,), -1.0, dtype=t, device="cuda")
        rwpt.rwpt_transfer_noalloc(cfg, n, xs[off:].data_ptr(), ms[off:].data_ptr(), res[off:].data_ptr(), 0.1, D)
        torch.cuda.synchronize()
        got = res.cpu().numpy()
        assert np.all(got[:off] == -1.0) and np.all(got[off + M.numel():] == -1.0)
        out.append(got[off:off + M.numel()])
    assert np.array_equal(out[0], out[1]) and np.all(np.isfinite(out[0]))
