"""Merged legs of batches without pre-smoothing, and with it beside: V(0,1) and
V(1,1) problems in one batch, against the CPU oracle value for value (FP64) and
the same problems solved alone (FP32 cycles)."""
import numpy as np
import pytest

from paper_0912_0180_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nu1", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("sizes", [(((352, 416), 6), ((208, 176), 5)), (((208, 240), 5), ((96, 80), 3))])
def test_batch_merge_v01(oracle_mod, sizes, nu1):
    import torch
    from paper_0912_0180_amd import hh
    print("case", sizes, nu1, flush=True)
    grids, bs, refs = [], [], []
    for k, (n, levels) in enumerate(sizes):
        hi = [-0.1 + m / 64 for m in n]
        d = W.base_desc(2, n, [-0.1] * 2, hi, [0.0] * 2, [v - 0.1 for v in hi], levels=levels, nu1=nu1[k])
        rng = np.random.default_rng(70 + k)
        N = int(np.prod(n))
        phi, b = 100.0 * (1 + 0.3 * rng.uniform(size=N)), rng.standard_normal(N) + 1j * rng.standard_normal(N)
        grids.append(hh.Grid(d, phi))
        bs.append(torch.from_numpy(b).cuda())
        refs.append(oracle_mod.Grid(d, phi).solve(b, method="bicgstab", tol=1e-30, max_matvec=6)[0])
    xs, _ = hh.solve_batch(grids, bs, tol=1e-30, max_matvec=6, vcycle_prec="c128")
    for x, ref in zip(xs, refs):
        assert np.array_equal(x.cpu().numpy(), ref)
    xs, infos = hh.solve_batch(grids, bs, tol=1e-30, max_matvec=6, vcycle_prec="c64")
    for g, b, x, i in zip(grids, bs, xs, infos):
        xa, ia = g.solve(b, tol=1e-30, max_matvec=6, vcycle_prec="c64")
        assert i["matvecs"] == ia["matvecs"] and torch.equal(x, xa)
