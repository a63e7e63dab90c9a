"""Tile shapes are timed the first time a level class is planned, on a stream of
the library's own.  Cycles of the same grid that are still running then keep
their values: a batch is planned behind cycles whose own plan merged the finest
levels and so has timed no shape of theirs."""
import numpy as np
import pytest

from paper_0912_0180_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["c64", "c128"])
@pytest.mark.parametrize("n,levels", [((208, 176), 5), ((144, 112), 4), ((96, 80), 3)])
def test_cycles_in_flight_keep_their_values(n, levels, prec):
    import torch
    from paper_0912_0180_amd import hh
    print("case", n, levels, prec, flush=True)
    lo = [-0.1] * 2
    hi = [lo[a] + n[a] / 64 for a in range(2)]
    d = W.base_desc(2, n, lo, hi, [0.0] * 2, [v - 0.1 for v in hi], levels=levels)
    rng = np.random.default_rng(17)
    N = int(np.prod(n))
    A, B = (hh.Grid(d, 100.0 * (1 + 0.3 * rng.uniform(size=N))) for _ in range(2))
    fs = [torch.from_numpy(rng.standard_normal(N) + 1j * rng.standard_normal(N)).cuda() for _ in range(8)]
    ref = [A.vcycle(f, prec).clone() for f in fs]
    torch.cuda.synchronize()
    outs = [torch.zeros_like(ref[0]) for _ in range(160)]
    for k, u in enumerate(outs):
        A.vcycle(fs[k % 8], prec, out=u)
    hh.solve_batch([A, B], [fs[0], fs[1]], tol=1e-30, max_matvec=4, vcycle_prec=prec)     # planned while they run
    torch.cuda.synchronize()
    for k, u in enumerate(outs):
        assert torch.equal(u, ref[k % 8]), k
