"""Merged legs of a batch, at the edges of what takes part in them: coarsest
sides that are no multiple of the tile, three and four merged up-levels, the
fewest levels that merge, problems beside them that do not, and batches the
rule leaves on the tiled legs.  FP64 against the CPU oracle value for value,
FP32 cycles against the same problems solved alone."""
import numpy as np
import pytest

from paper_0912_0180_amd import workloads as W

pytestmark = pytest.mark.gpu


def problem(n, levels, seed):
    h = 1.0 / 64
    lo = [-0.1] * 2
    hi = [lo[a] + h * n[a] for a in range(2)]
    d = W.base_desc(2, n, lo, hi, [0.0] * 2, [v - 0.1 for v in hi], levels=levels)
    rng = np.random.default_rng(seed)
    N = int(np.prod(n))
    return d, 100.0 * (1 + 0.3 * rng.uniform(size=N)), rng.standard_normal(N) + 1j * rng.standard_normal(N)


# (sides, levels) of each problem
BATCHES = {
    "four up-levels": [((352, 416), 6), ((480, 224), 6)],
    "fewest levels": [((208, 176), 5), ((176, 144), 5)],
    "mixed depths": [((192, 224), 5), ((576, 320), 7), ((256, 256), 6)],
    "beside tiled ones": [((208, 240), 5), ((96, 80), 3), ((48, 40), 2)],
    "no split coarsest": [((128, 160), 5), ((96, 128), 5)],
    "too many workgroups": [((480, 512), 5)] * 3,
}


@pytest.mark.parametrize("name", BATCHES)
def test_batch_merge(oracle_mod, name):
    import torch
    from paper_0912_0180_amd import hh
    print("case", name, flush=True)
    grids, bs, refs = [], [], []
    for k, (n, levels) in enumerate(BATCHES[name]):
        d, phi, b = problem(n, levels, 31 + k)
        grids.append(hh.Grid(d, phi))
        bs.append(torch.from_numpy(b).cuda())
        refs.append(oracle_mod.Grid(d, phi).solve(b, method="bicgstab", tol=1e-30, max_matvec=6)[0])
    xs, _ = hh.solve_batch(grids, bs, tol=1e-30, max_matvec=6, vcycle_prec="c128")
    for x, ref in zip(xs, refs):
        assert np.array_equal(x.cpu().numpy(), ref)
    xs, infos = hh.solve_batch(grids, bs, tol=1e-30, max_matvec=6, vcycle_prec="c64")
    for g, b, x, i in zip(grids, bs, xs, infos):
        xa, ia = g.solve(b, tol=1e-30, max_matvec=6, vcycle_prec="c64")
        assert i["matvecs"] == ia["matvecs"]
        assert np.array_equal(x.cpu().numpy(), xa.cpu().numpy())
