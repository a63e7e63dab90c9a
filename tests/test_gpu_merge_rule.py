"""Where the merged legs of one problem take level 0: not in FP64 over three
levels with more down-leg tiles than CUs (a workgroup takes a CU there, and they
would run in two rounds).  Either way the cycle is the oracle's."""
import numpy as np
import pytest

from paper_0912_0180_amd import workloads as W

pytestmark = pytest.mark.gpu


# sides, levels, (FP64, FP32) level 0 merged: 256, 260 and 272 tiles of 2 x 2
# coarsest points over three levels; 260 over two; more unknowns than the rule takes
@pytest.mark.parametrize("n,levels,merged", [((256, 256), 4, (True, True)), ((320, 200), 4, (False, True)),
                                             ((248, 264), 4, (False, True)), ((8192, 8), 4, (False, True)),
                                             ((160, 100), 3, (True, True)), ((272, 256), 5, (False, False))])
def test_level_0_and_values(oracle_mod, n, levels, merged):
    import torch
    from paper_0912_0180_amd import hh
    print("case", n, levels, flush=True)
    hi = [-0.1 + m / 64 for m in n]
    d = W.base_desc(2, n, [-0.1] * 2, hi, [-0.05] * 2, [v - 0.02 for v in hi], levels=levels)
    rng = np.random.default_rng(n[0])
    N = int(np.prod(n))
    phi, f = 100.0 * (1 + 0.3 * rng.uniform(size=N)), rng.standard_normal(N) + 1j * rng.standard_normal(N)
    g, o = hh.Grid(d, phi), oracle_mod.Grid(d, phi)
    fd = torch.from_numpy(f).cuda()
    ref = o.vcycle(f)
    u = g.vcycle(fd, "c128")
    assert np.array_equal(u.cpu().numpy(), ref)
    u32 = g.vcycle(fd, "c64").cpu().numpy()
    assert np.linalg.norm(u32 - ref) <= 1e-4 * np.linalg.norm(ref)     # FP32 rounding, cycle norm of order 100
    for prec, m in zip(("c128", "c64"), merged):
        r = g.profile_vcycle(fd, prec, reps=2)
        assert ((r["down_shape"] == -1), (r["up_shape"] == -1)) == (m, m), prec
    if g.N * 16 / 2 < 32 << 20:
        assert torch.equal(g.vcycle_noalloc(fd, "c128"), u)
