"""hh_profile_vcycle: it times the launches that the cycle makes (merged ones
where the cycle merges the finest leg), leaves V(f) in u, and leaves nothing
running on the stream."""
import numpy as np
import pytest

from paper_0912_0180_amd import workloads as W

pytestmark = pytest.mark.gpu


# sides, levels, and whether the finest down- and up-leg are part of a merged
# launch: coarsest 16^2 (k_coarse) below three and four levels, the tail kernel
# below two, a level 0 of more than 65,536 unknowns, and 3D
@pytest.mark.parametrize("n,levels,merged", [((128, 128), 4, (True, True)), ((256, 256), 5, (False, True)),
                                             ((128, 128), 5, (True, True)), ((272, 256), 5, (False, False)),
                                             ((32, 32, 32), 3, (False, False))])
@pytest.mark.parametrize("prec", ["c64", "c128"])
def test_profile_times_the_cycle_and_waits(n, levels, merged, prec):
    import torch
    from paper_0912_0180_amd import hh
    print("case", n, levels, prec, flush=True)
    dim = len(n)
    lo = [-0.1] * dim
    hi = [lo[a] + n[a] / 64 for a in range(dim)]
    d = W.base_desc(dim, n, lo, hi, [0.0] * dim, [v - 0.1 for v in hi], levels=levels)
    rng = np.random.default_rng(3)
    N = int(np.prod(n))
    g = hh.Grid(d, 100.0 * (1 + 0.3 * rng.uniform(size=N)))
    f = torch.from_numpy(rng.standard_normal(N) + 1j * rng.standard_normal(N)).cuda()
    ref = g.vcycle(f, prec)
    u = torch.zeros_like(ref)
    torch.cuda.synchronize()
    s, t = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(s):
        r = g.profile_vcycle(f, prec, reps=3, out=u)
        idle = s.query()
    with torch.cuda.stream(t):      # no wait for s between
        got = u.cpu()
    assert idle
    assert torch.equal(got, ref.cpu())
    assert ((r["down_shape"] == -1), (r["up_shape"] == -1)) == merged
    assert min(r["down_shape"], r["up_shape"]) >= -1 and min(r["down_groups"], r["up_groups"]) >= 1
    assert min(r["vcycle_us"], r["down_us"], r["up_us"]) > 0.0
